"""What the gradient call launches, recorded without a GPU (tests/host/record_launches.c takes the place of the
runtime's launch entry points): grids stay within what a launch may ask for, and buffers that were large enough stay so."""
import os
import shutil
import subprocess

import pytest

from paper_2601_04342_amd import binding, build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    if shutil.which("gcc") is None:
        pytest.skip("gcc not available")
    binding.library()   # built if it is not there
    exe = str(tmp_path_factory.mktemp("host") / "record_launches")
    subprocess.run(["gcc", "-O1", "-rdynamic", os.path.join(ROOT, "tests", "host", "record_launches.c"), "-o", exe,
                    "-ldl"], check=True, capture_output=True, text=True)

    def run(B, H, T, HW, d, chunk, overlap, saved, ws_bytes):
        """(status, [(x, y, z, kernel), ...]) of one rehyat_phi_backward call."""
        args = (B, H, T, HW, d, chunk, overlap, int(saved), ws_bytes)
        r = subprocess.run([exe, build.LIB, *map(str, args)], capture_output=True, text=True, timeout=120, check=True)
        *lines, status = r.stdout.splitlines()
        grids = [line.split() for line in lines]
        return int(status.split()[1]), [(int(x), int(y), int(z), name) for x, y, z, name in grids]

    return run


@pytest.mark.parametrize("saved", [False, True])
@pytest.mark.parametrize("B,H,d", [(1, 12, 128), (32767, 1, 64), (16384, 2, 64), (65535, 1, 64), (1, 65535, 128)])
def test_gradient_grids_stay_in_bounds(record, B, H, d, saved):
    """Up to 65,535 (batch, head)s are accepted; no launch asks for more rows or layers of blocks than that."""
    T, HW, chunk = 2, 1, 1
    need = binding.phi_backward_workspace_bytes(B, H, T, HW, d, chunk)
    status, launches = record(B, H, T, HW, d, chunk, 0, saved, need)
    assert status == binding.OK and len(launches) >= 6
    for x, y, z, name in launches:
        assert 1 <= x < 2**31 and 1 <= y <= 65535 and 1 <= z <= 65535, (x, y, z, name)


# bytes that the call asked for while every launch was of one side; launches with a saved forward pass
@pytest.mark.parametrize("B,H,T,HW,d,chunk,enough,launches", [
    (1, 12, 21, 1560, 128, 1, 498_432_000, 6),
    (1, 12, 21, 600, 128, 3, 215_623_680, 6),
    (1, 24, 21, 1560, 64, 1, 463_828_992, 6),
    (1, 22, 93, 16, 128, 1, 590_233_600, 8),     # the sums of both sides at once would take 831 MB
    (1, 12, 101, 50, 128, 1, 394_206_720, 8),
    (1, 2, 87, 105, 128, 1, 71_393_280, 6),
    (1, 6, 50, 60, 128, 1, 101_624_832, 8),
    (2, 8, 134, 2288, 64, 5, 2_698_715_136, 9),  # 1 / den and w beside everything else would take 25 MB more
    (1, 8, 25, 84, 128, 1, 74_008_576, 8),
    (1, 1, 8, 550, 128, 2, 32_701_440, 6),       # the layouts of the GPU test
    (1, 3, 28, 42, 64, 7, 8_114_176, 6),
    (2, 3, 50, 20, 64, 1, 24_033_792, 8),
    (1, 2, 40, 29, 128, 7, 18_940_928, 6),
    (64, 2, 4, 4105, 64, 1, 1_178_419_200, 9),
])
def test_gradient_takes_the_buffers_that_it_took(record, B, H, T, HW, d, chunk, enough, launches):
    need = binding.phi_backward_workspace_bytes(B, H, T, HW, d, chunk)
    assert need % 256 == 0 and 0 < need <= enough
    for saved, n in ((True, launches), (False, 10 if launches == 9 else 9)):
        status, got = record(B, H, T, HW, d, chunk, 0, saved, need)
        assert status == binding.OK and len(got) == n, [name for *_, name in got]
    assert record(B, H, T, HW, d, chunk, 0, True, need - 1) == (binding.E_WORKSPACE, [])
