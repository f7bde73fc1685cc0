"""What the gradient call launches, recorded without a GPU (tests/host/record_launches.c takes the place of the
runtime's launch entry points): grids stay within what a launch may ask for."""
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
