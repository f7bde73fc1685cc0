"""Tile-edge sizes of the loops that run the next tile's first products beside the current tile:
one tile, the fewest that enter the loop, odd and even counts, and last tiles of 1, 2, 63 and 64
rows, at both head widths, against the oracle with every component."""
import pytest
import torch

from tests import parity

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _announce(request):
    print(f"[gpu-test] {request.node.nodeid}", flush=True)
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("HW", [1, 63, 64, 65, 127, 128, 130, 191, 193, 256, 319, 386])
def test_key_tiles(HW, d):
    """Softmax windows of one to seven key tiles (below 448 keys: one group of waves), and chunk
    states over as many tiles."""
    parity.run_case(1, 1, 3, HW, d, 1, 0, 0, 4.0, seed=HW + d)
