"""Tile-edge sizes of the loops that run the next tile's first products beside the current tile:
one tile, the fewest that enter the loop, odd and even counts, and last tiles of 1, 2, 63 and 64
rows, at both head widths, against the oracle with every component."""
import pytest
import torch

from paper_2601_04342_amd import binding, synth
from tests import parity
from tests.test_gpu_backward import run_case

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _announce(request):
    print(f"[gpu-test] {request.node.nodeid}", flush=True)
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("HW", [1, 63, 64, 65, 127, 128, 130, 191, 193, 256, 319, 386])
def test_key_tiles(HW, d):
    """Softmax windows of one to seven key tiles (one group of waves), and chunk
    states over as many tiles."""
    parity.run_case(1, 1, 3, HW, d, 1, 0, 0, 4.0, seed=HW + d)


@pytest.mark.parametrize("d", [128, 64])
def test_chunk_states_are_reproducible(d):
    """Every CU runs state pieces of three and more tiles several times over: the same bits each time
    (a barrier that publishes a tile too early shows as rare differences)."""
    H, T, HW = 48, 4, 1300
    q, k, v = synth.make_qkv(1, H, T * HW, d, seed=d)
    phi = synth.make_phi(H, d, seed=1, gain=4.0)
    _, dk, dv, dphi = parity.to_device(q, k, v, phi)
    first = binding.state(dk, dv, dphi, T, HW, T)
    for i in range(20):
        again = binding.state(dk, dv, dphi, T, HW, T)
        assert all(torch.equal(a, b) for a, b in zip(again, first)), i


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("B,H,HW", [(1, 1, 32), (1, 1, 65), (16, 8, 33), (16, 8, 64), (16, 8, 97), (16, 8, 160)])
def test_weight_gradient_tiles(B, H, HW, d):
    """Weight gradients of pieces of one tile (one head; HW = 65 leaves a piece of two rows) and of two, four and
    five tiles with a last one of 2 or 64 rows (128 (b, h), one piece each); bars as for the other gradients."""
    run_case(B, H, 3, HW, d, 1, 0, 4.0, seed=HW + d)


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("nan", ["nan", "-nan", "inf - inf"])
def test_gate_of_every_nan_is_closed(nan, d):
    """As below, for NaN of either sign in the weights and for one that the products make."""
    B, H, T, HW = 1, 2, 3, 97
    q, k, v = synth.make_qkv(B, H, T * HW, d, seed=d)
    G = synth.make_grad_out(B, H, T * HW, d).to("cuda", torch.bfloat16)
    _, dk, dv, dphi = parity.to_device(q, k, v, synth.make_phi(H, d, seed=1, gain=4.0))
    dq = q.to("cuda", torch.bfloat16)
    runs = []
    for on in (True, False):
        phi = {n: t.clone() for n, t in dphi.items()}
        for side in "qk":
            phi[f"w1_{side}"][0, 5] = 0.0
            phi[f"b1_{side}"][0, 5] = -1.0
            if on and nan == "inf - inf":
                phi[f"w1_{side}"][0, 5, :2] = torch.tensor([float("inf"), float("-inf")], device="cuda")
                for x in (dq, dk):
                    x[..., :2] = x[..., :2].abs() + 0.5
                phi[f"b1_{side}"][0, 5] = 0.0
            elif on:
                phi[f"w1_{side}"][0, 5] = torch.tensor(0x7FC0 if nan == "nan" else -0x40, dtype=torch.int16).view(torch.bfloat16)
        runs.append(binding.phi_backward(dq, dk, dv, phi, G, T, HW, 1)[0])
    for n in runs[0]:
        assert torch.isfinite(runs[0][n]).all(), n
        assert torch.equal(runs[0][n], runs[1][n]), n


@pytest.mark.parametrize("d", [128, 64])
def test_gate_of_a_nan_is_closed(d):
    """A hidden unit that is NaN for every token is rectified to zero, and its gate is closed: the gradients are
    those of a unit that is negative everywhere, bit for bit."""
    B, H, T, HW = 1, 2, 3, 97
    q, k, v = synth.make_qkv(B, H, T * HW, d, seed=d)
    G = synth.make_grad_out(B, H, T * HW, d).to("cuda", torch.bfloat16)
    _, dk, dv, dphi = parity.to_device(q, k, v, synth.make_phi(H, d, seed=1, gain=4.0))
    dq = q.to("cuda", torch.bfloat16)
    runs = []
    for nan in (True, False):
        phi = {n: t.clone() for n, t in dphi.items()}
        for side in "qk":
            for unit in (5, 2 * d - 1):
                phi[f"w1_{side}"][0, unit] = float("nan") if nan else 0.0
                phi[f"b1_{side}"][0, unit] = -1.0
        runs.append(binding.phi_backward(dq, dk, dv, phi, G, T, HW, 1)[0])
    for n in runs[0]:
        assert torch.isfinite(runs[0][n]).all(), n
        assert torch.equal(runs[0][n], runs[1][n]), n


@pytest.mark.parametrize("d,HW,row", [
    (128, 97, 36), (64, 97, 36),        # the last tile holds rows 33 .. 96
    (128, 1000, 939), (64, 1700, 1639),   # two groups of waves
    (128, 40, 39), (64, 40, 39),        # fewer rows than a tile: the last one stands in for those beyond
])
def test_infinite_value_in_a_shared_row(d, HW, row):
    """A ragged last key tile holds rows that an earlier tile has taken already.  An infinity in such a row of V
    counts once: its column of the output is infinite, not NaN, and no other column changes."""
    q, k, v = synth.make_qkv(1, 1, HW, d, seed=HW + d)
    dq, dk, dv, dphi = parity.to_device(q, k, v, synth.make_phi(1, d, seed=1))
    want = binding.forward(dq, dk, dv, dphi, 1, HW, 1)
    dv[0, 0, row, 5] = float("inf")
    out = binding.forward(dq, dk, dv, dphi, 1, HW, 1)
    assert (out[..., 5] == float("inf")).all()
    rest = [c for c in range(d) if c != 5]
    assert torch.equal(out[..., rest], want[..., rest])


@pytest.mark.parametrize("d", [128, 64])
def test_infinite_value_in_a_state(d):
    """The same for chunk states, at every row: S is infinite where phi of the key is positive."""
    HW = 97
    _, k, v = synth.make_qkv(1, 1, HW, d, seed=d)
    phi = synth.make_phi(1, d, seed=1, gain=4.0)
    _, dk, dv, dphi = parity.to_device(k, k, v, phi)
    p = {n: t.double()[0] for n, t in phi.items()}
    psi = torch.relu(torch.relu(k[0, 0].double() @ p["w1_k"].T + p["b1_k"]) @ p["w2_k"].T + p["b2_k"])
    for row in range(HW):
        x = dv.clone()
        x[0, 0, row, 5] = float("inf")
        S, _ = binding.state(dk, x, dphi, 1, HW, 1)
        on = psi[row] > 0.02 * psi[row].max()   # well above what bf16 makes of zero
        assert (S[0, 0, :, 5].cpu()[on] == float("inf")).all(), row


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("row", [36, 96])
def test_infinite_gradient_in_a_shared_row(d, row):
    """An infinite dL/dy at a token whose row two tiles hold: the second layer's gradient keeps the infinities of
    the features that it opens (NaN only where they meet a closed hidden unit)."""
    B, H, T, HW = 16, 16, 2, 97
    q, k, v = synth.make_qkv(B, H, T * HW, d, seed=d)
    G = synth.make_grad_out(B, H, T * HW, d).to("cuda", torch.bfloat16)
    G[0, 0, HW + row, 5] = float("inf")
    _, dk, dv, dphi = parity.to_device(q, k, v, synth.make_phi(H, d, seed=1, gain=4.0))
    grads, _ = binding.phi_backward(q.to("cuda", torch.bfloat16), dk, dv, dphi, G, T, HW, 1)
    assert torch.isinf(grads["w2_q"][0]).any()
    assert torch.isfinite(grads["w2_q"][1:]).all()
