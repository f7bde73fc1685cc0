"""GPU parity of the feature-map gradient (rehyat_phi_backward, Eq. 19) against the fp64
gradient oracle, element by element, on the same seeded bf16-rounded inputs."""
import numpy as np
import pytest
import torch

from oracle import grad as ograd
from paper_2601_04342_amd import binding, synth
from tests import parity

pytestmark = pytest.mark.gpu

# Bars on each of the eight gradient tensors, relative to the tensor's own scale.  Every entry
# is a sum over tokens of signed products whose factors pass through bf16 on the GPU (MFMA
# operands): Phi_q/den, Phi_q, the states S_t and R_tau, dpsi, dU, and y_hat inside w -- up to
# six roundings of relative size <= 2^-8 (rms 2^-9 / sqrt 3 = 1.1e-3) along one path, fp32
# accumulation.  The terms of a sum have random signs, so the relative error of the sum stays at
# the level of one term's: about sqrt(6) * 1.1e-3 = 2.8e-3 in the Frobenius norm (4e-3 to 5e-3 when
# the roundings are replayed in numpy on the first cases below): the Frobenius bar leaves a factor
# two.  The largest single-entry error is the maximum over 10^4 - 10^6 entries of a roughly Gaussian
# error of that relative size, i.e. 4 - 5 standard deviations of an entry (1.6e-2 of max |ref| is the
# largest seen, on a 320x480 workload); its bar is set at six.  A wrong term, sign or index moves
# entries by O(1).  The hidden activations U are bf16 on both sides (hidden_round of the oracle), so
# the ReLU gates of the second layer are decided on the same values.
MAX_REL = 3e-2    # max |gpu - ref| <= MAX_REL * max |ref|
FRO_REL = 1e-2    # ||gpu - ref||_F <= FRO_REL * ||ref||_F


@pytest.fixture(autouse=True)
def _announce(request):
    print(f"[gpu-test] {request.node.nodeid}", flush=True)
    yield
    torch.cuda.synchronize()


def check_grads(grads, ref, label):
    worst = 0.0
    for name in synth.PHI_NAMES:
        g = grads[name].cpu().double().numpy()
        r = ref[name]
        assert np.isfinite(g).all(), (label, name)
        scale = np.abs(r).max()
        emax = np.abs(g - r).max()
        efro = np.linalg.norm(g - r) / max(np.linalg.norm(r), 1e-300)
        print(f"   {name}: max-abs err / max |ref| = {emax / max(scale, 1e-300):.2e}   "
              f"relative Frobenius = {efro:.2e}   max |ref| = {scale:.3e}", flush=True)
        if scale == 0.0:
            assert emax == 0.0, (label, name)
            continue
        assert emax <= MAX_REL * scale, (label, name, emax, scale)
        assert efro <= FRO_REL, (label, name, efro)
        worst = max(worst, efro)
    return worst


def run_case(B, H, T, HW, d, chunk, overlap, gain, seed, l1=False):
    N = T * HW
    q, k, v = synth.make_qkv(B, H, N, d, seed=seed)
    phi = synth.make_phi(H, d, seed=seed + 1, gain=gain)
    if l1:
        # G of the L1 loss of Eq. 19 against a random teacher: +-1/count, exact in bf16 for
        # a power-of-two count; the sign pattern comes from a seeded draw, not from y_hat
        G = torch.sign(synth.make_grad_out(B, H, N, d, seed=seed + 2)) / 65536.0
    else:
        G = synth.make_grad_out(B, H, N, d, seed=seed + 2)
    dq, dk, dv, dphi = parity.to_device(q, k, v, phi)
    dG = G.to("cuda", torch.bfloat16).contiguous()
    grads = {n: torch.full(t.shape, float("nan"), device="cuda", dtype=torch.float32)
             for n, t in dphi.items()}
    grads, y = binding.phi_backward(dq, dk, dv, dphi, dG, T, HW, chunk, overlap=overlap,
                                    out=parity.nan_like(dq), grads=grads)
    torch.cuda.synchronize()
    qn, kn, vn, pn = parity.oracle_inputs(q, k, v, phi)
    ref, y_ref = ograd.phi_backward(qn, kn, vn, pn, G.double().numpy(), T, HW, chunk, overlap,
                                        hidden_round="bf16")
    label = f"B{B} H{H} T{T} HW{HW} d{d} chunk{chunk} ov{overlap} gain{gain}"
    yerr = np.abs(y.float().cpu().double().numpy() - y_ref)
    assert np.isfinite(yerr).all(), label
    assert yerr.max() <= parity.OUT_MAX_ABS and yerr.mean() <= parity.OUT_MEAN_ABS, (label, yerr.max())
    return check_grads(grads, ref, label)


CASES = [
    # B, H, T, HW, d, chunk, overlap, gain
    (1, 2, 4, 64, 64, 1, 0, 8.0),
    (2, 3, 5, 77, 128, 2, 0, 4.0),      # T % chunk != 0, ragged tiles, batch sum
    (1, 2, 5, 77, 128, 2, 1, 4.0),      # overlapping windows: key segments lag the chunks
    (1, 2, 7, 50, 64, 3, 2, 6.0),
    (1, 2, 4, 30, 64, 1, 3, 6.0),       # overlap reaches the first frame: empty key segments
    (1, 2, 6, 700, 128, 1, 0, 2.0),     # many tiles per segment
    (1, 1, 4, 2000, 128, 1, 0, 2.0),    # few (b, h, segment): segments are split
    (1, 2, 40, 20, 64, 1, 0, 3.0),      # many short chunks (segments shorter than a tile)
    (2, 2, 6, 300, 64, 2, 1, 4.0),      # d = 64 with several tiles per segment, batch 2, overlap
    (1, 1, 2, 1, 128, 1, 0, 1.0),       # two tokens (small phi: with a dominant linear part the
                                        # single query's gradient is a difference of nearly equal terms)
]


@pytest.mark.parametrize("case", CASES)
def test_small_shapes_match_gradient_oracle(case):
    run_case(*case, seed=sum(case[:7]))


@pytest.mark.parametrize("case", [
    (2, 2, 6, 300, 128, 1, 0, 4.0),     # 58 partials per head: three batches of a reduction wave
    (3, 1, 5, 150, 64, 2, 0, 4.0),      # 36 partials of three batch elements, 12 each
    (5, 1, 2, 60, 64, 1, 0, 4.0),       # a batch element has fewer partials than a block has waves
])
def test_partial_sums_over_batch_and_pieces(case):
    run_case(*case, seed=sum(case[:7]))


def test_l1_distillation_gradient():
    run_case(1, 2, 5, 200, 128, 1, 0, 4.0, seed=5, l1=True)


def test_one_chunk_gives_zero_gradients():
    B, H, T, HW, d = 1, 2, 3, 100, 128
    q, k, v = synth.make_qkv(B, H, T * HW, d, seed=3)
    phi = synth.make_phi(H, d, seed=4, gain=4.0)
    dq, dk, dv, dphi = parity.to_device(q, k, v, phi)
    dG = synth.make_grad_out(B, H, T * HW, d).to("cuda", torch.bfloat16)
    grads = {n: torch.full(t.shape, float("nan"), device="cuda", dtype=torch.float32)
             for n, t in dphi.items()}
    grads, y = binding.phi_backward(dq, dk, dv, dphi, dG, T, HW, T, grads=grads)
    torch.cuda.synchronize()
    for n in synth.PHI_NAMES:
        assert (grads[n] == 0).all(), n
    assert torch.equal(y, binding.forward(dq, dk, dv, dphi, T, HW, T))


def test_backward_is_reproducible_and_leaves_inputs_alone():
    B, H, T, HW, d = 1, 2, 5, 150, 128
    q, k, v = synth.make_qkv(B, H, T * HW, d, seed=8)
    phi = synth.make_phi(H, d, seed=9, gain=4.0)
    dq, dk, dv, dphi = parity.to_device(q, k, v, phi)
    dG = synth.make_grad_out(B, H, T * HW, d).to("cuda", torch.bfloat16)
    keep = [t.clone() for t in (dq, dk, dv, dG)]
    g1, y1 = binding.phi_backward(dq, dk, dv, dphi, dG, T, HW, 1)
    g2, y2 = binding.phi_backward(dq, dk, dv, dphi, dG, T, HW, 1)
    torch.cuda.synchronize()
    for n in synth.PHI_NAMES:
        assert torch.equal(g1[n], g2[n]), n
    assert torch.equal(y1, y2)
    for a, b in zip(keep, (dq, dk, dv, dG)):
        assert torch.equal(a, b)


def test_workspace_too_small_is_refused():
    B, H, T, HW, d = 1, 2, 4, 64, 64
    q, k, v = synth.make_qkv(B, H, T * HW, d)
    phi = synth.make_phi(H, d)
    dq, dk, dv, dphi = parity.to_device(q, k, v, phi)
    dG = dq.clone()
    need = binding.phi_backward_workspace_bytes(B, H, T, HW, d, 1)
    ws = torch.empty(need - 256, device="cuda", dtype=torch.uint8)
    with pytest.raises(binding.RehyatError) as e:
        binding.phi_backward(dq, dk, dv, dphi, dG, T, HW, 1, workspace=ws)
    assert e.value.code == binding.E_WORKSPACE


def full_size_case(name, overlap, heads, seed_g=2):
    """A benchmark-size workload in the launch configuration bench.py --mode backward times;
    the oracle evaluates the first `heads` heads completely (gradients are per head, B = 1)."""
    w = synth.WORKLOADS[name]
    q, k, v, phi = synth.make_workload(w)
    G = synth.make_grad_out(w.B, w.H, w.N, w.d, seed=seed_g)
    dq, dk, dv, dphi = parity.to_device(q, k, v, phi)
    dG = G.to("cuda", torch.bfloat16).contiguous()
    grads = {n: torch.full(t.shape, float("nan"), device="cuda", dtype=torch.float32)
             for n, t in dphi.items()}
    grads, y = binding.phi_backward(dq, dk, dv, dphi, dG, w.T, w.HW, w.chunk, overlap=overlap,
                                    out=parity.nan_like(dq), grads=grads)
    torch.cuda.synchronize()
    for n in synth.PHI_NAMES:
        assert torch.isfinite(grads[n]).all(), n
    assert torch.isfinite(y.float()).all()
    hs = slice(0, heads)
    qn, kn, vn, pn = parity.oracle_inputs(q, k, v, phi, heads=hs)
    ref, y_ref = ograd.phi_backward(qn, kn, vn, pn, G[:, hs].double().numpy(), w.T, w.HW, w.chunk,
                                    overlap, hidden_round="bf16")
    yerr = np.abs(y[:, hs].float().cpu().double().numpy() - y_ref)
    assert yerr.max() <= parity.OUT_MAX_ABS and yerr.mean() <= parity.OUT_MEAN_ABS, yerr.max()
    check_grads({n: g[hs] for n, g in grads.items()}, ref, f"{name} ov{overlap}")


def test_wan480p_every_entry_of_every_gradient():
    """The 480p layer shape (B=1, H=12, d=128, 32,760 tokens, chunk 1): all 2.37 M gradient
    entries against the oracle."""
    full_size_case("wan480p", 0, 12)


def test_p320_chunk3_overlap1_gradients():
    """320x480 shape with the paper's preferred T_c = 3, T_o = 1 (section 4.1): key segments
    lag the chunks by one frame."""
    full_size_case("p320_t21_c3", 1, 4)


@pytest.mark.parametrize("case", [
    # the sums of both sides share their launches here, tokens carry a scale and a weight; pieces of fewer than 64
    # tokens, of 64, one more, ragged; an empty key segment (the window of chunk 1 still holds everything)
    (1, 2, 4, 37, 128, 1, 0), (1, 1, 3, 64, 128, 1, 0), (2, 1, 5, 65, 64, 1, 1), (1, 3, 4, 129, 128, 1, 1),
    (1, 1, 9, 200, 64, 2, 0),
])
def test_saved_forward_pass_at_the_edges_of_tiles(case):
    B, H, T, HW, d, chunk, overlap = case
    q, k, v = synth.make_qkv(B, H, T * HW, d, seed=sum(case))
    phi = synth.make_phi(H, d, seed=sum(case) + 1, gain=4.0)
    G = synth.make_grad_out(B, H, T * HW, d, seed=sum(case) + 2)
    dq, dk, dv, dphi = parity.to_device(q, k, v, phi)
    dG = G.to("cuda", torch.bfloat16).contiguous()
    out, comps = binding.forward(dq, dk, dv, dphi, T, HW, chunk, overlap=overlap, debug=True)
    need = binding.phi_backward_workspace_bytes(B, H, T, HW, d, chunk)
    ws = torch.full((need + 4096,), 255, device="cuda", dtype=torch.uint8)   # NaN wherever nothing was written
    grads, _ = binding.phi_backward(dq, dk, dv, dphi, dG, T, HW, chunk, overlap=overlap, workspace=ws[:need],
                                    saved=(out, comps["nS"], comps["nL"]))
    torch.cuda.synchronize()
    assert (ws[need:] == 255).all()
    ref, _ = ograd.phi_backward(*parity.oracle_inputs(q, k, v, phi), G.double().numpy(), T, HW, chunk, overlap,
                                hidden_round="bf16")
    check_grads(grads, ref, str(case))


def test_saved_forward_pass_gives_the_same_gradients():
    """The distillation step has already run the forward pass: handing its output and the
    components n^S, n^L to the gradient call skips the attention kernel there."""
    B, H, T, HW, d, chunk, overlap = 1, 2, 5, 300, 128, 2, 1
    q, k, v = synth.make_qkv(B, H, T * HW, d, seed=21)
    phi = synth.make_phi(H, d, seed=22, gain=4.0)
    dq, dk, dv, dphi = parity.to_device(q, k, v, phi)
    dG = synth.make_grad_out(B, H, T * HW, d, seed=23).to("cuda", torch.bfloat16)
    g_full, y_full = binding.phi_backward(dq, dk, dv, dphi, dG, T, HW, chunk, overlap=overlap)
    out, comps = binding.forward(dq, dk, dv, dphi, T, HW, chunk, overlap=overlap, debug=True)
    keep = out.clone()
    g_saved, y_saved = binding.phi_backward(dq, dk, dv, dphi, dG, T, HW, chunk, overlap=overlap,
                                            saved=(out, comps["nS"], comps["nL"]))
    torch.cuda.synchronize()
    assert torch.equal(y_saved, keep)            # the saved output is an input: untouched
    # the two forward passes may split the chunk-state sums differently: equal up to that rounding
    assert (y_full.float() - keep.float()).abs().max() <= 2.0 ** -7 * keep.float().abs().max()
    for n in synth.PHI_NAMES:
        a, b = g_full[n].double(), g_saved[n].double()
        assert torch.isfinite(b).all(), n
        assert (a - b).norm() <= 2e-3 * a.norm(), (n, float((a - b).norm() / a.norm()))


@pytest.mark.parametrize("d,H,HW", [(128, 256, 2048), (64, 512, 1024)])
def test_bias_gradient_sums_stay_short(d, H, HW):
    """Every query of chunk 1 contributes the same gradient, so db2_q is HW times that of one query,
    up to the roundings of the sum alone.  A lane sums 16 features of a 32-token block, then the
    blocks of its piece (half the tokens each of two lanes), then pieces: no term passes more than
    16 + HW / 32 + 8 additions, of a relative rounding of 2^-24 each (all terms have one sign)."""
    T, N = 2, 2 * HW
    gen = torch.Generator(device="cuda").manual_seed(7)
    row = lambda n: torch.randn(1, H, n, d, generator=gen, device="cuda").to(torch.bfloat16)
    q = row(1).expand(1, H, N, d).contiguous()
    k, v = row(N), row(N)
    G = (row(1) / 64).expand(1, H, N, d).contiguous()
    dphi = binding.phi_to_device(synth.make_phi(H, d, seed=8, gain=4.0))
    one = torch.zeros_like(G)
    one[:, :, HW] = G[:, :, HW]
    full = binding.phi_backward(q, k, v, dphi, G, T, HW, 1)[0]["b2_q"]
    single = binding.phi_backward(q, k, v, dphi, one, T, HW, 1)[0]["b2_q"]
    torch.cuda.synchronize()
    assert (single != 0).float().mean() > 0.1
    want = single.double() * HW
    err = (full.double() - want).abs()
    bound = (16 + HW / 32 + 8) * 2.0 ** -24
    worst = (err / want.abs().clamp_min(1e-300)).max().item()
    print(f"   worst relative error {worst:.2e}, bound {bound:.2e}", flush=True)
    assert (err <= bound * want.abs()).all(), worst


def test_saved_forward_pass_of_more_batch_heads_than_half_a_grid():
    """32,800 (batch, head)s: the two passes that share a launch would need more rows of blocks than the 65,535 of a
    grid if one lay behind the other.  Three batch elements carry the same G, the others none, so every entry is three
    times that of a call with one, up to the two additions (each rounds to 2^-24)."""
    B, H, T, HW, d = 16400, 2, 2, 1, 64
    N = T * HW
    q, k, v = synth.make_qkv(1, H, N, d, seed=31)
    phi = synth.make_phi(H, d, seed=32, gain=4.0)
    dq, dk, dv, dphi = parity.to_device(q, k, v, phi)
    dG = synth.make_grad_out(1, H, N, d, seed=33).to("cuda", torch.bfloat16)
    out, comps = binding.forward(dq, dk, dv, dphi, T, HW, 1, debug=True)
    one, _ = binding.phi_backward(dq, dk, dv, dphi, dG, T, HW, 1, saved=(out, comps["nS"], comps["nL"]))
    many = lambda t: t.expand(B, *t.shape[1:]).contiguous()
    G = torch.zeros_like(many(dG))
    G[[0, B // 2, B - 1]] = dG[0]
    got, _ = binding.phi_backward(many(dq), many(dk), many(dv), dphi, G, T, HW, 1,
                                  saved=(many(out), many(comps["nS"]), many(comps["nL"])))
    torch.cuda.synchronize()
    for n in synth.PHI_NAMES:
        want = 3.0 * one[n].double()
        assert (want != 0).any(), n
        assert ((got[n].double() - want).abs() <= 2.0 ** -22 * want.abs()).all(), n


@pytest.mark.parametrize("saved", [False, True])
@pytest.mark.parametrize("case,copies", [
    ((1, 1, 8, 550, 128, 2, 0), 1),     # sums of both sides, within what the weight gradients' sums take later
    ((1, 3, 28, 42, 64, 7, 1), 1),      # and the activation gradients
    ((1, 2, 40, 29, 128, 7, 2), 1),     # short pieces, empty key segments
    ((2, 3, 50, 20, 64, 1, 0), 1),      # one area of sums, larger than the activation gradients
    ((1, 2, 4, 4105, 64, 1, 0), 64),    # activation gradients of one side after the other
])
def test_every_layout_of_the_workspace(case, copies, saved):
    """What lies over what differs with the sizes: gradients against the oracle, in a workspace of exactly the stated size
    that holds NaN wherever the call has not written.  Of `copies` equal batch elements two carry a G."""
    B, H, T, HW, d, chunk, overlap = case
    q, k, v = synth.make_qkv(B, H, T * HW, d, seed=sum(case))
    phi = synth.make_phi(H, d, seed=sum(case) + 1, gain=4.0)
    G = synth.make_grad_out(B, H, T * HW, d, seed=sum(case) + 2)
    dq, dk, dv, dphi = parity.to_device(q, k, v, phi)
    dG = G.to("cuda", torch.bfloat16).contiguous()
    many = lambda t: t.expand(copies, *t.shape[1:]).contiguous() if copies > 1 else t
    fwd = None
    if saved:
        out, comps = binding.forward(dq, dk, dv, dphi, T, HW, chunk, overlap=overlap, debug=True)
        fwd = many(out), many(comps["nS"]), many(comps["nL"])
    if copies > 1:
        G = 2.0 * G
        one, dG = dG, torch.zeros_like(many(dG))
        dG[[0, copies - 1]] = one[0]
    need = binding.phi_backward_workspace_bytes(B * copies, H, T, HW, d, chunk)
    ws = torch.full((need + 4096,), 255, device="cuda", dtype=torch.uint8)
    grads, _ = binding.phi_backward(many(dq), many(dk), many(dv), dphi, dG, T, HW, chunk, overlap=overlap,
                                    workspace=ws[:need], saved=fwd)
    torch.cuda.synchronize()
    assert (ws[need:] == 255).all()
    ref, _ = ograd.phi_backward(*parity.oracle_inputs(q, k, v, phi), G.double().numpy(), T, HW, chunk, overlap,
                                hidden_round="bf16")
    check_grads(grads, ref, f"{case} x {copies}, saved {saved}")
