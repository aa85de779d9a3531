"""GPU parity of the 8-bit attention backward (Algorithm 3) against the
oracle, through the C ABI.  Both sides take the same O and L (the oracle's
forward); dQ, dK, dV must match within the oracle's per-element tolerance
(codes of P^ and dS^ whose pre-rounding value lies near a rounding midpoint
may take either neighbour on the GPU) plus 2e-5 of the tensor's largest
magnitude for fp32 rounding and summation order."""
import numpy as np
import pytest

import oracle
from paper_2505_11594_amd import binding as bd
from paper_2505_11594_amd import workloads as wl

from _gpu import to_dev, torch_dev, say

pytestmark = pytest.mark.gpu


def make_case(B, H, N, D, in_dtype, seed, causal, k_bias_var=1.0, outlier_frac=0.0):
    q, k, v = wl.make_inputs(B, H, N, D, in_dtype, seed=seed, k_bias_var=k_bias_var, outlier_frac=outlier_frac)
    rng = np.random.default_rng(seed + 3)
    do = wl.to_bits(rng.standard_normal((B, H, N, D)).astype(np.float32), in_dtype)
    o, lse, _, _ = oracle.attn_int8(q, k, v, in_dtype, causal, 128)
    return q, k, v, do, o.reshape(B, H, N, D), lse.reshape(B, H, N)


def gpu_bwd(q, k, v, do, o, lse, in_dtype, causal, flags=0):
    torch = torch_dev()
    od = torch.from_numpy(o).to("cuda")
    ld = torch.from_numpy(lse).to("cuda")
    r = bd.sage_attn_int8_bwd(to_dev(q, in_dtype), to_dev(k, in_dtype), to_dev(v, in_dtype), od, ld,
                              to_dev(do, in_dtype), causal=causal, flags=flags)
    torch.cuda.synchronize()
    return [x.cpu().numpy() for x in r]


def check_grads(got, ref, tol, label):
    """Per element: |got - ref| <= the oracle's tolerance + 2e-5 of max |ref|.
    Also reports the tolerance's tightness: the largest error over the bar,
    and the error over the tolerance where the error exceeds 2e-5 of max |ref|
    (a code that took its other accepted neighbour)."""
    for name, g, r, t in zip(("dQ", "dK", "dV"), got, ref, tol):
        err = np.abs(g - r)
        floor = 2e-5 * np.abs(r).max()
        lim = t + floor
        flip = err > floor
        say("%s %s: max err %.3g (max |ref| %.3g), elements with a tolerance %d, max err/bar %.3f, "
            "elements beyond 2e-5 of max|ref| %d (max err/tolerance there %.3f)" %
            (label, name, float(err.max()), float(np.abs(r).max()), int((t > 0).sum()), float((err / lim).max()),
             int(flip.sum()), float((err[flip] / np.maximum(t[flip], 1e-30)).max()) if flip.any() else 0.0))
        assert np.all(err <= lim), "%s %s: %d elements over, worst %.3g" % (label, name, int((err > lim).sum()),
                                                                           float(err.max()))


@pytest.mark.parametrize("N", [1, 100, 257, 640])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("causal", [False, True])
def test_bwd_edge_shapes(N, D, causal):
    in_dtype = 1 if (N + D) % 2 else 0
    say("bwd edge N=%d D=%d causal=%d dtype=%d" % (N, D, causal, in_dtype))
    q, k, v, do, o, lse = make_case(1, 2, N, D, in_dtype, seed=1100 + N, causal=causal, k_bias_var=4.0,
                                    outlier_frac=0.02)
    got = gpu_bwd(q, k, v, do, o, lse, in_dtype, causal)
    *ref, tol = oracle.attn_int8_bwd(q, k, v, do, o, lse, in_dtype, causal, 128)
    check_grads(got, ref, tol, "edge")


def test_bwd_no_smooth_k():
    q, k, v, do, o, lse = make_case(1, 2, 300, 128, 1, seed=1110, causal=False, k_bias_var=4.0)
    got = gpu_bwd(q, k, v, do, o, lse, 1, False, flags=bd.SAGE_NO_SMOOTH_K)
    *ref, tol = oracle.attn_int8_bwd(q, k, v, do, o, lse, 1, False, 128, flags=oracle.NO_SMOOTH_K)
    check_grads(got, ref, tol, "no smooth-K")


@pytest.mark.parametrize("causal", [False, True])
def test_bwd_longer_sequence(causal):
    q, k, v, do, o, lse = make_case(1, 2, 2048, 128, 1, seed=1120 + causal, causal=causal)
    got = gpu_bwd(q, k, v, do, o, lse, 1, causal)
    *ref, tol = oracle.attn_int8_bwd(q, k, v, do, o, lse, 1, causal, 128)
    check_grads(got, ref, tol, "N=2048")


def test_bwd_deterministic_and_workspace_variant():
    torch = torch_dev()
    B, H, N, D = 1, 2, 1024, 128
    q, k, v, do, o, lse = make_case(B, H, N, D, 1, seed=1130, causal=False)
    a = gpu_bwd(q, k, v, do, o, lse, 1, False)
    b = gpu_bwd(q, k, v, do, o, lse, 1, False)
    ws = torch.empty(bd.attn_int8_bwd_workspace_size(B, H, N, D, bd.SAGE_IN_BF16), dtype=torch.uint8, device="cuda")
    c = bd.sage_attn_int8_bwd(to_dev(q, 1), to_dev(k, 1), to_dev(v, 1), torch.from_numpy(o).cuda(),
                              torch.from_numpy(lse).cuda(), to_dev(do, 1), workspace=ws)
    torch.cuda.synchronize()
    for x, y, z in zip(a, b, c):
        assert np.array_equal(x, y) and np.array_equal(x, z.cpu().numpy())


def test_bwd_zero_do_and_doubling():
    """Closed forms on the GPU: dO = 0 gives zero gradients; doubling dO
    doubles every gradient bit for bit."""
    q, k, v, do, o, lse = make_case(1, 1, 300, 128, 1, seed=1140, causal=True)
    z = gpu_bwd(q, k, v, np.zeros_like(do), o, lse, 1, True)
    assert not any(x.any() for x in z)
    a = gpu_bwd(q, k, v, do, o, lse, 1, True)
    d2 = wl.to_bits(wl.from_bits(do, 1) * np.float32(2.0), 1)
    b = gpu_bwd(q, k, v, d2, o, lse, 1, True)
    for x, y in zip(a, b):
        assert np.array_equal(2 * x, y)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("causal", [False, True])
def test_bwd_workspace_selects_stored_or_recomputed_ds(D, causal):
    """The minimum workspace makes the dQ kernel recompute S, dP and dS; each
    head's worth of workspace beyond it lets the dK kernel store dS^ for the
    dQ kernel, heads in groups of that many.  dK and dV are the same bits on
    every path, dQ the same bits on every stored path, and all of them match
    the oracle."""
    torch = torch_dev()
    B, H, N = 1, 3, 300
    say("bwd workspace paths D=%d causal=%d" % (D, causal))
    q, k, v, do, o, lse = make_case(B, H, N, D, 1, seed=1150 + D + causal, causal=causal, k_bias_var=4.0)
    lo = bd.attn_int8_bwd_min_workspace_size(B, H, N, D, bd.SAGE_IN_BF16)
    hi = bd.attn_int8_bwd_workspace_size(B, H, N, D, bd.SAGE_IN_BF16)
    assert 0 < lo < hi and (hi - lo) % (B * H) == 0
    per_head = (hi - lo) // (B * H)
    *ref, tol = oracle.attn_int8_bwd(q, k, v, do, o, lse, 1, causal, 128)
    args = [to_dev(q, 1), to_dev(k, 1), to_dev(v, 1), torch.from_numpy(o).cuda(), torch.from_numpy(lse).cuda(),
            to_dev(do, 1)]
    runs = {}
    for heads in (0, 1, 2, 3):
        ws = torch.empty(lo + heads * per_head, dtype=torch.uint8, device="cuda")
        r = bd.sage_attn_int8_bwd(*args, causal=causal, workspace=ws)
        torch.cuda.synchronize()
        runs[heads] = [x.cpu().numpy() for x in r]
        check_grads(runs[heads], ref, tol, "heads stored %d" % heads)
    for heads in (1, 2, 3):
        assert np.array_equal(runs[heads][1], runs[0][1]) and np.array_equal(runs[heads][2], runs[0][2])
        assert np.array_equal(runs[heads][0], runs[1][0])
    with pytest.raises(RuntimeError):
        bd.sage_attn_int8_bwd(*args, causal=causal, workspace=torch.empty(lo - 256, dtype=torch.uint8, device="cuda"))


def test_bwd_long_sequence_head_grouped_stored_ds():
    """N = 8192 (the long-sequence regime of the bench workload) on two heads,
    with a workspace between the minimum and the recommended size: the dK
    kernel stores dS^ for one head at a time and the dQ kernel sums from the
    stored codes, heads in groups of one (Algorithm 3).  Every element of dQ,
    dK and dV against the oracle; the recommended workspace (both heads at
    once) gives the same bits."""
    torch = torch_dev()
    B, H, N, D = 1, 2, 8192, 128
    say("bwd N=%d H=%d D=%d, head-grouped stored dS" % (N, H, D))
    q, k, v, do, o, lse = make_case(B, H, N, D, 1, seed=1160, causal=False, k_bias_var=4.0, outlier_frac=0.01)
    lo = bd.attn_int8_bwd_min_workspace_size(B, H, N, D, bd.SAGE_IN_BF16)
    hi = bd.attn_int8_bwd_workspace_size(B, H, N, D, bd.SAGE_IN_BF16)
    per_head = (hi - lo) // (B * H)
    args = [to_dev(q, 1), to_dev(k, 1), to_dev(v, 1), torch.from_numpy(o).cuda(), torch.from_numpy(lse).cuda(),
            to_dev(do, 1)]
    ws = torch.empty(lo + per_head, dtype=torch.uint8, device="cuda")
    g1 = [x.cpu().numpy() for x in bd.sage_attn_int8_bwd(*args, causal=False, workspace=ws)]
    del ws
    ws = torch.empty(hi, dtype=torch.uint8, device="cuda")
    g2 = [x.cpu().numpy() for x in bd.sage_attn_int8_bwd(*args, causal=False, workspace=ws)]
    torch.cuda.synchronize()
    for x, y in zip(g1, g2):
        assert np.array_equal(x, y)
    *ref, tol = oracle.attn_int8_bwd(q, k, v, do, o, lse, 1, False, 128)
    check_grads(g1, ref, tol, "N=8192 head-grouped")


@pytest.mark.parametrize("N", [1, 129, 300])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("stored", [False, True])
def test_bwd_many_heads_same_bits(N, D, causal, stored):
    """The dK kernel runs eight waves per key block where its grid leaves CUs
    idle and four otherwise, and large calls quantize in separate launches: two
    heads alone and 400 copies of them give the same bits, with the stored dS^
    state and without."""
    torch = torch_dev()
    say("int8 bwd many heads N=%d D=%d causal=%d stored=%d" % (N, D, causal, stored))
    g = torch.Generator(device="cuda").manual_seed(50 + N)
    dt = torch.bfloat16 if N % 2 else torch.float16
    q, k, v, dout = (torch.randn((1, 2, N, D), generator=g, device="cuda").to(dt) for _ in range(4))

    def grads(q, k, v, dout):
        o, lse = bd.sage_attn_int8_fwd(q, k, v, causal=causal)
        B, H = q.shape[:2]
        size = bd.attn_int8_bwd_workspace_size if stored else bd.attn_int8_bwd_min_workspace_size
        ws = torch.empty(size(B, H, N, D), dtype=torch.uint8, device="cuda")
        return (o, lse) + tuple(bd.sage_attn_int8_bwd(q, k, v, o, lse, dout, causal=causal, workspace=ws))

    few = grads(q, k, v, dout)
    many = grads(*(x.repeat(400, 1, 1, 1) for x in (q, k, v, dout)))
    torch.cuda.synchronize()
    for a, b in zip(few, many):
        assert torch.equal(b, a.expand_as(b))


@pytest.mark.parametrize("N", [1, 129, 257])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("stored", [False, True])
def test_bwd_reads_nothing_behind_its_tensors(N, D, causal, stored):
    """Inputs that are the front of larger tensors: the ragged last block's rows
    past N of the last head lie behind them.  NaN there and in the workspace
    beforehand gives the bits of zeros there."""
    torch = torch_dev()
    say("int8 bwd NaN behind its tensors N=%d D=%d causal=%d stored=%d" % (N, D, causal, stored))
    g = torch.Generator(device="cuda").manual_seed(80 + N)
    x = [torch.randn((1, 2, N, D), generator=g, device="cuda").to(torch.bfloat16) for _ in range(4)]
    x += list(bd.sage_attn_int8_fwd(*x[:3], causal=causal))
    size = bd.attn_int8_bwd_workspace_size if stored else bd.attn_int8_bwd_min_workspace_size

    def grads(behind, ws_byte):
        def front(t):
            big = torch.full((t.numel() + 128 * D,), behind, dtype=t.dtype, device="cuda")
            big[:t.numel()] = t.flatten()
            return big[:t.numel()].view(t.shape)
        q, k, v, dout, o, lse = (front(t) for t in x)
        ws = torch.full((size(1, 2, N, D, bd.SAGE_IN_BF16),), ws_byte, dtype=torch.uint8, device="cuda")
        return bd.sage_attn_int8_bwd(q, k, v, o, lse, dout, causal=causal, workspace=ws)

    ref, got = grads(0.0, 0), grads(float("nan"), 255)
    torch.cuda.synchronize()
    for a, b in zip(ref, got):
        assert torch.isfinite(a).all() and torch.equal(a, b)
