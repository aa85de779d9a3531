"""Workloads of the attention library as its users call it, for timing and comparing builds.

A case is one call (or, for training, one forward and its backward) through
the public binding, on seeded inputs of the kinds that
``paper_2505_11594_amd/workloads.py`` describes: normal Q, K, V, with or without
a per-channel bias on K and 1% of large rows.  ``listed()`` holds the fixed
cases, ``draw(rng)`` one more of the same ranges.  ``exact`` evaluates the
method's definition in 64-bit torch: the codes of the inputs follow their
32-bit definition, everything after them is fp64.

Fields of a case
  op      "fp4" (one sage_attn_fp4_fwd), "bf16", "int8" (forward with L),
          "int8_train" (forward, then backward; returns O, L, dQ, dK, dV)
  entry   how the fp4 and int8 forwards get their workspace: "alloc" inside the
          call, "ws" from the caller (kept between calls), "noalloc" from the library
  fmt     "mx" (MXFP4) or "nv16" (16-element blocks, E4M3 scales)
  bkv     keys per KV tile
"""
import math

import torch

from paper_2505_11594_amd import binding as bd

BASE = {"op": "fp4", "entry": "ws", "B": 1, "H": 1, "N": 128, "D": 128, "causal": False, "dtype": "bf16",
        "fmt": "mx", "bkv": 128, "wg256": False, "smooth_q": False, "out_f32": False, "k_bias": 0.0,
        "outliers": False}


def _case(**kw):
    c = dict(BASE)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: one head, one tile of queries; launches and latency are all there is
        _case(name="mx_b1h1n128d64_fp16", entry="alloc", H=1, N=128, D=64, dtype="fp16", bkv=64, out_f32=True),
        # 32 heads split over 8 GPUs: four heads of a middling sequence on one card
        _case(name="mx_b1h4n4096d128", H=4, N=4096, bkv=256, k_bias=1.0),
        # a ragged batch of prompts, causal, on the library's own scratch, default tile
        _case(name="mx_b2h24n1237d128_causal", entry="noalloc", B=2, H=24, N=1237, causal=True, k_bias=1.0),
        # prefill batch
        _case(name="mx_b4h32n4096d128", B=4, H=32, N=4096, bkv=256, k_bias=4.0),
        # long non-causal sequence with outlier rows, the benchmark's workload and launch shape
        _case(name="mx_b1h32n32768d128_wg256", H=32, N=32768, bkv=256, wg256=True, out_f32=True, outliers=True),
        # causal prefill, large batch
        _case(name="mx_b8h32n8192d128_causal", B=8, H=32, N=8192, bkv=256, causal=True, k_bias=1.0),
        # smoothing Q beside smoothing K
        _case(name="mx_b4h32n4096d128_smoothq", B=4, H=32, N=4096, bkv=256, smooth_q=True, k_bias=4.0),
        # the 16-element format at head dimension 64 (video-like: 24 heads, long, non-causal)
        _case(name="nv16_b1h24n19200d64", H=24, N=19200, D=64, fmt="nv16", k_bias=4.0),
        # the 16-bit kernel on the same kind of prefill batch
        _case(name="bf16_b4h32n4096d128", op="bf16", entry="alloc", B=4, H=32, N=4096),
        # 8-bit forward with its log-sum-exp, for evaluation during training
        _case(name="int8_b2h32n8192d128", op="int8", B=2, H=32, N=8192, k_bias=1.0, out_f32=True),
        # one 8-bit training step of an attention layer
        _case(name="int8_train_b1h32n8192d128", op="int8_train", H=32, N=8192, k_bias=1.0, out_f32=True),
        # the same, causal, ragged, D = 64, fp16, a small batch of short sequences
        _case(name="int8_train_b2h12n1000d64_causal_fp16", op="int8_train", B=2, H=12, N=1000, D=64, causal=True,
              dtype="fp16", out_f32=True),
    ]


# attention operations of one pass, over 4 B H N^2 D
_OPS = {"fp4": 1.0, "bf16": 1.0, "int8": 1.0, "int8_train": 3.5}
# rough cost of one pass against an MXFP4 forward of the same shape (keeps drawn cases below the largest listed one)
_COST = {"fp4": 1.0, "bf16": 2.5, "int8": 1.7, "int8_train": 12.0}


def draw(rng):
    while True:
        op = rng.choice(["fp4", "fp4", "fp4", "fp4", "fp4", "bf16", "int8", "int8_train"])
        D = rng.choice([128, 128, 64])
        N = int(round(math.exp(rng.uniform(math.log(100), math.log(32768)))))
        if rng.random() < 0.3:
            N = max(128, N // 128 * 128)
        BH = int(round(math.exp(rng.uniform(0.0, math.log(256)))))
        H = min(BH, rng.choice([1, 4, 8, 12, 24, 32]))
        c = _case(op=op, entry=rng.choice(["ws", "ws", "alloc"]), B=max(1, BH // H), H=H, N=N, D=D,
                  causal=rng.random() < 0.4, dtype=rng.choice(["bf16", "bf16", "fp16"]),
                  out_f32=rng.random() < 0.5, k_bias=rng.choice([0.0, 1.0, 4.0]), outliers=rng.random() < 0.2)
        if op == "fp4":
            c["fmt"] = rng.choice(["mx", "mx", "mx", "nv16"])
            c["bkv"] = rng.choice([256, 256, 128, 64]) if c["fmt"] == "mx" else rng.choice([128, 64])
            c["smooth_q"] = rng.random() < 0.25
            c["wg256"] = c["bkv"] == 256 and not c["causal"] and not c["smooth_q"] and rng.random() < 0.3
        elif op == "bf16":
            c["dtype"], c["entry"], c["k_bias"], c["outliers"] = "bf16", "alloc", 0.0, False
        elif op == "int8":
            c["bkv"] = rng.choice([128, 128, 64])
        else:
            c["out_f32"], c["outliers"] = True, False
        cost = _COST[op] * c["B"] * H * float(N) * N * D * (6.0 if c["fmt"] == "nv16" else 1.0)
        if cost < 0.25 * 32 * 32768.0 ** 2 * 128 and c["B"] * H * N * D < 2 ** 27:
            return c


def _inputs(case, seed):
    """Q, K, V (and dO for training) on the GPU, from the seed alone."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    B, H, N, D = case["B"], case["H"], case["N"], case["D"]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float16
    x = [torch.randn((B, H, N, D), generator=g, device="cuda") for _ in range(3)]
    if case["k_bias"] > 0:
        x[1] += torch.randn((B, H, 1, D), generator=g, device="cuda") * math.sqrt(case["k_bias"])
    if case["outliers"]:
        for t in x[:2]:
            big = torch.rand((B, H, N, 1), generator=g, device="cuda") < 0.01
            t *= torch.where(big, 20.0, 1.0)
    if case["op"] == "int8_train":
        x.append(torch.randn((B, H, N, D), generator=g, device="cuda"))
    return [t.to(dt).contiguous() for t in x]


def _fmt(case):
    f = bd.SAGE_FMT_MXFP4 if case["fmt"] == "mx" else bd.SAGE_FMT_NV16_E4M3
    f |= bd.bkv_flag(case["bkv"])
    if case["wg256"]:
        f |= bd.SAGE_WG256
    if case["smooth_q"]:
        f |= bd.SAGE_SMOOTH_Q
    return f


def prepare(case, seed):
    x = _inputs(case, seed)
    s = {"case": case, "x": x, "fmt": 0, "ws": None, "out": None}
    B, H, N, D, op = case["B"], case["H"], case["N"], case["D"], case["op"]
    byts = lambda n: torch.empty(n, dtype=torch.uint8, device="cuda")
    odt = torch.float32 if case["out_f32"] else x[0].dtype
    if case["entry"] != "alloc" or op == "int8_train":
        s["out"] = torch.empty((B, H, N, D), dtype=odt, device="cuda")
    if op == "fp4":
        s["fmt"] = _fmt(case)
        if case["entry"] == "ws":
            s["ws"] = byts(bd.attn_fp4_workspace_size(B, H, N, D, s["fmt"] | (4 if case["dtype"] == "bf16" else 0)))
    elif op != "bf16":
        s["fmt"] = bd.SAGE_BKV64 if case["bkv"] == 64 else 0
        if case["entry"] == "ws" or op == "int8_train":
            s["ws"] = byts(bd.attn_int8_workspace_size(B, H, N, D, s["fmt"]))
            s["lse"] = torch.empty((B, H, N), dtype=torch.float32, device="cuda")
        if op == "int8_train":
            s["bws"] = byts(bd.attn_int8_bwd_workspace_size(B, H, N, D, 0))
            s["grads"] = [torch.empty((B, H, N, D), dtype=torch.float32, device="cuda") for _ in range(3)]
    return s


def run(s):
    c, (q, k, v) = s["case"], s["x"][:3]
    if c["op"] == "fp4":
        if c["entry"] == "noalloc":
            return bd.sage_attn_fp4_fwd_noalloc(q, k, v, c["causal"], s["fmt"], c["out_f32"], out=s["out"])
        return bd.sage_attn_fp4_fwd(q, k, v, c["causal"], s["fmt"], c["out_f32"], out=s["out"], workspace=s["ws"])
    if c["op"] == "bf16":
        return bd.sage_attn_bf16_fwd(q, k, v, c["causal"], c["out_f32"], out=s["out"])
    if s["ws"] is None:
        return bd.sage_attn_int8_fwd(q, k, v, c["causal"], s["fmt"], c["out_f32"])
    o, lse = bd.sage_attn_int8_fwd(q, k, v, c["causal"], s["fmt"], c["out_f32"], out=s["out"], lse_out=s["lse"],
                                   workspace=s["ws"])
    if c["op"] == "int8":
        return o, lse
    grads = bd.sage_attn_int8_bwd(q, k, v, o, lse, s["x"][3], c["causal"], 0, workspace=s["bws"], out=s["grads"])
    return (o, lse) + tuple(grads)


def work(case):
    B, H, N, D = case["B"], case["H"], case["N"], case["D"]
    pairs = N * (N + 1) / 2 if case["causal"] else float(N) * N
    n = B * H * N * D
    byts = 6 * n + (4 if case["out_f32"] else 2) * n
    if case["op"] in ("int8", "int8_train"):
        byts += 4 * B * H * N
    if case["op"] == "int8_train":
        byts += 2 * n + 12 * n                       # dO, and dQ, dK, dV in fp32
    return {"bytes": byts, "flops": 4.0 * _OPS[case["op"]] * B * H * pairs * D}


def tolerance(case):
    """About four times the distance measured between the library and ``exact``:
    a few of P's codes round the other way near a midpoint (fp4 with fp32 output
    2e-4, int8 7e-4, gradients 1.6e-3), the bf16 kernel rounds P to bf16
    (2.3e-3 with its output), and a 16-bit output rounds once more (bf16 1.7e-3,
    fp16 2.9e-4)."""
    rel = {"fp4": 8e-4, "bf16": 9e-3, "int8": 3e-3, "int8_train": 6.5e-3}[case["op"]]
    if case["op"] != "bf16" and not case["out_f32"]:
        rel = max(rel, 7e-3 if case["dtype"] == "bf16" else 1.2e-3)
    return {"rel": rel}


# ---------------------------------------------------------------- the definition in 64 bits
def _e2m1(y):
    """Nearest E2M1 value, ties to the even code, saturating at 6."""
    a = y.abs()
    step = torch.where(a < 2, 0.5, torch.where(a < 4, 1.0, 2.0)).to(y.dtype)
    return torch.copysign((torch.round(a / step) * step).clamp(max=6.0), y)


def _e4m3(s):
    return s.clamp(max=448.0).to(torch.float32).to(torch.float8_e4m3fn).to(s.dtype)


def _phi(x, nv):
    """Dequantized microscaling FP4 of fp32 x, blocks along the last axis, in fp64."""
    shape = x.shape
    n = 16 if nv else 32
    x = torch.nn.functional.pad(x, (0, -shape[-1] % n)).unflatten(-1, (-1, n))
    am = x.abs().amax(-1, keepdim=True)
    if nv:
        s = _e4m3(am / 6.0)
        r = torch.where(s > 0, 1.0 / s, 0.0)
        q = _e2m1(x * r).double() * s.double()
    else:
        m, ex = torch.frexp(am)
        s = torch.exp2(torch.where(am > 0, ex - 3 + (m > 0.75).int(), -127).clamp(-127, 127).double())
        q = _e2m1(x.double() / s) * s
    return q.flatten(-2)[..., :shape[-1]]


def _psi(x, rows):
    """INT8 codes (fp64) and scales per block of `rows` rows of fp32 [N, D]; scales repeated per row."""
    N, D = x.shape
    p = torch.nn.functional.pad(x, (0, 0, 0, -N % rows)).view(-1, rows * D)
    s = p.abs().amax(-1, keepdim=True) / 127.0
    r = torch.where(s > 0, 1.0 / s, 0.0)
    codes = torch.round(p * r).view(-1, D)[:N]
    return codes.double(), s.expand(-1, rows).reshape(-1)[:N].double()


def _smooth(k):
    mean = k.double().mean(0).float()
    return k.float() - mean, mean.double()


def _mask(u, i0, causal):
    if causal:
        q = torch.arange(i0, i0 + u.shape[0], device=u.device)[:, None]
        u.masked_fill_(torch.arange(u.shape[1], device=u.device)[None, :] > q, -math.inf)
    return u


def _c2(D):
    return float(torch.tensor(1.0 / (math.log(2.0) * math.sqrt(D)), dtype=torch.float32))


def _tiles(u, bkv, fill):
    return torch.nn.functional.pad(u, (0, -u.shape[1] % bkv), value=fill).unflatten(1, (-1, bkv))


def _fp4_head(q, k, v, c, chunk):
    nv, bkv, N, D = c["fmt"] == "nv16", c["bkv"], c["N"], c["D"]
    ks, _ = _smooth(k)
    kq, vq = _phi(ks, nv), _phi(v.float().t().contiguous(), nv).t().contiguous()
    out = torch.empty((N, D), dtype=torch.float64, device=q.device)
    for i0 in range(0, N, chunk):                    # chunks of whole 128-row query blocks
        qf = q[i0:i0 + chunk].float()
        n = qf.shape[0]
        if c["smooth_q"]:
            means = torch.stack([b.double().mean(0).float() for b in qf.split(128)])
            rep = means.repeat_interleave(128, 0)[:n]
            S = _phi(qf - rep, nv) @ kq.t() + (means.double() @ ks.double().t()).repeat_interleave(128, 0)[:n]
        else:
            S = _phi(qf, nv) @ kq.t()
        u = _mask(S.mul_(_c2(D)), i0, c["causal"])
        M = u.amax(1, keepdim=True)
        l = torch.exp2(u - M).sum(1, keepdim=True)
        u = _tiles(u, bkv, -math.inf)                # [n, tiles, bkv]
        t = u.amax(2, keepdim=True)
        w = torch.exp2(t - M[:, :, None])            # 0 for tiles that are masked whole
        t = torch.where(torch.isinf(t), 0.0, t)
        n2 = 16 if nv else 32
        y = torch.exp2(u.sub_(t)).unflatten(2, (-1, n2))
        bm = y.amax(3, keepdim=True)
        if nv:
            s = _e4m3((2688.0 * bm / 6.0).float()).double()
            P = torch.where(s > 0, _e2m1(2688.0 * y / s), 0.0) * s / 2688.0
        else:
            s = torch.exp2(torch.ceil(torch.log2(bm) - 1e-12).clamp(min=-126.0))
            P = _e2m1(6.0 * y / s) * s / 6.0
        P = (P.flatten(2) * w).flatten(1)[:, :N]
        out[i0:i0 + n] = (P @ vq) / l
    return out


def _bf16_head(q, k, v, c, chunk):
    out = torch.empty((c["N"], c["D"]), dtype=torch.float64, device=q.device)
    kd, vd = k.double(), v.double()
    for i0 in range(0, c["N"], chunk):
        u = _mask((q[i0:i0 + chunk].double() @ kd.t()) / math.sqrt(c["D"]), i0, c["causal"])
        out[i0:i0 + chunk] = torch.softmax(u, 1) @ vd
    return out


def _int8_head(q, k, v, c, chunk):
    N, D, bkv = c["N"], c["D"], c["bkv"]
    ks, _ = _smooth(k)
    (qi, sq), (ki, sk), (vi, sv) = _psi(q.float(), 128), _psi(ks, bkv), _psi(v.float(), bkv)
    out = torch.empty((N, D), dtype=torch.float64, device=q.device)
    lse = torch.empty(N, dtype=torch.float64, device=q.device)
    for i0 in range(0, N, chunk):
        u = (qi[i0:i0 + chunk] @ ki.t()) * (sq[i0:i0 + chunk, None] * sk[None, :] * _c2(D))
        u = _mask(u, i0, c["causal"])
        M = u.amax(1, keepdim=True)
        l = torch.exp2(u - M).sum(1, keepdim=True)
        lse[i0:i0 + chunk] = ((M + torch.log2(l)) * math.log(2.0))[:, 0]
        u = _tiles(u, bkv, -math.inf)
        t = u.amax(2, keepdim=True)
        w = torch.exp2(t - M[:, :, None]) / 127.0
        P = torch.round(127.0 * torch.exp2(u - torch.where(torch.isinf(t), 0.0, t))) * w
        out[i0:i0 + chunk] = ((P.flatten(1)[:, :N] * sv[None, :]) @ vi) / l
    return out, lse


def _psi_blocks(x):
    """Dequantized INT8 of x [128, N] (fp64), one scale per 128 columns."""
    N = x.shape[1]
    t = _tiles(x, 128, 0.0)
    s = t.abs().amax((0, 2), keepdim=True) / 127.0
    return (torch.round(torch.where(s > 0, t / s, 0.0)) * s).flatten(1)[:, :N]


def _bwd_head(q, k, v, g, o, lse, c):
    N, D = c["N"], c["D"]
    ks, km = _smooth(k)
    deq = lambda p: p[0] * p[1][:, None]
    Q, K, G = _psi(q.float(), 128), _psi(ks, 128), deq(_psi(g.float(), 128))
    Qd, Kd, vd, gd = deq(Q), deq(K), v.double(), g.double()
    drow = (gd * o).sum(1, keepdim=True)
    r = 1.0 / math.sqrt(D)
    dq, dk, dv = (torch.zeros((N, D), dtype=torch.float64, device=q.device) for _ in range(3))
    for i0 in range(0, N, 128):
        sl = slice(i0, min(N, i0 + 128))
        u = _mask((Q[0][sl] @ K[0].t()) * (Q[1][sl, None] * K[1][None, :] * _c2(D)), i0, c["causal"])
        P = torch.exp2(u - (lse[sl, None] / math.log(2.0)))
        dS = P * (gd[sl] @ vd.t() - drow[sl])
        dv += _psi_blocks(P).t() @ G[sl]
        dSq = _psi_blocks(dS)
        dq[sl] = (dSq @ Kd + dS.sum(1, keepdim=True) * km[None, :]) * r
        dk += (dSq.t() @ Qd[sl]) * r
    return dq, dk, dv


def exact(case, seed):
    c = case
    B, H, N, D = c["B"], c["H"], c["N"], c["D"]
    pairs = float(B) * H * N * N
    if pairs > 4e10 or (c["op"] == "int8_train" and pairs > 4e9):
        return None                                  # over about 20 seconds in fp64
    x = [t.view(B * H, N, D) for t in _inputs(c, seed)]
    chunk = max(128, min(4096, (1 << 26) // N) // 128 * 128)
    outs = None
    for b in range(B * H):
        q, k, v = (t[b] for t in x[:3])
        if c["op"] == "fp4":
            r = (_fp4_head(q, k, v, c, chunk),)
        elif c["op"] == "bf16":
            r = (_bf16_head(q, k, v, c, chunk),)
        else:
            r = _int8_head(q, k, v, c, chunk)
            if c["op"] == "int8_train":
                r = r + _bwd_head(q, k, v, x[3][b], r[0], r[1], c)
        if outs is None:
            outs = [torch.empty((B * H,) + t.shape, dtype=torch.float64, device=q.device) for t in r]
        for o, t in zip(outs, r):
            o[b] = t
    outs = [o.view((B, H) + o.shape[1:]) for o in outs]
    return outs[0] if len(outs) == 1 else tuple(outs)
