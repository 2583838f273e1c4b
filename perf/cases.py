"""The calls whose speed matters to a user of the library: one case per use, each through a public entry point
(paper_2602_10016_amd.binding for single calls, paper_2602_10016_amd.autograd for training steps).

    listed()            the named cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) inputs on the GPU, and the buffers a program keeps between calls
    run(state)          one pass; returns its outputs
    work(case)          bytes and flops the pass cannot do without
    tolerance(case)     how far another correct implementation may be
    exact(case, seed)   the outputs in 64 bits, by plain torch

History lengths are the quantiles of the case's length distribution in an order drawn from the seed, so that every
seed has the same number of tokens (and the same work) and a different packing.
"""
import math
import statistics

import numpy as np
import torch

from paper_2602_10016_amd import autograd as ka
from paper_2602_10016_amd import binding as kb

ACTS = {"softmax": kb.ACT_SOFTMAX, "gelu": kb.ACT_GELU, "gelu_tanh": kb.ACT_GELU_TANH, "silu": kb.ACT_SILU,
        "gelu_poly": kb.ACT_GELU_POLY}


def _gdpa(name, op, B, H, d, n, dist, lo, hi, act, dtype="bf16"):
    """op: fwd, bwd, train (n dense queries per example over a jagged history), seed (n batch-shared queries),
    pffn (the jagged history asks, n context keys per example answer)."""
    return dict(name=name, op=op, dtype=dtype, B=B, H=H, d=d, n=n, dist=dist, lo=lo, hi=hi, act=act)


def _swa(name, op, B, H, d, dist, lo, hi, left, right):
    return dict(name=name, op=op, dtype="bf16", B=B, H=H, d=d, dist=dist, lo=lo, hi=hi, left=left, right=right)


def _sumkron(name, B, S, T, D, k):
    return dict(name=name, op="sumkron", dtype="bf16", B=B, S=S, T=T, D=D, k=k)


def listed():
    return [
        # The smallest call: a two-example fp32 evaluation, dense histories.  Launches and host time count.
        _gdpa("fwd_fp32_tiny", "fwd", 2, 2, 32, 8, "uniform", 64, 64, "gelu", "fp32"),
        # One serving request: a few users, their context tokens over their histories.
        _gdpa("fwd_request", "fwd", 12, 4, 64, 32, "uniform", 64, 1024, "gelu"),
        # A ranking batch: forward at serving time ...
        _gdpa("fwd_batch", "fwd", 256, 4, 64, 32, "uniform", 64, 1024, "gelu"),
        # ... and its backward in training.
        _gdpa("bwd_batch", "bwd", 256, 4, 64, 32, "uniform", 64, 1024, "gelu"),
        # The large jagged batch of the benchmark (log-normal histories): forward ...
        _gdpa("fwd_large", "fwd", 1024, 8, 128, 64, "lognormal", 32, 4096, "gelu"),
        # ... and, for a quarter of the batch (one micro-batch), backward.
        _gdpa("bwd_large", "bwd", 256, 8, 128, 64, "lognormal", 32, 4096, "gelu"),
        # Multi-head attention pooling in a 256-wide layer of 8 heads: a training step under softmax.
        _gdpa("train_heads_of_32", "train", 512, 8, 32, 32, "lognormal", 32, 4096, "softmax"),
        # Sliding-window self-attention over the history (previous 256 events): serving ...
        _swa("swa_fwd", "swa_fwd", 128, 4, 128, "uniform", 256, 2048, 255, 0),
        # ... and a training step of the same layer.
        _swa("swa_train", "swa_train", 128, 4, 128, "uniform", 256, 2048, 255, 0),
        # The feed-forward direction: every event of the history asks a few context tokens; a training step.
        _gdpa("pffn_train", "pffn", 128, 4, 128, 32, "uniform", 256, 2048, "gelu"),
        # Hierarchical seed pooling, first stage: 256 shared seeds over every history; a training step.
        _gdpa("seed_train", "seed", 256, 8, 128, 256, "lognormal", 32, 4096, "softmax"),
        # Hierarchical seed pooling, last stage: the 256 pooled seeds compressed to 32 tokens; a training step.
        _sumkron("sumkron_train", 1024, 256, 32, 384, 8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["fp32", "fwd", "fwd", "bwd", "bwd", "train", "swa_fwd", "swa_train", "pffn", "seed", "sumkron"])
    if op == "sumkron":
        # widths in use are multiples of 128; any batch size (an even one with 16 output tokens: whole 32-row blocks)
        T, B = rng.choice([16, 32, 32]), _log_int(rng, 8, 1024)
        return {k: v for k, v in _sumkron("", B + (B % 2 if T == 16 else 0), rng.choice([128, 256]), T,
                                          rng.choice([128, 256, 384]), rng.randint(2, 8)).items() if k != "name"}
    d = rng.choice([32, 64, 128])
    H = rng.choice([2, 4, 8])
    dist, lo, hi = rng.choice([("uniform", 64, 1024), ("uniform", 256, 2048), ("lognormal", 32, 4096)])
    if op.startswith("swa"):
        left = _log_int(rng, 32, 512)
        c = _swa("", op, _log_int(rng, 4, 256), H, d, dist, lo, hi, left, rng.choice([0, 0, left]))
    elif op == "fp32":
        c = _gdpa("", "fwd", _log_int(rng, 1, 128), H, d, _log_int(rng, 4, 64), "uniform", 64, 1024, rng.choice(sorted(ACTS)), "fp32")
    elif op == "pffn":
        c = _gdpa("", "pffn", _log_int(rng, 4, 512), H, d, _log_int(rng, 8, 64), dist, lo, hi, rng.choice(sorted(ACTS)))
    elif op == "seed":
        c = _gdpa("", "seed", _log_int(rng, 4, 256), H, d, _log_int(rng, 96, 320), dist, lo, hi, "softmax")
    else:
        c = _gdpa("", op, _log_int(rng, 2, 1024), H, d, _log_int(rng, 8, 64), dist, lo, hi, rng.choice(sorted(ACTS)))
    # no larger than the listed ones
    flops = {"fp32": 4e9}.get(op, 2.5e11)
    while c["B"] > 1 and (work(c)["flops"] > flops or work(c)["bytes"] > 1.2e9):
        c["B"] = max(1, c["B"] // 2)
    return {k: v for k, v in c.items() if k != "name"}


# ---- sizes ----

def _lengths(case):
    B, lo, hi = case["B"], case["lo"], case["hi"]
    u = [(i + 0.5) / B for i in range(B)]
    if case["dist"] == "uniform":
        return [lo + min(hi - lo, int(x * (hi - lo + 1))) for x in u]
    nd = statistics.NormalDist(math.log(800.0), 1.0)  # median 800, sigma 1
    return [min(hi, max(lo, round(math.exp(nd.inv_cdf(x))))) for x in u]


def _packed(case, seed):
    lens = np.random.default_rng(seed).permutation(np.asarray(_lengths(case), dtype=np.int64))
    off = np.zeros(len(lens) + 1, dtype=np.int64)
    np.cumsum(lens, out=off[1:])
    return lens, off


def _scale(case):
    if case.get("act", "softmax") == "softmax":
        return 1.0 / math.sqrt(case["d"])
    return 1.0 / case["hi"]


def work(case):
    if case["op"] == "sumkron":
        B, S, T, D, k = (case[x] for x in ("B", "S", "T", "D", "k"))
        weights = k * S * T + k * D * D
        # x, z, w read, y written; x, z, w, dy read, dx, dz, dw written
        return {"bytes": 2 * (3 * B * S * D + 2 * B * T * D + 4 * weights), "flops": 2 * B * k * T * D * (4 * S + 3 * D)}
    H, d = case["H"], case["d"]
    lens = _lengths(case)
    T = sum(lens)
    if case["op"].startswith("swa"):
        left, right = case["left"], case["right"]
        # pairs inside the window: each query's own position and the reach to both sides, cut at the edges
        side = lambda L, w: L * w - w * (w + 1) // 2 if w < L else L * (L - 1) // 2
        pairs = sum(L + side(L, left) + side(L, right) for L in lens)
        if case["op"] == "swa_fwd":
            return {"bytes": 2 * 4 * T * H * d, "flops": 4 * d * H * pairs}
        # the forward's, then q, k, v, o, d_o read and dq, dk, dv written
        return {"bytes": 2 * 12 * T * H * d, "flops": 14 * d * H * pairs}
    elt = 4 if case["dtype"] == "fp32" else 2
    n, B = case["n"], case["B"]
    q, kv = (T, B * n) if case["op"] == "pffn" else (B * n, T)
    fwd = (2 * q + 2 * kv) * H * d * elt
    bwd = ((4 if case["act"] == "softmax" else 3) * q + 4 * kv) * H * d * elt
    f = d * H * T * n
    if case["op"] == "fwd":
        return {"bytes": fwd, "flops": 4 * f}
    if case["op"] == "bwd":
        return {"bytes": bwd, "flops": 10 * f}
    if case["op"] == "seed":  # the queries are one block: read once, not per example
        fwd = (q + n + 2 * kv) * H * d * elt
        bwd = (2 * q + 2 * n + 4 * kv) * H * d * elt
    return {"bytes": fwd + bwd, "flops": 14 * f}


# ---- inputs ----

def _normal(gen, shape, sigma, dtype):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, sigma, generator=gen)


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if case["op"] == "sumkron":
        B, S, T, D, k = (case[x] for x in ("B", "S", "T", "D", "k"))
        bf = torch.bfloat16
        return dict(x=_normal(gen, (B, S, D), 1.0, bf), z=_normal(gen, (k, S, T), S ** -0.5, bf),
                    w=_normal(gen, (k, D, D), D ** -0.5, bf), dy=_normal(gen, (B, T, D), 1.0, bf))
    dtype = torch.float32 if case["dtype"] == "fp32" else torch.bfloat16
    sigma = 1.0 if case["dtype"] == "fp32" else 0.5
    B, H, d, n = case["B"], case["H"], case["d"], case.get("n")
    lens, off = _packed(case, seed)
    T = int(off[-1])
    q_rows, kv_rows, o_rows = {"pffn": (T, B * n if n else 0, T), "seed": (n, T, B * n if n else 0), "swa_fwd": (T, T, T),
                               "swa_train": (T, T, T)}.get(case["op"], (B * n if n else 0, T, B * n if n else 0))
    s = dict(q=_normal(gen, (q_rows, H, d), sigma, dtype), k=_normal(gen, (kv_rows, H, d), sigma, dtype),
             v=_normal(gen, (kv_rows, H, d), sigma, dtype), lens=lens, off=off)
    if case["op"] not in ("fwd", "swa_fwd"):
        s["d_o"] = _normal(gen, (o_rows, H, d), 1.0, dtype)
    return s


def _device_offsets(off):
    return torch.from_numpy(np.ascontiguousarray(off, dtype=np.int32)).cuda()


def prepare(case, seed):
    s = _inputs(case, seed)
    s["op"] = op = case["op"]
    if op == "sumkron":
        for t in (s["x"], s["z"], s["w"]):
            t.requires_grad_(True)
        return s
    s["scale"], s["max"] = _scale(case), int(s["lens"].max())
    s["offsets"] = _device_offsets(s["off"])
    B, H, d, n, longest = case["B"], case["H"], case["d"], case.get("n"), s["max"]
    T = int(s["off"][-1])
    buffer = lambda nbytes: torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    if op.startswith("swa"):
        s["window"] = (case["left"], case["right"])
    else:
        s["act"], s["n"] = ACTS[case["act"]], n
        s["softmax"] = case["act"] == "softmax"
    if op in ("fwd", "swa_fwd"):  # a serving program keeps its output and workspace
        s["out"] = torch.empty_like(s["q"])
        s["lse"] = None
        s["ws"] = buffer(kb.workspace_bytes(kb.OP_SWA_FWD, B, H, d, longest, longest, T, T) if op == "swa_fwd" else
                         kb.workspace_bytes(kb.OP_GDPA_FWD, B, H, d, n, longest, B * n, T))
    elif op == "bwd":  # gradients into buffers that are kept, the forward's results in hand
        s["out"] = tuple(torch.empty_like(s[x]) for x in "qkv")
        s["ws"] = buffer(kb.workspace_bytes(kb.OP_GDPA_BWD, B, H, d, n, longest, B * n, T))
        s["o"], s["lse"] = (kb.gdpa_fwd(s["q"], s["k"], s["v"], s["offsets"], s["scale"], s["act"], max_q=n, max_kv=longest)
                            if s["softmax"] else (None, None))
    elif op == "seed":
        s["ws"] = buffer(kb.workspace_bytes(kb.OP_SEED_FWD, B, H, d, n, longest, B * n, T))
        s["ws_bwd"] = buffer(kb.workspace_bytes(kb.OP_SEED_BWD, B, H, d, n, longest, B * n, T))
    else:
        if op == "pffn":
            s["kv_offsets"] = _device_offsets(np.arange(B + 1, dtype=np.int64) * n)
        for t in (s["q"], s["k"], s["v"]):
            t.requires_grad_(True)
    return s


# ---- one pass ----

def run(s):
    op = s["op"]
    if op == "sumkron":
        y = ka.sumkron_linear(s["x"], s["z"], s["w"])
        return (y.detach(), *torch.autograd.grad(y, (s["x"], s["z"], s["w"]), s["dy"]))
    q, k, v, off, scale, longest = s["q"], s["k"], s["v"], s["offsets"], s["scale"], s["max"]
    if op == "fwd":
        return kb.gdpa_fwd(q, k, v, off, scale, s["act"], max_q=s["n"], max_kv=longest, out=s["out"], want_lse=False,
                           workspace=s["ws"])[0]
    if op == "bwd":
        return kb.gdpa_bwd(q, k, v, s["d_o"], off, scale, s["act"], o=s["o"], lse=s["lse"], max_q=s["n"], max_kv=longest,
                           out=s["out"], workspace=s["ws"])
    if op == "swa_fwd":
        return kb.swa_fwd(q, k, v, off, *s["window"], scale, max_len=longest, out=s["out"], want_lse=False, workspace=s["ws"])[0]
    if op == "seed":
        o, lse = kb.seed_attn_fwd(q, k, v, off, scale, s["act"], max_kv=longest, workspace=s["ws"])
        return (o, lse, *kb.seed_attn_bwd(q, k, v, s["d_o"], off, scale, s["act"], o=o, lse=lse, max_kv=longest,
                                          workspace=s["ws_bwd"]))
    if op == "train":
        o = ka.gdpa(q, k, v, off, scale, s["act"], max_q=s["n"], max_kv=longest)
    elif op == "pffn":
        o = ka.gdpa(q, k, v, s["kv_offsets"], scale, s["act"], q_offsets=off, max_q=longest, max_kv=s["n"])
    else:
        o = ka.sliding_window_attention(q, k, v, off, *s["window"], scale, max_len=longest)
    return (o.detach(), *torch.autograd.grad(o, (q, k, v), s["d_o"]))


# ---- what is right ----

def tolerance(case):
    if case["dtype"] == "fp32":  # 2e-7 off 64 bits over 64 keys; up to sixteen times as many terms, summed in another order
        return {"rel": 2e-6}
    return {"rel": 1.2e-2}       # 2.1e-3 to 2.9e-3 off 64 bits: the weights and the results rounded to bf16


def _act64(name, x):
    """The score function and its slope."""
    if name == "gelu_poly":
        C = 3.875
        a = (3.9862210505e-01, -6.5595134356e-02, 9.2376422360e-03, -9.1053389233e-04, 5.8010079080e-05,
             -2.1110704002e-06, 3.2949778488e-08)
        t = x.clamp(-C, C)
        u = t * t
        p, dp = torch.zeros_like(u), torch.zeros_like(u)
        for i in range(6, -1, -1):
            dp = dp * u + p
            p = p * u + a[i]
        inside = ((x > -C) & (x < C)).to(x.dtype)
        cdf = 0.5 + t * p
        return x * cdf, cdf + x * (p + 2 * u * dp) * inside
    if name == "gelu":
        cdf = 0.5 * (1 + torch.erf(x / math.sqrt(2.0)))
        return x * cdf, cdf + x * torch.exp(-0.5 * x * x) / math.sqrt(2 * math.pi)
    if name == "gelu_tanh":
        c = math.sqrt(2 / math.pi)
        t = torch.tanh(c * (x + 0.044715 * x ** 3))
        return 0.5 * x * (1 + t), 0.5 * (1 + t) + 0.5 * x * (1 - t * t) * c * (1 + 3 * 0.044715 * x * x)
    sg = torch.sigmoid(x)  # silu
    return x * sg, sg + x * sg * (1 - sg)


def _sumkron64(case, seed):
    s = _inputs(case, seed)
    x, z, w, dy = (s[n].double() for n in ("x", "z", "w", "dy"))
    B, S, T, D, k = (case[n] for n in ("B", "S", "T", "D", "k"))
    y, dx, dz, dw = torch.zeros_like(dy), torch.zeros_like(x), torch.zeros_like(z), torch.zeros_like(w)
    for i in range(k):
        zt, wt = z[i].t().contiguous(), w[i].t().contiguous()
        u = torch.matmul(zt, x)                                   # [B, T, D]
        g = torch.matmul(dy.reshape(B * T, D), wt).reshape(B, T, D)
        y += torch.matmul(u.reshape(B * T, D), w[i]).reshape(B, T, D)
        dx += torch.matmul(z[i], g)
        dw[i] = torch.matmul(u.reshape(B * T, D).t().contiguous(), dy.reshape(B * T, D))
        xs = x.permute(1, 0, 2).reshape(S, B * D)
        gs = g.permute(0, 2, 1).reshape(B * D, T)
        dz[i] = torch.matmul(xs, gs)
    return y, dx, dz, dw


def exact(case, seed):
    if case["op"] == "sumkron":
        return _sumkron64(case, seed)
    s = _inputs(case, seed)
    op, H, B, n, scale = case["op"], case["H"], case["B"], case.get("n"), _scale(case)
    act = case.get("act", "softmax")
    q, k, v, off = s["q"], s["k"], s["v"], s["off"]
    grads = op not in ("fwd", "swa_fwd")
    heads = lambda t: t.double().permute(1, 0, 2).contiguous()    # [H, rows, d]
    rows = lambda t: t.permute(1, 0, 2)
    tr = lambda t: t.transpose(1, 2).contiguous()
    q_rows = B * n if op == "seed" else q.shape[0]
    o = torch.zeros((q_rows, *q.shape[1:]), dtype=torch.float64, device="cuda")
    lse = torch.zeros((H, q_rows), dtype=torch.float64, device="cuda")
    dq = torch.zeros(q.shape, dtype=torch.float64, device="cuda")
    dk = torch.zeros(k.shape, dtype=torch.float64, device="cuda") if grads else None
    dv = torch.zeros(k.shape, dtype=torch.float64, device="cuda") if grads else None
    for b in range(B):
        hist = slice(int(off[b]), int(off[b + 1]))
        mine = slice(b * n, (b + 1) * n) if n else None
        qs, ks = {"pffn": (hist, mine)}.get(op, (mine, hist) if n else (hist, hist))
        qq = slice(0, n) if op == "seed" else qs
        Q, K, V = heads(q[qq]), heads(k[ks]), heads(v[ks])
        S = torch.matmul(Q, tr(K)) * scale
        if op.startswith("swa"):
            t = torch.arange(S.shape[1], device="cuda")
            dist = t[:, None] - t[None, :]
            S.masked_fill_((dist > case["left"]) | (dist < -case["right"]), -math.inf)
        if act == "softmax":
            P, slope = torch.softmax(S, dim=2), None
            lse[:, qs] = torch.logsumexp(S, dim=2)
        else:
            P, slope = _act64(act, S)
        O = torch.matmul(P, V)
        o[qs] = rows(O)
        if not grads:
            continue
        dO = heads(s["d_o"][qs])
        dP = torch.matmul(dO, tr(V))
        dS = (P * (dP - (dO * O).sum(dim=2, keepdim=True)) if act == "softmax" else dP * slope) * scale
        dv[ks] = rows(torch.matmul(tr(P), dO))
        dk[ks] = rows(torch.matmul(tr(dS), Q))
        dq[qq] += rows(torch.matmul(dS, K))
    if not grads:
        return o
    if op == "bwd":
        return dq, dk, dv
    if op == "seed":
        return o, lse, dq, dk, dv
    return o, dq, dk, dv
