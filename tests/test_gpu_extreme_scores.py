"""Softmax with scores of -inf (single keys, the whole share of a wave, the first tiles, every key of a head), of +inf and NaN through
the launches that share an item's key tiles, own a pair of heads or both query blocks, against 64-bit numpy: a key that scores
-inf has weight 0, a query whose keys all do has output 0 and an LSE of -inf, +inf and NaN make the row NaN - of that head alone."""
import math

import numpy as np
import pytest
import torch

from paper_2602_10016_amd import workloads as W
from tests.helpers import TOL, offsets_dev, to_dev, to_np

pytestmark = pytest.mark.gpu


def make(B, H, d, n, longest, kinds):
    """q[..., 0] = 1, so that K[key, h, 0] = -inf, +inf or NaN is the score of a key; example b takes kind b % 8 in head b % H."""
    rng = np.random.default_rng(B + n + d)
    lengths = rng.integers(30, 200, size=B)
    lengths = np.minimum(lengths, longest)
    lengths[B // 2] = longest
    off = W.offsets_from_lengths(lengths)
    bf = lambda *s: W.round_to_bf16((rng.standard_normal(s) * 0.5).astype(np.float32))
    q, k, v, d_o = bf(B * n, H, d), bf(int(off[-1]), H, d), bf(int(off[-1]), H, d), bf(B * n, H, d)
    q[:, :, 0] = 1
    for b in range(B):
        rows, h, L = np.arange(off[b], off[b + 1]), b % H, lengths[b]
        tile, kind = np.arange(L) // 32, kinds[b % len(kinds)]
        if kind == "all":
            k[rows, h, 0] = -np.inf
        elif kind in ("even", "second", "first", "half"):
            gone = {"even": tile % 2 == 0, "second": tile % 4 == 1, "first": np.arange(L) < 64, "half": rng.random(L) < 0.5}[kind]
            gone[-1] = False if kind != "even" else gone[-1] and tile[-1] > 0
            if kind == "even" and gone.all():
                gone[0] = False
            k[rows[gone], h, 0] = -np.inf
        elif kind in ("inf", "nan"):
            k[rows[rng.integers(L)], h, 0] = np.inf if kind == "inf" else np.nan
    return q, k, v, d_o, off


def softmax(s):
    with np.errstate(invalid="ignore"):
        return softmax_of(s)


def softmax_of(s):
    m = s.max(axis=1, keepdims=True)
    e = np.exp(s - np.where(np.isfinite(m), m, 0))
    e[np.isneginf(s)] = 0
    total = e.sum(axis=1, keepdims=True)
    bad = np.isnan(m) | np.isposinf(m)
    p = np.where(total > 0, e / np.where(total > 0, total, 1), 0)
    lse = np.where(total > 0, np.where(np.isfinite(m), m, 0) + np.log(np.where(total > 0, total, 1)), -np.inf)
    return np.where(bad, np.nan, p), np.where(bad, np.nan, lse)[:, 0]


def close(got, ref, what):
    assert np.array_equal(np.isnan(got), np.isnan(ref)), f"{what}: NaN in other places"
    ok = ~np.isnan(ref)
    assert not ok.any() or np.all(np.isfinite(got[ok])) and np.abs(got[ok] - ref[ok]).max() <= TOL["bf16"] * (1 + np.abs(ref[ok]).max()), what


def scores(q, k, scale):
    with np.errstate(invalid="ignore"):
        return (q.astype(np.float64) @ k.astype(np.float64).T) * scale


# pairs: four and two waves with one query block, two, eight and four with two; both blocks at d = 64: two, four, eight waves;
# many items with two and four waves; few items with four and eight; a workgroup of two waves at d = 128
@pytest.mark.parametrize("B,H,d,n,longest", [(310, 4, 32, 20, 1100), (1030, 2, 32, 32, 200), (760, 2, 32, 40, 200), (255, 4, 32, 50, 1100), (600, 4, 32, 33, 1100),
                                             (130, 4, 64, 64, 200), (50, 4, 64, 40, 600), (80, 4, 64, 40, 1100), (515, 4, 64, 32, 200), (515, 4, 64, 20, 1100),
                                             (515, 4, 128, 20, 200), (16, 2, 64, 32, 200), (16, 2, 128, 64, 1100), (515, 4, 128, 50, 200)])
def test_forward(B, H, d, n, longest):
    from paper_2602_10016_amd import binding as kb
    q, k, v, _, off = make(B, H, d, n, longest, ["none", "all", "even", "second", "first", "half", "inf", "nan"])
    scale = 1 / math.sqrt(d)
    dev = [to_dev(x, "bf16") for x in (q, k, v)]
    o = torch.full_like(dev[0], 7.0)
    lse = torch.full((H, B * n), 7.0, device="cuda")
    kb.gdpa_fwd(*dev, offsets_dev(off), scale, kb.ACT_SOFTMAX, max_q=n, max_kv=longest, out=o, lse=lse)
    torch.cuda.synchronize()
    o, lse = to_np(o), to_np(lse)
    for b in range(B):
        rows, keys = slice(b * n, (b + 1) * n), slice(off[b], off[b + 1])
        for h in range(H):
            p, ref_lse = softmax(scores(q[rows, h], k[keys, h], scale))
            what = f"example {b} head {h}"
            close(o[rows, h], p @ v[keys, h].astype(np.float64), what)
            ok = ~np.isnan(ref_lse)
            assert np.array_equal(np.isneginf(lse[h, rows][ok]), np.isneginf(ref_lse[ok])), what
            ok &= np.isfinite(ref_lse)
            assert np.all(np.abs(lse[h, rows][ok] - ref_lse[ok]) <= 1e-2), what


# pairs with four and eight waves, single heads of 32 with four and eight, d = 64 with two, four and eight, d = 128 with four
@pytest.mark.parametrize("B,H,d,n,longest", [(1800, 2, 32, 20, 300), (1002, 2, 32, 32, 600), (70, 2, 32, 50, 200), (300, 2, 32, 20, 200), (260, 2, 64, 40, 200),
                                             (70, 2, 64, 40, 200), (70, 2, 64, 32, 200), (70, 2, 128, 20, 200), (40, 2, 128, 64, 200), (40, 2, 128, 40, 200)])
def test_backward(B, H, d, n, longest):
    from paper_2602_10016_amd import binding as kb
    q, k, v, d_o, off = make(B, H, d, n, longest, ["none", "even", "second", "first", "half"])
    scale = 1 / math.sqrt(d)
    qd, kd, vd, dod = (to_dev(x, "bf16") for x in (q, k, v, d_o))
    kvo = offsets_dev(off)
    o, lse = kb.gdpa_fwd(qd, kd, vd, kvo, scale, kb.ACT_SOFTMAX, max_q=n, max_kv=longest)
    out = tuple(torch.full_like(t, 7.0) for t in (qd, kd, vd))
    kb.gdpa_bwd(qd, kd, vd, dod, kvo, scale, kb.ACT_SOFTMAX, o=o, lse=lse, max_q=n, max_kv=longest, out=out)
    torch.cuda.synchronize()
    dq, dk, dv = (to_np(t) for t in out)
    for b in range(B):
        rows, keys = slice(b * n, (b + 1) * n), slice(off[b], off[b + 1])
        for h in range(H):
            Q, K, V, dO = (x.astype(np.float64) for x in (q[rows, h], k[keys, h], v[keys, h], d_o[rows, h]))
            p, _ = softmax(scores(Q, K, scale))
            dp = dO @ V.T
            ds = p * (dp - (p * dp).sum(axis=1, keepdims=True)) * scale
            what = f"example {b} head {h}"
            close(dv[keys, h], p.T @ dO, what + " dV")
            close(dk[keys, h], ds.T @ Q, what + " dK")
            with np.errstate(invalid="ignore"):
                close(dq[rows, h], ds @ K, what + " dQ")  # (channel 0 is NaN where a weight of 0 meets a key of -inf)


# as many items as heads go in pairs from: forward above 2048 short items (33..64 seeds 1500), backward above 3584 of 257..512 keys
@pytest.mark.parametrize("B,H,seeds,longest", [(1030, 2, 20, 90), (760, 2, 40, 90), (1800, 2, 32, 300)])
def test_shared_seeds_through_pairs_of_heads(oracle, B, H, seeds, longest):
    from paper_2602_10016_amd import binding as kb
    from tests.helpers import assert_close, assert_close_sums
    d, rng = 32, np.random.default_rng(seeds)
    lengths = rng.integers(0, 40, size=B)
    lengths[[3, B - 1]] = [longest, 65]
    wl = W.make("cfg5", seeds, B=B, H=H, d=d, Nq=seeds, lengths=("list", lengths), scale=1 / math.sqrt(d))
    e = W.round_to_bf16((rng.standard_normal((seeds, H, d)) * 0.5).astype(np.float32))
    ed, k, v, d_o = (to_dev(x, "bf16") for x in (e, wl.k, wl.v, wl.d_o))
    kvo = offsets_dev(wl.kv_offsets)
    o, lse = kb.seed_attn_fwd(ed, k, v, kvo, wl.scale, 0, max_kv=longest)
    d_e, dk, dv = kb.seed_attn_bwd(ed, k, v, d_o, kvo, wl.scale, 0, o=o, lse=lse, max_kv=longest)
    torch.cuda.synchronize()
    assert_close(to_np(o), oracle.seed_attn_fwd(e, wl.k, wl.v, wl.kv_offsets, wl.scale, 0)[0], TOL["bf16"], "O")
    refs = oracle.seed_attn_bwd(e, wl.k, wl.v, wl.d_o, wl.kv_offsets, wl.scale, 0)
    # (sums, dK and dV too: a history of a few keys has weights between 1/2 and 1, whose rounding is off by up to 2^-9; 40 seeds add up
    # to sqrt(40) 2^-9 / sqrt(3) = 0.007, a third of the element-wise tolerance, and there are 955 000 elements)
    for got, ref, name in zip((d_e, dk, dv), refs, ("dE", "dK", "dV")):
        assert_close_sums(to_np(got), ref, TOL["bf16"], name, offsets=None if name == "dE" else wl.kv_offsets)
