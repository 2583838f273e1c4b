"""The one-pass backward for 65..256 queries per example at head dimension 128 (whole histories, and ranges of them with
partial query gradients) against the CPU oracle, at the edges of its tiles, query blocks and ranges."""
import math

import numpy as np
import pytest
import torch

from paper_2602_10016_amd import workloads as W
from tests.helpers import TOL, assert_close, assert_close_sums, offsets_dev, to_dev, to_np

pytestmark = pytest.mark.gpu

# (B, H, queries, history lengths drawn from lo..hi, first lengths fixed): whole histories when a compute unit has
# enough work besides the longest one, ranges of 8 tiles (256 keys) else - one key more and less than a range, too
CASES = [
    (130, 8, 65, 1, 40, [0, 1, 31, 32, 33, 64]),
    (64, 4, 256, 20, 60, [0, 33, 60]),
    (5, 2, 256, 1, 700, [0, 255, 256, 257, 513]),
    (9, 3, 97, 1, 300, [256, 0, 1, 257]),
    (3, 1, 129, 500, 1100, [1025]),
    (4, 2, 255, 33, 64, [33]),
    # whole histories of several tiles (the ring of three stages wraps, items follow long ones): 1024 items and more
    (129, 8, 65, 0, 300, [97, 128, 129, 257, 0, 1]),
    (128, 8, 256, 0, 300, [300, 96, 128, 129, 0, 257]),
    # ranges of nine tiles (more than 4608 tiles in all)
    (40, 8, 100, 400, 450, [2300, 288, 289, 0, 577]),
]


@pytest.mark.parametrize("B,H,n,lo,hi,fixed", CASES)
@pytest.mark.parametrize("act", [0, 3])
@pytest.mark.parametrize("ragged", [False, True])
def test_backward_65_to_256_queries(oracle, B, H, n, lo, hi, fixed, act, ragged):
    from paper_2602_10016_amd import binding as kb
    rng = np.random.default_rng(1000 * B + n)
    lengths = np.concatenate([fixed, rng.integers(lo, hi + 1, size=B - len(fixed))]).astype(np.int64)
    wl = W.make("cfg5", B + n, B=B, H=H, d=128, Nq=n, lengths=("list", lengths), scale=1 / math.sqrt(128))
    q, d_o, q_off = wl.q, wl.d_o, None
    if ragged:  # an example without queries, one with a single one, one that ends a block of 32
        counts = rng.integers(1, n + 1, size=B)
        counts[:3] = [n, 0, 1]
        counts[-1] = 64
        q_off = W.offsets_from_lengths(counts)
        q, d_o = q[:q_off[-1]], d_o[:q_off[-1]]
    mk = wl.max_kv
    qd, k, v, dod = to_dev(q, "bf16"), to_dev(wl.k, "bf16"), to_dev(wl.v, "bf16"), to_dev(d_o, "bf16")
    kvo, qo = offsets_dev(wl.kv_offsets), offsets_dev(q_off)
    o, lse = kb.gdpa_fwd(qd, k, v, kvo, wl.scale, act, q_offsets=qo, max_q=n, max_kv=mk)
    out = tuple(torch.full_like(t, float("nan")) for t in (qd, k, v))
    got = kb.gdpa_bwd(qd, k, v, dod, kvo, wl.scale, act, o=o, lse=lse, q_offsets=qo, max_q=n, max_kv=mk, out=out)
    again = kb.gdpa_bwd(qd, k, v, dod, kvo, wl.scale, act, o=o, lse=lse, q_offsets=qo, max_q=n, max_kv=mk)
    torch.cuda.synchronize()
    refs = oracle.gdpa_bwd(q, wl.k, wl.v, d_o, wl.kv_offsets, wl.scale, act, q_offsets=q_off, max_q=n)
    for a, b, ref, name in zip(got, again, refs, ("dQ", "dK", "dV")):
        what = f"B={B} H={H} n={n} act={act} ragged={ragged} {name}"
        if name == "dQ" and act == 3 and mk > 512:
            # Scores of order one without a normaliser: dQ sums ~1000 products with a bf16-rounded dS, each off by at
            # most 2^-8 of itself and 2^-9 / sqrt(3) = 1.1e-3 RMS, so the sum is off by 1.1e-3 of its RMS (about 4
            # here: 5 standard deviations are 2.2e-2 absolute, also where the value is near zero), plus its own
            # rounding 2^-9 |r|: within 2e-2 (rms + |r|) with a factor of three to spare.
            assert_close_sums(to_np(a), ref, TOL["bf16"], what)
        elif n == 256 and B == 128 and (act == 3 or name != "dQ"):
            # 256 terms per dK and dV element (histories of one key: weights of one, dV of order 16), 300 per dQ element, each
            # with a bf16-rounded factor, in tens of millions of elements: off by 1.1e-3 of the RMS of its sums (as above),
            # here per example and head for dK and dV, so 2e-2 (rms + |r|) are 18 standard deviations, where
            # 2e-2 (1 + |r|) are 2.5 of the largest sums.  (The two-pass kernels have the same errors: 5.24e-4 RMS in dV.)
            assert_close_sums(to_np(a), ref, TOL["bf16"], what, offsets=None if name == "dQ" else wl.kv_offsets)
        else:
            assert_close(to_np(a), ref, TOL["bf16"], what)
        assert torch.equal(a, b), f"{name} differs between two runs"


@pytest.mark.parametrize("act", [1, 2, 4, 5, 6])
def test_backward_wide_every_score_function(oracle, act):
    from paper_2602_10016_amd import binding as kb
    wl = W.make("cfg5", act, B=6, H=2, d=128, Nq=70, lengths=("list", np.array([300, 0, 40, 257, 31, 64])), scale=0.09)
    q, k, v, d_o = (to_dev(x, "bf16") for x in (wl.q, wl.k, wl.v, wl.d_o))
    got = kb.gdpa_bwd(q, k, v, d_o, offsets_dev(wl.kv_offsets), wl.scale, act, max_q=70, max_kv=300)
    torch.cuda.synchronize()
    refs = oracle.gdpa_bwd(wl.q, wl.k, wl.v, wl.d_o, wl.kv_offsets, wl.scale, act, max_q=70)
    for a, ref, name in zip(got, refs, ("dQ", "dK", "dV")):
        # dQ: up to 300 products with a rounded dS at scores of order one, RMS about 4 - the bound above
        (assert_close_sums if name == "dQ" else assert_close)(to_np(a), ref, TOL["bf16"], f"act={act} {name}")


def test_workspace_of_the_largest_batch_serves_smaller_ones(oracle):
    """One buffer, sized for the largest batch, for calls with fewer examples and fewer tokens: accepted, and right."""
    from paper_2602_10016_amd import binding as kb
    n, H, d, longest = 70, 8, 128, 900
    ws = torch.empty(kb.workspace_bytes(kb.OP_GDPA_BWD, 150, H, d, n, longest, 150 * n, 150 * longest), dtype=torch.uint8, device="cuda")
    ws_seed = torch.empty(kb.workspace_bytes(kb.OP_SEED_BWD, 150, H, d, n, longest, 150 * n, 150 * longest), dtype=torch.uint8, device="cuda")
    for B, lengths in ((3, [900, 40, 1]), (2, [0, 333])):
        wl = W.make("cfg5", B, B=B, H=H, d=d, Nq=n, lengths=("list", np.array(lengths)), scale=1 / math.sqrt(d))
        q, k, v, d_o = (to_dev(x, "bf16") for x in (wl.q, wl.k, wl.v, wl.d_o))
        kvo = offsets_dev(wl.kv_offsets)
        o, lse = kb.gdpa_fwd(q, k, v, kvo, wl.scale, 0, max_q=n, max_kv=longest)
        got = kb.gdpa_bwd(q, k, v, d_o, kvo, wl.scale, 0, o=o, lse=lse, max_q=n, max_kv=longest, workspace=ws)
        refs = oracle.gdpa_bwd(wl.q, wl.k, wl.v, wl.d_o, wl.kv_offsets, wl.scale, 0, max_q=n)
        seeds = q[:n].contiguous()
        o, lse = kb.seed_attn_fwd(seeds, k, v, kvo, wl.scale, 0, max_kv=longest)
        got_seed = kb.seed_attn_bwd(seeds, k, v, d_o, kvo, wl.scale, 0, o=o, lse=lse, max_kv=longest, workspace=ws_seed)
        torch.cuda.synchronize()
        for a, ref, name in zip(got, refs, ("dQ", "dK", "dV")):
            assert_close(to_np(a), ref, TOL["bf16"], f"B={B} {name}")
        refs = oracle.gdpa_bwd(np.tile(wl.q[:n], (B, 1, 1)), wl.k, wl.v, wl.d_o, wl.kv_offsets, wl.scale, 0, max_q=n)
        for a, ref, name in zip(got_seed, (refs[0].reshape(B, n, H, d).sum(axis=0), *refs[1:]), ("dE", "dK", "dV")):
            (assert_close_sums if name == "dE" else assert_close)(to_np(a), ref, TOL["bf16"], f"B={B} seeds {name}")


@pytest.mark.parametrize("n", [65, 97, 250])
def test_padding_queries_add_nothing_at_keys_masked_by_infinity(n):
    """A key whose scores are -inf (a channel of -inf) has weight 0 for every query of the example, and so zero dK and dV:
    the rows that pad the queries to whole blocks, whose scores there are 0 * -inf, must not reach them.  (dQ is not
    compared: it adds 0 * -inf.)"""
    from paper_2602_10016_amd import binding as kb
    B, H, L = 3, 2, 70
    wl = W.make("cfg5", n, B=B, H=H, d=128, Nq=n, lengths=("list", np.full(B, L)), scale=1 / math.sqrt(128))
    q, k, v, d_o = (to_dev(x, "bf16") for x in (wl.q, wl.k, wl.v, wl.d_o))
    q[:, :, 0] = 1
    masked = torch.zeros(B * L, dtype=torch.bool, device="cuda")
    masked[[3, 40, L + 69, 2 * L]] = True
    k[masked, :, 0] = -torch.inf
    kvo = offsets_dev(wl.kv_offsets)
    o, lse = kb.gdpa_fwd(q, k, v, kvo, wl.scale, 0, max_q=n, max_kv=L)
    _, dk, dv = kb.gdpa_bwd(q, k, v, d_o, kvo, wl.scale, 0, o=o, lse=lse, max_q=n, max_kv=L)
    torch.cuda.synchronize()
    assert torch.isfinite(o).all() and torch.isfinite(dk).all() and torch.isfinite(dv).all()
    assert (dk[masked] == 0).all() and (dv[masked] == 0).all() and (dv[~masked] != 0).any()
