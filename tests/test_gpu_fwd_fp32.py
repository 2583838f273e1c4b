"""The fp32 forward on the matrix cores (head dimensions 32, 64, 128) against the CPU oracle at the edges of its query
blocks (16, 32), key steps (32) and shares of the waves."""
import numpy as np
import pytest
import torch

from paper_2602_10016_amd import workloads as W
from tests.helpers import TOL, assert_close, assert_lse_close, offsets_dev, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("n,ragged", [(1, False), (16, True), (17, False), (33, True)])
@pytest.mark.parametrize("act", [0, 3])
def test_fp32_forward(oracle, d, n, ragged, act):
    from paper_2602_10016_amd import binding as kb
    lengths = np.array([0, 1, 31, 32, 33, 64, 65, 600, 257])
    B, H = len(lengths), 3
    wl = W.make("cfg1", d + n, B=B, H=H, d=d, Nq=n, lengths=("list", lengths), scale=1 / np.sqrt(d) if act == 0 else 1 / 600)
    q, q_off = wl.q, None
    if ragged:
        counts = np.array([n, 0, 1, n, n - 1, 2, n, n // 2, n])
        q_off = W.offsets_from_lengths(counts)
        q = q[:q_off[-1]]
    o, lse = kb.gdpa_fwd(to_dev(q, "fp32"), to_dev(wl.k, "fp32"), to_dev(wl.v, "fp32"), offsets_dev(wl.kv_offsets), wl.scale, act,
                         q_offsets=offsets_dev(q_off), max_q=n, max_kv=600)
    torch.cuda.synchronize()
    o_ref, lse_ref = oracle.gdpa_fwd(q, wl.k, wl.v, wl.kv_offsets, wl.scale, act, q_offsets=q_off, max_q=n)
    assert_close(to_np(o), o_ref, TOL["fp32"], f"d={d} n={n} act={act} O")
    if act == 0:
        assert_lse_close(to_np(lse), lse_ref, TOL["fp32"])


@pytest.mark.parametrize("act", [1, 2, 4, 5, 6])
def test_fp32_forward_every_score_function_many_items(oracle, act):
    """Enough items for one wave each; a key with an infinite value past the end of a history must not matter."""
    from paper_2602_10016_amd import binding as kb
    wl = W.make("cfg1", act, B=540, H=8, d=32, Nq=5, lengths=("uniform", 0, 40), scale=0.2)
    k, v = wl.k.copy(), wl.v.copy()
    last = int(wl.kv_offsets[-1]) - 1
    v[last] = np.inf  # the last key belongs to the last example alone
    o, _ = kb.gdpa_fwd(to_dev(wl.q, "fp32"), to_dev(k, "fp32"), to_dev(v, "fp32"), offsets_dev(wl.kv_offsets), wl.scale, act, max_q=5, max_kv=40)
    torch.cuda.synchronize()
    keep = slice(0, int(np.flatnonzero(np.diff(wl.kv_offsets) > 0)[-1]) * 5)
    o_ref, _ = oracle.gdpa_fwd(wl.q, wl.k, wl.v, wl.kv_offsets, wl.scale, act, max_q=5)
    assert_close(to_np(o)[keep], o_ref[keep], TOL["fp32"], f"act={act} O")


# (first masked key, one past the last) of the histories below: 32 keys in the middle (the first step of a later wave), the
# first step of the first wave, every step of the third of sixteen waves (or of eight), all keys but the last, all keys
MASKS = [(64, 96), (0, 32), (64, 96), (0, 599), (0, 600), (0, 0)]


@pytest.mark.parametrize("d", [32, 64, 128, 40])  # (40: the scalar kernel, 64 keys at a time)
@pytest.mark.parametrize("n", [5, 20])
@pytest.mark.parametrize("infinite", [False, True])
def test_fp32_softmax_with_scores_of_minus_infinity(oracle, d, n, infinite):
    """Keys whose scores are -inf (a channel of -inf, or products beyond the fp32 range) have weight 0 wherever they lie;
    a query with no other key gets a zero row and lse = -inf, as an empty history does."""
    from paper_2602_10016_amd import binding as kb
    B, H, L = len(MASKS), 2, 600
    wl = W.make("cfg1", d + n, B=B, H=H, d=d, Nq=n, lengths=("list", np.full(B, L)), scale=1 / np.sqrt(d))
    q, k = wl.q.copy(), wl.k.copy()
    q[:, :, 0] = 1e30
    k[:, :, 0] = 0
    masked = np.zeros(B * L, dtype=bool)
    for b, (lo, hi) in enumerate(MASKS):
        masked[b * L + lo:b * L + hi] = True
    masked[2 * L + 64 + 256:2 * L + 96 + 256] = True   # the third of eight waves: its second step ...
    masked[2 * L + 64 + 512:2 * L + 96 + 512] = True   # ... and its third, which is the second of the third of sixteen
    k[masked, :, 0] = -1e30
    kd = to_dev(k, "fp32")
    if infinite:
        kd[torch.from_numpy(masked).cuda(), :, 0] = -torch.inf
    o, lse = kb.gdpa_fwd(to_dev(q, "fp32"), kd, to_dev(wl.v, "fp32"), offsets_dev(wl.kv_offsets), wl.scale, 0, max_q=n, max_kv=L)
    torch.cuda.synchronize()
    o_ref, lse_ref = oracle.gdpa_fwd(q, k, wl.v, wl.kv_offsets, wl.scale, 0, max_q=n)
    o_ref[4 * n:5 * n], lse_ref[:, 4 * n:5 * n] = 0, -np.inf
    assert_close(to_np(o), o_ref, TOL["fp32"], f"d={d} n={n} O")
    assert_lse_close(to_np(lse), lse_ref, TOL["fp32"])


def test_fp32_forward_with_a_bound_far_above_the_query_counts(oracle):
    """q_offsets with one query per example under a bound of 4096: one workgroup per block of the bound would be more
    threads than a launch may have (2^32)."""
    from paper_2602_10016_amd import binding as kb
    B, H, d = 70000, 8, 32
    wl = W.make("cfg1", 5, B=B, H=H, d=d, Nq=1, lengths=("list", np.full(B, 2)), scale=0.2)
    off = np.arange(B + 1)
    o, lse = kb.gdpa_fwd(to_dev(wl.q, "fp32"), to_dev(wl.k, "fp32"), to_dev(wl.v, "fp32"), offsets_dev(wl.kv_offsets), wl.scale, 0,
                         q_offsets=offsets_dev(off), max_q=4096, max_kv=2)
    torch.cuda.synchronize()
    o_ref, lse_ref = oracle.gdpa_fwd(wl.q, wl.k, wl.v, wl.kv_offsets, wl.scale, 0, q_offsets=off, max_q=1)
    assert_close(to_np(o), o_ref, TOL["fp32"], "O")
    assert_lse_close(to_np(lse), lse_ref, TOL["fp32"])
