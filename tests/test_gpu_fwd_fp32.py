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
