"""Streaming forward with heads in pairs (d = 32: many items, neighbouring heads with one score function) and with both
blocks of 33..64 queries in one wave (d = 32 pairs and d = 64), against the CPU oracle: every number of waves that share the
key tiles of an item, ragged query counts, histories around a tile and empty ones."""
import math

import numpy as np
import pytest
import torch

from paper_2602_10016_amd import workloads as W
from tests.helpers import TOL, assert_close, assert_lse_close, offsets_dev, to_dev, to_np

pytestmark = pytest.mark.gpu


def check(oracle, B, H, d, n, longest, act=0, head_act=None, seed=0):
    from paper_2602_10016_amd import binding as kb
    rng = np.random.default_rng(B + n + d + seed)
    lengths = rng.integers(0, 40, size=B)
    lengths[[3, B // 2, B - 1]] = [longest, 64, 65]
    lengths[rng.choice(B, 5, replace=False)] = 0
    counts = rng.integers(max(0, n - 3), n + 1, size=B)
    counts[[0, 3, B - 1]] = [0, n, n]
    softmax = act == 0 if head_act is None else 0 in head_act
    wl = W.make("cfg5", B + n, B=B, H=H, d=d, Nq=n, lengths=("list", lengths), scale=1 / math.sqrt(d) if softmax else 1 / longest)
    q_off = W.offsets_from_lengths(counts)
    q = wl.q[:q_off[-1]]
    qd, k, v = (to_dev(x, "bf16") for x in (q, wl.k, wl.v))
    o = torch.full_like(qd, float("nan"))
    lse = torch.full((H, qd.shape[0]), float("nan"), dtype=torch.float32, device="cuda")
    kb.gdpa_fwd(qd, k, v, offsets_dev(wl.kv_offsets), wl.scale, act, q_offsets=offsets_dev(q_off), max_q=n, max_kv=longest,
                head_act=head_act, out=o, lse=lse)
    torch.cuda.synchronize()
    o_ref, lse_ref = oracle.gdpa_fwd(q, wl.k, wl.v, wl.kv_offsets, wl.scale, act, q_offsets=q_off, max_q=n,
                                     **({} if head_act is None else dict(head_act=head_act)))
    assert_close(to_np(o), o_ref, TOL["bf16"], f"B={B} H={H} d={d} n={n} longest={longest} act={act}")
    for h in range(H):
        if (act if head_act is None else head_act[h]) == 0:
            assert_lse_close(to_np(lse)[h], lse_ref[h], 1e-2)


# items = B * H.  Up to 32 queries: pairs above 2048 items, or with histories beyond 1024 keys above 1024 where they are even, else
# 1216 (1456 with a form of GELU); 33..64: above 1500 or 1000 (two, four or eight waves by items and longest history)
@pytest.mark.parametrize("B,H,n,longest", [(1030, 2, 1, 90), (1030, 2, 32, 600), (260, 4, 31, 1100), (530, 4, 32, 1100), (330, 8, 17, 1100),
                                           (760, 2, 33, 90), (760, 2, 64, 600), (1060, 4, 40, 600), (255, 4, 64, 1100), (600, 4, 33, 1100),
                                           (1100, 4, 64, 1100), (510, 2, 50, 2100), (306, 4, 31, 1100), (366, 4, 31, 1100)])
@pytest.mark.parametrize("act", [0, 3])
def test_pairs_of_heads(oracle, B, H, n, longest, act):
    check(oracle, B, H, 32, n, longest, act)


@pytest.mark.parametrize("head_act", [[0, 0, 5, 5], [3, 3, 0, 0], [0, 3, 0, 3]])
@pytest.mark.parametrize("n", [20, 50])
def test_pairs_share_a_score_function_or_go_alone(oracle, head_act, n):
    check(oracle, 530, 4, 32, n, 200, act=3, head_act=head_act)


# both blocks above 140 short items or, with uneven histories beyond 1024 keys, 256; two items per (example, head) below
@pytest.mark.parametrize("B,H,n,longest", [(35, 4, 40, 90), (36, 4, 40, 90), (64, 4, 40, 1100), (65, 4, 40, 1100), (33, 4, 33, 90), (49, 4, 64, 1100), (130, 4, 64, 90), (130, 4, 40, 600), (130, 4, 64, 1100), (300, 4, 50, 600),
                                           (300, 4, 64, 1100), (180, 4, 64, 2100), (520, 4, 64, 1100)])
@pytest.mark.parametrize("act", [0, 3, 5])
def test_both_query_blocks_in_a_wave(oracle, B, H, n, longest, act):
    check(oracle, B, H, 64, n, longest, act)


# more than 2048 items of up to 32 queries: two waves, or four with long histories, share an item's key tiles; d = 128 and uneven
# long histories: eight up to 936 items
@pytest.mark.parametrize("B,d,n,longest", [(515, 64, 32, 90), (515, 64, 20, 1100), (515, 128, 20, 90), (515, 128, 32, 1100), (234, 128, 20, 1100),
                                           (235, 128, 20, 1100)])
@pytest.mark.parametrize("act", [0, 3])
def test_many_items_share_key_tiles(oracle, B, d, n, longest, act):
    check(oracle, B, 4, d, n, longest, act)
