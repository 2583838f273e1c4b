"""Backward of up to 64 queries per example with heads in pairs (d = 32: many items, neighbouring heads with one score
function) and with two, four or eight waves per item, against the CPU oracle: ragged query counts (none, all), histories
around a tile and empty ones."""
import math

import numpy as np
import pytest
import torch

from paper_2602_10016_amd import workloads as W
from tests.helpers import TOL, assert_close, offsets_dev, to_dev, to_np

pytestmark = pytest.mark.gpu


def check(oracle, B, H, d, n, longest, act=0, head_act=None):
    from paper_2602_10016_amd import binding as kb
    rng = np.random.default_rng(B + n + d)
    lengths = rng.integers(0, 40, size=B)
    lengths[[3, B // 2, B - 1]] = [longest, 64, 65]
    lengths[rng.choice(B, 2, replace=False)] = 0
    counts = rng.integers(max(0, n - 3), n + 1, size=B)
    counts[[0, 3, B - 1]] = [0, n, n]
    softmax = act == 0 if head_act is None else 0 in head_act
    wl = W.make("cfg5", B + n, B=B, H=H, d=d, Nq=n, lengths=("list", lengths), scale=1 / math.sqrt(d) if softmax else 1 / longest)
    q_off = W.offsets_from_lengths(counts)
    q, d_o = wl.q[:q_off[-1]], wl.d_o[:q_off[-1]]
    qd, dod, k, v = (to_dev(x, "bf16") for x in (q, d_o, wl.k, wl.v))
    kvo, qo = offsets_dev(wl.kv_offsets), offsets_dev(q_off)
    args = dict(q_offsets=qo, max_q=n, max_kv=longest, head_act=head_act)
    o, lse = kb.gdpa_fwd(qd, k, v, kvo, wl.scale, act, **args)
    out = tuple(torch.full_like(t, float("nan")) for t in (qd, k, v))
    got = kb.gdpa_bwd(qd, k, v, dod, kvo, wl.scale, act, o=o, lse=lse, out=out, **args)
    torch.cuda.synchronize()
    refs = oracle.gdpa_bwd(q, wl.k, wl.v, d_o, wl.kv_offsets, wl.scale, act, q_offsets=q_off, max_q=n,
                           **({} if head_act is None else dict(head_act=head_act)))
    for a, ref, name in zip(got, refs, ("dQ", "dK", "dV")):
        assert_close(to_np(a), ref, TOL["bf16"], f"B={B} H={H} d={d} n={n} longest={longest} act={act} {name}")


# items = B * H: pairs above 3584 items of 257..512 keys (four waves), 2000 of up to 1024, 768 of longer ones (eight)
@pytest.mark.parametrize("B,H,n,longest", [(1800, 2, 1, 300), (900, 4, 32, 300), (1002, 2, 32, 600), (251, 8, 20, 600), (100, 8, 31, 1100), (390, 2, 32, 1100),
                                           (260, 8, 32, 1100)])
@pytest.mark.parametrize("act", [0, 3, 5])
def test_pairs_of_heads(oracle, B, H, n, longest, act):
    check(oracle, B, H, 32, n, longest, act)


@pytest.mark.parametrize("head_act", [[0, 0, 5, 5], [3, 3, 0, 0], [0, 3, 0, 3]])
def test_pairs_share_a_score_function_or_go_alone(oracle, head_act):
    check(oracle, 900, 4, 32, 20, 300, act=3, head_act=head_act)


# ... and eight waves for 33..64 queries up to 576 items of them
@pytest.mark.parametrize("B,n", [(1024, 3), (288, 40), (289, 40)])
def test_even_histories(oracle, B, n):
    """Histories beyond 1024 keys whose longest is less than 2.5 times the mean: many pairs are issued in memory order."""
    from paper_2602_10016_amd import binding as kb
    H, d = 2, 32
    lengths = np.full(B, 500)
    lengths[[1, 7]] = [1025, 0]
    wl = W.make("cfg5", 5, B=B, H=H, d=d, Nq=n, lengths=("list", lengths), scale=0.2)
    q, k, v, d_o = (to_dev(a, "bf16") for a in (wl.q, wl.k, wl.v, wl.d_o))
    kvo = offsets_dev(wl.kv_offsets)
    o, lse = kb.gdpa_fwd(q, k, v, kvo, wl.scale, 0, max_q=n, max_kv=1025)
    got = kb.gdpa_bwd(q, k, v, d_o, kvo, wl.scale, 0, o=o, lse=lse, max_q=n, max_kv=1025)
    torch.cuda.synchronize()
    for a, ref, name in zip(got, oracle.gdpa_bwd(wl.q, wl.k, wl.v, wl.d_o, wl.kv_offsets, wl.scale, 0, max_q=n), ("dQ", "dK", "dV")):
        assert_close(to_np(a), ref, TOL["bf16"], name)


# eight waves: d = 32 up to 256 items in whole groups of eight examples (768 of long histories), d = 64 with up to 32 queries 256 so, beyond 512 keys 640 with softmax
# heads and 1024 without, all beyond 1024; two waves: d = 64 with 33..64 queries above 512 items (640 with histories beyond 512
# keys, 704 beyond 1024, 1400 beyond 2048), and with up to 32 queries above 2048 items of up to 256 keys
@pytest.mark.parametrize("B,H,d,n,longest", [(64, 4, 32, 32, 90), (65, 4, 32, 32, 90), (64, 4, 32, 64, 300), (65, 4, 32, 33, 300), (192, 4, 32, 20, 1100),
                                             (192, 4, 32, 64, 1100), (193, 4, 32, 40, 1100), (64, 4, 64, 32, 500), (65, 4, 64, 32, 500),
                                             (256, 4, 64, 17, 600), (257, 4, 64, 17, 600), (300, 4, 64, 32, 1100), (128, 4, 64, 64, 90),
                                             (129, 4, 64, 33, 90), (160, 4, 64, 40, 600), (161, 4, 64, 40, 600), (320, 4, 64, 40, 2100), (321, 4, 64, 40, 2100),
                                             (513, 4, 64, 20, 90), (160, 4, 64, 17, 600), (161, 4, 64, 17, 600), (176, 4, 64, 40, 1100), (177, 4, 64, 40, 1100),
                                             (350, 4, 64, 40, 2100), (351, 4, 64, 40, 2100), (81, 3, 64, 20, 90), (80, 3, 32, 40, 90), (81, 3, 32, 40, 90)])
@pytest.mark.parametrize("act", [0, 3])
def test_waves_per_item(oracle, B, H, d, n, longest, act):
    check(oracle, B, H, d, n, longest, act)
