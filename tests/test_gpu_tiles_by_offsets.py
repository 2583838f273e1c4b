"""Small launches of long query sequences find their tiles from the offsets: in the forward up to 1280 tiles of 128 queries, times heads, at d = 128 and
2048 at d = 32 and 64, in the two-pass backward 1536 and 3600, over at most 32 keys 2600 and 4096 (1280 for examples of less than a tile at d = 64
and 128), where the numbers without a tile cost no round.  Examples of less than a tile, of whole tiles and empty ones, first and last, in batches around
the 64 probes of a search step and of one, two and three steps, by both mappings, against the CPU oracle.  Which mapping a call took shows in its
workspace: by offsets nothing is written where the tile tables would be."""
import numpy as np
import pytest
import torch

from paper_2602_10016_amd import workloads as W
from tests.helpers import TOL, assert_close, assert_close_sums, offsets_dev, to_dev, to_np

pytestmark = pytest.mark.gpu


def ragged(rng, B, longest):
    lengths = rng.integers(0, longest + 1, size=B)
    special = [0, 128, 129, 127, 0, 256, 1, longest]
    lengths[:min(B, len(special))] = [min(x, longest) for x in special[-min(B, len(special)):]]
    rng.shuffle(lengths)
    if B > 2:
        lengths[0] = lengths[-1] = 0
    return lengths


def workspace(kb, op, *sizes):
    return torch.full((kb.workspace_bytes(op, *sizes),), 0xEE, dtype=torch.uint8, device="cuda")


def tables_written(ws, at):
    """Whether a launch has left tile tables at byte `at` of a workspace that was filled with 0xEE."""
    return bool(torch.any(ws[at:at + 4] != 0xEE))


def behind_order(B):
    return 256 + ((B + 1) * 4 + 255) // 256 * 256


def values(rng, rows, H, d):
    return W.round_to_bf16(rng.standard_normal((rows, H, d), dtype=np.float32) * 0.5)


# tables: whether the forward writes them, and the backward (over more than 32 keys in two passes)
@pytest.mark.parametrize("B,H,d,longest,keys,act,tables", [(1, 2, 64, 500, 20, 3, (False, False)), (63, 2, 128, 600, 32, 0, (False, False)), (64, 3, 32, 400, 48, 3, (False, False)),
                                                           (65, 1, 128, 700, 40, 0, (False, False)), (129, 4, 64, 300, 8, 0, (True, True)), (231, 1, 32, 150, 46, 0, (False, True)),
                                                           (1500, 1, 64, 140, 33, 0, (True, False)), (520, 4, 32, 300, 20, 3, (True, False)), (700, 2, 128, 300, 40, 0, (True, True)),
                                                           (4300, 1, 64, 200, 40, 3, (True, True))])
def test_long_query_sequences(oracle, B, H, d, longest, keys, act, tables):
    from paper_2602_10016_amd import binding as kb
    rng = np.random.default_rng(B + d)
    n_keys = rng.integers(0, keys + 1, size=B)
    n_keys[B // 2] = keys
    q_off, kv_off = W.offsets_from_lengths(ragged(rng, B, longest)), W.offsets_from_lengths(n_keys)
    q, k, v = values(rng, q_off[-1], H, d), values(rng, kv_off[-1], H, d), values(rng, kv_off[-1], H, d)
    d_o = values(rng, q_off[-1], H, d)
    scale = d ** -0.5 if act == 0 else 1.0 / keys
    tq, tk, tv, tdo = (to_dev(x, "bf16") for x in (q, k, v, d_o))
    how = dict(q_offsets=offsets_dev(q_off), max_q=longest, max_kv=keys)
    sizes = (B, H, d, longest, keys, tq.shape[0], tk.shape[0])
    ws, ws_bwd = workspace(kb, kb.OP_GDPA_FWD, *sizes), workspace(kb, kb.OP_GDPA_BWD, *sizes)
    o, lse = kb.gdpa_fwd(tq, tk, tv, offsets_dev(kv_off), scale, act, out=torch.full_like(tq, float("nan")), workspace=ws, **how)
    out = tuple(torch.full_like(t, float("nan")) for t in (tq, tk, tv))
    got = kb.gdpa_bwd(tq, tk, tv, tdo, offsets_dev(kv_off), scale, act, o=o, lse=lse, out=out, workspace=ws_bwd, **how)
    torch.cuda.synchronize()
    assert (tables_written(ws, 256), tables_written(ws_bwd, behind_order(B))) == tables
    o_ref, _ = oracle.gdpa_fwd(q, k, v, kv_off, scale, act, q_offsets=q_off, max_q=longest)
    refs = oracle.gdpa_bwd(q, k, v, d_o, kv_off, scale, act, q_offsets=q_off, max_q=longest)
    for a, ref, name in zip((o, got[0]), (o_ref, refs[0]), ("O", "dQ")):
        assert_close(to_np(a), ref, TOL["bf16"], f"B={B} H={H} d={d} {name}")
    for a, ref, name in zip(got[1:], refs[1:], ("dK", "dV")):  # sums over the queries with rounded factors: held to their RMS (see there)
        assert_close_sums(to_np(a), ref, TOL["bf16"], f"B={B} H={H} d={d} {name}", offsets=kv_off)


@pytest.mark.parametrize("B,H,d,longest,left,right,tables", [(1, 1, 64, 300, 40, 0, False), (64, 2, 64, 260, 127, 0, False), (65, 2, 128, 260, 31, 31, False), (66, 1, 32, 400, 255, 0, False),
                                                             (2200, 1, 64, 130, 20, 5, False), (4200, 1, 32, 60, 20, 0, False), (30, 2, 64, 900, 800, 0, False), (160, 1, 32, 200, 20, 0, True),
                                                             (5200, 1, 32, 60, 20, 0, True), (6000, 1, 64, 60, 9, 0, True)])
def test_sliding_window_backward(oracle, B, H, d, longest, left, right, tables):
    from paper_2602_10016_amd import binding as kb
    rng = np.random.default_rng(B + d)
    off = W.offsets_from_lengths(ragged(rng, B, longest))
    q, k, v, d_o = (values(rng, off[-1], H, d) for _ in range(4))
    tq, tk, tv, tdo = (to_dev(x, "bf16") for x in (q, k, v, d_o))
    o, lse = kb.swa_fwd(tq, tk, tv, offsets_dev(off), left, right, d ** -0.5, max_len=longest)
    out = tuple(torch.full_like(t, float("nan")) for t in (tq, tk, tv))
    ws = workspace(kb, kb.OP_SWA_BWD, B, H, d, longest, longest, tq.shape[0], tq.shape[0])
    got = kb.swa_bwd(tq, tk, tv, o, lse, tdo, offsets_dev(off), left, right, d ** -0.5, max_len=longest, out=out, workspace=ws)
    torch.cuda.synchronize()
    assert tables_written(ws, behind_order(B)) == tables
    refs = oracle.swa_bwd(q, k, v, d_o, off, left, right, d ** -0.5)
    for a, ref, name in zip(got, refs, ("dQ", "dK", "dV")):
        assert_close(to_np(a), ref, TOL["bf16"], f"B={B} H={H} d={d} window=({left}, {right}) {name}")


# 2 x 1700 and 2 x 1100 examples of less than a tile (3490 and 2260 tile-heads), 2 x 150 (300) and 2 x 200 of several tiles (1840); the line of d = 32 is 4096
@pytest.mark.parametrize("d,B,H,longest,tables", [(64, 1700, 2, 90, True), (128, 1100, 2, 90, True), (32, 1700, 2, 90, False), (64, 150, 2, 90, False), (128, 150, 2, 90, False),
                                                  (64, 200, 2, 700, False), (128, 200, 2, 700, False)])
def test_few_keys_of_short_examples_keep_the_tables(d, B, H, longest, tables):
    assert few_keys_by_tables(d, B, H, longest // 2, longest) == tables


# chunks of nearly equal lengths: one round of two workgroups per compute unit by tables and two of numbers; one of either
@pytest.mark.parametrize("d,B,H,shortest,longest,tables", [(128, 401, 1, 103, 129, True), (64, 217, 2, 104, 131, True), (128, 150, 1, 103, 129, False)])
def test_few_keys_of_nearly_equal_lengths(d, B, H, shortest, longest, tables):
    assert few_keys_by_tables(d, B, H, shortest, longest) == tables


def few_keys_by_tables(d, B, H, shortest, longest):
    from paper_2602_10016_amd import binding as kb
    rng = np.random.default_rng(B + d)
    lengths = rng.integers(shortest, longest + 1, size=B)
    lengths[0] = longest
    q_off, kv_off = W.offsets_from_lengths(lengths), W.offsets_from_lengths(np.full(B, 8))
    q, k, v, d_o = (to_dev(values(rng, int(n), H, d), "bf16") for n in (q_off[-1], kv_off[-1], kv_off[-1], q_off[-1]))
    ws = workspace(kb, kb.OP_GDPA_BWD, B, H, d, longest, 8, q.shape[0], k.shape[0])
    kb.gdpa_bwd(q, k, v, d_o, offsets_dev(kv_off), 0.1, 3, q_offsets=offsets_dev(q_off), max_q=longest, max_kv=8, workspace=ws)
    torch.cuda.synchronize()
    return tables_written(ws, behind_order(B))
