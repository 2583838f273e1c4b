"""Backward calls with many queries over at most 32 keys keep partial sums per workgroup.  Every workspace that was made for a
larger batch is accepted, and one with room for fewer partial sums gives the same gradients."""
import numpy as np
import pytest
import torch

from paper_2602_10016_amd import workloads as W
from tests.helpers import TOL, assert_close, offsets_dev, to_dev, to_np


def test_a_workspace_for_a_larger_batch_is_accepted():
    """(Misaligned workspace pointer: an accepted size ends in that error, and nothing is launched.)"""
    from paper_2602_10016_amd import binding as kb
    lib, P, max_kv = kb.raw(), 0x1000, 32
    for H, d in ((1, 32), (4, 128), (8, 64)):
        for op in (kb.OP_GDPA_BWD, kb.OP_SEED_BWD):
            sizes = [(B, 65 if op == kb.OP_SEED_BWD else mean) for B in (1, 3, 100, 128, 230, 240, 1000) for mean in (65, 600, 1152, 1300, 4000)]
            for B, mean in set(sizes):
                largest = kb.workspace_bytes(op, B, H, d, 65 if op == kb.OP_SEED_BWD else 4096, max_kv, B * mean, B * max_kv)
                for b, m in set(sizes):
                    if b > B or b * m > B * mean:
                        continue
                    if op == kb.OP_GDPA_BWD:
                        rc = lib.kunlun_gdpa_bwd(P, P, P, P, P, P, P, P, P, P, P, b, H, d, 4096, max_kv, b * m, b * max_kv, 0.1, 0, None, kb.BF16,
                                                 P + 16, largest, None)
                    else:
                        rc = lib.kunlun_seed_attn_bwd(P, P, P, P, P, P, P, P, P, P, b, H, d, 65, max_kv, b * max_kv, 0.1, 0, None, kb.BF16, P + 16,
                                                      largest, None)
                    assert rc == kb.ERR_ALIGN, (H, d, op, B, mean, b, m)


@pytest.mark.gpu
@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("tiles", [1, 2, 3, 5, 8])
def test_gradients_with_less_room(oracle, d, tiles):
    """Few examples: one tile per workgroup where the workspace has room, here for chunks of `tiles` tiles of 128 queries."""
    from paper_2602_10016_amd import binding as kb
    H, counts, keys = 2, np.array([1500, 0, 65, 1025, 128]), np.array([32, 5, 0, 17, 1])
    q_off = W.offsets_from_lengths(counts)
    total, B = int(q_off[-1]), len(counts)
    wl = W.make("cfg5", d + tiles, B=B, H=H, d=d, Nq=1500, lengths=("list", keys), scale=0.1)
    rng = np.random.default_rng(tiles)
    q, d_o = (W.round_to_bf16(rng.standard_normal((total, H, d)).astype(np.float32)) for _ in range(2))
    align = lambda n: (n + 255) // 256 * 256
    partial = lambda t: align((total // (128 * t) + B) * H * 2 * 32 * d * 4)
    args = (B, H, d, 1500, 32, total, int(keys.sum()))
    n = kb.workspace_bytes(kb.OP_GDPA_BWD, *args) - partial(1) + partial(tiles)
    memory = torch.full((n + 4096,), 0xEE, dtype=torch.uint8, device="cuda")
    qd, dod, k, v = (to_dev(x, "bf16") for x in (q, d_o, wl.k, wl.v))
    kvo, qo = offsets_dev(wl.kv_offsets), offsets_dev(q_off)
    o, lse = kb.gdpa_fwd(qd, k, v, kvo, 0.1, 0, q_offsets=qo, max_q=1500, max_kv=32)
    out = tuple(torch.full_like(t, float("nan")) for t in (qd, k, v))
    got = kb.gdpa_bwd(qd, k, v, dod, kvo, 0.1, 0, o=o, lse=lse, q_offsets=qo, max_q=1500, max_kv=32, out=out, workspace=memory[:n])
    torch.cuda.synchronize()
    refs = oracle.gdpa_bwd(q, wl.k, wl.v, d_o, wl.kv_offsets, 0.1, 0, q_offsets=q_off, max_q=1500)
    for a, ref, name in zip(got, refs, ("dQ", "dK", "dV")):
        assert_close(to_np(a), ref, TOL["bf16"], f"d={d} tiles={tiles} {name}")
    assert torch.all(memory[n:] == 0xEE)
