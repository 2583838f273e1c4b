"""More than 64 dense queries per example over uneven histories: query tiles in the order of the histories' lengths (more than 512
(example, head, tile) workgroups, counted with the examples rounded up to eight; histories beyond 256 keys, the longest at least 1.25 times the
mean), on both sides of that rule, against the CPU oracle."""
import math

import numpy as np
import pytest
import torch

from paper_2602_10016_amd import workloads as W
from tests.helpers import TOL, assert_close, offsets_dev, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,d,n,longest,act", [(65, 4, 128, 130, 600, 0), (64, 4, 128, 129, 600, 3), (67, 8, 64, 65, 500, 0), (33, 2, 64, 1000, 300, 0),
                                                 (131, 4, 32, 128, 700, 3), (17, 8, 32, 257, 257, 0), (90, 4, 64, 200, 256, 0)])
def test_dense_queries_over_uneven_histories(oracle, B, H, d, n, longest, act):
    from paper_2602_10016_amd import binding as kb
    rng = np.random.default_rng(B + n)
    lengths = np.minimum(longest, np.round(np.exp(rng.normal(math.log(longest / 4), 0.8, size=B)))).astype(np.int64)
    lengths[:4] = [0, 1, 33, longest]
    rng.shuffle(lengths)
    # (element-wise score functions with the 1 / tau scaling: at 1 / sqrt(d) a dQ element of 600 keys is a sum of terms of about 0.17 with
    # rounded factors, whose error of 2^-9 / sqrt(3) * 0.17 * sqrt(600) = 0.005 in the mean square exceeds 0.02 among millions of elements)
    wl = W.make("cfg2", B, B=B, H=H, d=d, Nq=n, lengths=("list", lengths), scale=1.0 / math.sqrt(d) if act == 0 else 1.0 / longest)
    q, k, v = (to_dev(x, "bf16") for x in (wl.q, wl.k, wl.v))
    d_o = torch.from_numpy(rng.standard_normal(wl.q.shape).astype(np.float32)).to(torch.bfloat16)
    off = offsets_dev(wl.kv_offsets)
    o, lse = kb.gdpa_fwd(q, k, v, off, wl.scale, act, max_q=n, max_kv=longest, out=torch.full_like(q, float("nan")))
    out = tuple(torch.full_like(t, float("nan")) for t in (q, k, v))
    got = kb.gdpa_bwd(q, k, v, d_o.cuda(), off, wl.scale, act, o=o, lse=lse, max_q=n, max_kv=longest, out=out)
    torch.cuda.synchronize()
    o_ref, _ = oracle.gdpa_fwd(wl.q, wl.k, wl.v, wl.kv_offsets, wl.scale, act, max_q=n)
    refs = oracle.gdpa_bwd(wl.q, wl.k, wl.v, d_o.double().numpy(), wl.kv_offsets, wl.scale, act, max_q=n)
    for a, ref, name in zip((o, *got), (o_ref, *refs), ("O", "dQ", "dK", "dV")):
        assert_close(to_np(a), ref, TOL["bf16"], f"B={B} H={H} d={d} n={n} act={act} {name}")


# one tile per example: the forward at d = 128 over up to 352 keys leaves more than 4608 of them (256 compute units) in the order of the tables where
# the longest history is at most 2.5 times the mean, and more than 7168 of any histories; a part of the batch is sorted, with the same bits
@pytest.mark.parametrize("B,d,n,shortest,longest,tables", [(5000, 128, 70, 1, 280, True), (5000, 128, 70, 150, 352, True), (5000, 64, 70, 1, 280, False), (2504, 128, 130, 1, 280, False),
                                                           (5000, 128, 65, 1, 360, False), (4600, 128, 65, 1, 280, False), (7400, 128, 65, -300, 300, True),
                                                           (7000, 128, 65, -300, 300, False)])
def test_many_short_histories_keep_the_tables(B, d, n, shortest, longest, tables):
    from paper_2602_10016_amd import binding as kb
    rng = np.random.default_rng(B + n)
    lengths = np.maximum(1, rng.integers(shortest, longest + 1, size=B))
    some = 64 * (8 if n <= 128 else 4) + 8  # more than 512 workgroups
    lengths[[0, some - 1]] = longest
    offsets = np.concatenate([[0], np.cumsum(lengths)])
    normal = lambda rows: torch.from_numpy(rng.standard_normal((rows, 1, d), dtype=np.float32)).to(torch.bfloat16).cuda()
    q, k, v = normal(B * n), normal(int(offsets[-1])), normal(int(offsets[-1]))

    def forward(examples):
        keys = int(offsets[examples])
        ws = torch.zeros(kb.workspace_bytes(kb.OP_GDPA_FWD, examples, 1, d, n, longest, examples * n, keys), dtype=torch.uint8, device="cuda")
        o, _ = kb.gdpa_fwd(q[:examples * n], k[:keys], v[:keys], offsets_dev(offsets[:examples + 1]), d ** -0.5, 0, max_q=n, max_kv=longest, workspace=ws)
        listed = ws[256:256 + 4 * examples].view(torch.int32).cpu()  # the first tile of every example, or the examples, longest history first
        return o, torch.equal(listed, torch.arange(examples, dtype=torch.int32) * ((n + 127) // 128))

    (o, by_tables), (part, part_by_tables) = forward(B), forward(some)
    assert by_tables == tables and not part_by_tables
    assert torch.equal(o[:some * n].view(torch.int16), part.view(torch.int16))
