"""The seed gradient at the edges of its summation groups (32 examples; one group is summed and rounded in one launch): bit for bit the
sum of the per-example query gradients in the documented order, so no tolerance."""
import numpy as np
import pytest
import torch

from paper_2602_10016_amd import binding as kb
from tests.helpers import offsets_dev

pytestmark = pytest.mark.gpu


# (3 seeds of 24 channels: fewer elements than a workgroup has threads, served by the generic kernels)
@pytest.mark.parametrize("dtype,H,d,n_seeds", [("bf16", 2, 32, 8), ("bf16", 1, 24, 3), ("fp32", 1, 32, 5), ("fp32", 3, 24, 3)])
@pytest.mark.parametrize("B", [1, 31, 32, 33, 64, 65])
def test_seed_gradient_is_the_sum_in_order(B, dtype, H, d, n_seeds):
    check(B, dtype, H, d, n_seeds)


# rows of 3.7, 4.1 and 33 MiB in bf16, 4.1 in fp32 and 4.3 of the generic kernels: read with streaming loads above 4 MiB
@pytest.mark.parametrize("B,dtype,H,d,n_seeds", [(34, "bf16", 4, 64, 224), (37, "bf16", 4, 64, 225), (65, "bf16", 8, 128, 256), (33, "fp32", 4, 64, 128),
                                                 (36, "bf16", 1, 24, 2600)])
def test_seed_gradient_of_many_rows(B, dtype, H, d, n_seeds):
    check(B, dtype, H, d, n_seeds)


def check(B, dtype, H, d, n_seeds):
    rng = np.random.default_rng(B * 100 + d)
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    off = np.concatenate([[0], np.cumsum(rng.integers(0, 70, size=B))]).astype(np.int32)
    off[-1] = max(off[-1], off[-2] + 1)
    normal = lambda *shape: torch.from_numpy(rng.standard_normal(shape, dtype=np.float32)).to(t).cuda()
    e, k, v = normal(n_seeds, H, d), normal(int(off[-1]), H, d), normal(int(off[-1]), H, d)
    d_o, kvo, longest = normal(B * n_seeds, H, d), offsets_dev(off), int(np.diff(off).max())
    o, lse = kb.seed_attn_fwd(e, k, v, kvo, 0.2, 0, max_kv=longest)
    out = tuple(torch.full_like(x, float("nan")) for x in (e, k, v))
    d_e = kb.seed_attn_bwd(e, k, v, d_o, kvo, 0.2, 0, o=o, lse=lse, max_kv=longest, out=out)[0]
    q = e.repeat(B, 1, 1).contiguous()
    o2, lse2 = kb.gdpa_fwd(q, k, v, kvo, 0.2, 0, max_q=n_seeds, max_kv=longest)
    dq = kb.gdpa_bwd(q, k, v, d_o, kvo, 0.2, 0, o=o2, lse=lse2, max_q=n_seeds, max_kv=longest)[0]
    rows = dq.float().view(B, -1)
    total = torch.zeros_like(rows[0])
    for g0 in range(0, B, 32):
        part = torch.zeros_like(rows[0])
        for b in range(g0, min(B, g0 + 32)):
            part = part + rows[b]
        total = total + part
    torch.cuda.synchronize()
    assert torch.equal(d_e.view(-1), total.to(t))
