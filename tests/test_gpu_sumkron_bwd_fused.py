"""SumKronLinear backward in two kernels (T = 32, S in {128, 256}, D in {128, 256, 384}, k <= 8) against the CPU oracle at
the edges of its groups of examples, pairs of factors and ranges, and the first shape beyond it (k = 9)."""
import math

import numpy as np
import pytest
import torch

from paper_2602_10016_amd import workloads as W
from tests.helpers import TOL, assert_close, assert_close_sums, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,S,D,k", [(1, 256, 128, 1), (5, 128, 256, 3), (4, 256, 384, 5), (7, 128, 384, 8), (3, 256, 256, 2),
                                     (9, 128, 128, 4), (70, 256, 128, 7), (3, 128, 128, 9)])
def test_sumkron_backward_fused(oracle, B, S, D, k):
    from paper_2602_10016_amd import binding as kb
    rng = np.random.default_rng(B + 10 * k)
    draw = lambda shape, sigma: W.round_to_bf16(rng.standard_normal(shape, dtype=np.float32) * np.float32(sigma))
    x, dy = draw((B, S, D), 1.0), draw((B, 32, D), 1.0)
    z, w = draw((k, S, 32), 1 / math.sqrt(S)), draw((k, D, D), 1 / math.sqrt(D))
    args = [to_dev(a, "bf16") for a in (x, z, w, dy)]
    got, again = kb.sumkron_bwd(*args), kb.sumkron_bwd(*args)
    torch.cuda.synchronize()
    for a, b, ref, name in zip(got, again, oracle.sumkron_bwd(x, z, w, dy), ("dX", "dZ", "dW")):
        # dZ, dW: sums over the batch of products with a bf16-rounded factor, off by 1.1e-3 of their RMS (tests/helpers.py)
        (assert_close if name == "dX" else assert_close_sums)(to_np(a), ref, TOL["bf16"], f"B={B} S={S} D={D} k={k} {name}")
        assert torch.equal(a, b), f"{name} differs between two runs"


def test_sumkron_backward_in_the_workspace_of_the_five_products(oracle):
    """A workspace too small for the two kernels: the five products run instead."""
    from paper_2602_10016_amd import binding as kb
    rng = np.random.default_rng(4)
    draw = lambda shape, sigma: W.round_to_bf16(rng.standard_normal(shape, dtype=np.float32) * np.float32(sigma))
    B, S, D, k = 2, 256, 128, 3
    x, dy, z, w = draw((B, S, D), 1.0), draw((B, 32, D), 1.0), draw((k, S, 32), 1 / math.sqrt(S)), draw((k, D, D), 1 / math.sqrt(D))
    # two copies of Z, U and G of every example in bf16, one fp32 partial sum of dW; the guard behind it must stay
    need = 2 * (k * S * 32 * 2) + 2 * (B * 32 * k * D * 2) + k * D * D * 4 + 256
    assert need < kb.sumkron_bwd_workspace_bytes(B, S, 32, D, k)
    ws = torch.full((need + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    got = kb.sumkron_bwd(*[to_dev(a, "bf16") for a in (x, z, w, dy)], workspace=ws[:need])
    torch.cuda.synchronize()
    assert torch.all(ws[need:] == 0x5A)
    for a, ref, name in zip(got, oracle.sumkron_bwd(x, z, w, dy), ("dX", "dZ", "dW")):
        (assert_close if name == "dX" else assert_close_sums)(to_np(a), ref, TOL["bf16"], name)


# (B, S, D, k) with several blocks of 32 channels per workgroup in the kernel of G and dX: while groups of four examples times
# the ways to cut the D / 32 blocks stay within 256 workgroups, a workgroup has 2 (B = 86), 4 and 12 of 12 blocks, 2 of 4
# (B = 262), 8 of 8; one, two and four examples per wave (k <= 2, <= 4, above)
@pytest.mark.parametrize("B,S,D,k", [(86, 256, 384, 5), (257, 128, 384, 3), (515, 256, 384, 2), (262, 128, 128, 8), (514, 128, 256, 4),
                                     (518, 256, 128, 1)])
def test_sumkron_backward_fused_over_several_channel_blocks(oracle, B, S, D, k):
    """dX of sampled examples against the oracle; dZ and dW, sums over all examples, against 64-bit torch products."""
    from paper_2602_10016_amd import binding as kb
    gen = torch.Generator(device="cuda").manual_seed(B + k)
    draw = lambda shape, sigma: torch.empty(shape, device="cuda").normal_(0, sigma, generator=gen).to(torch.bfloat16)
    x, dy = draw((B, S, D), 1.0), draw((B, 32, D), 1.0)
    z, w = draw((k, S, 32), 1 / math.sqrt(S)), draw((k, D, D), 1 / math.sqrt(D))
    dx, dz, dw = kb.sumkron_bwd(x, z, w, dy)
    torch.cuda.synchronize()
    some = sorted({0, 1, 3, 4, B // 2, B // 2 + 1, B - 6, B - 3, B - 2, B - 1})
    ref = oracle.sumkron_bwd(*(t.float().cpu().numpy() for t in (x[some], z, w, dy[some])))[0]
    assert_close(to_np(dx[some]), ref, TOL["bf16"], f"B={B} S={S} D={D} k={k} dX")
    assert torch.isfinite(dx).all()
    xd, dyd = x.double(), dy.double()
    for i in range(k):
        u = torch.matmul(z[i].double().t().contiguous(), xd)                                   # [B, 32, D]
        g = torch.matmul(dyd.reshape(B * 32, D), w[i].double().t().contiguous()).reshape(B, 32, D)
        ref_dx = torch.matmul(z[i].double(), g) if i == 0 else ref_dx + torch.matmul(z[i].double(), g)
        ref_dw = torch.matmul(u.reshape(B * 32, D).t().contiguous(), dyd.reshape(B * 32, D))
        ref_dz = torch.matmul(xd.permute(1, 0, 2).reshape(S, B * D), g.permute(0, 2, 1).reshape(B * D, 32))
        assert_close_sums(to_np(dw[i]), ref_dw.cpu().numpy(), TOL["bf16"], f"B={B} S={S} D={D} k={k} dW[{i}]")
        assert_close_sums(to_np(dz[i]), ref_dz.cpu().numpy(), TOL["bf16"], f"B={B} S={S} D={D} k={k} dZ[{i}]")
    assert_close(to_np(dx), ref_dx.cpu().numpy(), TOL["bf16"], f"B={B} S={S} D={D} k={k} dX, all examples")
