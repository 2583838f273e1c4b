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
