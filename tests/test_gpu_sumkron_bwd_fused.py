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
