"""Query-tiled sliding-window forward whose tiles are issued in several runs per XCD (d = 128, windows of up to 128 rows over long
sequences, 1025..1792 tiles times heads) and just outside that rule, against the CPU oracle: every tile is taken once, whatever
the number of heads and the remainder of the last run."""
import numpy as np
import pytest
import torch

from paper_2602_10016_amd import workloads as W
from tests.helpers import TOL, assert_close, assert_lse_close, offsets_dev, to_dev, to_np

pytestmark = pytest.mark.gpu


# (half a tile per example more than the rows fill) times heads: 1040, 1024 (in order), 1792, 1800 (in order), 1066 (short sequences,
# in order), 1208 with one head (32 runs), 1056
@pytest.mark.parametrize("B,H,mean,left,right", [(13, 8, 1212, 3, 0), (13, 8, 1199, 64, 64), (22, 8, 1240, 127, 1), (22, 8, 1247, 0, 0), (120, 2, 505, 9, 3),
                                                 (101, 1, 1467, 5, 5), (24, 8, 640, 128, 0)])
def test_forward(oracle, B, H, mean, left, right):
    from paper_2602_10016_amd import binding as kb
    rng = np.random.default_rng(B + H)
    lengths = rng.integers(mean * 7 // 10, mean * 13 // 10, size=B)
    lengths[[0, B // 2]] = [1, 129]
    lengths[1:B // 2] += (B * mean - lengths.sum()) // (B // 2 - 1)
    lengths[-1] += B * mean - lengths.sum()
    wl = W.make("cfg3", B, B=B, H=H, d=128, lengths=("list", lengths))
    q, k, v = (to_dev(x, "bf16") for x in (wl.q, wl.k, wl.v))
    o = torch.full_like(q, float("nan"))
    lse = torch.full((H, q.shape[0]), float("nan"), dtype=torch.float32, device="cuda")
    kb.swa_fwd(q, k, v, offsets_dev(wl.kv_offsets), left, right, wl.scale, max_len=int(lengths.max()), out=o, lse=lse)
    torch.cuda.synchronize()
    o_ref, lse_ref = oracle.swa_fwd(wl.q, wl.k, wl.v, wl.kv_offsets, left, right, wl.scale)
    assert_close(to_np(o), o_ref, TOL["bf16"], f"B={B} H={H} window=({left}, {right})")
    assert_lse_close(to_np(lse), lse_ref, 1e-2)
