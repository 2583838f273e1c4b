"""Sliding-window backward in two passes (at d = 128 the launches that the one-pass kernel is not asked for: few items, uneven lengths, or windows
of more than nine key tiles) in workgroups of two waves (64 rows; bounded windows reaching fewer than 704 rows at d = 64 and 448 at
d = 128, for half to one tile of 128 rows per compute unit 320 and 200, 112 for sequences of up to 256 rows) and of four (wider or unbounded windows, d = 32), against
the CPU oracle: sequences around 32, 64 and 128 rows, windows on both sides of the lines."""
import numpy as np
import pytest
import torch

from paper_2602_10016_amd import workloads as W
from tests.helpers import TOL, assert_close, offsets_dev, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("left,right", [(0, 0), (31, 0), (32, 32), (255, 0), (383, 0), (384, 0), (0, 383), (200, 184), (-1, 5)])
def test_swa_backward_around_the_two_wave_rule(oracle, d, left, right):
    from paper_2602_10016_amd import binding as kb
    lengths = np.array([1, 0, 31, 32, 33, 63, 64, 65, 127, 128, 129, 191, 193, 450])
    wl = W.make("cfg3", d + left, B=len(lengths), H=2, d=d, lengths=("list", lengths))
    q, k, v = (to_dev(x, "bf16") for x in (wl.q, wl.k, wl.v))
    rng = np.random.default_rng(d)
    d_o = torch.from_numpy(rng.standard_normal(wl.q.shape).astype(np.float32)).to(torch.bfloat16)
    off = offsets_dev(wl.kv_offsets)
    longest = int(lengths.max())
    o, lse = kb.swa_fwd(q, k, v, off, left, right, wl.scale, max_len=longest)
    out = tuple(torch.full_like(t, float("nan")) for t in (q, k, v))
    got = kb.swa_bwd(q, k, v, o, lse, d_o.cuda(), off, left, right, wl.scale, max_len=longest, out=out)
    torch.cuda.synchronize()
    refs = oracle.swa_bwd(wl.q, wl.k, wl.v, d_o.double().numpy(), wl.kv_offsets, left, right, wl.scale)
    for a, ref, name in zip(got, refs, ("dQ", "dK", "dV")):
        assert_close(to_np(a), ref, TOL["bf16"], f"d={d} window=({left}, {right}) {name}")


# 4 sequences of up to 1100 rows, 2 heads (40 tiles), and 20 of up to 900, 2 heads (about 240 tiles: one per compute unit)
@pytest.mark.parametrize("d,B,longest,left,right", [(64, 4, 1100, 703, 0), (64, 4, 1100, 352, 352), (128, 4, 1100, 447, 0), (128, 4, 1100, 0, 448),
                                                    (64, 20, 900, 319, 0), (64, 20, 900, 160, 160), (128, 20, 900, 199, 0), (128, 20, 900, 100, 100),
                                                    (64, 70, 256, 111, 0), (128, 70, 256, 112, 0)])
def test_swa_backward_around_the_lines_by_reach_and_size(oracle, d, B, longest, left, right):
    from paper_2602_10016_amd import binding as kb
    rng = np.random.default_rng(d + B)
    lengths = rng.integers(longest // 2, longest + 1, size=B)
    lengths[0] = longest
    wl = W.make("cfg3", d + left, B=B, H=2, d=d, lengths=("list", lengths))
    q, k, v = (to_dev(x, "bf16") for x in (wl.q, wl.k, wl.v))
    d_o = torch.from_numpy(rng.standard_normal(wl.q.shape).astype(np.float32)).to(torch.bfloat16)
    off = offsets_dev(wl.kv_offsets)
    o, lse = kb.swa_fwd(q, k, v, off, left, right, wl.scale, max_len=longest)
    out = tuple(torch.full_like(t, float("nan")) for t in (q, k, v))
    got = kb.swa_bwd(q, k, v, o, lse, d_o.cuda(), off, left, right, wl.scale, max_len=longest, out=out)
    torch.cuda.synchronize()
    refs = oracle.swa_bwd(wl.q, wl.k, wl.v, d_o.double().numpy(), wl.kv_offsets, left, right, wl.scale)
    for a, ref, name in zip(got, refs, ("dQ", "dK", "dV")):
        assert_close(to_np(a), ref, TOL["bf16"], f"d={d} B={B} window=({left}, {right}) {name}")
