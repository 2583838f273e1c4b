"""Sliding-window backward in one pass (d = 128, windows that put at most nine key tiles of 32 under a query tile, enough sequences
and heads for every compute unit), against the CPU oracle: windows on both sides of the line, one to nine tiles, reaching to the left,
to the right and to both sides, sequences around the tile size, empty ones among them."""
import numpy as np
import pytest
import torch

from paper_2602_10016_amd import workloads as W
from tests.helpers import TOL, assert_close, offsets_dev, to_dev, to_np
from tests.test_kernel_resources import spilled_vector_registers


def check(oracle, B, H, longest, left, right, seed):
    from paper_2602_10016_amd import binding as kb
    rng = np.random.default_rng(seed)
    lengths = rng.integers(1, longest + 1, size=B)
    special = [0, 1, 31, 32, 33, 63, 64, 65, 255, 256, 257, 287, 288, 289]
    lengths[rng.choice(B, size=len(special) + 1, replace=False)] = [min(x, longest) for x in special] + [longest]
    wl = W.make("cfg3", seed, B=B, H=H, d=128, lengths=("list", lengths))
    q, k, v = (to_dev(x, "bf16") for x in (wl.q, wl.k, wl.v))
    d_o = torch.from_numpy(rng.standard_normal(wl.q.shape).astype(np.float32)).to(torch.bfloat16)
    off = offsets_dev(wl.kv_offsets)
    o, lse = kb.swa_fwd(q, k, v, off, left, right, wl.scale, max_len=longest)
    out = tuple(torch.full_like(t, float("nan")) for t in (q, k, v))
    got = kb.swa_bwd(q, k, v, o, lse, d_o.cuda(), off, left, right, wl.scale, max_len=longest, out=out)
    torch.cuda.synchronize()
    refs = oracle.swa_bwd(wl.q, wl.k, wl.v, d_o.double().numpy(), wl.kv_offsets, left, right, wl.scale)
    for a, ref, name in zip(got, refs, ("dQ", "dK", "dV")):
        assert_close(to_np(a), ref, TOL["bf16"], f"B={B} H={H} window=({left}, {right}) {name}")


# tiles under a query tile: ceil(left / 32) + ceil(right / 32) + 1
@pytest.mark.gpu
@pytest.mark.parametrize("left,right", [(0, 0), (1, 0), (32, 0), (33, 31), (0, 64), (127, 0), (160, 40), (224, 0), (225, 0), (255, 0), (256, 0), (0, 256),
                                        (128, 128), (1, 224), (257, 0), (130, 129)])
def test_swa_backward_one_pass(oracle, left, right):
    check(oracle, 400, 2, 330, left, right, seed=1000 + left + right)


@pytest.mark.gpu
@pytest.mark.parametrize("B,H,longest,left,right", [(520, 1, 256, -1, 0), (264, 2, 96, -1, -1), (700, 1, 40, 5, 7), (75, 8, 1100, 255, 0)])
def test_swa_backward_one_pass_unbounded_short_and_long(oracle, B, H, longest, left, right):
    check(oracle, B, H, longest, left, right, seed=B + longest)


def test_the_one_pass_window_backward_keeps_its_registers(tmp_path):
    """A reload from scratch memory would also count among the vector-memory operations that the kernel's waits number."""
    spilled = spilled_vector_registers("attn_swa_bwd_band_mfma.hip", tmp_path)
    assert len(spilled) == 1 and not any(spilled.values()), spilled
