"""SumKronLinear forward in ranges of channel blocks (batches that would leave compute units empty): group tails, every number
of ranges, and workspaces with room for all, some or none of the partial sums, against the CPU oracle; nothing is written
behind the workspace that a call is told of."""
import numpy as np
import pytest
import torch

from paper_2602_10016_amd import workloads as W
from tests.helpers import TOL, assert_close, to_dev, to_np

pytestmark = pytest.mark.gpu


def align(n):
    return (n + 255) // 256 * 256


# groups of four examples x ranges <= 256, ranges divide D / 32 (12, 8 or 4)
@pytest.mark.parametrize("B,S,D,k", [(1, 256, 384, 8), (5, 256, 384, 3), (87, 128, 384, 2), (130, 128, 256, 1), (260, 128, 128, 2), (515, 128, 128, 2)])
@pytest.mark.parametrize("room", ["all", "two ranges", "none"])
def test_split_forward(oracle, B, S, D, k, room):
    from paper_2602_10016_amd import binding as kb
    T = 32
    rng = np.random.default_rng(B + S + D)
    bf = lambda shape, s: W.round_to_bf16((rng.standard_normal(shape) * s).astype(np.float32))
    x, z, w = bf((B, S, D), 1.0), bf((k, S, T), S ** -0.5), bf((k, D, D), D ** -0.5)
    need = align(k * T * S * 2) + align(k * D * D * 2) + 256
    nbytes = {"all": kb.sumkron_workspace_bytes(B, S, T, D, k), "two ranges": need + 2 * B * T * D * 4, "none": need}[room]
    memory = torch.full((nbytes + 4096,), 0xEE, dtype=torch.uint8, device="cuda")
    y = torch.full((B, T, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    got = kb.sumkron_fwd(*(to_dev(a, "bf16") for a in (x, z, w)), out=y, workspace=memory[:nbytes])
    torch.cuda.synchronize()
    assert_close(to_np(got), oracle.sumkron_fwd(x, z, w), TOL["bf16"], f"B={B} S={S} D={D} k={k} {room}")
    assert torch.all(memory[nbytes:] == 0xEE)


def test_a_call_allocates_for_its_own_batch():
    """B = 1024 cuts no ranges: the prepared copies of Z and W and the result, not the partial sums of a smaller batch; B = 8 has
    room for its twelve ranges."""
    from paper_2602_10016_amd import binding as kb
    S, T, D, k = 256, 32, 384, 8
    need = align(k * T * S * 2) + align(k * D * D * 2) + 256
    z, w = (torch.zeros(s, dtype=torch.bfloat16, device="cuda") for s in ((k, S, T), (k, D, D)))
    for B, partial in ((1024, 0), (8, 12 * 8 * T * D * 4)):
        x = torch.zeros((B, S, D), dtype=torch.bfloat16, device="cuda")
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        before = torch.cuda.memory_allocated()
        torch.cuda.reset_peak_memory_stats()
        y = kb.sumkron_fwd(x, z, w)
        taken = torch.cuda.max_memory_allocated() - before - y.numel() * 2
        assert need + partial <= taken <= need + partial + 4096, (B, taken, need + partial)
    assert kb.raw().kunlun_sumkron_batch_bytes(0, 0, 1, 8, 1, kb.BF16) == 0
    for B in (1, 5, 80, 170, 255, 256, 300, 512, 1024, 5000):
        assert kb.raw().kunlun_sumkron_batch_bytes(B, S, T, D, k, kb.BF16) <= kb.sumkron_workspace_bytes(B, S, T, D, k)
        assert kb.raw().kunlun_sumkron_batch_bytes(B, S, 16, D, k, kb.BF16) == kb.sumkron_workspace_bytes(B, S, 16, D, k)
