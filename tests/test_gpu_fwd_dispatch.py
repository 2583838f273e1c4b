"""Forward launches that share the key tiles of an item among waves (few items: 33..64 queries as two blocks, eight waves
for histories beyond 1024 keys) and those on either side of the rule, against the CPU oracle; and the short form of GELU
for small scores against the function itself, on both sides of its range."""
import math

import numpy as np
import pytest
import torch

from paper_2602_10016_amd import workloads as W
from tests.helpers import TOL, assert_close, assert_lse_close, offsets_dev, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("n", [1, 32, 33, 64])
@pytest.mark.parametrize("longest", [1024, 1025, 1100])
@pytest.mark.parametrize("act", [0, 3])
def test_key_split_forward(oracle, d, n, longest, act):
    from paper_2602_10016_amd import binding as kb
    lengths = np.array([longest, 0, 1, 31, 33, 200, 255, 257, 32])
    B, H = len(lengths), 2
    wl = W.make("cfg5", d + n, B=B, H=H, d=d, Nq=n, lengths=("list", lengths), scale=1 / math.sqrt(d) if act == 0 else 1 / longest)
    counts = np.array([n, n, 1, n, n, max(1, n - 1), n, 0, n])
    q_off = W.offsets_from_lengths(counts)
    q = wl.q[:q_off[-1]]
    qd, k, v = (to_dev(x, "bf16") for x in (q, wl.k, wl.v))
    o, lse = kb.gdpa_fwd(qd, k, v, offsets_dev(wl.kv_offsets), wl.scale, act, q_offsets=offsets_dev(q_off), max_q=n, max_kv=longest)
    torch.cuda.synchronize()
    o_ref, lse_ref = oracle.gdpa_fwd(q, wl.k, wl.v, wl.kv_offsets, wl.scale, act, q_offsets=q_off, max_q=n)
    assert_close(to_np(o), o_ref, TOL["bf16"], f"d={d} n={n} longest={longest} act={act}")
    if act == 0:
        assert_lse_close(to_np(lse), lse_ref, 1e-2)


# The largest launch that shares key tiles among four waves, for GELU (act 3) and for the others; at d = 128 with up to 32
# queries the line between four and two.
@pytest.mark.parametrize("d,n,blocks,act", [(128, 64, 512, 3), (64, 64, 1024, 3), (32, 64, 4096, 3), (128, 64, 256, 0), (64, 64, 512, 0),
                                            (32, 64, 768, 0), (64, 20, 2048, 0), (64, 20, 2048, 3), (128, 20, 256, 0), (128, 20, 2048, 0)])
@pytest.mark.parametrize("above", [False, True])
def test_both_sides_of_the_few_items_rule(oracle, d, n, blocks, act, above):
    """`blocks` = examples x heads x blocks of 32 queries is the largest launch that shares key tiles among waves."""
    from paper_2602_10016_amd import binding as kb
    H = 4
    B = blocks // H // ((n + 31) // 32) + (1 if above else 0)
    wl = W.make("cfg5", blocks, B=B, H=H, d=d, Nq=n, lengths=("uniform", 0, 50), scale=0.1)
    q, k, v = (to_dev(x, "bf16") for x in (wl.q, wl.k, wl.v))
    o, _ = kb.gdpa_fwd(q, k, v, offsets_dev(wl.kv_offsets), wl.scale, act, max_q=n, max_kv=50)
    torch.cuda.synchronize()
    o_ref, _ = oracle.gdpa_fwd(wl.q, wl.k, wl.v, wl.kv_offsets, wl.scale, act, max_q=n)
    assert_close(to_np(o), o_ref, TOL["bf16"], f"d={d} n={n} B={B} act={act}")


@pytest.mark.parametrize("d,n,act", [(32, 20, 0), (32, 64, 3), (64, 20, 3), (64, 20, 0), (64, 64, 0), (128, 20, 0), (128, 40, 3)])
def test_key_split_of_sorted_items(oracle, d, n, act):
    """Long histories above one item per compute unit: eight waves share the key tiles of items in sorted order."""
    from paper_2602_10016_amd import binding as kb
    B, H = 100, 4
    rng = np.random.default_rng(d + n)
    lengths = rng.integers(0, 60, size=B)
    lengths[[5, 50, 99]] = [1100, 300, 700]
    wl = W.make("cfg5", d + n, B=B, H=H, d=d, Nq=n, lengths=("list", lengths), scale=1 / math.sqrt(d) if act == 0 else 1 / 1100)
    q, k, v = (to_dev(x, "bf16") for x in (wl.q, wl.k, wl.v))
    ws = torch.full((kb.workspace_bytes(kb.OP_GDPA_FWD, B, H, d, n, 1100, B * n, k.shape[0]),), 0xEE, dtype=torch.uint8, device="cuda")
    o, lse = kb.gdpa_fwd(q, k, v, offsets_dev(wl.kv_offsets), wl.scale, act, max_q=n, max_kv=1100, workspace=ws)
    torch.cuda.synchronize()
    order = ws[256:256 + 4 * B].cpu().numpy().view(np.int32)
    assert order[0] == 5 and np.array_equal(np.sort(order), np.arange(B)), "the items were not sorted"
    o_ref, lse_ref = oracle.gdpa_fwd(wl.q, wl.k, wl.v, wl.kv_offsets, wl.scale, act, max_q=n)
    assert_close(to_np(o), o_ref, TOL["bf16"], f"d={d} n={n} act={act}")
    if act == 0:
        assert_lse_close(to_np(lse), lse_ref, 1e-2)


@pytest.mark.parametrize("scale", [1.0, 1 / 32])
def test_gelu_of_small_and_large_scores_is_the_function_rounded_once(scale):
    """One key e_0, value e_0, queries (x / scale) e_0: O[0] = bf16(gelu(x)) and, with dO = e_0, dQ[0] = bf16(gelu'(x)) scale.
    With the small scale, examples whose scores all lie inside [-1, 1] take the short form, the others (also with one score
    just outside) the general."""
    from paper_2602_10016_amd import binding as kb
    n, d = 64, 32
    inside = torch.linspace(-1, 1, 40 * n).view(40, n)
    wide = torch.linspace(-6, 6, 40 * n).view(40, n)
    edge = inside.clone()
    edge[:, 7] = 1.0078125  # the bf16 value after 1
    x = torch.cat([inside, wide, edge]).to(torch.bfloat16).cuda()
    B = x.shape[0]
    q = torch.zeros((B * n, 1, d), dtype=torch.bfloat16, device="cuda")
    q[:, 0, 0] = x.reshape(-1) / scale  # a power of two: exact
    k = torch.zeros((B, 1, d), dtype=torch.bfloat16, device="cuda")
    k[:, 0, 0] = 1
    d_o = torch.zeros_like(q)
    d_o[:, 0, 0] = 1
    off = torch.arange(B + 1, dtype=torch.int32, device="cuda")
    o, _ = kb.gdpa_fwd(q, k, k.clone(), off, scale, kb.ACT_GELU, max_q=n, max_kv=1)
    dq, _, _ = kb.gdpa_bwd(q, k, k.clone(), d_o, off, scale, kb.ACT_GELU, max_q=n, max_kv=1)
    torch.cuda.synchronize()
    t = x.double().reshape(-1)
    cdf = 0.5 * (1 + torch.erf(t / math.sqrt(2)))
    for got, want in ((o[:, 0, 0].double(), t * cdf), (dq[:, 0, 0].double() / scale, cdf + t * torch.exp(-t * t / 2) / math.sqrt(2 * math.pi))):
        # half a unit in the last place of bf16 (2^-9 of the value, rounded up to the next power of two: 2^-8), plus the
        # stated error 7.5e-8 of the general form's cdf times |x| <= 6 and fp32 rounding
        assert torch.all((got - want).abs() <= 2.0 ** -8 * want.abs() + 6e-7)
        assert torch.all((got - want).abs() <= 2.0 ** -9 * 2.0 ** torch.ceil(torch.log2(want.abs().clamp_min(1e-30))) + 6e-7)
