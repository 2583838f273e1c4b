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


def prepared(kind, lengths, H, left, right):
    """Inputs and the forward's results; q[..., 0] = 1 under "masked keys", so that K[key, h, 0] = -inf masks a key."""
    from paper_2602_10016_amd import binding as kb
    rng = np.random.default_rng(left + 3 * right + len(kind))
    total = int(lengths.sum())
    q, k, v, d_o = (W.round_to_bf16(rng.standard_normal((total, H, 128), dtype=np.float32) * (4 if kind == "large scores" else 0.5)) for _ in range(4))
    if kind == "masked keys":
        q[..., 0] = 1
        k[rng.random(k.shape[:2]) < 0.3, 0] = -np.inf
        k[rng.random(k.shape[0]) < 0.002] = -np.inf  # (in every head)
    scale = {"tiny scale": 1e-7, "negative scale": -0.2}.get(kind, 128 ** -0.5)
    off = W.offsets_from_lengths(lengths)
    dev = [to_dev(x, "bf16") for x in (q, k, v)]
    o, lse = kb.swa_fwd(*dev, offsets_dev(off), left, right, scale, max_len=int(lengths.max()))
    return off, scale, (*dev, o, lse, to_dev(d_o, "bf16"))


def bits(t):
    return torch.where(t.isnan(), torch.full_like(t, float("nan")), t).view(torch.int16)


# 512 items: one pass; a sequence by itself has too few of them and goes through the two-pass kernels
@pytest.mark.gpu
@pytest.mark.parametrize("kind,left,right", [("ordinary", 255, 0), ("ordinary", 128, 128), ("ordinary", 40, 0), ("ordinary", 0, 0), ("ordinary", 100, 31),
                                             ("tiny scale", 255, 0), ("negative scale", 100, 31), ("large scores", 255, 0), ("large scores", 20, 20),
                                             ("masked keys", 255, 0), ("masked keys", 60, 60)])
def test_one_pass_and_two_passes_give_the_same_bits(kind, left, right):
    from paper_2602_10016_amd import binding as kb
    B, H = 128, 4
    lengths = np.random.default_rng(left).integers(200, 331, size=B)
    some = [0, 1, 17, 40, 63, 90, B - 1]
    lengths[some] = [330, 1, 31, 33, 288, 289, 64]
    off, scale, (q, k, v, o, lse, d_o) = prepared(kind, lengths, H, left, right)
    total, order_end = int(off[-1]), 256 + ((B + 1) * 4 + 255) // 256 * 256
    ws = torch.full((kb.workspace_bytes(kb.OP_SWA_BWD, B, H, 128, 330, 330, total, total),), 0xEE, dtype=torch.uint8, device="cuda")
    got = kb.swa_bwd(q, k, v, o, lse, d_o, offsets_dev(off), left, right, scale, max_len=330, workspace=ws)
    assert torch.all(ws[order_end:] == 0xEE), "the two passes leave delta here: the one-pass kernel did not run"
    for b in some:
        n, at = int(lengths[b]), slice(int(off[b]), int(off[b + 1]))
        ws = torch.full((kb.workspace_bytes(kb.OP_SWA_BWD, 1, H, 128, n, n, n, n),), 0xEE, dtype=torch.uint8, device="cuda")
        own = kb.swa_bwd(*(x[at].contiguous() for x in (q, k, v, o)), lse[:, at].contiguous(), d_o[at].contiguous(), offsets_dev(np.array([0, n])),
                         left, right, scale, max_len=n, workspace=ws)
        assert torch.any(ws[512:] != 0xEE), "the one-pass kernel ran"
        for a, ref, name in zip(got, own, ("dQ", "dK", "dV")):
            assert torch.equal(bits(a[at]), bits(ref)), f"{kind} window=({left}, {right}) sequence of {n} rows {name}"


# 1384 items of up to 22 rows: the two passes by offsets, in workgroups of two waves; 2400 of 100 to 120 rows and 2080 of 73 to 91: two
# passes by tables; short sequences in one pass: few and many items, up to 32 rows, and beside one of 130 rows.  Windows to the right over short
# sequences, whose first steps only take up key tiles: 19 items per compute unit of four tiles, of two, six of four tiles, and few of
# three in two passes; seven of two tiles and 30 of two in one
@pytest.mark.gpu
@pytest.mark.parametrize("B,H,lo,hi,left,right,one_pass", [(346, 4, 1, 22, 20, 20, False), (600, 4, 100, 120, 63, 0, False), (520, 4, 73, 91, 90, 90, False),
                                                           (256, 2, 100, 120, 255, 0, True), (1536, 4, 100, 120, 63, 0, True), (4096, 1, 8, 32, 31, 0, True),
                                                           (600, 4, 100, 130, 63, 0, True), (1659, 3, 91, 114, -1, 122, False), (674, 8, 36, 42, -1, 1, False),
                                                           (194, 8, 98, 122, 40, 20, False), (300, 2, 130, 160, 20, 120, False), (450, 4, 40, 60, 20, 20, True),
                                                           (3840, 2, 56, 62, 40, 40, True)])
def test_which_short_sequences_take_one_pass(B, H, lo, hi, left, right, one_pass):
    from paper_2602_10016_amd import binding as kb
    lengths = np.random.default_rng(B).integers(lo, hi + 1, size=B)
    lengths[B // 2] = hi
    off, scale, (q, k, v, o, lse, d_o) = prepared("ordinary", lengths, H, left, right)
    total, order_end = int(off[-1]), 256 + ((B + 1) * 4 + 255) // 256 * 256
    ws = torch.full((kb.workspace_bytes(kb.OP_SWA_BWD, B, H, 128, hi, hi, total, total),), 0xEE, dtype=torch.uint8, device="cuda")
    kb.swa_bwd(q, k, v, o, lse, d_o, offsets_dev(off), left, right, scale, max_len=hi, workspace=ws)
    assert bool(torch.all(ws[order_end:] == 0xEE)) == one_pass


# 8.4 million sequences, most of them empty: as workgroups of 512 threads more work items than one launch may have
@pytest.mark.gpu
def test_more_sequences_than_one_pass_can_launch():
    from paper_2602_10016_amd import binding as kb
    B, rows = 8_400_000, 100_000
    rng = np.random.default_rng(0)
    lengths = np.zeros(B, dtype=np.int64)
    lengths[rng.choice(B, size=rows, replace=False)] = 1
    q, k, v, d_o = (to_dev(W.round_to_bf16(rng.standard_normal((rows, 1, 128), dtype=np.float32)), "bf16") for _ in range(4))
    lse = ((q.float() * k.float()).sum(dim=2) * 0.1).T.contiguous()
    dq, dk, dv = kb.swa_bwd(q, k, v, v.clone(), lse, d_o, offsets_dev(W.offsets_from_lengths(lengths)), 31, 0, 0.1, max_len=1)
    torch.cuda.synchronize()
    # one key each: P = 1 up to the rounding of a score of a few units in 32 bits, dS = 0 up to that of dP
    assert torch.allclose(dv.float(), d_o.float(), rtol=1e-2, atol=0) and max(float(t.abs().max()) for t in (dq, dk)) < 1e-3


def test_the_one_pass_window_backward_keeps_its_registers(tmp_path):
    """A reload from scratch memory would also count among the vector-memory operations that the kernel's waits number."""
    spilled = spilled_vector_registers("attn_swa_bwd_band_mfma.hip", tmp_path)
    assert len(spilled) == 1 and not any(spilled.values()), spilled
