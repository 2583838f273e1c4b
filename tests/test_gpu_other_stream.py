"""Calls on a stream that is not the current one, without a workspace: the workspace that the call allocates is not handed out
again before that stream has reached the call's kernels."""
import pytest
import torch

from paper_2602_10016_amd import binding as kb

pytestmark = pytest.mark.gpu


class PythonOnly:
    def __getattr__(self, name):
        return lambda *args: None


@pytest.mark.parametrize("native", [True, False])
def test_a_workspace_is_kept_until_its_stream_has_used_it(monkeypatch, native):
    if not native:
        monkeypatch.setattr(kb, "_native", PythonOnly())
    gen = torch.Generator(device="cuda").manual_seed(0)
    r = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0, 0.1, generator=gen)
    x, z, w = r(8, 256, 384), r(8, 256, 32), r(8, 384, 384)
    want = kb.sumkron_fwd(x, z, w)
    nbytes = kb.raw().kunlun_sumkron_batch_bytes(8, 256, 32, 384, 8, kb.BF16)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    probe = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    address = probe.data_ptr()
    del probe  # the only free block of this size: the call's workspace
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        torch.cuda._sleep(100_000_000)  # tens of milliseconds ahead of the call
    got = kb.sumkron_fwd(x, z, w, stream=stream)
    assert not stream.query(), "the stream was to be busy still"
    other = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")  # on the current stream, at once
    assert other.data_ptr() != address
    torch.cuda.synchronize()
    assert torch.equal(got, want)


def test_the_count_of_violations_is_read_behind_its_kernel():
    offsets = torch.tensor([0, 5, 3, 9], dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        torch.cuda._sleep(100_000_000)
    assert kb.check_offsets(offsets, 9, 5, stream=stream) > 0
