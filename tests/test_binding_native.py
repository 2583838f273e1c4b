"""The native marshalling of the entry points (csrc/torch_call.cpp) against the Python code behind it: what it accepts gives
the same results, and what it does not accept it leaves to that code (None), without touching anything."""
import enum

import numpy as np
import pytest
import torch

from paper_2602_10016_amd import binding as kb

H, D, N, B, T = 2, 64, 8, 3, 40


def arguments(device, dtype=torch.bfloat16):
    gen = torch.Generator().manual_seed(0)
    r = lambda *s: torch.randn(*s, generator=gen).to(dtype).to(device)
    i = lambda *x: torch.tensor(x, dtype=torch.int32, device=device)
    return dict(q=r(B * N, H, D), seed=r(N, H, D), k=r(T, H, D), v=r(T, H, D), d_o=r(B * N, H, D), d_t=r(T, H, D), off=i(0, 15, 15, T),
                qo=i(0, N, 2 * N, 3 * N), x=r(B, 64, 128), z=r(2, 64, 32), w=r(2, 128, 128), dy=r(B, 32, 128))


def calls(a, act=kb.ACT_SOFTMAX, scale=0.1, n=N, longest=25, stream=None):
    """Every entry point once, outputs allocated by the call."""
    o, lse = kb.gdpa_fwd(a["q"], a["k"], a["v"], a["off"], scale, act, max_q=n, max_kv=longest, stream=stream)
    so, slse = kb.seed_attn_fwd(a["seed"], a["k"], a["v"], a["off"], scale, act, max_kv=longest, stream=stream)
    wo, wlse = kb.swa_fwd(a["k"], a["k"], a["v"], a["off"], 7, 2, scale, max_len=longest, stream=stream)
    return [o, lse, so, slse, wo, wlse,
            *kb.gdpa_fwd(a["q"], a["k"], a["v"], a["off"], scale, act, q_offsets=a["qo"], max_q=n, max_kv=longest, stream=stream),
            *kb.gdpa_bwd(a["q"], a["k"], a["v"], a["d_o"], a["off"], scale, act, o=o, lse=lse, max_q=n, max_kv=longest, stream=stream),
            *kb.seed_attn_bwd(a["seed"], a["k"], a["v"], a["d_o"], a["off"], scale, act, o=so, lse=slse, max_kv=longest, stream=stream),
            *kb.swa_bwd(a["k"], a["k"], a["v"], wo, wlse, a["d_t"], a["off"], 7, 2, scale, max_len=longest, stream=stream),
            kb.sumkron_fwd(a["x"], a["z"], a["w"], stream=stream), *kb.sumkron_bwd(a["x"], a["z"], a["w"], a["dy"], stream=stream)]


class PythonOnly:
    def __getattr__(self, name):
        return lambda *args: None


def native_fwd(a, **change):
    p = dict(q=a["q"], k=a["k"], v=a["v"], off=a["off"], scale=0.1, act=3, qo=None, max_q=N, max_kv=25, out=None, lse=None, want_lse=False, ws=None, stream=None)
    p.update(change)
    return kb._native.gdpa_fwd(*p.values())


def test_host_tensors_and_wrong_types_are_left_to_the_python_code():
    a = arguments("cpu")
    assert native_fwd(a) is None
    assert native_fwd(a, q=None) is None and native_fwd(a, q="x") is None
    assert kb._native.sumkron_fwd(a["x"], a["z"], a["w"], None, None, None) is None
    with pytest.raises(TypeError):
        kb._native.gdpa_fwd(a["q"])


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("stream", [False, True])
def test_same_results(monkeypatch, dtype, stream):
    a = arguments("cuda", dtype)
    torch.cuda.synchronize()
    s = torch.cuda.Stream() if stream else None
    got = calls(a, stream=s)
    torch.cuda.synchronize()
    monkeypatch.setattr(kb, "_native", PythonOnly())
    want = calls(a, stream=s)
    torch.cuda.synchronize()
    assert len(got) == len(want)
    for g, w in zip(got, want):
        assert g.dtype == w.dtype and g.shape == w.shape and not g.requires_grad and torch.equal(g, w)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_every_entry_point_goes_the_native_way(monkeypatch, dtype):
    a, native, taken = arguments("cuda", dtype), kb._native, []

    class Recorder:
        def __getattr__(self, name):
            def call(*args):
                done = getattr(native, name)(*args)
                assert done is not None, name
                taken.append(name)
                return done
            return call

    monkeypatch.setattr(kb, "_native", Recorder())
    calls(a)
    torch.cuda.synchronize()
    assert sorted(set(taken)) == sorted(["gdpa_fwd", "gdpa_bwd", "seed_attn_fwd", "seed_attn_bwd", "swa_fwd", "swa_bwd", "sumkron_fwd", "sumkron_bwd"])


@pytest.mark.gpu
def test_given_outputs_come_back_themselves():
    a = arguments("cuda")
    out, lse = torch.empty_like(a["q"]), torch.empty((H, B * N), device="cuda")
    ws = torch.empty(1 << 16, dtype=torch.uint8, device="cuda")
    got = native_fwd(a, out=out, lse=lse, ws=ws)
    assert got[0] is out and got[1] is lse
    assert native_fwd(a)[1] is None and native_fwd(a, want_lse=True)[1].shape == (H, B * N)
    grads = [torch.empty_like(a[x]) for x in ("q", "k", "v")]
    got = kb.gdpa_bwd(a["q"], a["k"], a["v"], a["d_o"], a["off"], 0.1, 3, max_q=N, max_kv=25, out=grads)
    assert isinstance(got, tuple) and all(x is y for x, y in zip(got, grads))
    p = torch.nn.Parameter(a["q"])  # a parameter is an ordinary tensor here
    assert native_fwd(a, q=p)[0].requires_grad is False


class Sub(torch.Tensor):
    pass


class Act(enum.IntEnum):
    GELU = 3


@pytest.mark.gpu
def test_what_is_not_plain_is_left_to_the_python_code(monkeypatch):
    a = arguments("cuda")
    q = a["q"]
    odd = [dict(q=q.as_subclass(Sub)), dict(act=Act.GELU), dict(scale=np.float64(0.1)), dict(max_q=np.int64(N)), dict(max_q=True),
           dict(off=a["off"].long()), dict(q=q.half()), dict(k=a["k"].float()), dict(q=q[:, :, :32]), dict(q=q.transpose(0, 1)),
           dict(v=a["v"][:-1]), dict(qo=a["off"][:2].contiguous()), dict(off=a["off"].cpu()), dict(out=torch.empty_like(q)[:-1]), dict(lse=torch.empty(H, 3, device="cuda")),
           dict(ws=torch.empty(8, dtype=torch.uint8, device="cuda")), dict(ws=torch.empty(1 << 16, device="cuda")), dict(max_q=N + 1), dict(act=99),
           dict(max_q=None), dict(scale=float("nan")), dict(max_kv=-1), dict(max_kv=1 << 40), dict(stream=7)]
    for change in odd:
        assert native_fwd(a, **change) is None, change

    def outcome(change):
        p = dict(dict(q=q, k=a["k"], v=a["v"], off=a["off"], scale=0.1, act=3, max_q=N, max_kv=25), **change)
        names = dict(qo="q_offsets", ws="workspace")
        kw = {names.get(x, x): y for x, y in p.items() if x not in ("q", "k", "v", "off", "scale", "act")}
        try:
            return kb.gdpa_fwd(p["q"], p["k"], p["v"], p["off"], p["scale"], p["act"], **kw)[0].float().cpu()
        except Exception as e:
            return type(e), str(e)

    both = [[outcome(c) for c in odd]]
    monkeypatch.setattr(kb, "_native", PythonOnly())
    both.append([outcome(c) for c in odd])
    for change, x, y in zip(odd, *both):
        assert torch.equal(x, y) if isinstance(x, torch.Tensor) else x == y, change


@pytest.mark.gpu
def test_transforms_see_the_python_code():
    a = arguments("cuda")
    def f(q):
        assert native_fwd(a, q=q) is None
        return q
    torch.func.vmap(f)(a["q"].unsqueeze(0))
    torch.func.grad(lambda q: f(q).sum())(a["q"].float())
