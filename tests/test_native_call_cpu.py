"""The native marshalling (csrc/torch_call.cpp) on the CPU: built for host tensors, in front of a library of stubs that note
their arguments, call back into Python in the middle of the call (the interpreter's lock is free there, as for another thread)
and return the status they are told."""
import ctypes
import gc
import importlib.machinery
import importlib.util
import os
import re
import subprocess
import types
import weakref

import pytest
import torch

from paper_2602_10016_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
H, D, N, B, T = 2, 64, 8, 3, 40
ENTRIES = ["gdpa_fwd", "gdpa_bwd", "seed_attn_fwd", "seed_attn_bwd", "swa_fwd", "swa_bwd", "sumkron_fwd", "sumkron_bwd"]


def stub_source():
    """Every entry point of include/kunlun.h that returns a status: arguments as text into a buffer, then the hook."""
    header = open(os.path.join(ROOT, "include", "kunlun.h")).read()
    code = ['#include "kunlun.h"', "#include <stdio.h>", "char noted[4096]; int calls, status; void (*hook)(void);",
            "size_t kunlun_workspace_bytes(int op, int B, int H, int d, int mq, int mk, int64_t tq, int64_t tk) { return 1000 + op; }",
            "size_t kunlun_sumkron_batch_bytes(int B, int S, int T, int D, int k, int dtype) { return 2000; }",
            "size_t kunlun_sumkron_bwd_workspace_bytes(int B, int S, int T, int D, int k, int dtype) { return 3000; }"]
    for name in ENTRIES:
        args = re.search(rf"^int kunlun_{name}\(([^)]*)\);", header, flags=re.M).group(1)
        formats, values = [], []
        for arg in args.split(","):
            kind, var = arg.replace("\n", " ").strip().rsplit(" ", 1)
            var = var.lstrip("*")
            pointer = "*" in arg
            formats.append("%p" if pointer else {"float": "%.9g"}.get(kind, "%lld"))
            values.append(f"(void*){var}" if pointer else f"(double){var}" if kind == "float" else f"(long long){var}")
        code.append(f'int kunlun_{name}({args}) {{ ++calls; snprintf(noted, sizeof noted, "{" ".join(formats)}", {", ".join(values)}); '
                    "if (hook) hook(); return status; }")
    return "\n".join(code)


class Stub:
    def __init__(self, folder):
        source, library, module = (os.path.join(folder, f) for f in ("stub.c", "libkunlun_stub.so", "_torch_call.so"))
        with open(source, "w") as f:
            f.write(stub_source())
        subprocess.run(["gcc", "-shared", "-fPIC", f"-I{ROOT}/include", source, "-o", library], check=True)
        build._build_torch_call(out=module, library=library, extra=["-O0", "-DKUNLUN_CALL_DEVICE=CPU"])
        loader = importlib.machinery.ExtensionFileLoader("_torch_call", module)
        self.native = importlib.util.module_from_spec(importlib.util.spec_from_loader("_torch_call", loader))
        self.lib = ctypes.CDLL(library)
        self.reset()

    def reset(self, status=0, hook=None):
        self.hook = ctypes.CFUNCTYPE(None)(hook) if hook else None
        ctypes.c_void_p.in_dll(self.lib, "hook").value = ctypes.cast(self.hook, ctypes.c_void_p).value if hook else None
        ctypes.c_int.in_dll(self.lib, "status").value = status
        ctypes.c_int.in_dll(self.lib, "calls").value = 0

    @property
    def calls(self):
        return ctypes.c_int.in_dll(self.lib, "calls").value

    @property
    def noted(self):
        return (ctypes.c_char * 4096).in_dll(self.lib, "noted").value.decode().split()


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    return Stub(str(tmp_path_factory.mktemp("native")))


@pytest.fixture
def stub(built):
    built.reset()
    return built


STREAM = types.SimpleNamespace(cuda_stream=0x5EED)


def arguments(name, dtype=torch.bfloat16, **change):
    """The arguments of a native entry point by name, in its order."""
    r = lambda *s: torch.zeros(*s, dtype=dtype)
    i = lambda *x: torch.tensor(x, dtype=torch.int32)
    off, lse = i(0, 15, 15, T), torch.zeros(H, B * N)
    kv = dict(k=r(T, H, D), v=r(T, H, D))
    gdpa = dict(q=r(B * N, H, D), **kv)
    seed = dict(e_seed=r(N, H, D), **kv)
    swa = dict(q=r(T, H, D), **kv)
    sk = dict(x=r(B, 64, 128), z=r(2, 64, 32), w=r(2, 128, 128))
    o, d_o = r(B * N, H, D), r(B * N, H, D)
    tail = dict(workspace=None, stream=STREAM)
    fwd_tail = dict(out=None, lse=None, want_lse=True, **tail)
    a = {"gdpa_fwd": dict(**gdpa, kv_offsets=off, scale=0.1, act=3, q_offsets=None, max_q=N, max_kv=25, **fwd_tail),
         "gdpa_bwd": dict(**gdpa, d_o=d_o, kv_offsets=off, scale=0.1, act=0, o=o, lse=lse, q_offsets=None, max_q=N, max_kv=25, out=None, **tail),
         "seed_attn_fwd": dict(**seed, kv_offsets=off, scale=0.1, act=0, max_kv=25, **fwd_tail),
         "seed_attn_bwd": dict(**seed, d_o=d_o, kv_offsets=off, scale=0.1, act=0, o=o, lse=lse, max_kv=25, out=None, **tail),
         "swa_fwd": dict(**swa, offsets=off, window_left=7, window_right=2, scale=0.1, max_len=25, **fwd_tail),
         "swa_bwd": dict(**swa, o=r(T, H, D), lse=torch.zeros(H, T), d_o=r(T, H, D), offsets=off, window_left=7, window_right=2, scale=0.1,
                         max_len=25, out=None, **tail),
         "sumkron_fwd": dict(**sk, out=None, **tail),
         "sumkron_bwd": dict(**sk, dy=r(B, 32, 128), **tail)}[name]
    assert set(change) <= set(a)
    a.update(change)
    return a


def gradients(a):
    return [torch.zeros_like(t) for t in list(a.values())[:3]]


@pytest.mark.parametrize("name", ["gdpa_bwd", "seed_attn_bwd", "swa_bwd"])
def test_gradients_of_a_list_outlive_its_change_during_the_call(stub, name):
    a = arguments(name)
    a["out"] = gradients(a)
    alive, pointers = [weakref.ref(t) for t in a["out"]], [t.data_ptr() for t in a["out"]]
    during = []

    def another_thread():
        a["out"].clear()
        gc.collect()
        during.extend(w() is not None for w in alive)

    stub.reset(hook=another_thread)
    got = getattr(stub.native, name)(*a.values())
    assert during == [True] * 3
    assert [id(g) for g in got] == [id(w()) for w in alive] and [g.data_ptr() for g in got] == pointers


@pytest.mark.parametrize("name", ENTRIES)
def test_memory_that_may_not_be_had_is_an_error(stub, name):
    a = arguments(name)
    torch._C._set_throw_on_mutable_data_ptr(list(a.values())[1])
    with pytest.raises(RuntimeError):
        getattr(stub.native, name)(*a.values())
    assert stub.calls == 0


@pytest.mark.parametrize("name", ENTRIES)
def test_a_refused_launch_raises_without_a_second_call(stub, name):
    """The launchers report after kernels are enqueued: the Python code behind must not make the call again."""
    from paper_2602_10016_amd import binding as kb
    stub.reset(status=kb.ERR_LAUNCH)
    with pytest.raises(kb.KunlunError) as error:
        getattr(stub.native, name)(*arguments(name).values())
    assert error.value.status == kb.ERR_LAUNCH and stub.calls == 1
    for status in (kb.ERR_NULL, kb.ERR_SHAPE, kb.ERR_UNSUPPORTED, kb.ERR_ALIGN, kb.ERR_WORKSPACE):  # of an argument: nothing is enqueued
        stub.reset(status=status)
        assert getattr(stub.native, name)(*arguments(name).values()) is None and stub.calls == 1


def parameters(name):
    """Names of the C parameters, in order."""
    header = open(os.path.join(ROOT, "include", "kunlun.h")).read()
    return [p.rsplit(" ", 1)[1].lstrip("*") for p in re.search(rf"^int kunlun_{name}\(([^)]*)\);", header, flags=re.M).group(1).replace("\n", " ").split(",")]


def expected(name, a, result, dtype):
    """C parameter -> value that the call must have received."""
    pointer = lambda t: 0 if t is None else t.data_ptr()
    given = {k: pointer(v) if isinstance(v, torch.Tensor) or v is None else v for k, v in a.items() if k not in ("out", "want_lse", "stream", "workspace")}
    results = [pointer(t) for t in (result if isinstance(result, tuple) else (result,))]
    want = dict(given, stream=0x5EED, dtype=1 if dtype == torch.float32 else 0, head_act=0, H=H, d=D, B=B, total_q=B * N, total_kv=T, n_seeds=N, total=T)
    if name.startswith("sumkron"):
        want.update(S=64, T=32, D=128, k_=2, y=results[0])
        want.update(zip(("dx", "dz", "dw"), results) if name == "sumkron_bwd" else ())
    elif name.endswith("fwd"):
        want.update(o=results[0], lse=results[1])
    else:
        want.update(zip(("d_e" if name == "seed_attn_bwd" else "dq", "dk", "dv"), results))
    return want


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("given", [False, True])
@pytest.mark.parametrize("name", ENTRIES)
def test_every_entry_point_takes_its_plain_arguments(stub, name, given, dtype):
    """The call is made, once, with every argument in its place; outputs and workspace that are given are the ones that are used."""
    a = arguments(name, dtype)
    if given:
        a["workspace"] = torch.zeros(5000, dtype=torch.uint8)
        if "q_offsets" in a:
            a["q_offsets"] = torch.tensor([0, N, 2 * N, 3 * N], dtype=torch.int32)
        if name.endswith("bwd") and "out" in a:
            a["out"] = gradients(a)
        elif "out" in a:
            rows = T if name == "swa_fwd" else B * N
            a["out"] = torch.zeros(B, 32, 128, dtype=dtype) if name == "sumkron_fwd" else torch.zeros(rows, H, D, dtype=dtype)
            if "lse" in a:
                a["lse"] = torch.zeros(H, rows)
    result = getattr(stub.native, name)(*a.values())
    assert result is not None and stub.calls == 1
    flat = list(result) if isinstance(result, tuple) else [result]
    if given and "out" in a:
        outs = a["out"] if isinstance(a["out"], list) else [a["out"]]
        assert [id(x) for x in flat[:len(outs)]] == [id(x) for x in outs]
    want, got = expected(name, a, result, dtype), dict(zip(parameters(name), stub.noted))
    if name.startswith("sumkron"):  # (there k is a number, not a tensor)
        want["k"] = want.pop("k_")
    for parameter, text in got.items():
        if parameter == "workspace":
            assert int(text, 16) == a["workspace"].data_ptr() if given else int(text, 16) != 0
        elif parameter == "workspace_bytes":
            assert int(text) == (5000 if given else {"gdpa_fwd": 1000, "gdpa_bwd": 1001, "swa_fwd": 1002, "swa_bwd": 1003, "seed_attn_fwd": 1004,
                                                     "seed_attn_bwd": 1005, "sumkron_fwd": 2000, "sumkron_bwd": 3000}[name])
        elif parameter == "scale":
            assert float(text) == pytest.approx(0.1, rel=1e-7)
        else:
            value = 0 if text == "(nil)" else int(text, 16) if text.startswith("0x") else int(text)
            assert value == want[parameter], parameter


class Sub(torch.Tensor):
    pass


def odd(x):
    """Arguments of other kinds in the place of x."""
    if isinstance(x, torch.Tensor):
        yield from (None, "x", x.double(), x.half(), x.long(), x.float() if x.dtype != torch.float32 else x.bfloat16(), x.unsqueeze(0), x[:-1],
                    torch.cat([x, x[:1]]), torch.stack([x, x], -1)[..., 0], x.as_subclass(Sub), x[:0])
        if x.dim() > 1:
            yield from (x.transpose(0, 1), x.transpose(0, 1).contiguous(), x[:, :1].contiguous(), x[..., :-8].contiguous())
    elif isinstance(x, (int, float)) and not isinstance(x, bool):
        yield from (None, "x", [], 1 << 40, 2.5, torch.zeros(2))


@pytest.mark.parametrize("name", ENTRIES)
def test_nothing_is_accepted_that_the_python_code_refuses(stub, name, monkeypatch):
    """Every argument in turn replaced by others: what the Python code refuses for any other reason than the device, the native
    call leaves to it, without making the call."""
    from paper_2602_10016_amd import binding as kb
    monkeypatch.setattr(kb, "_native", types.SimpleNamespace(**{n: lambda *args: None for n in ENTRIES}))

    def refused(a):
        try:
            getattr(kb, name)(**a)
        except Exception as e:
            return "CUDA" not in str(e)
        raise AssertionError("host tensors were accepted")

    assert not refused(arguments(name))
    cases = [(key, value) for key, x in arguments(name).items() for value in odd(x)]
    grads = lambda i, value: [value if i == j else g for j, g in enumerate(gradients(arguments(name)))]
    if name.endswith("bwd") and "out" in arguments(name):
        cases += [("out", grads(i, value)) for i in range(3) for value in odd(gradients(arguments(name))[i])]
        cases += [("out", gradients(arguments(name))[:2]), ("out", 5)]
    elif "out" in arguments(name):
        shape = (B, 32, 128) if name == "sumkron_fwd" else (T if name == "swa_fwd" else B * N, H, D)
        cases += [("out", value) for value in odd(torch.zeros(shape, dtype=torch.bfloat16)) if value is not None]
        if "lse" in arguments(name):
            cases += [("lse", value) for value in odd(torch.zeros(H, shape[0])) if value is not None]
    cases += [("workspace", value) for value in ("x", torch.zeros(5000), torch.zeros(5000, 2, dtype=torch.uint8)[:, 0])]
    if "q_offsets" in arguments(name):
        cases += [("q_offsets", value) for value in odd(torch.tensor([0, N, 2 * N, 3 * N], dtype=torch.int32)) if value is not None]
    n = 0
    for key, value in cases:
        a = arguments(name, **{key: value})
        stub.reset()
        if refused(a):
            n += 1
            assert getattr(stub.native, name)(*a.values()) is None and stub.calls == 0, (key, value)
    assert n > 20
