"""Build libkunlun.so (HIP, gfx950 only) in-tree with hipcc, and _torch_call.so (the entry points' marshalling) with g++."""
import os
import platform
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor
from importlib import metadata

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libkunlun.so")
TORCH_CALL = os.path.join(HERE, "_torch_call.so")
MADE_FOR = os.path.join(OBJ, "made_for")  # the torch and Python that _torch_call.so was compiled against
SOURCES = ["api.hip", "static_scratch.hip", "sched.hip", "stream_probe.hip", "scalar_kernels.hip", "attn_fwd_fp32_mfma.hip", "attn_fwd_mfma.hip", "attn_fwd_ring_mfma.hip", "attn_swa_band_mfma.hip", "attn_swa_bwd_band_mfma.hip", "attn_bwd_mfma.hip", "attn_bwd_pair_mfma.hip", "attn_bwd_wide_mfma.hip", "attn_bwd_tiled_mfma.hip", "sumkron.hip", "sumkron_fused.hip", "sumkron_bwd_fused.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# -packed-fp32-ops off: the compiler must not form packed fp32 instructions on this target.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
         "-packed-fp32-ops", "-Wall", "-Wno-unused-command-line-argument", "-Wno-unknown-attributes"]


def _deps_mtime():
    paths = [os.path.join(CSRC, f) for f in os.listdir(CSRC)]
    paths.append(os.path.join(os.path.dirname(HERE), "include", "kunlun.h"))
    return max(os.path.getmtime(p) for p in paths)


def _installed():
    return f"torch {metadata.version('torch')}, Python {platform.python_version()}"


def _made_for():
    if not os.path.exists(MADE_FOR):
        return None
    with open(MADE_FOR) as f:
        return f.read()


def _compile(src, extra=()):
    obj = os.path.join(OBJ, src.replace(".hip", ".o"))
    cmd = [HIPCC, *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
    warn = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip())
    return obj, warn


def _build_torch_call(out=TORCH_CALL, library=LIB, extra=()):
    """The CPython module of the entry points' accepted case: host code only, against torch's C++ headers and the library."""
    from torch.utils.cpp_extension import include_paths, library_paths
    dirs = [*include_paths(), sysconfig.get_paths()["include"]]
    libs = library_paths()[0]
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", *extra, *[f"-I{d}" for d in dirs], os.path.join(CSRC, "torch_call.cpp"),
           "-o", out, f"-L{os.path.dirname(library)}", f"-l:{os.path.basename(library)}", "-Wl,-rpath,$ORIGIN", f"-L{libs}", "-ltorch_python",
           "-ltorch_cpu", "-lc10"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed on torch_call.cpp:\n{r.stdout}\n{r.stderr}")


def build(force: bool = False, verbose: bool = False, extra=()) -> str:
    """Compile every source and link libkunlun.so and _torch_call.so.  Skips what is newer than every source
    unless force is set; _torch_call.so also has to be made for the installed torch and Python."""
    newer = [not force and os.path.exists(f) and os.path.getmtime(f) >= _deps_mtime() for f in (LIB, TORCH_CALL)]
    if not newer[0]:
        _build_library(verbose, extra)
    if not all(newer) or _made_for() != _installed():
        _build_torch_call()
        os.makedirs(os.path.dirname(MADE_FOR), exist_ok=True)
        with open(MADE_FOR, "w") as f:
            f.write(_installed())
    return LIB


def _build_library(verbose, extra):
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        results = list(ex.map(lambda s: _compile(s, extra), SOURCES))
    if verbose:
        for _, w in results:
            if w:
                print(w)
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *[o for o, _ in results]]
    subprocess.run(cmd, check=True)


if __name__ == "__main__":
    print(build(force=True, verbose=True))
