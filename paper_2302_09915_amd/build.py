"""Builds libtamoe.so (the C-ABI library of HIP kernels) in-tree with hipcc for gfx950, and the native half of
the Python binding."""
from __future__ import annotations

import glob
import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtamoe.so")
# yardstick kernels that only bench.py calls: a library of their own, nothing shared with libtamoe.so
BENCH_CSRC = os.path.join(HERE, "csrc_bench")
BENCH_LIB = os.path.join(HERE, "libtamoe_bench.so")
# native half of the Python binding: host code over torch's C++ tensors that links libtamoe.so, for this Python
NATIVE_SRC = os.path.join(HERE, "csrc_py", "native.cpp")
NATIVE_LIB = os.path.join(HERE, "_native" + sysconfig.get_config_var("EXT_SUFFIX"))

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # the compiler must not form packed fp32 instructions from ordinary float code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wextra", "-Wno-unused-parameter",
]
OBJ_DIR = os.path.join(HERE, "_build")


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.cpp")))


def bench_sources():
    return sorted(glob.glob(os.path.join(BENCH_CSRC, "*.hip")))


def _headers():
    return (glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(ROOT, "include", "*.h"))
            + glob.glob(os.path.join(BENCH_CSRC, "*.h")) + glob.glob(os.path.join(os.path.dirname(NATIVE_SRC), "*.h")))


def _fresh(obj: str, src: str) -> bool:
    """True if obj is newer than its source and every header."""
    if not os.path.exists(obj):
        return False
    t = os.path.getmtime(obj)
    return all(os.path.getmtime(f) < t for f in [src, *_headers()])


def _run(cmd, verbose: bool) -> subprocess.CompletedProcess:
    if verbose:
        print(" ".join(cmd), flush=True)
    return subprocess.run(cmd, capture_output=True, text=True)


def _compile(hipcc: str, src: str, verbose: bool, incremental: bool = False):
    obj = os.path.join(OBJ_DIR, os.path.basename(src) + ".o")
    if incremental and _fresh(obj, src):
        return obj, subprocess.CompletedProcess([], 0, "", "")
    # .cpp files hold host code only but share the HIP headers
    inc = ["-I", BENCH_CSRC] if os.path.dirname(src) == BENCH_CSRC else ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    cmd = [hipcc, *HIPCC_FLAGS, *inc, "-x", "hip", "-c", src, "-o", obj]
    return obj, _run(cmd, verbose)


def _torch_dir() -> str:
    import torch

    return os.path.dirname(torch.__file__)


def _rocm_dir() -> str:
    hipcc = shutil.which("hipcc")
    return os.path.dirname(os.path.dirname(os.path.realpath(hipcc))) if hipcc else "/opt/rocm"


def _native_object() -> str:
    """Named after everything outside the sources that the code in it depends on."""
    import torch

    abi = int(torch._C._GLIBCXX_USE_CXX11_ABI)
    return os.path.join(OBJ_DIR, f"native-{sys.implementation.cache_tag}-torch-{torch.__version__}-abi{abi}.o")


def _compile_native(verbose: bool, incremental: bool = False):
    import torch

    obj = _native_object()
    if incremental and _fresh(obj, NATIVE_SRC):
        return obj, subprocess.CompletedProcess([], 0, "", "")
    cmd = [shutil.which("g++") or "c++", "-O2", "-std=c++17", "-fPIC", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           f'-DTAMOE_TORCH_VERSION="{torch.__version__}"', "-I", os.path.join(ROOT, "include"),
           "-isystem", os.path.join(_torch_dir(), "include"), "-isystem", sysconfig.get_paths()["include"],
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", "-isystem", os.path.join(_rocm_dir(), "include"), "-c", NATIVE_SRC, "-o", obj]
    return obj, _run(cmd, verbose)


def _link_native(obj: str, verbose: bool) -> subprocess.CompletedProcess:
    return _run([shutil.which("g++") or "c++", "-shared", "-L", HERE, "-L", os.path.join(_torch_dir(), "lib"),
                 "-Wl,-rpath,$ORIGIN", obj, "-ltamoe", "-ltorch_cpu", "-ltorch_hip", "-lc10", "-lc10_hip", "-ltorch_python", "-o", NATIVE_LIB], verbose)


def _finish_native(compiled, verbose: bool) -> None:
    """Links the native half of the binding.  Without it the binding works, so what stands in the way of it (no g++,
    no headers of torch or Python) is reported and does not fail the build; an older one does not stay behind."""
    for old in (NATIVE_LIB, os.path.join(HERE, "_native.so")):   # the latter: any Python would load it
        if os.path.exists(old):
            os.remove(old)
    try:
        obj, res = compiled.result()
        if res.returncode == 0:
            res = _link_native(obj, verbose)
        why = res.stdout + res.stderr if res.returncode != 0 else ""
    except (ImportError, AttributeError, OSError) as e:
        why = f"{type(e).__name__}: {e}\n"
    if why:
        sys.stderr.write(f"{why}the native half of the binding was not built\n")


def build(verbose: bool = False, jobs: int = 0, incremental: bool = False) -> str:
    """Compiles every source of csrc/ to an object (in parallel: the gate's tile code is instantiated
    in one translation unit per element type) and links libtamoe.so.  incremental: keep the objects
    that are newer than their source and every header (for development; the default rebuilds all)."""
    from concurrent.futures import ThreadPoolExecutor

    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    os.makedirs(OBJ_DIR, exist_ok=True)
    srcs = sources() + bench_sources()
    jobs = jobs or max(1, min(len(srcs), os.cpu_count() or 1, 8))
    with ThreadPoolExecutor(max_workers=jobs) as pool:
        native = pool.submit(_compile_native, verbose, incremental)
        done = list(pool.map(lambda src: _compile(hipcc, src, verbose, incremental), srcs))
    objs, bench_objs = [], []
    for src, (obj, res) in zip(srcs, done):
        if res.returncode != 0:
            sys.stderr.write(res.stdout + res.stderr)
            raise RuntimeError(f"hipcc failed compiling {src}")
        if verbose and res.stderr.strip():
            sys.stderr.write(res.stderr)
        (bench_objs if os.path.dirname(src) == BENCH_CSRC else objs).append(obj)
    for out, parts in ((LIB, objs), (BENCH_LIB, bench_objs)):
        res = _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *parts, "-o", out], verbose)
        if res.returncode != 0:
            sys.stderr.write(res.stdout + res.stderr)
            raise RuntimeError(f"hipcc failed linking {out}")
    _finish_native(native, verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True, incremental="--incremental" in sys.argv[1:]))
