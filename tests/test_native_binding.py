"""The native half of the binding against the Python path: same results bit for bit, same errors."""
import os
import shutil
import subprocess
import sys
import sysconfig
import types
import warnings

import numpy as np
import pytest
import torch

import paper_2302_09915_amd as T

CALLS = {"gate": 7, "gate_dispatch": 9, "aux_loss": 6, "dispatch": 7, "combine": 6, "combine_bwd": 8, "dispatch_bwd": 5,
         "gate_bwd": 9}


@pytest.mark.parametrize("name", sorted(CALLS))
def test_leaves_the_unusual_to_python(name):
    """Host tensors, other objects and wrong counts are none of its business, and no error stays behind."""
    native, n = getattr(T._fast(), name), CALLS[name]
    class Sub(torch.Tensor):
        pass
    for arg in (torch.zeros(4, 4), torch.zeros(4, 4).as_subclass(Sub), torch.zeros(4, 4, device="meta"), None, 1, 1.5, "x",
                np.zeros(3), object()):
        assert native(*[arg] * n) is NotImplemented
    for count in (0, 1, n - 1, n + 1):
        assert native(*[torch.zeros(2, 2)] * count) is NotImplemented


def test_bound_arguments():
    """What ctypes would be given, and nothing else; a status comes back, which the caller turns into an error."""
    import ctypes

    bind, null = T._fast().bind, ctypes.c_void_p(None)
    good = (null, 0, ctypes.c_void_p(16), None, T.F32, -1, 8, 1, null, ctypes.c_void_p(0))
    call = bind("tamoe_combine", good)
    assert call() == T.INVALID_ARG and call() == T.INVALID_ARG
    with pytest.raises(TypeError):
        call(1)
    for name, args in (("tamoe_version", ()), ("tamoe_combine", good[:-1]), ("tamoe_combine", good + (None,)), ("tamoe_combine", list(good)),
                       ("tamoe_combine", (1.5,) + good[1:]), ("tamoe_combine", good[:4] + (1 << 40,) + good[5:]),
                       ("tamoe_combine", good[:1] + (1 << 70,) + good[2:]), ("tamoe_combine", good[:1] + (None,) + good[2:]),
                       ("tamoe_renorm_topk", (None, 1, True, None, None)), ("tamoe_gate_bwd", (None,) * 5 + (1, 1, 2, 2, 1, None, None))):
        assert bind(name, args) is NotImplemented, (name, args)
    assert bind() is NotImplemented and bind("tamoe_combine") is NotImplemented and bind(1, good) is NotImplemented
    zero = bind("tamoe_gate_bwd", (None,) * 5 + (0.5, 0, 2, 2, 1, None, None))   # no tokens: nothing is launched
    assert zero() == T.OK


def test_host_tensors_raise_as_before():
    f, i = torch.zeros(4, 4), torch.zeros(4, 2, dtype=torch.int32)
    for call in (lambda: T.gate(f, f, 2, 2, ws=f), lambda: T.aux_loss(f[0], i, None, 2, 4), lambda: T.dispatch(f, i, i, 4, 2, ws=f),
                 lambda: T.combine(f, 4, i, f), lambda: T.tamoe_combine_bwd(f, f, 4, i, f, f, f),
                 lambda: T.tamoe_dispatch_bwd(f, 4, i, f), lambda: T.tamoe_gate_bwd(f, i, f, None, i, 1.0, 2, f)):
        with pytest.raises(T.TamoeError, match="must be a device tensor") as e:
            call()
        assert e.value.status == T.INVALID_ARG


@pytest.mark.parametrize("stand_in", [None, types.SimpleNamespace(torch_version="0.0"), types.SimpleNamespace()])
def test_works_without_a_native_half_that_fits(stand_in, monkeypatch):
    """Missing, of another torch or of an older build: one warning, then the Python path answers."""
    monkeypatch.setitem(sys.modules, "paper_2302_09915_amd._native", stand_in)
    monkeypatch.setattr(T, "_native_half", None)
    with pytest.warns(RuntimeWarning, match="native half"):
        assert T._fast() is None
    f, i = torch.zeros(4, 4), torch.zeros(4, 2, dtype=torch.int32)
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        for call in (lambda: T.gate(f, f, 2, 2, ws=f), lambda: T.aux_loss(f[0], i, None, 2, 4), lambda: T.dispatch(f, i, i, 4, 2, ws=f),
                     lambda: T.combine(f, 4, i, f), lambda: T.tamoe_combine_bwd(f, f, 4, i, f, f, f)):
            with pytest.raises(T.TamoeError, match="must be a device tensor"):
                call()


def test_build_without_a_host_compiler(tmp_path, monkeypatch):
    """The library is built and a stale native half does not stay; its object depends on torch and Python."""
    from concurrent.futures import Future

    from paper_2302_09915_amd import build as B

    assert torch.__version__ in B._native_object() and sys.implementation.cache_tag in B._native_object()
    for name, path in (("HERE", str(tmp_path)), ("NATIVE_LIB", str(tmp_path / "_native.so.tagged"))):
        monkeypatch.setattr(B, name, path)
    for result in (("x.o", subprocess.CompletedProcess([], 1, "", "no headers\n")), FileNotFoundError("c++"), ImportError("torch")):
        for stale in ("_native.so", "_native.so.tagged"):
            (tmp_path / stale).write_text("old")
        done = Future()
        done.set_exception(result) if isinstance(result, Exception) else done.set_result(result)
        B._finish_native(done, False)
        assert os.listdir(tmp_path) == []


def test_daemon_threads_at_the_end_of_the_interpreter(tmp_path):
    """Threads that are outside the interpreter lock when the program ends do not abort it."""
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not found")
    src = tmp_path / "spin.cpp"
    src.write_text('''
#include "unlocked.h"
#include <stdexcept>
#include <unistd.h>
static PyObject* spin(PyObject*, PyObject* fail) {
    try {
        unlocked([&] { usleep(2000); if (fail != Py_None) throw std::runtime_error(""); return 0; });
    } catch (abi::__forced_unwind&) { throw;
    } catch (...) { return PyLong_FromLong(1); }
    Py_RETURN_NONE;
}
static PyMethodDef m[] = {{"spin", spin, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
static PyModuleDef d = {PyModuleDef_HEAD_INIT, "spin", nullptr, -1, m, nullptr, nullptr, nullptr, nullptr};
PyMODINIT_FUNC PyInit_spin() { return PyModule_Create(&d); }
''')
    here = os.path.join(os.path.dirname(T.__file__), "csrc_py")
    subprocess.run([cxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-I", here, "-I", sysconfig.get_paths()["include"], str(src),
                    "-o", str(tmp_path / "spin.so")], check=True)
    prog = ("import threading, time, spin\n"
            "assert spin.spin(None) is None and spin.spin(1) == 1\n"
            "def f(x):\n    while True: spin.spin(x)\n"
            "for i in range(8): threading.Thread(target=f, args=(None if i % 2 else 1,), daemon=True).start()\n"
            "time.sleep(0.05)\n")
    for _ in range(3):
        r = subprocess.run([sys.executable, "-c", prog], cwd=tmp_path, capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stderr


def _layer(dtype, S, d, N, P, k, stream=None):
    g = torch.Generator(device="cuda").manual_seed(S + N)
    x = torch.randn(S, d, device="cuda", generator=g).to(dtype)
    w = torch.nn.Parameter(torch.randn(N, d, device="cuda", generator=g).to(dtype))
    pen = torch.rand(N, device="cuda", generator=g)
    cap = torch.full((N,), max(1, S * k // N), dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()          # the inputs may be used on another stream than their own
    a = T.gate(x, w, P, k, stream=stream)
    out = {"gate." + n: v for n, v in a.items()}
    out["loss"] = T.aux_loss(a["m"], a["c_expert"], pen, P, S, stream=stream)
    b = T.dispatch(x, a["topk_idx"], cap, N, P, stream=stream)
    torch.cuda.synchronize()
    K = int(b["send_count_dev"].sum())
    out.update({"dispatch." + n: v[:K] if n == "send" else v for n, v in b.items()})
    out["y"] = T.combine(b["send"], K, b["slot"], a["topk_w"], stream=stream)
    f = T.gate_dispatch(x, w, P, k, pen, cap, False, stream=stream)
    assert f["logits"] is None
    out.update({"fused." + n: v[:K] if n == "send" else v for n, v in f.items() if v is not None})
    d_recv, d_w = torch.empty_like(b["send"]), torch.empty_like(a["topk_w"])
    T.tamoe_combine_bwd(x, b["send"], K, b["slot"], a["topk_w"], d_recv, d_w, stream)
    d_x, d_lg = torch.empty_like(x), torch.empty_like(a["logits"])
    T.tamoe_dispatch_bwd(d_recv, K, b["slot"], d_x, stream)
    T.tamoe_gate_bwd(a["logits"], a["topk_idx"], d_w, pen, a["c_expert"], 0.5, P, d_lg, stream)
    out.update(d_recv=d_recv[:K], d_w=d_w, d_x=d_x, d_lg=d_lg)
    torch.cuda.synchronize()
    return out


def _count_answers(monkeypatch):
    """Calls of every native function that were not left to the Python path."""
    native, answered = T._fast(), {name: 0 for name in CALLS}

    class Proxy:
        def __getattr__(self, name):
            def call(*args):
                r = getattr(native, name)(*args)
                answered[name] += r is not NotImplemented
                return r
            return call

    monkeypatch.setattr(T, "_fast", lambda: Proxy())
    return answered


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(1, 8, 2, 2, 1), (333, 40, 12, 4, 3), (1024, 256, 64, 8, 2)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
def test_same_as_the_python_path(dtype, shape, monkeypatch):
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    answered = _count_answers(monkeypatch)
    fast = [_layer(dtype, *shape), _layer(dtype, *shape, stream=side), _layer(dtype, *shape, stream=side.cuda_stream)]
    with torch.cuda.stream(side):
        fast.append(_layer(dtype, *shape))
    assert answered == {name: 4 for name in CALLS}      # the native half made every call, four layers long
    seen = []
    monkeypatch.setattr(T, "_fast", lambda: seen.append(0) or None)
    slow = _layer(dtype, *shape)
    assert len(seen) == len(CALLS) and answered == {name: 4 for name in CALLS}
    for out in fast:
        assert list(out) == list(slow)
        for n, v in slow.items():
            assert out[n].dtype == v.dtype and out[n].shape == v.shape and torch.equal(out[n], v), n


@pytest.mark.gpu
def test_takes_ordinary_calls_and_leaves_the_others():
    native = T._fast()
    x = torch.randn(64, 32, device="cuda")
    w = torch.randn(8, 32, device="cuda")
    ws = T.workspace(64, 32, 8, 2, 2, T.F32)
    assert type(native.gate(x, w, 2, 2, True, ws, None)) is dict
    class Sub(torch.Tensor):
        pass
    class Mode(torch.overrides.TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))
    for a in ((x.t(), w), (x.double(), w.double()), (x, w.half()), (x, w[:, :16].contiguous()), (x.as_subclass(Sub), w)):
        assert native.gate(*a, 2, 2, True, ws, None) is NotImplemented
    assert native.gate(x, w, 2, 2.0, True, ws, None) is NotImplemented
    assert native.gate(x, w, 2, 2, True, ws.float(), None) is NotImplemented
    assert native.gate(x, w, 2, 2, True, ws, object()) is NotImplemented
    assert native.gate(x, w, 2, 2, torch.ones(2), ws, None) is NotImplemented
    with Mode():
        assert native.gate(x, w, 2, 2, True, ws, None) is NotImplemented
        watched = T.gate(x, w, 2, 2)["logits"]
    assert torch.equal(watched, T.gate(x, w, 2, 2)["logits"])
    # the library's own refusals come through with their status
    assert native.gate(x, w, 2, 9, True, ws, None) in (T.UNSUPPORTED, T.INVALID_ARG)
    with pytest.raises(T.TamoeError) as e:
        T.gate(x, w, 2, 2, ws=ws[:1])
    assert e.value.status == T.WORKSPACE_TOO_SMALL and e.value.message
    # recv too short for K_rows
    with pytest.raises(T.TamoeError, match="hold K_rows rows"):
        T.combine(x, 65, torch.zeros(4, 2, dtype=torch.int32, device="cuda"), torch.zeros(4, 2, device="cuda"))
    with pytest.raises(T.TamoeError, match="hold K_rows rows"):
        T.combine(x, 1 << 62, torch.zeros(4, 2, dtype=torch.int32, device="cuda"), torch.zeros(4, 2, device="cuda"))
    # recorded, not made
    loss = torch.full((1,), 7.0, device="cuda")
    m, c = torch.rand(8, device="cuda"), torch.ones(8, dtype=torch.int32, device="cuda")
    call = T.bind(T.tamoe_aux_loss, m, c, None, 2, 8, loss)
    assert loss.item() == 7.0
    call()
    assert torch.equal(loss, T.aux_loss(m, c, None, 2, 8))


@pytest.mark.gpu
def test_new_tensors_are_seen_by_what_watches_torch():
    """A profiler and a tracer see the outputs being made, and under a transform, where new tensors are wrapped and have no
    address, the helpers refuse."""
    x, w = torch.randn(64, 32, device="cuda"), torch.randn(8, 32, device="cuda")
    plain = T.gate(x, w, 2, 2)
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CPU]) as prof:
        profiled = T.gate(x, w, 2, 2)
    assert {e.key: e.count for e in prof.key_averages()}.get("aten::empty", 0) >= len(plain)
    assert all(torch.equal(profiled[n], v) for n, v in plain.items())
    with warnings.catch_warnings():
        warnings.simplefilter("ignore")
        traced = torch.jit.trace(lambda v: T.gate(v, w, 2, 2)["topk_w"], (x,), check_trace=False)
    assert "aten::empty" in str(traced.graph)
    with pytest.raises(RuntimeError):
        torch.func.grad(lambda v: v.sum() + T.gate(x, w, 2, 2)["topk_w"].sum())(torch.ones(2, device="cuda"))
    assert torch.equal(T.gate(x, w, 2, 2)["topk_w"], plain["topk_w"])
