// Native half of the Python binding: checks and unwraps tensors, allocates the outputs of the allocating
// helpers and calls the C entry points (include/tamoe.h).
//
// A layer of a few thousand tokens is a handful of launches of 3 to 10 us each.  Checking and converting some
// forty tensors and allocating eighteen outputs in Python took longer than that.  Host time, whatever the sizes:
// gate + aux_loss + dispatch + combine 79 -> 38 us, the three backward entry points 29 -> 13 us.  Without
// the dispatcher for each output, unless something watches torch, Python for the stream and ctypes for bound calls: gate_dispatch 17.0 -> 14.7,
// a bound call of one launch 3.0 -> 2.75.
//
// Every function returns NotImplemented when anything about its arguments is out of the ordinary (a type, a
// layout, a device, a subclass, a mode that watches torch's functions, an exception on the way); the caller
// then takes the Python path, which checks everything again and raises what it has to.  Nothing has been
// launched by then.  A status other than TAMOE_OK is returned as an int.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/hip/EmptyTensor.h>
#include <ATen/record_function.h>
#include <Python.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>

#include <memory>
#include <tuple>
#include <type_traits>
#include <utility>

#include "tamoe.h"
#include "unlocked.h"

namespace {

PyObject* g_tensor = nullptr;          // torch.Tensor
PyObject* g_parameter = nullptr;       // torch.nn.Parameter

struct Slow {};                        // thrown where the Python path has to decide

const at::Tensor& tensor(PyObject* o) {
    PyObject* t = reinterpret_cast<PyObject*>(Py_TYPE(o));
    if (t != g_tensor && t != g_parameter) throw Slow{};
    const at::Tensor& v = THPVariable_Unpack(o);
    if (!v.is_cuda() || !v.is_contiguous()) throw Slow{};
    return v;
}
const at::Tensor& tensor(PyObject* o, at::ScalarType dt) {
    const at::Tensor& v = tensor(o);
    if (v.scalar_type() != dt) throw Slow{};
    return v;
}
template <class P = void>
P* ptr(const at::Tensor& t) { return static_cast<P*>(t.data_ptr()); }
template <class P>
P* ptr(PyObject* o, at::ScalarType dt) { return ptr<P>(tensor(o, dt)); }
template <class P>
P* ptr_or_null(PyObject* o, at::ScalarType dt) { return o == Py_None ? nullptr : ptr<P>(o, dt); }

int64_t integer(PyObject* o) {
    if (!PyLong_CheckExact(o)) throw Slow{};
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw Slow{};
    return v;
}
int small(PyObject* o) {
    const int64_t v = integer(o);
    if (v < INT32_MIN || v > INT32_MAX) throw Slow{};
    return (int)v;
}
int storage(const at::Tensor& t) {
    switch (t.scalar_type()) {
        case at::kFloat: return TAMOE_F32;
        case at::kBFloat16: return TAMOE_BF16;
        case at::kHalf: return TAMOE_F16;
        default: throw Slow{};
    }
}
bool truth(PyObject* o) {
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw Slow{};
    return v != 0;
}
int dim32(int64_t v) {
    if (v > INT32_MAX) throw Slow{};
    return (int)v;
}
void matrix(const at::Tensor& t) {
    if (t.dim() != 2) throw Slow{};
}
void holds_rows(const at::Tensor& t, int64_t rows, int64_t d) {
    int64_t n;
    if (__builtin_mul_overflow(rows, d, &n) || t.numel() < n) throw Slow{};
}

// hipStream_t of `stream`: None (the current stream of the current device), an object with cuda_stream, or an int
void* stream_of(PyObject* stream) {
    PyObject* v;
    if (stream == Py_None) {
        return c10::hip::getCurrentHIPStream().stream();
    } else if (PyLong_CheckExact(stream)) {
        v = Py_NewRef(stream);
    } else {
        v = PyObject_GetAttrString(stream, "cuda_stream");
    }
    if (v == nullptr) throw Slow{};
    void* p = PyLong_Check(v) ? PyLong_AsVoidPtr(v) : nullptr;
    const bool bad = !PyLong_Check(v) || PyErr_Occurred() != nullptr;
    Py_DECREF(v);
    if (bad) throw Slow{};
    return p;
}

struct Out {
    at::TensorOptions f32, i32, u8, x;
    explicit Out(const at::Tensor& t)
        : f32(at::TensorOptions().device(t.device()).dtype(at::kFloat)),
          i32(f32.dtype(at::kInt)), u8(f32.dtype(at::kByte)), x(f32.dtype(t.scalar_type())) {}
};

// Does something in torch look at operators or replace them: a profiler, a tracer, a transform of torch.func?
bool watched() {
    return at::hasCallbacks() || !(c10::impl::tls_local_dispatch_key_set().included_ - c10::default_included_set).empty();
}
// at::empty without the dispatcher (a fourth of its time) where nothing depends on it: not watched, and new tensors are not filled.
at::Tensor empty(at::IntArrayRef sizes, const at::TensorOptions& o) {
    if (at::globalContext().deterministicAlgorithms() || watched()) return at::empty(sizes, o);
    return at::detail::empty_cuda(sizes, c10::typeMetaToScalarType(o.dtype()), o.device(), std::nullopt);
}

PyObject* interned(const char* text) { return PyUnicode_InternFromString(text); }
// Keys of the results, made once.
#define KEY(name) PyObject* const k_##name = interned(#name)
struct Keys {
    KEY(topk_idx);
    KEY(topk_w);
    KEY(m);
    KEY(c_expert);
    KEY(c_device);
    KEY(logits);
    KEY(loss);
    KEY(send);
    KEY(slot);
    KEY(kept_expert);
    KEY(expert_offset);
    KEY(send_count_dev);
};
#undef KEY
const Keys* g_keys = nullptr;

struct Dict {
    PyObject* d = PyDict_New();
    ~Dict() {
        if (d != nullptr && PyGILState_Check()) Py_DECREF(d);   // not in a thread that the interpreter ends (unlocked)
    }
    void put(PyObject* key, const at::Tensor& t) { put(key, THPVariable_Wrap(t)); }
    void none(PyObject* key) { put(key, Py_NewRef(Py_None)); }
    void put(PyObject* key, PyObject* v) {
        const bool bad = d == nullptr || v == nullptr || key == nullptr || PyDict_SetItem(d, key, v) != 0;
        Py_XDECREF(v);
        if (bad) throw Slow{};
    }
    PyObject* release() {
        PyObject* r = d;
        d = nullptr;
        return r;
    }
};

// a workspace that is given, or a new one
at::Tensor workspace(PyObject* ws, int64_t S, int d, int N, int P, int k, int dtype, const Out& o) {
    if (ws != Py_None) return tensor(ws, at::kByte);
    return unlocked([&] { return empty({(int64_t)tamoe_workspace_bytes(S, d, N, P, k, dtype)}, o.u8); });
}

template <class F>
PyObject* guarded(Py_ssize_t n, Py_ssize_t want, F body) {
    if (n == want && !at::impl::torch_function_mode_enabled() && !c10::impl::dispatch_mode_enabled()) {
        try {
            return body();
        } catch (abi::__forced_unwind&) {   // the thread is being ended (unlocked)
            throw;
        } catch (...) {   // Slow, or an error of the allocator: the Python path meets it again
        }
        PyErr_Clear();
    }
    return Py_NewRef(Py_NotImplemented);
}

struct Gate {   // what the gate and the fused call share
    const at::Tensor &x, &w;
    int64_t S;
    int d, N, P, k, dt;
    Out o;
    Gate(PyObject* const* a)
        : x(tensor(a[0])), w(tensor(a[1])), S(0), d(0), N(0), P(small(a[2])), k(small(a[3])), dt(storage(x)), o(x) {
        matrix(x);
        matrix(w);
        if (w.scalar_type() != x.scalar_type() || w.size(1) != x.size(1) || k < 0 || P < 0) throw Slow{};
        S = x.size(0);
        d = dim32(x.size(1));
        N = dim32(w.size(0));
    }
};
struct GateOut {
    at::Tensor idx, wgt, m, ce, cd, lg;
    GateOut(const Gate& g, bool logits)
        : idx(empty({g.S, g.k}, g.o.i32)), wgt(empty({g.S, g.k}, g.o.f32)), m(empty({g.N}, g.o.f32)),
          ce(empty({g.N}, g.o.i32)), cd(empty({g.P}, g.o.i32)) {
        if (logits) lg = empty({g.S, g.N}, g.o.f32);
    }
    float* logits() const { return lg.defined() ? ptr<float>(lg) : nullptr; }
    void fill(Dict& r) const {
        r.put(g_keys->k_topk_idx, idx);
        r.put(g_keys->k_topk_w, wgt);
        r.put(g_keys->k_m, m);
        r.put(g_keys->k_c_expert, ce);
        r.put(g_keys->k_c_device, cd);
        if (lg.defined()) r.put(g_keys->k_logits, lg);
        else r.none(g_keys->k_logits);
    }
};
struct DispatchOut {
    at::Tensor send, slot, kept, off, cnt;
    DispatchOut(const Out& o, int64_t S, int64_t k, int64_t d, int64_t N, int64_t P)
        : send(empty({S * k, d}, o.x)), slot(empty({S, k}, o.i32)), kept(empty({N}, o.i32)),
          off(empty({N + 1}, o.i32)), cnt(empty({P}, o.i32)) {}
    void fill(Dict& r) const {
        r.put(g_keys->k_send, send);
        r.put(g_keys->k_slot, slot);
        r.put(g_keys->k_kept_expert, kept);
        r.put(g_keys->k_expert_offset, off);
        r.put(g_keys->k_send_count_dev, cnt);
    }
};

// gate(x, w, P, k, want_logits, ws, stream) -> dict
PyObject* n_gate(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 7, [&]() -> PyObject* {
        const Gate g(a);
        const bool logits = truth(a[4]);
        const GateOut q = unlocked([&] { return GateOut(g, logits); });
        const at::Tensor ws = workspace(a[5], g.S, g.d, g.N, g.P, g.k, g.dt, g.o);
        void* st = stream_of(a[6]);
        Dict r;
        q.fill(r);
        const int rc = unlocked([&] {
            return tamoe_gate(ptr(g.x), ptr(g.w), g.dt, g.S, g.d, g.N, g.P, g.k, q.logits(), ptr<int32_t>(q.idx),
                              ptr<float>(q.wgt), ptr<float>(q.m), ptr<int32_t>(q.ce), ptr<int32_t>(q.cd), ptr(ws),
                              (size_t)ws.numel(), st);
        });
        return rc == TAMOE_OK ? r.release() : PyLong_FromLong(rc);
    });
}

// gate_dispatch(x, w, P, k, penalty, cap, want_logits, ws, stream) -> dict
PyObject* n_gate_dispatch(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 9, [&]() -> PyObject* {
        const Gate g(a);
        const float* pen = ptr_or_null<float>(a[4], at::kFloat);
        const int32_t* cap = ptr<int32_t>(a[5], at::kInt);
        const bool logits = truth(a[6]);
        struct Outputs {
            GateOut q;
            at::Tensor loss;
            DispatchOut p;
        };
        const Outputs all = unlocked([&] {
            return Outputs{GateOut(g, logits), empty({1}, g.o.f32), DispatchOut(g.o, g.S, g.k, g.d, g.N, g.P)};
        });
        const GateOut& q = all.q;
        const at::Tensor& loss = all.loss;
        const DispatchOut& p = all.p;
        const at::Tensor ws = workspace(a[7], g.S, g.d, g.N, g.P, g.k, g.dt, g.o);
        void* st = stream_of(a[8]);
        Dict r;
        q.fill(r);
        r.put(g_keys->k_loss, loss);
        p.fill(r);
        const int rc = unlocked([&] {
            return tamoe_gate_dispatch(ptr(g.x), ptr(g.w), g.dt, g.S, g.d, g.N, g.P, g.k, pen, cap, q.logits(),
                                       ptr<int32_t>(q.idx), ptr<float>(q.wgt), ptr<float>(q.m), ptr<int32_t>(q.ce),
                                       ptr<int32_t>(q.cd), ptr<float>(loss), ptr(p.send), ptr<int32_t>(p.slot),
                                       ptr<int32_t>(p.kept), ptr<int32_t>(p.off), ptr<int32_t>(p.cnt), ptr(ws),
                                       (size_t)ws.numel(), st);
        });
        return rc == TAMOE_OK ? r.release() : PyLong_FromLong(rc);
    });
}

// aux_loss(m, c_expert, penalty, P, S, stream) -> tensor
PyObject* n_aux_loss(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 6, [&]() -> PyObject* {
        const at::Tensor& m = tensor(a[0], at::kFloat);
        const int32_t* ce = ptr<int32_t>(a[1], at::kInt);
        const float* pen = ptr_or_null<float>(a[2], at::kFloat);
        const int P = small(a[3]);
        const int64_t S = integer(a[4]);
        if (m.dim() < 1) throw Slow{};
        const int N = dim32(m.size(0));
        const at::Tensor loss = unlocked([&] { return empty({1}, Out(m).f32); });
        void* st = stream_of(a[5]);
        const int rc = unlocked([&] { return tamoe_aux_loss(ptr<float>(m), ce, pen, N, P, S, ptr<float>(loss), st); });
        return rc == TAMOE_OK ? THPVariable_Wrap(loss) : PyLong_FromLong(rc);
    });
}

// dispatch(x, topk_idx, cap, N, P, ws, stream) -> dict
PyObject* n_dispatch(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 7, [&]() -> PyObject* {
        const at::Tensor& x = tensor(a[0]);
        const at::Tensor& idx = tensor(a[1], at::kInt);
        const int32_t* cap = ptr<int32_t>(a[2], at::kInt);
        const int N = small(a[3]), P = small(a[4]), dt = storage(x);
        matrix(x);
        matrix(idx);
        if (N < 0 || P < 0) throw Slow{};
        const int64_t S = x.size(0);
        const int d = dim32(x.size(1)), k = dim32(idx.size(1));
        const Out o(x);
        const DispatchOut p = unlocked([&] { return DispatchOut(o, S, k, d, N, P); });
        const at::Tensor ws = workspace(a[5], S, d, N, P, k, dt, o);
        void* st = stream_of(a[6]);
        Dict r;
        p.fill(r);
        const int rc = unlocked([&] {
            return tamoe_dispatch(ptr(x), ptr<int32_t>(idx), cap, dt, S, d, N, P, k, ptr(p.send), ptr<int32_t>(p.slot),
                                  ptr<int32_t>(p.kept), ptr<int32_t>(p.off), ptr<int32_t>(p.cnt), ptr(ws),
                                  (size_t)ws.numel(), st);
        });
        return rc == TAMOE_OK ? r.release() : PyLong_FromLong(rc);
    });
}

// combine(recv, K_rows, slot, topk_w, d or None, stream) -> tensor
PyObject* n_combine(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 6, [&]() -> PyObject* {
        const at::Tensor& recv = tensor(a[0]);
        const int64_t K = integer(a[1]);
        const at::Tensor& slot = tensor(a[2], at::kInt);
        const float* w = ptr<float>(a[3], at::kFloat);
        matrix(slot);
        if (a[4] == Py_None) matrix(recv);
        const int64_t S = slot.size(0);
        const int d = dim32(a[4] == Py_None ? recv.size(1) : integer(a[4])), k = dim32(slot.size(1));
        if (d < 0) throw Slow{};
        holds_rows(recv, K, d);
        const at::Tensor y = unlocked([&] { return empty({S, d}, Out(recv).x); });
        const int dt = storage(y);
        void* st = stream_of(a[5]);
        const int rc = unlocked([&] { return tamoe_combine(ptr(recv), K, ptr<int32_t>(slot), w, dt, S, d, k, ptr(y), st); });
        return rc == TAMOE_OK ? THPVariable_Wrap(y) : PyLong_FromLong(rc);
    });
}

// combine_bwd(dy, recv, K_rows, slot, topk_w, d_recv, d_topk_w, stream) -> None
PyObject* n_combine_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 8, [&]() -> PyObject* {
        const at::Tensor &dy = tensor(a[0]), &recv = tensor(a[1]), &d_recv = tensor(a[5]);
        const int64_t K = integer(a[2]);
        const at::Tensor& slot = tensor(a[3], at::kInt);
        const float* w = ptr<float>(a[4], at::kFloat);
        float* d_w = ptr<float>(a[6], at::kFloat);
        matrix(dy);
        matrix(slot);
        const int d = dim32(dy.size(1)), k = dim32(slot.size(1));
        if (recv.scalar_type() != dy.scalar_type() || d_recv.scalar_type() != dy.scalar_type()) throw Slow{};
        holds_rows(recv, K, d);
        holds_rows(d_recv, K, d);
        const int dt = storage(dy);
        void* st = stream_of(a[7]);
        const int rc = unlocked([&] {
            return tamoe_combine_bwd(ptr(dy), ptr(recv), K, ptr<int32_t>(slot), w, dt, slot.size(0), d, k, ptr(d_recv), d_w,
                                     st);
        });
        return rc == TAMOE_OK ? Py_NewRef(Py_None) : PyLong_FromLong(rc);
    });
}

// dispatch_bwd(d_send, K_rows, slot, d_x, stream) -> None
PyObject* n_dispatch_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 5, [&]() -> PyObject* {
        const at::Tensor &d_send = tensor(a[0]), &d_x = tensor(a[3]);
        const int64_t K = integer(a[1]);
        const at::Tensor& slot = tensor(a[2], at::kInt);
        matrix(d_x);
        matrix(slot);
        const int d = dim32(d_x.size(1)), k = dim32(slot.size(1));
        if (d_send.scalar_type() != d_x.scalar_type()) throw Slow{};
        holds_rows(d_send, K, d);
        const int dt = storage(d_x);
        void* st = stream_of(a[4]);
        const int rc = unlocked([&] {
            return tamoe_dispatch_bwd(ptr(d_send), K, ptr<int32_t>(slot), dt, slot.size(0), d, k, ptr(d_x), st);
        });
        return rc == TAMOE_OK ? Py_NewRef(Py_None) : PyLong_FromLong(rc);
    });
}

// gate_bwd(logits, topk_idx, d_topk_w, penalty, c_expert, loss_scale, P, d_logits, stream) -> None
PyObject* n_gate_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 9, [&]() -> PyObject* {
        const at::Tensor &lg = tensor(a[0], at::kFloat), &idx = tensor(a[1], at::kInt);
        const float* d_w = ptr_or_null<float>(a[2], at::kFloat);
        const float* pen = ptr_or_null<float>(a[3], at::kFloat);
        const int32_t* ce = ptr<int32_t>(a[4], at::kInt);
        const double scale = PyFloat_AsDouble(a[5]);
        if (scale == -1.0 && PyErr_Occurred()) throw Slow{};
        const int P = small(a[6]);
        float* out = ptr<float>(a[7], at::kFloat);
        matrix(lg);
        matrix(idx);
        const int N = dim32(lg.size(1)), k = dim32(idx.size(1));
        void* st = stream_of(a[8]);
        const int rc = unlocked([&] {
            return tamoe_gate_bwd(ptr<float>(lg), ptr<int32_t>(idx), d_w, pen, ce, (float)scale, lg.size(0), N, P, k, out, st);
        });
        return rc == TAMOE_OK ? Py_NewRef(Py_None) : PyLong_FromLong(rc);
    });
}

// ---- bound calls ----
// A C entry point with its arguments, called without any.
template <class T>
T unmarshal(PyObject* o) {   // what ctypes would be given
    if constexpr (std::is_pointer_v<T>) {
        if (o == Py_None) return nullptr;
        PyObject* v = PyLong_Check(o) ? Py_NewRef(o) : PyObject_GetAttrString(o, "value");   // ctypes.c_void_p
        if (v == nullptr) throw Slow{};
        void* p = v == Py_None ? nullptr : PyLong_Check(v) ? PyLong_AsVoidPtr(v) : nullptr;
        const bool bad = (v != Py_None && !PyLong_Check(v)) || PyErr_Occurred() != nullptr;
        Py_DECREF(v);
        if (bad) throw Slow{};
        return static_cast<T>(p);
    } else if constexpr (std::is_floating_point_v<T>) {
        if (!PyFloat_CheckExact(o)) throw Slow{};
        return (T)PyFloat_AS_DOUBLE(o);
    } else {
        const int64_t v = integer(o);
        if ((int64_t)(T)v != v || (std::is_unsigned_v<T> && v < 0)) throw Slow{};
        return (T)v;
    }
}
template <auto Fn>
struct Bound;
template <class... A, int (*Fn)(A...)>
struct Bound<Fn> {
    using Args = std::tuple<A...>;
    static constexpr const char* kName = "tamoe bound call";
    static PyObject* call(PyObject* self, PyObject*) {
        const Args* a = static_cast<const Args*>(PyCapsule_GetPointer(self, kName));
        if (a == nullptr) return nullptr;
        return PyLong_FromLong(unlocked([&] { return std::apply(Fn, *a); }));
    }
    static void drop(PyObject* self) { delete static_cast<Args*>(PyCapsule_GetPointer(self, kName)); }
    template <size_t... I>
    static PyObject* make(PyObject* args, std::index_sequence<I...>) {
        if (PyTuple_GET_SIZE(args) != (Py_ssize_t)sizeof...(A)) throw Slow{};
        auto a = std::make_unique<Args>(Args{unmarshal<A>(PyTuple_GET_ITEM(args, I))...});
        static PyMethodDef def = {"bound", call, METH_NOARGS, nullptr};
        PyObject* self = PyCapsule_New(a.get(), kName, drop);
        if (self == nullptr) throw Slow{};
        a.release();
        PyObject* f = PyCFunction_New(&def, self);
        Py_DECREF(self);
        if (f == nullptr) throw Slow{};
        return f;
    }
    static PyObject* make(PyObject* args) { return make(args, std::index_sequence_for<A...>{}); }
};
struct Entry {
    const char* name;
    PyObject* (*make)(PyObject*);
};
#define ENTRY(name) {#name, Bound<name>::make}
const Entry g_entries[] = {ENTRY(tamoe_gate),           ENTRY(tamoe_select),          ENTRY(tamoe_aux_loss),    ENTRY(tamoe_dispatch),
                           ENTRY(tamoe_dispatch_padded), ENTRY(tamoe_dispatch_static), ENTRY(tamoe_gate_dispatch), ENTRY(tamoe_combine),
                           ENTRY(tamoe_combine_bwd),    ENTRY(tamoe_dispatch_bwd),    ENTRY(tamoe_gate_bwd),    ENTRY(tamoe_regroup),
                           ENTRY(tamoe_renorm_topk),    ENTRY(tamoe_renorm_topk_bwd)};

// bind(name, marshalled arguments) -> a function without arguments that returns the status
PyObject* n_bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
    try {
        if (n == 2 && PyUnicode_Check(a[0]) && PyTuple_CheckExact(a[1]))
            for (const Entry& e : g_entries)
                if (PyUnicode_CompareWithASCIIString(a[0], e.name) == 0) return e.make(a[1]);
    } catch (...) {   // the caller keeps its own way of calling
    }
    PyErr_Clear();
    return Py_NewRef(Py_NotImplemented);
}

#define FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(n_##name)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {FAST(gate),        FAST(gate_dispatch), FAST(aux_loss),     FAST(dispatch), FAST(combine),
                           FAST(combine_bwd), FAST(dispatch_bwd),  FAST(gate_bwd),     FAST(bind),     {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

PyObject* attribute(const char* module, const char* name) {
    PyObject* m = PyImport_ImportModule(module);
    if (m == nullptr) return nullptr;
    PyObject* v = PyObject_GetAttrString(m, name);
    Py_DECREF(m);
    return v;
}

}  // namespace

PyMODINIT_FUNC PyInit__native() {
    g_tensor = attribute("torch", "Tensor");
    g_parameter = attribute("torch.nn", "Parameter");
    if (g_tensor == nullptr || g_parameter == nullptr) return nullptr;
    static const Keys keys;
    g_keys = &keys;
    PyObject* m = PyModule_Create(&g_module);
    if (m != nullptr && PyModule_AddStringConstant(m, "torch_version", TAMOE_TORCH_VERSION) != 0) Py_CLEAR(m);
    return m;
}
