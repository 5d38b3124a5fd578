// Python module _launch: the per-call path of the ctypes binding (binding.py) as native code.
//
// A call of the binding costs the host a dozen tensor checks, one to four allocations and a ctypes
// call before its kernel is queued, in Python more than the small kernels run.  The
// functions here do the same checks and allocations on the tensors' C++ objects and call the library
// through the addresses that bind() was given.  Host time per call, Python path -> this one: forward
// 14.1 -> 6.0 us, backward 20.2 -> 10.5, without allocation 21.6 -> 7.6, one inference step 14.1 -> 6.2, ten
// in one call 82 -> 24.  They decide nothing: a call that is not plainly valid
// (another tensor type, a failed check, an argument that does not convert, an active mode, another
// current device) gets None, and the Python code goes through it in full, which also words the
// errors.  Otherwise they return the outputs, or the library's status code if that is not 0.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/EmptyTensor.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/hip/EmptyTensor.h>
#include <ATen/record_function.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <vector>

#include "hmar_attn.h"

namespace {

decltype(&hmar_attn_fwd_masked) g_fwd = nullptr;
decltype(&hmar_attn_bwd_masked) g_bwd = nullptr;
decltype(&hmar_attn_bwd_noalloc) g_bwd_noalloc = nullptr;
decltype(&hmar_attn_bwd_workspace_bytes_masked) g_ws_bytes = nullptr;
decltype(&hmar_attn_steps_fwd) g_steps = nullptr;
decltype(&hmar_attn_step_fwd_rows) g_rows = nullptr;

// A build for tests on hosts without a GPU (-DHMAR_LAUNCH_HOST) takes host tensors and the null stream.
#ifdef HMAR_LAUNCH_HOST
bool on_gpu(const at::Tensor&) { return true; }
bool current(const at::Device&) { return true; }
void* stream_of(const at::Tensor&) { return nullptr; }
#else
bool on_gpu(const at::Tensor& t) { return t.is_cuda(); }
bool current(const at::Device& d) { return d.index() == c10::hip::current_device(); }
void* stream_of(const at::Tensor& q) { return c10::hip::getCurrentHIPStream(q.device().index()).stream(); }
#endif

// Under a function transform (torch.func.grad and its like) an operation gives a wrapper without memory of its own,
// whatever it was given.
bool has_memory(const at::Tensor& t) { return t.unsafeGetTensorImpl()->has_storage(); }

// A plain tensor with memory of its own (no subclass, no wrapper of a function transform), or null.
const at::Tensor* plain(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !on_gpu(t) || t.layout() != at::kStrided || !has_memory(t)) return nullptr;
    return &t;
}

// the same, contiguous, of this type and shape, on this device
const at::Tensor* checked(PyObject* o, at::ScalarType type, at::IntArrayRef shape, at::Device device) {
    const at::Tensor* t = plain(o);
    return t && t->scalar_type() == type && t->sizes() == shape && t->device() == device && t->is_contiguous() ? t : nullptr;
}

const at::Tensor* checked_q(PyObject* o) {
    const at::Tensor* t = plain(o);
    return t && t->scalar_type() == at::kBFloat16 && t->dim() == 4 && t->is_contiguous() ? t : nullptr;
}

// The outputs and the launch below are what the caller sees only if no mode wants to see the calls.
bool ready(const at::Tensor& q) {
    return !at::impl::torch_function_mode_enabled() && !c10::impl::TorchDispatchModeTLS::any_modes_set() &&
           current(q.device());
}

bool to_int(PyObject* o, int64_t* out) {
    if (!PyLong_CheckExact(o)) return false;
    *out = PyLong_AsLongLong(o);
    if (*out == -1 && PyErr_Occurred()) { PyErr_Clear(); return false; }
    return *out >= INT32_MIN && *out <= INT32_MAX;
}

bool to_scale(PyObject* o, float* out) {
    if (!PyFloat_CheckExact(o)) return false;
    *out = (float)PyFloat_AS_DOUBLE(o);
    return true;
}

struct Sizes { const int32_t* array; int32_t count; int64_t L; };
bool to_sizes(PyObject* address, PyObject* count, PyObject* L, Sizes* out) {
    int64_t n = 0;
    if (!to_int(count, &n) || !PyLong_CheckExact(address)) return false;
    out->array = static_cast<const int32_t*>(PyLong_AsVoidPtr(address));
    out->count = (int32_t)n;
    out->L = PyLong_AsLongLong(L);
    if (PyErr_Occurred()) { PyErr_Clear(); return false; }
    return out->array != nullptr;
}

// New tensors: at::empty, without its way through the dispatcher (0.3 us of a call's 5 each) where nothing waits on
// that way; looked up once a call (0.05 us).  What can wait there:
//  - dispatch keys beyond the ones every thread has (function transforms, dispatch modes and the like add theirs);
//  - observers of operators (the profiler);
//  - the fill that torch.use_deterministic_algorithms asks of new memory (torch.utils.deterministic's
//    fill_uninitialized_memory), which is part of the operator: a row list leaves rows unwritten.
// (A kernel that a program registers in place of aten::empty's own is not looked for.)
bool nothing_waits() {
    return (c10::impl::tls_local_dispatch_key_set().included_ - c10::default_included_set).empty() && !at::hasCallbacks() &&
           !(at::globalContext().deterministicAlgorithms() && at::globalContext().deterministicFillUninitializedMemory());
}
at::Tensor fresh(at::IntArrayRef shape, at::ScalarType type, const at::Tensor& q, bool direct) {
    if (!direct) return at::empty(shape, q.options().dtype(type));
#ifdef HMAR_LAUNCH_HOST
    return at::Tensor(at::detail::empty_cpu(shape, type));
#else
    return at::Tensor(at::detail::empty_cuda(shape, type, q.device(), std::nullopt));
#endif
}

// an output tensor the caller gave (checked), or a new one (direct: nothing_waits())
bool output(PyObject* given, at::ScalarType type, at::IntArrayRef shape, const at::Tensor& q, bool direct, at::Tensor* out) {
    if (given == Py_None) {
        *out = fresh(shape, type, q, direct);
        return has_memory(*out);
    }
    const at::Tensor* t = checked(given, type, shape, q.device());
    if (!t) return false;
    *out = *t;
    return true;
}

PyObject* result(hmar_status code, std::initializer_list<at::Tensor> outs) {
    if (code != HMAR_OK) return PyLong_FromLong(code);
    PyObject* r = PyTuple_New((Py_ssize_t)outs.size());
    if (!r) return nullptr;
    Py_ssize_t i = 0;
    for (const at::Tensor& t : outs) {
        PyObject* o = THPVariable_Wrap(t);
        if (!o) { Py_DECREF(r); return nullptr; }
        PyTuple_SET_ITEM(r, i++, o);
    }
    return r;
}

// Exceptions of the tensor library (out of memory above all) are met again, and reported, by the Python path.
template <typename F>
PyObject* guarded(F&& body) {
    try {
        return body();
    } catch (const std::exception&) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

// The GIL is free while this lives.  Everything that can throw or needs Python (pointers and sizes of tensors, the
// stream) is fetched before; should the call throw all the same, the GIL is taken again on the way out.
struct GilReleased {
    PyThreadState* state = PyEval_SaveThread();
    GilReleased() = default;
    GilReleased(const GilReleased&) = delete;
    GilReleased& operator=(const GilReleased&) = delete;
    ~GilReleased() { PyEval_RestoreThread(state); }
};
template <typename F>
hmar_status without_gil(F&& call) {
    const GilReleased released;
    return call();
}

float* floats(const at::Tensor& t) { return static_cast<float*>(t.data_ptr()); }

// bind(addresses of the library's functions)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 6) { PyErr_SetString(PyExc_TypeError, "bind takes six addresses"); return nullptr; }
    void* p[6];
    for (int i = 0; i < 6; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (!p[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address");
            return nullptr;
        }
    }
    g_fwd = reinterpret_cast<decltype(g_fwd)>(p[0]);
    g_bwd = reinterpret_cast<decltype(g_bwd)>(p[1]);
    g_bwd_noalloc = reinterpret_cast<decltype(g_bwd_noalloc)>(p[2]);
    g_ws_bytes = reinterpret_cast<decltype(g_ws_bytes)>(p[3]);
    g_steps = reinterpret_cast<decltype(g_steps)>(p[4]);
    g_rows = reinterpret_cast<decltype(g_rows)>(p[5]);
    Py_RETURN_NONE;
}

// fwd(Q, K, V, O, LSE, sizes address, count, L, mask kind, scale)
PyObject* fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        Sizes s; int64_t kind; float scale;
        if (n != 10 || !g_fwd || !to_sizes(a[5], a[6], a[7], &s) || !to_int(a[8], &kind) || !to_scale(a[9], &scale)) Py_RETURN_NONE;
        const at::Tensor* q = checked_q(a[0]);
        if (!q || q->size(2) != s.L || !ready(*q)) Py_RETURN_NONE;
        const at::Tensor* k = checked(a[1], at::kBFloat16, q->sizes(), q->device());
        const at::Tensor* v = checked(a[2], at::kBFloat16, q->sizes(), q->device());
        const bool direct = nothing_waits();
        at::Tensor o, lse;
        if (!k || !v || !output(a[3], at::kBFloat16, q->sizes(), *q, direct, &o) ||
            !output(a[4], at::kFloat, q->sizes().slice(0, 3), *q, direct, &lse))
            Py_RETURN_NONE;
        void* stream = stream_of(*q);
        const void *Q = q->data_ptr(), *K = k->data_ptr(), *V = v->data_ptr();
        void* O = o.data_ptr();
        float* LSE = floats(lse);
        const int32_t B = (int32_t)q->size(0), H = (int32_t)q->size(1), D = (int32_t)q->size(3);
        const hmar_status code = without_gil([&] {
            return g_fwd(Q, K, V, O, LSE, s.array, s.count, (int32_t)kind, B, H, D, scale, stream);
        });
        return result(code, {o, lse});
    });
}

// bwd(Q, K, V, O, dO, LSE, dQ, dK, dV, workspace, sizes address, count, L, mask kind, scale)
PyObject* bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        Sizes s; int64_t kind; float scale;
        if (n != 15 || !g_bwd || !to_sizes(a[10], a[11], a[12], &s) || !to_int(a[13], &kind) || !to_scale(a[14], &scale)) Py_RETURN_NONE;
        const at::Tensor* q = checked_q(a[0]);
        if (!q || q->size(2) != s.L || !ready(*q)) Py_RETURN_NONE;
        const at::Tensor* in[4];                          // K, V, O, dO
        for (int i = 0; i < 4; ++i)
            if (!(in[i] = checked(a[1 + i], at::kBFloat16, q->sizes(), q->device()))) Py_RETURN_NONE;
        const at::Tensor* lse = checked(a[5], at::kFloat, q->sizes().slice(0, 3), q->device());
        if (!lse) Py_RETURN_NONE;
        const bool direct = nothing_waits();
        at::Tensor out[3], ws;
        for (int i = 0; i < 3; ++i)
            if (!output(a[6 + i], at::kBFloat16, q->sizes(), *q, direct, &out[i])) Py_RETURN_NONE;
        const int32_t B = (int32_t)q->size(0), H = (int32_t)q->size(1), D = (int32_t)q->size(3);
        if (a[9] == Py_None) {
            const int64_t need = (int64_t)g_ws_bytes(s.array, s.count, (int32_t)kind, B, H, D);
            ws = fresh({need < 16 ? 16 : need}, at::kByte, *q, direct);
            if (!has_memory(ws)) Py_RETURN_NONE;
        } else {
            const at::Tensor* t = plain(a[9]);
            if (!t || t->device() != q->device()) Py_RETURN_NONE;
            ws = *t;
        }
        void* stream = stream_of(*q);
        const void *Q = q->data_ptr(), *K = in[0]->data_ptr(), *V = in[1]->data_ptr(), *O = in[2]->data_ptr(), *dO = in[3]->data_ptr();
        const float* LSE = floats(*lse);
        void *dQ = out[0].data_ptr(), *dK = out[1].data_ptr(), *dV = out[2].data_ptr(), *workspace = ws.data_ptr();
        const size_t ws_bytes = (size_t)ws.numel() * ws.element_size();
        const hmar_status code = without_gil([&] {
            return g_bwd(Q, K, V, O, dO, LSE, dQ, dK, dV, s.array, s.count, (int32_t)kind, B, H, D, scale, workspace, ws_bytes, stream);
        });
        return result(code, {out[0], out[1], out[2]});
    });
}

// bwd_noalloc(Q, K, V, O, dO, LSE, dQ, dK, dV, sizes address, count, L, scale)
PyObject* bwd_noalloc(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        Sizes s; float scale;
        if (n != 13 || !g_bwd_noalloc || !to_sizes(a[9], a[10], a[11], &s) || !to_scale(a[12], &scale)) Py_RETURN_NONE;
        const at::Tensor* q = checked_q(a[0]);
        if (!q || q->size(2) != s.L || !ready(*q)) Py_RETURN_NONE;
        const at::Tensor* t[9] = {q};
        for (int i = 1; i < 9; ++i) {
            t[i] = i == 5 ? checked(a[5], at::kFloat, q->sizes().slice(0, 3), q->device())
                          : checked(a[i], at::kBFloat16, q->sizes(), q->device());
            if (!t[i]) Py_RETURN_NONE;
        }
        void* stream = stream_of(*q);
        void* p[9];
        for (int i = 0; i < 9; ++i) p[i] = t[i]->data_ptr();
        const int32_t B = (int32_t)q->size(0), H = (int32_t)q->size(1), D = (int32_t)q->size(3);
        const hmar_status code = without_gil([&] {
            return g_bwd_noalloc(p[0], p[1], p[2], p[3], p[4], static_cast<const float*>(p[5]), p[6], p[7], p[8], s.array, s.count,
                                 B, H, D, scale, stream);
        });
        if (code != HMAR_OK) return PyLong_FromLong(code);
        return PyTuple_Pack(3, a[6], a[7], a[8]);
    });
}

// The tensors of one inference step; false if a check fails.
struct Step { at::Tensor q, k, v, o, lse; int64_t n_prev; };       // owners: lists can change while the GIL is free
bool to_step(PyObject* Q, PyObject* K, PyObject* V, PyObject* n_prev, PyObject* O, PyObject* LSE, bool direct, Step* s) {
    const at::Tensor* q = checked_q(Q);
    if (!q || !to_int(n_prev, &s->n_prev)) return false;
    const int64_t kv[4] = {q->size(0), q->size(1), s->n_prev + q->size(2), q->size(3)};
    const at::Tensor* k = checked(K, at::kBFloat16, kv, q->device());
    const at::Tensor* v = checked(V, at::kBFloat16, kv, q->device());
    if (!k || !v || !output(O, at::kBFloat16, q->sizes(), *q, direct, &s->o) ||
        !output(LSE, at::kFloat, q->sizes().slice(0, 3), *q, direct, &s->lse))
        return false;
    s->q = *q;
    s->k = *k;
    s->v = *v;
    return true;
}

// step(Q, K, V, n_prev, O, LSE, scale)
PyObject* step(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        Step s; float scale;
        if (n != 7 || !g_steps || !to_scale(a[6], &scale)) Py_RETURN_NONE;
        const at::Tensor* q = checked_q(a[0]);
        if (!q || !ready(*q) || !to_step(a[0], a[1], a[2], a[3], a[4], a[5], nothing_waits(), &s)) Py_RETURN_NONE;
        void* stream = stream_of(*q);
        const void *Q = q->data_ptr(), *K = s.k.data_ptr(), *V = s.v.data_ptr();
        void* O = s.o.data_ptr();
        float* LSE = floats(s.lse);
        const int32_t n_prev = (int32_t)s.n_prev, n_cur = (int32_t)q->size(2);
        const int32_t B = (int32_t)q->size(0), H = (int32_t)q->size(1), D = (int32_t)q->size(3);
        const hmar_status code = without_gil([&] {
            return g_steps(&Q, &K, &V, &O, &LSE, &n_prev, &n_cur, 1, B, H, D, scale, stream);
        });
        return result(code, {s.o, s.lse});
    });
}

// rows(Q, K, V, n_prev, rows, O, LSE, scale)
PyObject* rows(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        Step s; float scale;
        if (n != 8 || !g_rows || !to_scale(a[7], &scale)) Py_RETURN_NONE;
        const at::Tensor* q = checked_q(a[0]);
        if (!q || !ready(*q) || !to_step(a[0], a[1], a[2], a[3], a[5], a[6], nothing_waits(), &s)) Py_RETURN_NONE;
        const at::Tensor* r = plain(a[4]);
        if (!r || r->device() != q->device() || r->scalar_type() != at::kInt || r->dim() != 1 || !r->is_contiguous() ||
            r->numel() < 1 || r->numel() > q->size(2))
            Py_RETURN_NONE;
        void* stream = stream_of(*q);
        const void *Q = q->data_ptr(), *K = s.k.data_ptr(), *V = s.v.data_ptr();
        void* O = s.o.data_ptr();
        float* LSE = floats(s.lse);
        const int32_t* list = static_cast<const int32_t*>(r->data_ptr());
        const int32_t n_rows = (int32_t)r->numel(), n_cur = (int32_t)q->size(2);
        const int32_t B = (int32_t)q->size(0), H = (int32_t)q->size(1), D = (int32_t)q->size(3);
        const hmar_status code = without_gil([&] {
            return g_rows(Q, K, V, O, LSE, list, n_rows, (int32_t)s.n_prev, n_cur, B, H, D, scale, stream);
        });
        return result(code, {s.o, s.lse});
    });
}

// steps(Qs, Ks, Vs, n_prevs, Os, LSEs, scale): exact lists or tuples; Os, LSEs lists or None; gives two lists
PyObject* steps(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        float scale;
        if (n != 7 || !g_steps || !to_scale(a[6], &scale)) Py_RETURN_NONE;
        for (int i = 0; i < 6; ++i)
            if (!(PyList_CheckExact(a[i]) || PyTuple_CheckExact(a[i]) || (i > 3 && a[i] == Py_None))) Py_RETURN_NONE;
        const Py_ssize_t count = PySequence_Fast_GET_SIZE(a[0]);
        if (count < 1) Py_RETURN_NONE;
        for (int i = 1; i < 6; ++i)
            if (a[i] != Py_None && PySequence_Fast_GET_SIZE(a[i]) != count) Py_RETURN_NONE;
        std::vector<Step> s((size_t)count);
        std::vector<const void*> Q((size_t)count), K((size_t)count), V((size_t)count);
        std::vector<void*> O((size_t)count);
        std::vector<float*> LSE((size_t)count);
        std::vector<int32_t> n_prev((size_t)count), n_cur((size_t)count);
        const at::Tensor* first = checked_q(PySequence_Fast_GET_ITEM(a[0], 0));
        if (!first || !ready(*first)) Py_RETURN_NONE;
        const at::Tensor q0 = *first;
        const bool direct = nothing_waits();
        for (Py_ssize_t i = 0; i < count; ++i) {
            auto item = [&](int k) { return a[k] == Py_None ? Py_None : PySequence_Fast_GET_ITEM(a[k], i); };
            Step& x = s[(size_t)i];
            if (!to_step(item(0), item(1), item(2), item(3), item(4), item(5), direct, &x)) Py_RETURN_NONE;
            if (x.q.size(0) != q0.size(0) || x.q.size(1) != q0.size(1) || x.q.size(3) != q0.size(3) ||
                x.q.device() != q0.device())
                Py_RETURN_NONE;
            Q[(size_t)i] = x.q.data_ptr(); K[(size_t)i] = x.k.data_ptr(); V[(size_t)i] = x.v.data_ptr();
            O[(size_t)i] = x.o.data_ptr(); LSE[(size_t)i] = floats(x.lse);
            n_prev[(size_t)i] = (int32_t)x.n_prev; n_cur[(size_t)i] = (int32_t)x.q.size(2);
        }
        void* stream = stream_of(q0);
        const int32_t B = (int32_t)q0.size(0), H = (int32_t)q0.size(1), D = (int32_t)q0.size(3);
        const hmar_status code = without_gil([&] {
            return g_steps(Q.data(), K.data(), V.data(), O.data(), LSE.data(), n_prev.data(), n_cur.data(), (int32_t)count, B, H, D,
                           scale, stream);
        });
        if (code != HMAR_OK) return PyLong_FromLong(code);
        PyObject *os = PyList_New(count), *lses = PyList_New(count);
        if (!os || !lses) { Py_XDECREF(os); Py_XDECREF(lses); return nullptr; }
        for (Py_ssize_t i = 0; i < count; ++i) {
            PyObject *o = THPVariable_Wrap(s[(size_t)i].o), *l = THPVariable_Wrap(s[(size_t)i].lse);
            if (!o || !l) { Py_XDECREF(o); Py_XDECREF(l); Py_DECREF(os); Py_DECREF(lses); return nullptr; }
            PyList_SET_ITEM(os, i, o);
            PyList_SET_ITEM(lses, i, l);
        }
        PyObject* r = PyTuple_Pack(2, os, lses);
        Py_DECREF(os);
        Py_DECREF(lses);
        return r;
    });
}

#define HMAR_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(name)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {HMAR_METHOD(bind), HMAR_METHOD(fwd), HMAR_METHOD(bwd), HMAR_METHOD(bwd_noalloc), HMAR_METHOD(step),
                           HMAR_METHOD(rows), HMAR_METHOD(steps), {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_launch", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__launch(void) { return PyModule_Create(&g_module); }
