// Host path of the binding's small calls: argument checks, output allocation and the call into the C ABI
// without the interpreter in between.  A call of a few seeds is bound by its host side: of the 8.9 us of an
// 8-seed forward through Python and ctypes, 3.5 us are the launch itself.
//
// Every function here takes the arguments that nearly every call has -- plain contiguous tensors of the
// expected types and shapes on one GPU, no mode that wants to see the allocations -- and returns None for
// anything else: the Python code of the binding, which is complete by itself, then takes the call and
// raises what there is to raise.  A failed library call returns its status, an int.
#include "../../include/fsa.h"

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

namespace {

using at::Tensor;

PyObject* raw_stream = nullptr;                        // device index -> current stream's handle

// Addresses of the C ABI's entry points, set by bind(), with the types that fsa.h declares them with.
#define FSA_HOST_ENTRIES(X) X(fsa_sample_mean_fwd) X(fsa_sample_wmean_fwd) X(fsa_mean_replay_fwd) X(fsa_mean_bwd) \
                            X(fsa_mean_bwd_ws) X(fsa_mean_bwd_lp_ws) X(fsa_wmean_bwd_ws) \
                            X(fsa_mean_bwd_dense) X(fsa_mean_bwd_dense_workspace_bytes) X(fsa_mean_bwd_dense_pays)
struct {
#define FSA_HOST_MEMBER(name) decltype(&::name) name;
    FSA_HOST_ENTRIES(FSA_HOST_MEMBER)
#undef FSA_HOST_MEMBER
} abi;

// The tensor behind an argument, or nullptr for anything but a plain tensor or parameter.
const Tensor* tensor_of(PyObject* o) { return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }

bool plain(const Tensor* t, int64_t dim) { return t && t->is_cuda() && t->dim() == dim && t->is_contiguous(); }
bool plain(const Tensor* t, int64_t dim, at::ScalarType type) { return plain(t, dim) && t->scalar_type() == type; }
bool together(const Tensor& a, const Tensor& b) { return a.get_device() == b.get_device(); }

int float_code(const Tensor& t) {                      // fsa.h's dtype code, -1 for none
    switch (t.scalar_type()) {
        case at::kFloat: return FSA_F32;
        case at::kBFloat16: return FSA_BF16;
        case at::kHalf: return FSA_F16;
        default: return -1;
    }
}

bool observed() { return at::impl::torch_function_mode_enabled() || c10::impl::dispatch_mode_enabled(); }

// 1 or 2 fanouts from a list or tuple of plain ints; returns how many, 0 if they are anything else.
int fanouts_of(PyObject* seq, int32_t (&fan)[2]) {
    if (!PyList_CheckExact(seq) && !PyTuple_CheckExact(seq)) return 0;
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(seq);
    if (n < 1 || n > 2) return 0;
    for (Py_ssize_t i = 0; i < n; ++i) {
        PyObject* k = PySequence_Fast_GET_ITEM(seq, i);
        if (!PyLong_CheckExact(k)) return 0;
        int over = 0;
        const long v = PyLong_AsLongAndOverflow(k, &over);
        if (over || v < 1 || v > FSA_KMAX) return 0;         // the library refuses it: not here
        fan[i] = (int32_t)v;
    }
    return (int)n;
}

// Current stream of t's device; false with an error set.
bool stream_of(const Tensor& t, void** stream) {
    PyObject* index = PyLong_FromLong(t.get_device());
    if (!index) return false;
    PyObject* h = PyObject_CallOneArg(raw_stream, index);
    Py_DECREF(index);
    if (!h) return false;
    *stream = PyLong_AsVoidPtr(h);
    Py_DECREF(h);
    return !PyErr_Occurred();
}

PyObject* wrap(const Tensor& t) {
    if (t.defined()) return THPVariable_Wrap(t);
    Py_RETURN_NONE;
}

template <size_t N> PyObject* tuple_of(const Tensor (&t)[N]) {
    PyObject* r = PyTuple_New(N);
    if (!r) return nullptr;
    for (size_t i = 0; i < N; ++i) {
        PyObject* o = wrap(t[i]);
        if (!o) { Py_DECREF(r); return nullptr; }
        PyTuple_SET_ITEM(r, i, o);
    }
    return r;
}

template <typename T = void> T* data(const Tensor& t) { return t.defined() ? static_cast<T*>(t.data_ptr()) : nullptr; }
template <typename T = void> T* data(const Tensor* t) { return t ? static_cast<T*>(t->data_ptr()) : nullptr; }

// Allocations (which may wait for the driver) and the C call, with other threads free to run meanwhile.
template <typename F> int without_gil(F f) {
    struct Released {
        PyThreadState* state = PyEval_SaveThread();
        ~Released() { PyEval_RestoreThread(state); }
    } released;
    return f();
}

// What no check here foresees is the Python code's to report.
template <typename F> PyObject* or_none(F f) {
    try {
        return f();
    } catch (const std::exception&) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

// (indptr, indices, edge_weight | None, x, seeds, fanouts, seed, emit_h1, emit_ids)
//   -> (out, out_h1, ids1, ids2), weighted: (..., w1, w2)
PyObject* sample_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 9) Py_RETURN_NONE;
    return or_none([&]() -> PyObject* {
        const Tensor *indptr = tensor_of(a[0]), *indices = tensor_of(a[1]), *x = tensor_of(a[3]), *seeds = tensor_of(a[4]);
        const bool weighted = a[2] != Py_None;
        const Tensor* edge_w = weighted ? tensor_of(a[2]) : nullptr;
        int32_t fan[2] = {0, 0};
        const int hops = fanouts_of(a[5], fan);
        if (!hops || !PyLong_CheckExact(a[6]) || !PyBool_Check(a[7]) || !PyBool_Check(a[8]) || observed()) Py_RETURN_NONE;
        if (!plain(indptr, 1) || !plain(indices, 1, at::kInt) || !plain(x, 2) || !plain(seeds, 1, at::kInt)) Py_RETURN_NONE;
        const int itype = indptr->scalar_type() == at::kLong ? FSA_I64 : FSA_I32;
        const int code = float_code(*x);
        const int64_t B = seeds->size(0), N = x->size(0), D = x->size(1);
        if ((itype == FSA_I32 && indptr->scalar_type() != at::kInt) || code < 0 || indptr->size(0) != N + 1) Py_RETURN_NONE;
        if (!together(*x, *indptr) || !together(*x, *indices) || !together(*x, *seeds)) Py_RETURN_NONE;
        if (weighted && (!plain(edge_w, 1, at::kFloat) || edge_w->size(0) != indices->size(0) || !together(*x, *edge_w))) Py_RETURN_NONE;
        void* stream;
        if (!stream_of(*x, &stream)) return nullptr;
        const uint64_t seed = PyLong_AsUnsignedLongLongMask(a[6]);
        const bool emit_ids = a[8] == Py_True, two = hops == 2;
        const auto rows = at::TensorOptions().dtype(x->dtype()).device(x->device());
        const auto ids = rows.dtype(at::kInt), weights = rows.dtype(at::kFloat);
        const bool emit_h1 = two && a[7] == Py_True;
        Tensor o[6];
        const int rc = without_gil([&] {
            o[0] = at::empty({B, D}, rows);
            if (emit_h1) o[1] = at::empty({B, fan[0], D}, rows);
            if (emit_ids) o[2] = at::empty({B, fan[0]}, ids);
            if (emit_ids && two) o[3] = at::empty({B, fan[0], fan[1]}, ids);
            if (weighted && emit_ids) o[4] = at::empty({B, fan[0]}, weights);
            if (weighted && emit_ids && two) o[5] = at::empty({B, fan[0], fan[1]}, weights);
            return weighted ? abi.fsa_sample_wmean_fwd(data(indptr), itype, data<int32_t>(indices), data<float>(edge_w), N, data(x), code, D,
                                                   data<int32_t>(seeds), B, fan, hops, seed, data(o[0]), data(o[1]),
                                                   data<int32_t>(o[2]), data<int32_t>(o[3]), data<float>(o[4]), data<float>(o[5]), stream)
                            : abi.fsa_sample_mean_fwd(data(indptr), itype, data<int32_t>(indices), N, data(x), code, D, data<int32_t>(seeds), B,
                                                  fan, hops, seed, data(o[0]), data(o[1]), data<int32_t>(o[2]), data<int32_t>(o[3]),
                                                  stream);
        });
        if (rc != FSA_OK) return PyLong_FromLong(rc);
        if (weighted) return tuple_of(o);
        const Tensor four[4] = {o[0], o[1], o[2], o[3]};
        return tuple_of(four);
    });
}

// (x, ids1, ids2 | None, emit_h1) -> (out, out_h1)
PyObject* replay_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 4) Py_RETURN_NONE;
    return or_none([&]() -> PyObject* {
        const Tensor *x = tensor_of(a[0]), *ids1 = tensor_of(a[1]);
        const bool two = a[2] != Py_None;
        const Tensor* ids2 = two ? tensor_of(a[2]) : nullptr;
        if (!PyBool_Check(a[3]) || observed() || !plain(x, 2) || !plain(ids1, 2, at::kInt)) Py_RETURN_NONE;
        const int64_t B = ids1->size(0), k1 = ids1->size(1), N = x->size(0), D = x->size(1);
        const int code = float_code(*x);
        if (code < 0 || !together(*x, *ids1)) Py_RETURN_NONE;
        if (two && (!plain(ids2, 3, at::kInt) || ids2->size(0) != B || ids2->size(1) != k1 || !together(*x, *ids2))) Py_RETURN_NONE;
        const int64_t k2 = two ? ids2->size(2) : 0;
        if (k1 < 1 || k1 > FSA_KMAX || k2 > FSA_KMAX || (two && k2 < 1)) Py_RETURN_NONE;
        void* stream;
        if (!stream_of(*x, &stream)) return nullptr;
        const auto rows = at::TensorOptions().dtype(x->dtype()).device(x->device());
        const bool emit_h1 = two && a[3] == Py_True;
        Tensor o[2];
        const int rc = without_gil([&] {
            o[0] = at::empty({B, D}, rows);
            if (emit_h1) o[1] = at::empty({B, k1, D}, rows);
            return abi.fsa_mean_replay_fwd(data(x), code, D, N, data<int32_t>(ids1), data<int32_t>(ids2), B, (int32_t)k1, (int32_t)k2,
                                       data(o[0]), data(o[1]), stream);
        });
        return rc != FSA_OK ? PyLong_FromLong(rc) : tuple_of(o);
    });
}

// Which backward entry point a call goes to.
enum { kPlain, kWorkspace, kLowPrecision, kWeighted };

// (kind, grad_out, ids1, w1 | None, ids2 | None, w2 | None, grad_h1 | None, grad_x, workspace | None) -> 0
PyObject* bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 9) Py_RETURN_NONE;
    return or_none([&]() -> PyObject* {
        const long kind = PyLong_CheckExact(a[0]) ? PyLong_AsLong(a[0]) : -1;
        const Tensor* t[9] = {};
        for (int i = 1; i < 9; ++i) {
            if (a[i] == Py_None) continue;
            t[i] = tensor_of(a[i]);
            if (!t[i] || !t[i]->is_cuda() || !t[i]->is_contiguous()) Py_RETURN_NONE;
        }
        const Tensor *g = t[1], *ids1 = t[2], *w1 = t[3], *ids2 = t[4], *w2 = t[5], *gh = t[6], *gx = t[7], *ws = t[8];
        if (kind < kPlain || kind > kWeighted || observed() || !plain(g, 2) || !plain(ids1, 2, at::kInt) || !plain(gx, 2)) Py_RETURN_NONE;
        const int64_t B = ids1->size(0), k1 = ids1->size(1), D = g->size(1), N = gx->size(0);
        const int g_code = float_code(*g), x_code = float_code(*gx);
        if (g_code < 0 || x_code < 0 || (kind != kLowPrecision && (g_code != FSA_F32 || x_code != FSA_F32))) Py_RETURN_NONE;
        if (g->size(0) != B || gx->size(1) != D || (ids2 && (ids2->dim() != 3 || ids2->scalar_type() != at::kInt || ids2->size(0) != B || ids2->size(1) != k1))) Py_RETURN_NONE;
        const int64_t k2 = ids2 ? ids2->size(2) : 0;
        if (k1 < 1 || k1 > FSA_KMAX || k2 > FSA_KMAX || (ids2 && k2 < 1)) Py_RETURN_NONE;
        if (gh && (gh->dim() != 3 || gh->scalar_type() != g->scalar_type() || gh->size(0) != B || gh->size(1) != k1 || gh->size(2) != D)) Py_RETURN_NONE;
        if ((kind == kWeighted) != (w1 != nullptr) || (w1 && (!plain(w1, 2, at::kFloat) || w1->size(0) != B || w1->size(1) != k1))) Py_RETURN_NONE;
        if ((w1 && ids2) != (w2 != nullptr) || (w2 && (!plain(w2, 3, at::kFloat) || w2->size(0) != B || w2->size(1) != k1 || w2->size(2) != k2))) Py_RETURN_NONE;
        for (int i = 1; i < 9; ++i) {
            if (t[i] && !together(*gx, *t[i])) Py_RETURN_NONE;
        }
        void* stream;
        if (!stream_of(*gx, &stream)) return nullptr;
        const int64_t ws_bytes = ws ? (int64_t)ws->nbytes() : 0;
        const int32_t f1 = (int32_t)k1, f2 = (int32_t)k2;
        const int32_t *i1 = data<int32_t>(ids1), *i2 = data<int32_t>(ids2);
        const int rc = without_gil([&]() -> int {
            switch (kind) {
                case kPlain: return abi.fsa_mean_bwd(data<float>(g), data<float>(gh), i1, i2, B, f1, f2, D, data<float>(gx), N, stream);
                case kWorkspace: return abi.fsa_mean_bwd_ws(data<float>(g), data<float>(gh), i1, i2, B, f1, f2, D, data<float>(gx), N, data(ws), ws_bytes, stream);
                case kLowPrecision: return abi.fsa_mean_bwd_lp_ws(data(g), data(gh), g_code, i1, i2, B, f1, f2, D, data(gx), x_code, N, data(ws), ws_bytes, stream);
                default: return abi.fsa_wmean_bwd_ws(data<float>(g), data<float>(gh), i1, i2, data<float>(w1), data<float>(w2), B, f1, f2, D, data<float>(gx), N, data(ws), ws_bytes, stream);
            }
        });
        return PyLong_FromLong(rc);
    });
}

// (grad_out, ids1, ids2 | None, grad_h1 | None, num_nodes) -> grad_x of fsa_mean_bwd_dense, or False where it does not pay
PyObject* grad_dense(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 5) Py_RETURN_NONE;
    return or_none([&]() -> PyObject* {
        const Tensor *g = tensor_of(a[0]), *ids1 = tensor_of(a[1]);
        const bool two = a[2] != Py_None, slots = a[3] != Py_None;
        const Tensor *ids2 = two ? tensor_of(a[2]) : nullptr, *gh = slots ? tensor_of(a[3]) : nullptr;
        if (!PyLong_CheckExact(a[4]) || observed() || !plain(g, 2) || !plain(ids1, 2, at::kInt) || float_code(*g) < 0) Py_RETURN_NONE;
        const int64_t B = ids1->size(0), k1 = ids1->size(1), D = g->size(1), N = PyLong_AsLongLong(a[4]);
        if (N < 1 || g->size(0) != B || !together(*g, *ids1)) { PyErr_Clear(); Py_RETURN_NONE; }
        if (two && (!plain(ids2, 3, at::kInt) || ids2->size(0) != B || ids2->size(1) != k1 || !together(*g, *ids2))) Py_RETURN_NONE;
        const int64_t k2 = two ? ids2->size(2) : 0;
        if (k1 < 1 || k1 > FSA_KMAX || k2 > FSA_KMAX || (two && k2 < 1)) Py_RETURN_NONE;
        if (slots && (!two || !plain(gh, 3, g->scalar_type()) || gh->size(0) != B || gh->size(1) != k1 || gh->size(2) != D || !together(*g, *gh))) Py_RETURN_NONE;
        if (!abi.fsa_mean_bwd_dense_pays(B, (int32_t)k1, (int32_t)k2, D, float_code(*g), N)) Py_RETURN_FALSE;
        const int64_t need = abi.fsa_mean_bwd_dense_workspace_bytes(B, (int32_t)k1, (int32_t)k2, D, N);
        void* stream;
        if (!stream_of(*g, &stream)) return nullptr;
        const auto rows = at::TensorOptions().dtype(g->dtype()).device(g->device());
        Tensor grad_x, ws;                                   // (the workspace may go once the call is queued: same stream)
        const int rc = without_gil([&] {
            grad_x = at::empty({N, D}, rows);
            ws = at::empty({need}, rows.dtype(at::kByte));
            return abi.fsa_mean_bwd_dense(data(g), data(gh), float_code(*g), data<int32_t>(ids1), data<int32_t>(ids2), B, (int32_t)k1, (int32_t)k2, D,
                                          data(grad_x), N, data(ws), need, stream);
        });
        return rc != FSA_OK ? PyLong_FromLong(rc) : wrap(grad_x);
    });
}

// (raw_stream, {entry point: address})
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 2 || !PyDict_Check(a[1])) { PyErr_SetString(PyExc_TypeError, "a stream function and the entry points' addresses"); return nullptr; }
#define FSA_HOST_BIND(name)                                                                                             \
    {                                                                                                                   \
        PyObject* at = PyDict_GetItemString(a[1], #name);                                                               \
        if (!at) { PyErr_SetString(PyExc_TypeError, "no address for " #name); return nullptr; }                         \
        abi.name = reinterpret_cast<decltype(abi.name)>(PyLong_AsVoidPtr(at));                                          \
        if (PyErr_Occurred()) return nullptr;                                                                           \
    }
    FSA_HOST_ENTRIES(FSA_HOST_BIND)
#undef FSA_HOST_BIND
    Py_INCREF(a[0]);
    Py_XDECREF(raw_stream);
    raw_stream = a[0];
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(bind)), METH_FASTCALL, nullptr},
    {"sample_fwd", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(sample_fwd)), METH_FASTCALL, nullptr},
    {"replay_fwd", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(replay_fwd)), METH_FASTCALL, nullptr},
    {"bwd", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(bwd)), METH_FASTCALL, nullptr},
    {"grad_dense", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(grad_dense)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fsa_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fsa_host() { return PyModule_Create(&module); }
