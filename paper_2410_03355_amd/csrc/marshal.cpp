// The host half of the step calls: checks, outputs and the call of the C entry points, without the interpreter in between.
//
// Small calls are bound by the host: 64 rows of 1024 logits take 8 us on the device, and checking five tensors,
// allocating two, asking for the stream and converting fourteen arguments takes 12 us in Python.  Calls one after the
// other, through Python and ctypes / through here: 64 rows of 1024 fp32 12.5 / 7.8 us, one tree of 60 on V = 16384 bf16
// 19.5 / 15.3, 16 trees under greedy decoding 20.2 / 11.8; from some 50 us on the device upwards there is no difference.
//
// Every function here takes the ordinary call alone: plain dense device tensors of the right types and shapes, no
// stream or output of the caller's, no interpreter modes, nothing empty.  For anything else it returns None and has done
// nothing; binding.py then goes through its own checks, which word the errors.  Otherwise the result is what the
// entry's Python function returns, or the C entry's status as an int where that is not zero.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <climits>

#include "lantern.h"

namespace {

// The entry points, in the library that binding.py has loaded (set once, before the first call).
decltype(&lantern_verify) c_verify;
decltype(&lantern_verify_rows) c_verify_rows;
decltype(&lantern_decide_rows) c_decide_rows;
decltype(&lantern_verify_greedy) c_verify_greedy;
decltype(&lantern_verify_greedy_rows) c_verify_greedy_rows;
decltype(&lantern_verify_trees) c_verify_trees;
decltype(&lantern_verify_trees_greedy) c_verify_trees_greedy;
decltype(&lantern_verify_trees_sequential) c_verify_trees_sequential;
decltype(&lantern_verify_trees_sequential_workspace_bytes) c_sequential_bytes;
decltype(&lantern_accept_chains) c_accept_chains;
decltype(&lantern_accept_trees) c_accept_trees;

// Interpreter modes see every torch call of the Python functions: with one active those run.
bool modes_active() {
    return at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set();
}

// A plain device tensor, or null: no subclass, no wrapper of a transformation, memory of its own.
const at::Tensor* plain(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    static const c10::DispatchKeySet wrappers({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched,
                                               c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize,
                                               c10::DispatchKey::Batched});
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage() || t.key_set().has_any(wrappers))
        return nullptr;
    return &t;
}
const at::Tensor* plain(PyObject* o, at::ScalarType type) {   // contiguous as well
    const at::Tensor* t = plain(o);
    return t && t->scalar_type() == type && t->is_contiguous() ? t : nullptr;
}

bool real(PyObject* o, float* out) {
    if (PyFloat_CheckExact(o)) {
        *out = (float)PyFloat_AS_DOUBLE(o);
        return true;
    }
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    const long v = PyLong_AsLongAndOverflow(o, &over);
    *out = (float)(double)v;
    return !over;
}
// A whole number in [1, INT_MAX].
bool count(PyObject* o, int* out) {
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    const long v = PyLong_AsLongAndOverflow(o, &over);
    if (over || v < 1 || v > INT_MAX) return false;
    *out = (int)v;
    return true;
}
bool bound_name(PyObject* o, int* out) {
    if (!PyUnicode_CheckExact(o)) return false;
    if (PyUnicode_CompareWithASCIIString(o, "tvd") == 0) *out = LANTERN_DIV_TVD;
    else if (PyUnicode_CompareWithASCIIString(o, "jsd") == 0) *out = LANTERN_DIV_JSD;
    else return false;
    return true;
}

// Logit rows, tokens, table and draws of a call.
struct Call {
    const at::Tensor* target = nullptr;
    const void* draft = nullptr;
    const int32_t *tokens = nullptr, *knn = nullptr, *row_index = nullptr;
    const float* uniforms = nullptr;
    lantern_dtype dtype = LANTERN_F32;
    int R = 0, V = 0, N = 0, k = 0, divergence = LANTERN_DIV_TVD;
    int64_t stride = 0;
    float delta = 0.f;

    bool rows(PyObject* t_obj, PyObject* g_obj) {
        target = plain(t_obj);
        if (!target || target->dim() != 2 || target->stride(1) != 1) return false;
        if (target->scalar_type() == at::kFloat) dtype = LANTERN_F32;
        else if (target->scalar_type() == at::kBFloat16) dtype = LANTERN_BF16;
        else return false;
        const int64_t r = target->size(0), v = target->size(1);
        if (r < 1 || r > INT_MAX || v < 1 || v > INT_MAX) return false;
        R = (int)r;
        V = (int)v;
        stride = R > 1 ? target->stride(0) : V;
        if (!g_obj) return true;
        const at::Tensor* g = plain(g_obj);
        if (!g || g->scalar_type() != target->scalar_type() || g->sizes() != target->sizes() || g->strides() != target->strides())
            return false;
        draft = g->const_data_ptr();
        return true;
    }
    bool rest(PyObject* index, PyObject* tok, PyObject* table, PyObject* delta_obj, PyObject* uni) {
        const at::Tensor* t = plain(tok, at::kInt);
        const at::Tensor* q = plain(table, at::kInt);
        if (!t || !q || t->numel() < 1 || t->numel() > INT_MAX || q->dim() != 2 || q->size(0) != V || q->size(1) < 1 ||
            q->size(1) > INT_MAX || !real(delta_obj, &delta))
            return false;
        N = (int)t->numel();
        k = (int)q->size(1);
        tokens = t->const_data_ptr<int32_t>();
        knn = q->const_data_ptr<int32_t>();
        if (index == Py_None) {
            if (R != N) return false;
        } else {
            const at::Tensor* i = plain(index, at::kInt);
            if (!i || i->numel() != N) return false;
            row_index = i->const_data_ptr<int32_t>();
        }
        if (!uni) return true;
        const at::Tensor* u = plain(uni, at::kFloat);
        if (!u || u->numel() != 2 * (int64_t)N) return false;
        uniforms = u->const_data_ptr<float>();
        return true;
    }
    at::Tensor ints(at::IntArrayRef size) const {
        return at::empty(size, at::TensorOptions().dtype(at::kInt).device(target->device()));
    }
};

// Parents of B trees of M nodes, B * M of them.
const int32_t* parents(PyObject* par, int N, int M, int* B) {
    const at::Tensor* p = plain(par, at::kInt);
    if (!p || p->numel() != N || N % M) return nullptr;
    *B = N / M;
    return p->const_data_ptr<int32_t>();
}

void* current_stream() { return c10::hip::getCurrentHIPStream().stream(); }
int32_t* data(at::Tensor& t) { return t.mutable_data_ptr<int32_t>(); }

// Runs `work` without the interpreter's lock.  It allocates, calls the entry point and returns its status.  False:
// it threw, so the call is left to the Python function, which meets the same error and reports it.
template <typename F>
bool unlocked(F work, int* status) {
    bool ok = true;
    Py_BEGIN_ALLOW_THREADS
    try {
        *status = work();
    } catch (...) {
        ok = false;
    }
    Py_END_ALLOW_THREADS
    return ok;
}

template <typename... T>
PyObject* result(int status, T&... tensors) {
    if (status != LANTERN_OK) return PyLong_FromLong(status);
    PyObject* out = PyTuple_New(sizeof...(T));
    if (!out) return nullptr;
    Py_ssize_t i = 0;
    for (at::Tensor* t : {&tensors...}) {
        PyObject* o = nullptr;
        try {
            o = THPVariable_Wrap(std::move(*t));
        } catch (...) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, "an output could not be returned");
        }
        if (!o) {
            Py_DECREF(out);
            return nullptr;
        }
        PyTuple_SET_ITEM(out, i++, o);
    }
    return out;
}

// The arguments as in the Python functions, positional, without outputs and stream.
#define ORDINARY(n, ...)                                              \
    try {                                                             \
        if (nargs != (n) || modes_active() || !(__VA_ARGS__)) Py_RETURN_NONE; \
    } catch (...) { /* a tensor without plain sizes or memory */       \
        Py_RETURN_NONE;                                               \
    }
#define RUN(...) \
    if (!unlocked([&]() -> int { __VA_ARGS__ }, &status)) Py_RETURN_NONE;

// target, draft, tokens, knn, delta, uniforms
PyObject* verify(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    Call c;
    ORDINARY(6, c.rows(a[0], a[1]) && c.rest(Py_None, a[2], a[3], a[4], a[5]))
    at::Tensor acc, res;
    int status = 0;
    RUN(acc = c.ints({c.N}); res = c.ints({c.N});
        return c_verify(c.target->const_data_ptr(), c.draft, c.dtype, c.N, c.V, c.stride, c.tokens, c.knn, c.k, c.delta,
                        c.uniforms, data(acc), data(res), current_stream());)
    return result(status, acc, res);
}

// target, draft, row_index, tokens, knn, delta, uniforms, divergence
PyObject* verify_rows(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    Call c;
    ORDINARY(8, a[2] != Py_None && c.rows(a[0], a[1]) && c.rest(a[2], a[3], a[4], a[5], a[6]) && bound_name(a[7], &c.divergence))
    at::Tensor acc, res;
    int status = 0;
    RUN(acc = c.ints({c.N}); res = c.ints({c.N});
        return c_verify_rows(c.target->const_data_ptr(), c.draft, c.dtype, c.R, c.V, c.stride, c.row_index, c.N, c.tokens,
                             c.knn, c.k, c.divergence, c.delta, c.uniforms, data(acc), data(res), current_stream());)
    return result(status, acc, res);
}

// target, draft, row_index, tokens, knn, delta, uniforms, divergence
PyObject* decide_rows(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    Call c;
    ORDINARY(8, c.rows(a[0], a[1]) && c.rest(a[2], a[3], a[4], a[5], a[6]) && bound_name(a[7], &c.divergence))
    at::Tensor acc;
    int status = 0;
    RUN(acc = c.ints({c.N});
        return c_decide_rows(c.target->const_data_ptr(), c.draft, c.dtype, c.R, c.V, c.stride, c.row_index, c.N, c.tokens,
                             c.knn, c.k, c.divergence, c.delta, c.uniforms, data(acc), nullptr, current_stream());)
    PyObject* one = result(status, acc);
    if (!one || status != LANTERN_OK) return one;
    PyObject* out = PyTuple_GET_ITEM(one, 0);
    Py_INCREF(out);
    Py_DECREF(one);
    return out;
}

// target, tokens, knn, delta
PyObject* verify_greedy(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    Call c;
    ORDINARY(4, c.rows(a[0], nullptr) && c.rest(Py_None, a[1], a[2], a[3], nullptr))
    at::Tensor acc, tok;
    int status = 0;
    RUN(acc = c.ints({c.N}); tok = c.ints({c.N});
        return c_verify_greedy(c.target->const_data_ptr(), c.dtype, c.N, c.V, c.stride, c.tokens, c.knn, c.k, c.delta,
                               data(acc), data(tok), nullptr, current_stream());)
    return result(status, acc, tok);
}

// target, row_index, tokens, knn, delta
PyObject* verify_greedy_rows(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    Call c;
    ORDINARY(5, a[1] != Py_None && c.rows(a[0], nullptr) && c.rest(a[1], a[2], a[3], a[4], nullptr))
    at::Tensor acc, tok;
    int status = 0;
    RUN(acc = c.ints({c.N}); tok = c.ints({c.N});
        return c_verify_greedy_rows(c.target->const_data_ptr(), c.dtype, c.R, c.V, c.stride, c.row_index, c.N, c.tokens,
                                    c.knn, c.k, c.delta, data(acc), data(tok), current_stream());)
    return result(status, acc, tok);
}

// target, draft, row_index, parent, M, tokens, knn, delta, uniforms, divergence
PyObject* verify_trees(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    Call c;
    int M = 0, B = 0;
    const int32_t* par = nullptr;
    ORDINARY(10, c.rows(a[0], a[1]) && c.rest(a[2], a[5], a[6], a[7], a[8]) && bound_name(a[9], &c.divergence) &&
                     count(a[4], &M) && (par = parents(a[3], c.N, M, &B)))
    at::Tensor acc, len, path, next;
    int status = 0;
    RUN(acc = c.ints({c.N}); len = c.ints({B}); path = c.ints({B, M}); next = c.ints({B});
        return c_verify_trees(c.target->const_data_ptr(), c.draft, c.dtype, c.R, c.V, c.stride, c.row_index, par, B, M,
                              c.tokens, c.knn, c.k, c.divergence, c.delta, c.uniforms, data(acc), data(len), data(path),
                              data(next), current_stream());)
    return result(status, acc, len, path, next);
}

// target, draft, row_index, parent, M, tokens, knn, delta, uniforms, divergence, workspace
PyObject* verify_trees_sequential(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    Call c;
    int M = 0, B = 0;
    const int32_t* par = nullptr;
    const at::Tensor* given = nullptr;
    ORDINARY(11, c.rows(a[0], a[1]) && c.rest(a[2], a[5], a[6], a[7], a[8]) && bound_name(a[9], &c.divergence) &&
                     count(a[4], &M) && (par = parents(a[3], c.N, M, &B)) &&
                     (a[10] == Py_None || (given = plain(a[10]))))
    at::Tensor len, path, next, work;
    int status = 0;
    RUN(if (given) work = *given;
        else work = at::empty({(int64_t)std::max<size_t>(c_sequential_bytes(B, M, c.V), 256)},
                              at::TensorOptions().dtype(at::kByte).device(c.target->device()));
        len = c.ints({B}); path = c.ints({B, M}); next = c.ints({B});
        return c_verify_trees_sequential(c.target->const_data_ptr(), c.draft, c.dtype, c.R, c.V, c.stride, c.row_index, par,
                                         B, M, c.tokens, c.knn, c.k, c.divergence, c.delta, c.uniforms, data(len), data(path),
                                         data(next), work.mutable_data_ptr(), work.numel() * work.element_size(),
                                         current_stream());)
    return result(status, len, path, next);
}

// target, row_index, parent, M, tokens, knn, delta
PyObject* verify_trees_greedy(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    Call c;
    int M = 0, B = 0;
    const int32_t* par = nullptr;
    ORDINARY(7, c.rows(a[0], nullptr) && c.rest(a[1], a[4], a[5], a[6], nullptr) && count(a[3], &M) &&
                    (par = parents(a[2], c.N, M, &B)))
    at::Tensor acc, tok, len, path, next;
    int status = 0;
    RUN(acc = c.ints({c.N}); tok = c.ints({c.N}); len = c.ints({B}); path = c.ints({B, M}); next = c.ints({B});
        return c_verify_trees_greedy(c.target->const_data_ptr(), c.dtype, c.R, c.V, c.stride, c.row_index, par, B, M, c.tokens,
                                     c.knn, c.k, c.delta, data(acc), data(tok), data(len), data(path), data(next),
                                     current_stream());)
    return result(status, acc, tok, len, path, next);
}

// accept, resample, L
PyObject* accept_chains(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    Call c;
    int L = 0;
    const at::Tensor *acc = nullptr, *res = nullptr;
    ORDINARY(3, (acc = plain(a[0], at::kInt)) && (res = plain(a[1], at::kInt)) && count(a[2], &L) && acc->numel() >= 1 &&
                    acc->numel() == res->numel() && acc->numel() <= INT_MAX && acc->numel() % L == 0)
    c.target = acc;
    const int B = (int)(acc->numel() / L);
    at::Tensor kept, next;
    int status = 0;
    RUN(kept = c.ints({B}); next = c.ints({B});
        return c_accept_chains(acc->const_data_ptr<int32_t>(), res->const_data_ptr<int32_t>(), B, L, data(kept), data(next),
                               current_stream());)
    return result(status, kept, next);
}

// accept, resample, parent, M
PyObject* accept_trees(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    Call c;
    int M = 0, B = 0;
    const at::Tensor *acc = nullptr, *res = nullptr;
    const int32_t* par = nullptr;
    ORDINARY(4, (acc = plain(a[0], at::kInt)) && (res = plain(a[1], at::kInt)) && count(a[3], &M) && acc->numel() >= 1 &&
                    acc->numel() == res->numel() && acc->numel() <= INT_MAX &&
                    (par = parents(a[2], (int)acc->numel(), M, &B)))
    c.target = acc;
    at::Tensor len, path, next;
    int status = 0;
    RUN(len = c.ints({B}); path = c.ints({B, M}); next = c.ints({B});
        return c_accept_trees(acc->const_data_ptr<int32_t>(), res->const_data_ptr<int32_t>(), par, B, M, data(len), data(path),
                              data(next), current_stream());)
    return result(status, len, path, next);
}

// bind({"lantern_verify": address, ...})
PyObject* bind(PyObject*, PyObject* table) {
    const auto set = [&](auto& f, const char* name) {
        PyObject* v = PyDict_Check(table) ? PyDict_GetItemString(table, name) : nullptr;
        f = v ? reinterpret_cast<std::decay_t<decltype(f)>>(PyLong_AsVoidPtr(v)) : nullptr;
        if (!f && !PyErr_Occurred()) PyErr_SetString(PyExc_KeyError, name);
        return f != nullptr;
    };
    if (set(c_verify, "lantern_verify") && set(c_verify_rows, "lantern_verify_rows") &&
        set(c_decide_rows, "lantern_decide_rows") && set(c_verify_greedy, "lantern_verify_greedy") &&
        set(c_verify_greedy_rows, "lantern_verify_greedy_rows") && set(c_verify_trees, "lantern_verify_trees") &&
        set(c_verify_trees_greedy, "lantern_verify_trees_greedy") &&
        set(c_verify_trees_sequential, "lantern_verify_trees_sequential") &&
        set(c_sequential_bytes, "lantern_verify_trees_sequential_workspace_bytes") &&
        set(c_accept_chains, "lantern_accept_chains") && set(c_accept_trees, "lantern_accept_trees"))
        Py_RETURN_NONE;
    return nullptr;
}

#define FAST(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"bind", bind, METH_O, nullptr}, FAST(verify), FAST(verify_rows), FAST(decide_rows),
                         FAST(verify_greedy), FAST(verify_greedy_rows), FAST(verify_trees), FAST(verify_trees_sequential),
                         FAST(verify_trees_greedy), FAST(accept_chains), FAST(accept_trees), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// BUILT_FOR: the versions that these libraries' interfaces were compiled for (binding.py compares them).
PyMODINIT_FUNC PyInit__marshal() {
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "BUILT_FOR", LANTERN_BUILT_FOR) != 0) Py_CLEAR(m);
    return m;
}
