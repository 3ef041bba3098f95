// Argument marshalling of the three calls of a layer in native code: checks, output tensors, pointers and strides, the library call.
// In Python (binding.py) they cost 9 us a call, more than the kernels of the smallest layer: 26 us for three calls, 14 of them kernels.
//
// Nothing is decided here.  Each function takes the ordinary case, plain torch.Tensor arguments that pass every check, and returns
// None for anything else, and where torch throws before the launch: the Python function then goes on as if this module were not there,
// and raises what it raises.  After the launch nothing returns None, which would launch again.
// The library's entry points are handed over as addresses by bind(), from the one copy of the library that binding.py loaded.
#define PY_SSIZE_T_CLEAN
#include <ATen/ATen.h>
#include <Python.h>
#include <cxxabi.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

namespace {

using AppendFn = int32_t (*)(void *, const void *, const void *, int64_t, int64_t, int32_t, void *);
using PoolSelectFn = int32_t (*)(const void *, const void *, int64_t, int64_t, const void *, float *, int32_t *, int32_t *, float *, void *);
using ForwardFn = int32_t (*)(const void *, const void *, int64_t, int64_t, const void *, const int32_t *, const int32_t *, void *, int64_t, int64_t,
                              float *, float, void *);
AppendFn append_fn = nullptr;
PoolSelectFn pool_select_fn = nullptr;
ForwardFn forward_fn = nullptr;

// Geom._plan(): address of its C struct, heads, query blocks, head_dim, topk, tokens a frame, query frames, bf16
struct Plan {
    const void *geom;
    int64_t heads, n_qb, d, topk, frame, q_frames;
    at::ScalarType type;
    bool take(PyObject *t) {
        if (!PyTuple_CheckExact(t) || PyTuple_GET_SIZE(t) != 8) return false;
        int64_t v[8];
        for (int i = 0; i < 8; ++i) {
            v[i] = PyLong_AsLongLong(PyTuple_GET_ITEM(t, i));
            if (v[i] == -1 && PyErr_Occurred()) { PyErr_Clear(); return false; }
        }
        geom = (const void *)v[0];
        heads = v[1]; n_qb = v[2]; d = v[3]; topk = v[4]; frame = v[5]; q_frames = v[6];
        type = v[7] ? at::kBFloat16 : at::kFloat;
        return true;
    }
};

bool plain(PyObject *x) { return THPVariable_CheckExact(x); }
// [frames * frame][heads][d] of the element type on the GPU, d contiguous
bool tokens(const at::Tensor &x, const Plan &p, int64_t frames) {
    return x.is_cuda() && x.layout() == at::kStrided && x.dim() == 3 && x.stride(2) == 1 && x.scalar_type() == p.type &&
           x.size(0) == frames * p.frame && x.size(1) == p.heads && x.size(2) == p.d;
}
bool whole(const at::Tensor &x, at::ScalarType type, int64_t numel) {
    return x.is_cuda() && x.layout() == at::kStrided && x.scalar_type() == type && x.is_contiguous() && x.numel() == numel;
}
bool address(PyObject *x, void *&out) {
    out = PyLong_AsVoidPtr(x);
    if (!out && PyErr_Occurred()) { PyErr_Clear(); return false; }
    return true;
}

// What torch throws becomes None.  A thread that asks for the interpreter lock while the interpreter shuts down is ended by unwinding its
// stack, which must not be held up: the process would abort.  Hence, too, no handler around the lock given up and taken back.
#define LCSA_OR_NONE catch (abi::__forced_unwind &) { throw; } catch (...) { PyErr_Clear(); Py_RETURN_NONE; }

// Outputs are allocated without the interpreter lock, as torch.empty does it: a first allocation takes long.  False where torch throws.
template <typename F> bool allocated(F &&outputs) {
    try {
        outputs();
        return true;
    } catch (abi::__forced_unwind &) {
        throw;
    } catch (...) {
        return false;
    }
}

// The result as a Python object, or null with a Python error set.
PyObject *wrapped(at::Tensor &&x) {
    try {
        return THPVariable_Wrap(std::move(x));
    } catch (abi::__forced_unwind &) {
        throw;
    } catch (python_error &e) {
        e.restore();
    } catch (...) {
        PyErr_SetString(PyExc_RuntimeError, "a result could not be handed to Python");
    }
    return nullptr;
}

// append(plan, cache, k, v, n_frames, stream) -> status
PyObject *append(PyObject *, PyObject *const *a, Py_ssize_t n) {
    Plan p;
    void *cache, *stream;
    if (n != 6 || !p.take(a[0]) || !address(a[1], cache) || !plain(a[2]) || !plain(a[3]) || !PyLong_CheckExact(a[4]) || !address(a[5], stream)) Py_RETURN_NONE;
    const int64_t frames = PyLong_AsLongLong(a[4]);
    if (frames < 1 || frames > (1 << 30)) { PyErr_Clear(); Py_RETURN_NONE; }
    const void *kp, *vp;
    int64_t st, sh;
    try {
        const at::Tensor &k = THPVariable_Unpack(a[2]), &v = THPVariable_Unpack(a[3]);
        if (!tokens(k, p, frames) || !tokens(v, p, frames) || k.stride(0) != v.stride(0) || k.stride(1) != v.stride(1)) Py_RETURN_NONE;
        kp = k.data_ptr(); vp = v.data_ptr();
        st = k.stride(0); sh = k.stride(1);
    } LCSA_OR_NONE
    int32_t status;
    Py_BEGIN_ALLOW_THREADS
    status = append_fn(cache, kp, vp, st, sh, (int32_t)frames, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

// pool_select(plan, q, cache, want_gap, stream) -> (pooled_q, sel_idx, sel_cnt, gap) or status
PyObject *pool_select(PyObject *, PyObject *const *a, Py_ssize_t n) {
    Plan p;
    void *cache, *stream;
    if (n != 5 || !p.take(a[0]) || !plain(a[1]) || !address(a[2], cache) || !PyBool_Check(a[3]) || !address(a[4], stream)) Py_RETURN_NONE;
    const bool want_gap = a[3] == Py_True;
    at::Tensor pooled, idx, cnt, gap;
    at::TensorOptions on;
    const void *qp;
    int64_t st, sh;
    try {
        const at::Tensor &q = THPVariable_Unpack(a[1]);
        if (!tokens(q, p, p.q_frames)) Py_RETURN_NONE;
        on = on.device(q.device());
        qp = q.data_ptr();
        st = q.stride(0); sh = q.stride(1);
    } LCSA_OR_NONE
    int32_t status;
    bool launched;
    Py_BEGIN_ALLOW_THREADS
    float *pp, *gp = nullptr;
    int32_t *ip, *cp;
    launched = allocated([&] {
        pooled = at::empty({p.heads, p.n_qb, p.d}, on.dtype(at::kFloat));
        idx = at::empty({p.heads, p.n_qb, p.topk}, on.dtype(at::kInt));
        cnt = at::empty({p.heads, p.n_qb}, on.dtype(at::kInt));
        if (want_gap) gap = at::empty({p.heads, p.n_qb}, on.dtype(at::kFloat));
        pp = (float *)pooled.data_ptr(); ip = (int32_t *)idx.data_ptr(); cp = (int32_t *)cnt.data_ptr();
        if (want_gap) gp = (float *)gap.data_ptr();
    });
    if (launched) status = pool_select_fn(p.geom, qp, st, sh, cache, pp, ip, cp, gp, stream);
    Py_END_ALLOW_THREADS
    if (!launched) { PyErr_Clear(); Py_RETURN_NONE; }
    if (status != 0) return PyLong_FromLong(status);
    PyObject *out = PyTuple_New(4);
    if (!out) return nullptr;
    at::Tensor *results[4] = {&pooled, &idx, &cnt, &gap};
    for (int i = 0; i < 4; ++i) {
        PyObject *x = Py_None;
        if (results[i]->defined()) x = wrapped(std::move(*results[i]));
        else Py_INCREF(Py_None);
        if (!x) { Py_DECREF(out); return nullptr; }
        PyTuple_SET_ITEM(out, i, x);
    }
    return out;
}

// forward(plan, q, cache, sel_idx, sel_cnt, o or None, lse or None, scale, stream) -> o or status
PyObject *forward(PyObject *, PyObject *const *a, Py_ssize_t n) {
    Plan p;
    void *cache, *stream;
    if (n != 9 || !p.take(a[0]) || !plain(a[1]) || !address(a[2], cache) || !plain(a[3]) || !plain(a[4]) || !(a[5] == Py_None || plain(a[5])) ||
        !(a[6] == Py_None || plain(a[6])) || !PyFloat_CheckExact(a[7]) || !address(a[8], stream))
        Py_RETURN_NONE;
    const float scale = (float)PyFloat_AS_DOUBLE(a[7]);
    const bool own_o = a[5] == Py_None;
    at::Tensor o;
    at::TensorOptions as_q;
    const void *qp;
    const int32_t *ip, *cp;
    float *lse = nullptr;
    int64_t rows, st, sh;
    try {
        const at::Tensor &q = THPVariable_Unpack(a[1]), &idx = THPVariable_Unpack(a[3]), &cnt = THPVariable_Unpack(a[4]);
        // sel_cnt's number of values is not checked by the Python function either
        if (!tokens(q, p, p.q_frames) || !whole(idx, at::kInt, p.heads * p.n_qb * p.topk) || !whole(cnt, at::kInt, cnt.numel())) Py_RETURN_NONE;
        if (a[6] != Py_None) {
            const at::Tensor &l = THPVariable_Unpack(a[6]);
            if (!whole(l, at::kFloat, q.size(0) * p.heads) || l.dim() != 2 || l.size(0) != q.size(0)) Py_RETURN_NONE;
            lse = (float *)l.data_ptr();
        }
        if (!own_o) {
            o = THPVariable_Unpack(a[5]);
            if (!tokens(o, p, p.q_frames)) Py_RETURN_NONE;
        }
        as_q = as_q.device(q.device()).dtype(q.scalar_type());
        rows = q.size(0);
        qp = q.data_ptr();
        ip = (const int32_t *)idx.data_ptr(); cp = (const int32_t *)cnt.data_ptr();
        st = q.stride(0); sh = q.stride(1);
    } LCSA_OR_NONE
    int32_t status;
    bool launched;
    Py_BEGIN_ALLOW_THREADS
    void *op;
    launched = allocated([&] {
        if (own_o) o = at::empty({rows, p.heads, p.d}, as_q);
        op = o.data_ptr();
    });
    if (launched) status = forward_fn(p.geom, qp, st, sh, cache, ip, cp, op, o.stride(0), o.stride(1), lse, scale, stream);
    Py_END_ALLOW_THREADS
    if (!launched) { PyErr_Clear(); Py_RETURN_NONE; }
    if (status != 0) return PyLong_FromLong(status);
    if (!own_o) { Py_INCREF(a[5]); return a[5]; }
    return wrapped(std::move(o));
}

// bind(addresses of lcsa_kv_cache_append, lcsa_pool_select_blocks, lcsa_sparse_attn_fwd)
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n) {
    void *f[3];
    if (n != 3) { PyErr_SetString(PyExc_TypeError, "bind: three addresses"); return nullptr; }
    for (int i = 0; i < 3; ++i)
        if (!address(a[i], f[i]) || !f[i]) { PyErr_SetString(PyExc_TypeError, "bind: three addresses"); return nullptr; }
    append_fn = (AppendFn)f[0];
    pool_select_fn = (PoolSelectFn)f[1];
    forward_fn = (ForwardFn)f[2];
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, nullptr},
    {"append", (PyCFunction)(void (*)(void))append, METH_FASTCALL, nullptr},
    {"pool_select", (PyCFunction)(void (*)(void))pool_select, METH_FASTCALL, nullptr},
    {"forward", (PyCFunction)(void (*)(void))forward, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

extern "C" __attribute__((visibility("default"))) PyObject *PyInit__marshal() {
    PyObject *m = PyModule_Create(&module);
    // of the headers it was built with: tensors are read by their layout there
    if (m && PyModule_AddStringConstant(m, "torch_version", TORCH_VERSION) != 0) { Py_DECREF(m); return nullptr; }
    return m;
}
