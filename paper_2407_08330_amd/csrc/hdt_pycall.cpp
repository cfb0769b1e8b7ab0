// The three calls that every layer of a model makes, for Python: hdt_build_layout, hdt_attn_fwd and hdt_attn_bwd on plain torch
// tensors.  Checks, output tensors, addresses, stream and the call into libhdt in one piece of native code.
//
// A layer of a thousand positions is bound by the host: its kernels take 8 us each, and a call from the interpreter took 8.1 us
// (forward: two outputs 3.0, the launch 3.0, checks 1.0, ctypes 0.7), 11.5 (backward) and 6.7 (deferred build with its
// destruction); from here 5.2, 6.9 and 4.3.  A build that is waited for and a forward, 1000 positions x 12 heads: 25.4 -> 20.1
// us; with the backward, one head of 512 in fp32: 38.7 -> 28.3.
//
// Nothing is decided here that binding.py does not decide: a call whose arguments are not the plain case (a tensor subclass, a
// wrong shape or type, a tensor that has no storage, a torch function mode, ...) returns None before it has done anything, and
// binding.py's own path takes it, errors included.
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "hdt.h"

namespace {

decltype(&hdt_build_layout) build_layout_fn;
decltype(&hdt_attn_fwd) fwd_fn;
decltype(&hdt_attn_fwd_ws) fwd_ws_fn;
decltype(&hdt_attn_bwd) bwd_fn;
decltype(&hdt_attn_bwd_workspace_bytes) bwd_bytes_fn;

// What is not plain is refused by return values: a C++ exception takes 1.5 us, and the calls that the general path takes then
// pay for it (us, no native form - refused by an exception - by return values: forward with a numpy scale 9.0 - 10.8 - 9.1, backward
// 13.3 - 15.0 - 13.2, on another stream with a temporary workspace 19.4 - 21.1 - 19.7, deferred build with a numpy number 6.9 - 8.5 - 7.0).

const at::Tensor *plain(PyObject *o) { return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }

bool whole(PyObject *o, int64_t *v)
{
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    *v = PyLong_AsLongLongAndOverflow(o, &over);
    return !over;
}

bool whole32(PyObject *o, int32_t *v)
{
    int64_t w;
    if (!whole(o, &w) || w != (int32_t)w) return false;
    *v = (int32_t)w;
    return true;
}

bool address(PyObject *o, void **p)
{
    *p = nullptr;
    if (o == Py_None) return true;
    if (!PyLong_CheckExact(o)) return false;
    *p = PyLong_AsVoidPtr(o);
    if (*p || !PyErr_Occurred()) return true;
    PyErr_Clear();
    return false;
}

// a raw stream handle, or None: the current stream of the current device
bool stream_of(PyObject *o, hipStream_t *st)
{
    void *p;
    if (!address(o, &p)) return false;
    *st = o == Py_None ? c10::hip::getCurrentHIPStream().stream() : (hipStream_t)p;
    return true;
}

bool dense(const at::Tensor &t) { return t.is_cuda() && t.is_contiguous(); }

bool has_shape(const at::Tensor &t, int64_t b, int64_t h, int64_t n, int64_t d)
{
    const auto s = t.sizes();
    return s.size() == 4 && s[0] == b && s[1] == h && s[2] == n && s[3] == d;
}

// what the arguments of an attention call have in common
struct Call {
    const at::Tensor *q, *k, *v;
    void *layout;
    int64_t batch, n_pos, n_kv, heads, head_dim;
    float scale;
    hdt_dtype_t dtype;

    // a: (layout, batch, n_pos, n_kv, q, k, v, scale, ...)
    bool plain_case(PyObject *const *a)
    {
        if (!PyFloat_CheckExact(a[7])) return false;
        scale = (float)PyFloat_AS_DOUBLE(a[7]);
        if (!(q = plain(a[4])) || !(k = plain(a[5])) || !(v = plain(a[6]))) return false;
        if (!address(a[0], &layout) || !whole(a[1], &batch) || !whole(a[2], &n_pos) || !whole(a[3], &n_kv)) return false;
        if (q->dim() != 4 || q->scalar_type() != k->scalar_type() || q->scalar_type() != v->scalar_type()) return false;
        heads = q->size(1), head_dim = q->size(3);
        if (heads > INT32_MAX || head_dim > INT32_MAX) return false;
        if (q->scalar_type() == at::kBFloat16) dtype = HDT_BF16;
        else if (q->scalar_type() == at::kFloat) dtype = HDT_F32;
        else return false;
        return like_q(*q) && like_k(*k) && like_k(*v);
    }
    bool like_q(const at::Tensor &t) const { return dense(t) && has_shape(t, batch, heads, n_pos, head_dim); }
    bool like_k(const at::Tensor &t) const { return dense(t) && has_shape(t, batch, heads, n_kv, head_dim); }
};

// the caller's tensor (a plain one, or None), or a new one
at::Tensor given_or(PyObject *o, const at::Tensor &like) { return o == Py_None ? at::empty_like(like) : THPVariable_Unpack(o); }

bool plain_or_none(PyObject *o) { return o == Py_None || THPVariable_CheckExact(o); }

// runs f, which returns NULL without a Python error where the general path has to take the call; None then
template <typename F>
PyObject *guarded(F f)
{
    try {
        PyObject *r = at::impl::torch_function_mode_enabled() ? nullptr : f();
        if (r || PyErr_Occurred()) return r;
    } catch (...) {  // (torch's own exceptions: the general path meets them again and reports them)
        PyErr_Clear();
    }
    Py_RETURN_NONE;
}

PyObject *results(hdt_status_t st, std::initializer_list<at::Tensor> ts)
{
    if (st != HDT_OK) return PyLong_FromLong(st);
    PyObject *out = PyTuple_New((Py_ssize_t)ts.size());
    if (!out) return nullptr;
    Py_ssize_t i = 0;
    for (const at::Tensor &t : ts) {
        PyObject *w = THPVariable_Wrap(t);
        if (!w) {
            Py_DECREF(out);
            return nullptr;
        }
        PyTuple_SET_ITEM(out, i++, w);
    }
    return out;
}

// (layout, batch, n_pos, n_kv, q, k, v, scale, o, lse, workspace, stream) -> (o, lse), a status, or None
PyObject *attn_fwd(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 12) Py_RETURN_NONE;
    return guarded([&]() -> PyObject * {
        Call c;
        hipStream_t st;
        if (!c.plain_case(a) || !plain_or_none(a[8]) || !plain_or_none(a[9]) || !plain_or_none(a[10]) || !stream_of(a[11], &st)) return nullptr;
        const at::Tensor &q = *c.q, &k = *c.k, &v = *c.v;
        const void *pq = q.data_ptr(), *pk = k.data_ptr(), *pv = v.data_ptr();
        at::Tensor o = given_or(a[8], q);
        at::Tensor lse = a[9] == Py_None ? at::empty({c.batch, c.heads, c.n_pos}, q.options().dtype(at::kFloat))
                                        : THPVariable_Unpack(a[9]);
        void *po = o.data_ptr();
        float *pl = (float *)lse.data_ptr(), *pw = nullptr;
        size_t bytes = 0;
        if (a[10] != Py_None) {
            const at::Tensor &w = THPVariable_Unpack(a[10]);
            pw = (float *)w.data_ptr();
            bytes = (size_t)w.numel() * w.element_size();
        }
        hdt_status_t r;
        Py_BEGIN_ALLOW_THREADS
        r = a[10] != Py_None ? fwd_ws_fn((const hdt_layout_t *)c.layout, pq, pk, pv, po, pl, (int32_t)c.heads, (int32_t)c.head_dim,
                                         c.dtype, c.scale, pw, bytes, st)
                             : fwd_fn((const hdt_layout_t *)c.layout, pq, pk, pv, po, pl, (int32_t)c.heads, (int32_t)c.head_dim,
                                      c.dtype, c.scale, st);
        Py_END_ALLOW_THREADS
        return results(r, {o, lse});
    });
}

// (layout, batch, n_pos, n_kv, q, k, v, scale, o, lse, d_o, dq, dk, dv, workspace, stream) -> (dq, dk, dv), a status, or None
PyObject *attn_bwd(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 16) Py_RETURN_NONE;
    return guarded([&]() -> PyObject * {
        // a temporary workspace comes from the stream the kernels run on: the current one, that is
        if (a[14] == Py_None && a[15] != Py_None) return nullptr;
        Call c;
        hipStream_t st;
        if (!c.plain_case(a) || !plain(a[8]) || !plain(a[9]) || !plain(a[10]) || !stream_of(a[15], &st)) return nullptr;
        for (int i = 11; i <= 14; i++)
            if (!plain_or_none(a[i])) return nullptr;
        const at::Tensor &q = *c.q, &k = *c.k, &v = *c.v, &o = *plain(a[8]), &lse = *plain(a[9]), &d_o = *plain(a[10]);
        if (o.scalar_type() != q.scalar_type() || d_o.scalar_type() != q.scalar_type() || !c.like_q(o) || !c.like_q(d_o)) return nullptr;
        const void *pq = q.data_ptr(), *pk = k.data_ptr(), *pv = v.data_ptr(), *po = o.data_ptr(), *pd = d_o.data_ptr();
        const float *pl = (const float *)lse.data_ptr();
        at::Tensor dq = given_or(a[11], q), dk = given_or(a[12], k), dv = given_or(a[13], k), w;
        if (a[14] == Py_None) {
            size_t need;
            Py_BEGIN_ALLOW_THREADS  // (waits for the report of a cross-attention build)
            need = bwd_bytes_fn((const hdt_layout_t *)c.layout, (int32_t)c.heads, (int32_t)c.head_dim, c.dtype);
            Py_END_ALLOW_THREADS
            w = at::empty({(int64_t)std::max<size_t>(need, 16)}, q.options().dtype(at::kByte));
        } else {
            w = THPVariable_Unpack(a[14]);
        }
        void *pdq = dq.data_ptr(), *pdk = dk.data_ptr(), *pdv = dv.data_ptr(), *pw = w.data_ptr();
        const size_t bytes = (size_t)w.numel() * w.element_size();
        hdt_status_t r;
        Py_BEGIN_ALLOW_THREADS
        r = bwd_fn((const hdt_layout_t *)c.layout, pq, pk, pv, po, pl, pd, pdq, pdk, pdv, (int32_t)c.heads, (int32_t)c.head_dim,
                   c.dtype, c.scale, pw, bytes, st);
        Py_END_ALLOW_THREADS
        return results(r, {dq, dk, dv});
    });
}

// (level, parent, tile_m, tile_n, force_dense, no_sort, windowed, edges, deferred, capacity, stream)
//   -> (handle, batch, n_pos), a status, or None
PyObject *build_layout(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 11) Py_RETURN_NONE;
    return guarded([&]() -> PyObject * {
        hdt_layout_opts_t opts = {};
        hipStream_t st;
        for (int i = 4; i <= 8; i++)
            if (i != 7 && !PyBool_Check(a[i])) return nullptr;
        if (!plain(a[0]) || !plain(a[1]) || !whole32(a[2], &opts.tile_m) || !whole32(a[3], &opts.tile_n) || !whole32(a[7], &opts.edges) ||
            !whole(a[9], &opts.capacity))
            return nullptr;
        opts.force_dense = a[4] == Py_True;
        opts.no_sort = a[5] == Py_True;
        opts.windowed = a[6] == Py_True;
        opts.deferred = a[8] == Py_True;
        const at::Tensor &level = *plain(a[0]), &parent = *plain(a[1]);
        if (level.scalar_type() != at::kInt || parent.scalar_type() != at::kInt || level.dim() != 2 || !dense(level) || !dense(parent) ||
            level.sizes() != parent.sizes())
            return nullptr;
        const int64_t B = level.size(0), N = level.size(1);
        if (B > INT32_MAX || N > INT32_MAX || !stream_of(a[10], &st)) return nullptr;
        const int32_t *pl = B * N ? (const int32_t *)level.data_ptr() : nullptr, *pp = B * N ? (const int32_t *)parent.data_ptr() : nullptr;
        hdt_layout_t *h = nullptr;
        hdt_status_t r;
        Py_BEGIN_ALLOW_THREADS
        r = build_layout_fn(pl, pp, (int32_t)B, (int32_t)N, &opts, st, &h);
        Py_END_ALLOW_THREADS
        if (r != HDT_OK) return PyLong_FromLong(r);
        return Py_BuildValue("(KLL)", (unsigned long long)(uintptr_t)h, (long long)B, (long long)N);
    });
}

// the addresses of libhdt's functions, in the order of the pointers above
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 5) {
        PyErr_SetString(PyExc_TypeError, "bind takes five addresses");
        return nullptr;
    }
    void *p[5];
    for (int i = 0; i < 5; i++)
        if (!(p[i] = PyLong_AsVoidPtr(a[i]))) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "bind: NULL");
            return nullptr;
        }
    build_layout_fn = (decltype(build_layout_fn))p[0];
    fwd_fn = (decltype(fwd_fn))p[1];
    fwd_ws_fn = (decltype(fwd_ws_fn))p[2];
    bwd_fn = (decltype(bwd_fn))p[3];
    bwd_bytes_fn = (decltype(bwd_bytes_fn))p[4];
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, nullptr},
    {"build_layout", (PyCFunction)(void (*)(void))build_layout, METH_FASTCALL, nullptr},
    {"attn_fwd", (PyCFunction)(void (*)(void))attn_fwd, METH_FASTCALL, nullptr},
    {"attn_bwd", (PyCFunction)(void (*)(void))attn_bwd, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_hdt_pycall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__hdt_pycall()
{
    PyObject *m = PyModule_Create(&module);
    // (binding.py uses the module under this torch alone: nothing else says that its tensors are laid out as in these headers)
    if (m && PyModule_AddStringConstant(m, "torch_version", HDT_TORCH_VERSION) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
