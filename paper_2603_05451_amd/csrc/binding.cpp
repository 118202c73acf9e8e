// The well-formed calls of the Python binding, marshalled natively: a small call's time is its marshalling (per call, 60 in a row: forward
// and backward of 2 heads x 128 tokens 25 us for 15 us of kernels, a decode step of 8 x 16 heads against 273 keys 11.8 for 6.9; what an
// argument costs is its attributes read from Python and its ctypes conversion).  Every function here does what its namesake in
// __init__.py does for plain torch tensors that pass all of that function's checks, and returns None for anything else, without having
// done anything: the Python text then runs and raises what there is to raise.  An int is the library's error code.
#include <Python.h>
#include <ATen/ATen.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

#include "../../include/attn.h"

namespace {

// entry points of libattn.so, which the package loads: addresses given once (bind)
decltype(&attn_fwd_dtype) p_fwd = nullptr;
decltype(&attn_bwd_phases) p_bwd_phases = nullptr;
decltype(&attn_bwd_dtype) p_bwd_dtype = nullptr;
decltype(&attn_bwd_workspace_bytes) p_bwd_bytes = nullptr;
decltype(&attn_varlen_fwd_dtype) p_varlen_fwd = nullptr;
decltype(&attn_varlen_bwd_dtype) p_varlen_bwd = nullptr;
decltype(&attn_varlen_workspace_bytes) p_varlen_bytes = nullptr;
decltype(&attn_fwd_strided) p_fwd_strided = nullptr;
decltype(&attn_bwd_strided) p_bwd_strided = nullptr;
decltype(&attn_strided_workspace_bytes) p_strided_bytes = nullptr;
PyObject *get_device = nullptr, *get_stream = nullptr;      // torch._C._cuda_getDevice, _cuda_getCurrentRawStream
PyTypeObject* parameter = nullptr;                          // torch.nn.Parameter

using Sizes = std::initializer_list<int64_t>;

// A plain tensor (no subclass that may have a say in what happens to it), or null.
const at::Tensor* plain(PyObject* x)
{
    if (Py_TYPE(x) != (PyTypeObject*)THPVariableClass && Py_TYPE(x) != parameter) return nullptr;
    return &THPVariable_Unpack(x);
}

// Arguments of one call.  `ok` falls with the first that is not as the Python text wants it.
struct Call {
    bool ok = true;
    at::ScalarType type = at::kBFloat16;
    int dtype = ATTN_BF16;
    attn_strides_t strides[8];
    int nstrides = 0;

    bool fits(int64_t x)
    {
        if (x < 0 || x > 0x7fffffff) ok = false;
        return ok;
    }
    // the first tensor gives the element type
    const at::Tensor* first(PyObject* x, int64_t dims)
    {
        const at::Tensor* t = plain(x);
        if (!t || t->dim() != dims || !t->is_cuda()) { ok = false; return nullptr; }
        type = t->scalar_type();
        if (type != at::kBFloat16 && type != at::kHalf) ok = false;
        dtype = type == at::kHalf ? ATTN_F16 : ATTN_BF16;
        for (int64_t n : t->sizes()) fits(n);
        return ok ? t : nullptr;
    }
    const at::Tensor* other(PyObject* x, int64_t dims)
    {
        const at::Tensor* t = ok ? plain(x) : nullptr;
        if (!t || t->dim() != dims) { ok = false; return nullptr; }
        for (int64_t n : t->sizes()) fits(n);
        return ok ? t : nullptr;
    }
    void* dense(const at::Tensor& t, Sizes shape, at::ScalarType as)
    {
        if (!ok || !t.is_cuda() || t.scalar_type() != as || !t.is_contiguous() || t.sizes() != at::IntArrayRef(shape)) { ok = false; return nullptr; }
        return t.data_ptr();
    }
    void* view(const at::Tensor& t, Sizes shape)
    {
        if (!ok || !t.is_cuda() || t.scalar_type() != type || t.sizes() != at::IntArrayRef(shape) || (t.stride(3) != 1 && t.size(3) != 1)) { ok = false; return nullptr; }
        strides[nstrides++] = {t.stride(0), t.stride(1), t.stride(2)};
        return t.data_ptr();
    }
    // an optional output: the caller's, or (made by `make`, once every check has passed) a new one
    at::Tensor given(PyObject* x)
    {
        if (x == Py_None || !ok) return at::Tensor();
        const at::Tensor* t = plain(x);
        if (!t) ok = false;
        return t ? *t : at::Tensor();
    }
    double number(PyObject* x)
    {
        if (PyFloat_CheckExact(x)) return PyFloat_AS_DOUBLE(x);
        ok = false;
        return 0;
    }
    int truth(PyObject* x)
    {
        if (x == Py_True || x == Py_False) return x == Py_True;
        ok = false;
        return 0;
    }
    // the stream's handle, or the current one of the current device; called after every other check
    void* stream(PyObject* x)
    {
        PyObject* h = nullptr;
        if (x != Py_None) {
            h = PyObject_GetAttrString(x, "cuda_stream");
        } else if (PyObject* d = PyObject_CallNoArgs(get_device)) {
            h = PyObject_CallOneArg(get_stream, d);
            Py_DECREF(d);
        }
        void* s = h && PyLong_Check(h) ? PyLong_AsVoidPtr(h) : nullptr;
        if (!h || !PyLong_Check(h) || PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        Py_XDECREF(h);
        return s;
    }
};

int size(const at::Tensor* t, int dim) { return (int)t->size(dim); }       // (Call::fits)

at::Tensor make(const at::Tensor& like, Sizes shape) { return at::empty(shape, like.options().requires_grad(false)); }
at::Tensor make_f32(const at::Tensor& like, Sizes shape) { return at::empty(shape, like.options().requires_grad(false).dtype(at::kFloat)); }
at::Tensor make_bytes(const at::Tensor& like, size_t n)
{
    return at::empty({(int64_t)(n < 256 ? 256 : n)}, like.options().requires_grad(false).dtype(at::kByte));
}

// What goes back: the caller's own objects, or new tensors.
PyObject* out(PyObject* mine, const at::Tensor& t)
{
    if (mine != Py_None) { Py_INCREF(mine); return mine; }
    return THPVariable_Wrap(t);
}
PyObject* outs(int rc, std::initializer_list<std::pair<PyObject*, const at::Tensor*>> list)
{
    if (rc != ATTN_OK) return PyLong_FromLong(rc);
    PyObject* r = PyTuple_New((Py_ssize_t)list.size());
    Py_ssize_t i = 0;
    for (const auto& x : list) PyTuple_SET_ITEM(r, i++, out(x.first, *x.second));
    return r;
}

// Other Python threads run while this lives: allocations, which may wait for memory, and the library's call, as with torch.empty and ctypes.
struct Unlocked {
    PyThreadState* state = PyEval_SaveThread();
    Unlocked() = default;
    Unlocked(const Unlocked&) = delete;
    ~Unlocked() { PyEval_RestoreThread(state); }
};

#define NOT_HERE Py_RETURN_NONE

// q, k, v, scale, causal, o, lse, stream
PyObject* fwd(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    Call c;
    if (n != 8) NOT_HERE;
    const at::Tensor *q = c.first(a[0], 4), *k = c.other(a[1], 4), *v = c.other(a[2], 4);
    if (!c.ok) NOT_HERE;
    const int B = size(q, 0), N = size(q, 1), H = size(q, 2), dqk = size(q, 3), Hkv = size(k, 2), dv = size(v, 3);
    const double scale = c.number(a[3]);
    const int causal = c.truth(a[4]);
    at::Tensor o = c.given(a[5]), lse = c.given(a[6]);
    void *qp = c.dense(*q, {B, N, H, dqk}, c.type), *kp = c.dense(*k, {B, N, Hkv, dqk}, c.type), *vp = c.dense(*v, {B, N, Hkv, dv}, c.type);
    if (o.defined()) c.dense(o, {B, N, H, dv}, c.type);
    if (lse.defined()) c.dense(lse, {B, H, N}, at::kFloat);
    if (!c.ok) NOT_HERE;
    void* s = c.stream(a[7]);
    if (!c.ok) NOT_HERE;
    int rc;
    {
        Unlocked threads;
        if (!o.defined()) o = make(*q, {B, N, H, dv});
        if (!lse.defined()) lse = make_f32(*q, {B, H, N});
        rc = p_fwd(c.dtype, qp, kp, vp, o.data_ptr(), (float*)lse.data_ptr(), B, H, Hkv, N, dqk, dv, (float)scale, causal, s);
    }
    return outs(rc, {{a[5], &o}, {a[6], &lse}});
    END_HANDLE_TH_ERRORS
}

// q, k, v, o, do, lse, scale, causal, dq, dk, dv, workspace, stream, phases
PyObject* bwd(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    Call c;
    if (n != 14 || !PyLong_CheckExact(a[13])) NOT_HERE;
    const at::Tensor *q = c.first(a[0], 4), *k = c.other(a[1], 4), *v = c.other(a[2], 4), *o = c.other(a[3], 4), *g = c.other(a[4], 4), *lse = c.other(a[5], 3);
    if (!c.ok) NOT_HERE;
    const long phases = PyLong_AsLong(a[13]);
    if (PyErr_Occurred()) { PyErr_Clear(); NOT_HERE; }
    const int B = size(q, 0), N = size(q, 1), H = size(q, 2), dqk = size(q, 3), Hkv = size(k, 2), dvd = size(v, 3);
    const double scale = c.number(a[6]);
    const int causal = c.truth(a[7]);
    at::Tensor dq = c.given(a[8]), dk = c.given(a[9]), dv = c.given(a[10]), ws = c.given(a[11]);
    void *qp = c.dense(*q, {B, N, H, dqk}, c.type), *kp = c.dense(*k, {B, N, Hkv, dqk}, c.type), *vp = c.dense(*v, {B, N, Hkv, dvd}, c.type),
         *op = c.dense(*o, {B, N, H, dvd}, c.type), *gp = c.dense(*g, {B, N, H, dvd}, c.type), *lp = c.dense(*lse, {B, H, N}, at::kFloat);
    if (dq.defined()) c.dense(dq, {B, N, H, dqk}, c.type);
    if (dk.defined()) c.dense(dk, {B, N, Hkv, dqk}, c.type);
    if (dv.defined()) c.dense(dv, {B, N, Hkv, dvd}, c.type);
    if (!c.ok || (phases != ATTN_BWD_ALL && (c.type == at::kHalf || phases < 0 || phases > ATTN_BWD_ALL))) NOT_HERE;
    const size_t need = p_bwd_bytes(B, H, Hkv, N, dqk, dvd);
    if (need == 0 || (ws.defined() && !ws.is_cuda())) NOT_HERE;
    void* s = c.stream(a[12]);
    if (!c.ok) NOT_HERE;
    int rc;
    {
        Unlocked threads;
        if (!dq.defined()) dq = make(*q, {B, N, H, dqk});
        if (!dk.defined()) dk = make(*q, {B, N, Hkv, dqk});
        if (!dv.defined()) dv = make(*q, {B, N, Hkv, dvd});
        if (!ws.defined()) ws = make_bytes(*q, need);
        const size_t bytes = (size_t)ws.numel() * ws.element_size();
        rc = c.type == at::kHalf
            ? p_bwd_dtype(c.dtype, qp, kp, vp, op, gp, (float*)lp, dq.data_ptr(), dk.data_ptr(), dv.data_ptr(), B, H, Hkv, N, dqk, dvd, (float)scale, causal,
                          ws.data_ptr(), bytes, s)
            : p_bwd_phases(qp, kp, vp, op, gp, (float*)lp, dq.data_ptr(), dk.data_ptr(), dv.data_ptr(), B, H, Hkv, N, dqk, dvd, (float)scale, causal,
                           ws.data_ptr(), bytes, s, (int)phases);
    }
    return outs(rc, {{a[8], &dq}, {a[9], &dk}, {a[10], &dv}});
    END_HANDLE_TH_ERRORS
}

// Boundaries [B + 1] on the device; both given here (tables kept in a workspace: the Python text).
const int* boundaries(Call& c, PyObject* x, int B)
{
    const at::Tensor* t = c.ok ? plain(x) : nullptr;
    if (!t) { c.ok = false; return nullptr; }
    return (const int*)c.dense(*t, {(int64_t)B + 1}, at::kInt);
}

// q, k, v, cu_seqlens, scale, causal, o, lse, workspace, stream, cu_seqlens_k
PyObject* varlen_fwd(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    Call c;
    if (n != 11) NOT_HERE;
    const at::Tensor *q = c.first(a[0], 3), *k = c.other(a[1], 3), *v = c.other(a[2], 3), *cu = c.other(a[3], 1);
    if (!c.ok) NOT_HERE;
    const int T = size(q, 0), H = size(q, 1), dqk = size(q, 2), Tk = size(k, 0), Hkv = size(k, 1), dv = size(v, 2), B = size(cu, 0) - 1;
    const double scale = c.number(a[4]);
    const int causal = c.truth(a[5]);
    const int *cq = boundaries(c, a[3], B), *ck = a[10] == Py_None ? cq : boundaries(c, a[10], B);
    at::Tensor o = c.given(a[6]), lse = c.given(a[7]), ws = c.given(a[8]);
    void *qp = c.dense(*q, {T, H, dqk}, c.type), *kp = c.dense(*k, {Tk, Hkv, dqk}, c.type), *vp = c.dense(*v, {Tk, Hkv, dv}, c.type);
    if (o.defined()) c.dense(o, {T, H, dv}, c.type);
    if (lse.defined()) c.dense(lse, {H, T}, at::kFloat);
    if (!c.ok || B < 1) NOT_HERE;
    const size_t need = ws.defined() ? 0 : p_varlen_bytes(B, T, Tk, H, Hkv, dqk, dv, 0);
    void* s = c.stream(a[9]);
    if (!c.ok) NOT_HERE;
    int rc;
    {
        Unlocked threads;
        if (!o.defined()) o = make(*q, {T, H, dv});
        if (!lse.defined()) lse = make_f32(*q, {H, T});
        if (!ws.defined()) ws = make_bytes(*q, need);
        rc = p_varlen_fwd(c.dtype, qp, kp, vp, o.data_ptr(), (float*)lse.data_ptr(), cq, ck, B, T, Tk, H, Hkv, dqk, dv, (float)scale, causal,
                          ws.data_ptr(), (size_t)ws.numel(), s);
    }
    return outs(rc, {{a[6], &o}, {a[7], &lse}});
    END_HANDLE_TH_ERRORS
}

// q, k, v, o, d_o, lse, cu_seqlens, scale, causal, dq, dk, dv, workspace, stream, cu_seqlens_k
PyObject* varlen_bwd(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    Call c;
    if (n != 15) NOT_HERE;
    const at::Tensor *q = c.first(a[0], 3), *k = c.other(a[1], 3), *v = c.other(a[2], 3), *o = c.other(a[3], 3), *g = c.other(a[4], 3), *lse = c.other(a[5], 2),
                     *cu = c.other(a[6], 1);
    if (!c.ok) NOT_HERE;
    const int T = size(q, 0), H = size(q, 1), dqk = size(q, 2), Tk = size(k, 0), Hkv = size(k, 1), dvd = size(v, 2), B = size(cu, 0) - 1;
    const double scale = c.number(a[7]);
    const int causal = c.truth(a[8]);
    const int *cq = boundaries(c, a[6], B), *ck = a[14] == Py_None ? cq : boundaries(c, a[14], B);
    at::Tensor dq = c.given(a[9]), dk = c.given(a[10]), dv = c.given(a[11]), ws = c.given(a[12]);
    void *qp = c.dense(*q, {T, H, dqk}, c.type), *kp = c.dense(*k, {Tk, Hkv, dqk}, c.type), *vp = c.dense(*v, {Tk, Hkv, dvd}, c.type),
         *op = c.dense(*o, {T, H, dvd}, c.type), *gp = c.dense(*g, {T, H, dvd}, c.type), *lp = c.dense(*lse, {H, T}, at::kFloat);
    if (dq.defined()) c.dense(dq, {T, H, dqk}, c.type);
    if (dk.defined()) c.dense(dk, {Tk, Hkv, dqk}, c.type);
    if (dv.defined()) c.dense(dv, {Tk, Hkv, dvd}, c.type);
    if (!c.ok || B < 1) NOT_HERE;
    const size_t need = ws.defined() ? 0 : p_varlen_bytes(B, T, Tk, H, Hkv, dqk, dvd, 1);
    void* s = c.stream(a[13]);
    if (!c.ok) NOT_HERE;
    int rc;
    {
        Unlocked threads;
        if (!dq.defined()) dq = make(*q, {T, H, dqk});
        if (!dk.defined()) dk = make(*q, {Tk, Hkv, dqk});
        if (!dv.defined()) dv = make(*q, {Tk, Hkv, dvd});
        if (!ws.defined()) ws = make_bytes(*q, need);
        rc = p_varlen_bwd(c.dtype, qp, kp, vp, op, gp, (float*)lp, dq.data_ptr(), dk.data_ptr(), dv.data_ptr(), cq, ck, B, T, Tk, H, Hkv, dqk, dvd,
                          (float)scale, causal, ws.data_ptr(), (size_t)ws.numel(), s);
    }
    return outs(rc, {{a[9], &dq}, {a[10], &dk}, {a[11], &dv}});
    END_HANDLE_TH_ERRORS
}

// q, k, v, scale, causal, o, lse, workspace, stream
PyObject* fwd_strided(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    Call c;
    if (n != 9) NOT_HERE;
    const at::Tensor *q = c.first(a[0], 4), *k = c.other(a[1], 4), *v = c.other(a[2], 4);
    if (!c.ok) NOT_HERE;
    const int B = size(q, 0), N = size(q, 1), H = size(q, 2), dqk = size(q, 3), Nk = size(k, 1), Hkv = size(k, 2), dv = size(v, 3);
    const double scale = c.number(a[3]);
    const int causal = c.truth(a[4]);
    at::Tensor o = c.given(a[5]), lse = c.given(a[6]), ws = c.given(a[7]);
    if (o.defined() && o.dim() != 4) NOT_HERE;
    void *qp = c.view(*q, {B, N, H, dqk}), *kp = c.view(*k, {B, Nk, Hkv, dqk}), *vp = c.view(*v, {B, Nk, Hkv, dv});
    if (o.defined()) c.view(o, {B, N, H, dv});
    if (lse.defined()) c.dense(lse, {B, H, N}, at::kFloat);
    if (!c.ok) NOT_HERE;
    const size_t need = ws.defined() ? 0 : p_strided_bytes(B, H, Hkv, N, Nk, dqk, dv, 0);
    void* s = c.stream(a[8]);
    if (!c.ok) NOT_HERE;
    int rc;
    {
        Unlocked threads;
        if (!o.defined()) { o = make(*q, {B, N, H, dv}); c.view(o, {B, N, H, dv}); }
        if (!lse.defined()) lse = make_f32(*q, {B, H, N});
        if (!ws.defined()) ws = make_bytes(*q, need);
        const attn_strides_t* st = c.strides;
        rc = p_fwd_strided(c.dtype, qp, st, kp, st + 1, vp, st + 2, o.data_ptr(), st + 3, (float*)lse.data_ptr(), B, H, Hkv, N, Nk, dqk, dv, (float)scale,
                           causal, ws.data_ptr(), (size_t)ws.numel(), s);
    }
    return outs(rc, {{a[5], &o}, {a[6], &lse}});
    END_HANDLE_TH_ERRORS
}

// q, k, v, o, d_o, lse, scale, causal, dq, dk, dv, workspace, stream
PyObject* bwd_strided(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    Call c;
    if (n != 13) NOT_HERE;
    const at::Tensor *q = c.first(a[0], 4), *k = c.other(a[1], 4), *v = c.other(a[2], 4), *o = c.other(a[3], 4), *g = c.other(a[4], 4), *lse = c.other(a[5], 3);
    if (!c.ok) NOT_HERE;
    const int B = size(q, 0), N = size(q, 1), H = size(q, 2), dqk = size(q, 3), Nk = size(k, 1), Hkv = size(k, 2), dvd = size(v, 3);
    const double scale = c.number(a[6]);
    const int causal = c.truth(a[7]);
    at::Tensor dq = c.given(a[8]), dk = c.given(a[9]), dv = c.given(a[10]), ws = c.given(a[11]);
    for (const at::Tensor* t : {&dq, &dk, &dv}) if (t->defined() && t->dim() != 4) NOT_HERE;
    void *qp = c.view(*q, {B, N, H, dqk}), *kp = c.view(*k, {B, Nk, Hkv, dqk}), *vp = c.view(*v, {B, Nk, Hkv, dvd}), *op = c.view(*o, {B, N, H, dvd}),
         *gp = c.view(*g, {B, N, H, dvd}), *lp = c.dense(*lse, {B, H, N}, at::kFloat);
    // (checked here; their strides are taken below, in the order of the call, once the missing ones exist)
    const int inputs = c.nstrides;
    if (dq.defined()) c.view(dq, {B, N, H, dqk});
    if (dk.defined()) c.view(dk, {B, Nk, Hkv, dqk});
    if (dv.defined()) c.view(dv, {B, Nk, Hkv, dvd});
    if (!c.ok) NOT_HERE;
    const size_t need = ws.defined() ? 0 : p_strided_bytes(B, H, Hkv, N, Nk, dqk, dvd, 1);
    void* s = c.stream(a[12]);
    if (!c.ok) NOT_HERE;
    int rc;
    {
        Unlocked threads;
        if (!dq.defined()) dq = make(*q, {B, N, H, dqk});
        if (!dk.defined()) dk = make(*q, {B, Nk, Hkv, dqk});
        if (!dv.defined()) dv = make(*q, {B, Nk, Hkv, dvd});
        if (!ws.defined()) ws = make_bytes(*q, need);
        c.nstrides = inputs;
        c.view(dq, {B, N, H, dqk});
        c.view(dk, {B, Nk, Hkv, dqk});
        c.view(dv, {B, Nk, Hkv, dvd});
        const attn_strides_t* st = c.strides;
        rc = p_bwd_strided(c.dtype, qp, st, kp, st + 1, vp, st + 2, op, st + 3, gp, st + 4, (float*)lp, dq.data_ptr(), st + 5, dk.data_ptr(), st + 6,
                           dv.data_ptr(), st + 7, B, H, Hkv, N, Nk, dqk, dvd, (float)scale, causal, ws.data_ptr(), (size_t)ws.numel(), s);
    }
    return outs(rc, {{a[8], &dq}, {a[9], &dk}, {a[10], &dv}});
    END_HANDLE_TH_ERRORS
}

// bind(ten addresses, in the order below; _cuda_getDevice, _cuda_getCurrentRawStream, Parameter)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    void** const to[] = {(void**)&p_fwd, (void**)&p_bwd_phases, (void**)&p_bwd_dtype, (void**)&p_bwd_bytes, (void**)&p_varlen_fwd, (void**)&p_varlen_bwd,
                         (void**)&p_varlen_bytes, (void**)&p_fwd_strided, (void**)&p_bwd_strided, (void**)&p_strided_bytes};
    if (n != 13 || !PyType_Check(a[12])) { PyErr_SetString(PyExc_TypeError, "bind: ten addresses, two functions, a type"); return nullptr; }
    for (int i = 0; i < 10; ++i) {
        *to[i] = PyLong_AsVoidPtr(a[i]);
        if (PyErr_Occurred()) return nullptr;
    }
    for (int i = 10; i < 13; ++i) Py_INCREF(a[i]);
    get_device = a[10];
    get_stream = a[11];
    parameter = (PyTypeObject*)a[12];
    Py_RETURN_NONE;
}

#define METHOD(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(bind), METHOD(fwd), METHOD(bwd), METHOD(varlen_fwd), METHOD(varlen_bwd), METHOD(fwd_strided), METHOD(bwd_strided),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject* PyInit__binding() { return PyModule_Create(&module); }
