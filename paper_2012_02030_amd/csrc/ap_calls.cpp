// Host path of the attention calls: from torch tensors to one C-ABI call, in native code.
//
// The binding's own marshalling (shape checks, three or four small arrays, ~30 converted arguments,
// attribute lookups) takes longer than the kernels of a short call: 16 us a forward call in which
// the kernels take 5 to 9 us.  The functions here do the same for the ordinary form of a call: plain
// torch tensors on a GPU, in the shapes, types and strides that the binding accepts, no outputs
// supplied by the caller, no tensor mode or transform active.  Anything else returns None before
// anything was done, and the binding's general path takes the call, or refuses it with its own
// message.  A call returns its output tensors, or the C ABI's status if that is not AP_OK.
//
// The library is not linked: the binding hands over the addresses of the functions of the library
// that it has loaded.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstring>
#include <initializer_list>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_strided.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "ap.h"

namespace {

struct Api {
    decltype(&ap_sparse_attn_fwd) fwd;
    decltype(&ap_sparse_attn_fwd_cropped) fwd_cropped;
    decltype(&ap_fwd_split_workspace_bytes) split_bytes;
    decltype(&ap_sparse_attn_fwd_split) split;
    decltype(&ap_sparse_attn_decode) decode;
    decltype(&ap_sparse_attn_entmax15_fwd) entmax_fwd;
    decltype(&ap_bwd_workspace_bytes) bwd_bytes;
    decltype(&ap_sparse_attn_bwd) bwd;
    decltype(&ap_sparse_attn_bwd_sched) bwd_sched;
    decltype(&ap_entmax15_bwd_workspace_bytes) entmax_bytes;
    decltype(&ap_sparse_attn_entmax15_bwd) entmax_bwd;
} api;
bool bound = false;
PyObject* get_device = nullptr;                              // torch._C._cuda_getDevice
PyObject* get_stream = nullptr;                              // torch._C._cuda_getCurrentRawStream

// A tensor whose memory a kernel can use as it stands: exactly torch.Tensor (or Parameter), strided, on a
// GPU, and no wrapper of a transform.
const at::Tensor* plain(PyObject* o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage()) return nullptr;
    using K = c10::DispatchKey;
    const auto ks = t.unsafeGetTensorImpl()->key_set();
    for (K k : {K::Python, K::FuncTorchBatched, K::FuncTorchGradWrapper, K::BatchedNestedTensor, K::Functionalize})
        if (ks.has(k)) return nullptr;
    return &t;
}

bool modes_active()
{
    return at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set() ||
           c10::impl::tls_local_dispatch_key_set().included_.has(c10::DispatchKey::FuncTorchDynamicLayerFrontMode);
}

bool to_int(PyObject* o, long* v)
{
    if (!PyLong_CheckExact(o)) return false;
    *v = PyLong_AsLong(o);
    if (*v == -1 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return *v >= -2147483647L && *v <= 2147483647L;
}

struct Lay {
    const int32_t* row_ptr;
    const int32_t* col_idx;
    const uint64_t* bitmaps;
    long H, Lq, Lk, bm, bn;
};
bool read_layout(PyObject* o, Lay* l)
{
    if (!PyTuple_Check(o) || PyTuple_GET_SIZE(o) != 9) return false;
    const at::Tensor* t[3];
    for (int k = 0; k < 3; ++k)
        if (!(t[k] = plain(PyTuple_GET_ITEM(o, k)))) return false;
    long* const out[5] = {&l->H, &l->Lq, &l->Lk, &l->bm, &l->bn};
    for (int k = 0; k < 5; ++k)
        if (!to_int(PyTuple_GET_ITEM(o, 4 + k), out[k])) return false;
    l->row_ptr = (const int32_t*)t[0]->data_ptr();
    l->col_idx = (const int32_t*)t[1]->data_ptr();
    l->bitmaps = (const uint64_t*)t[2]->data_ptr();
    return true;
}

// A schedule, or None (*p stays null).  One that was built with another `causal` is refused by the general path.
bool read_sched(PyObject* o, bool causal, ap_schedule* s, const ap_schedule** p)
{
    *p = nullptr;
    if (o == Py_None) return true;
    if (!PyTuple_Check(o) || PyTuple_GET_SIZE(o) != 6) return false;
    if (PyTuple_GET_ITEM(o, 4) != (causal ? Py_True : Py_False)) return false;
    const at::Tensor* t[4];
    for (int k = 0; k < 4; ++k)
        if (!(t[k] = plain(PyTuple_GET_ITEM(o, k)))) return false;
    s->cnt = (int32_t*)t[0]->data_ptr();
    s->start = (int32_t*)t[1]->data_ptr();
    s->cols = (int32_t*)t[2]->data_ptr();
    s->bitmaps = (uint64_t*)t[3]->data_ptr();
    *p = s;
    return true;
}

struct Transposed {
    const int32_t* ptr[3];
};
bool read_transposed(PyObject* o, Transposed* x)
{
    if (!PyTuple_Check(o) || PyTuple_GET_SIZE(o) != 3) return false;
    for (int k = 0; k < 3; ++k) {
        const at::Tensor* t = plain(PyTuple_GET_ITEM(o, k));
        if (!t) return false;
        x->ptr[k] = (const int32_t*)t->data_ptr();
    }
    return true;
}

// causal and softmax_scale as the binding's arguments have them, and torch's current stream.  A stream of the
// caller's own is not taken: outputs and scratch memory are allocated here, and those belong to the current stream.
struct Common {
    bool causal;
    float scale;
    void* stream;
};
bool read_common(PyObject* causal, PyObject* scale, PyObject* stream, Common* c)
{
    if (causal != Py_True && causal != Py_False) return false;
    c->causal = causal == Py_True;
    if (!PyFloat_CheckExact(scale) || stream != Py_None) return false;
    c->scale = (float)PyFloat_AS_DOUBLE(scale);
    PyObject* d = PyObject_CallNoArgs(get_device);
    PyObject* s = d ? PyObject_CallOneArg(get_stream, d) : nullptr;
    Py_XDECREF(d);
    if (s && PyLong_Check(s)) c->stream = PyLong_AsVoidPtr(s);
    Py_XDECREF(s);
    if (!s || PyErr_Occurred()) {                            // the general path meets it again and reports it
        PyErr_Clear();
        return false;
    }
    return true;
}

// Q [B,H,Lq,D], K and V [B,H,Lk,D] of one type with a contiguous last dimension, on one device
struct Qkv {
    const at::Tensor *q, *k, *v;
    int64_t B, H, Lq, Lk, D;
};
bool read_qkv(PyObject* Q, PyObject* K, PyObject* V, Qkv* x)
{
    if (!(x->q = plain(Q)) || !(x->k = plain(K)) || !(x->v = plain(V))) return false;
    if (x->q->dim() != 4 || x->k->dim() != 4 || x->v->dim() != 4) return false;
    const auto qs = x->q->sizes(), ks = x->k->sizes();
    x->B = qs[0], x->H = qs[1], x->Lq = qs[2], x->D = qs[3], x->Lk = ks[2];
    if (ks[0] != x->B || ks[1] != x->H || ks[3] != x->D || x->v->sizes() != ks) return false;
    for (const int64_t n : {x->B, x->H, x->Lq, x->Lk, x->D})
        if (n > 2147483647LL) return false;
    for (const at::Tensor* t : {x->q, x->k, x->v})
        if (t->stride(3) != 1 || t->scalar_type() != x->q->scalar_type() || t->device() != x->q->device()) return false;
    return true;
}
bool same_sizes(const Qkv& x, const Lay& l) { return l.H == x.H && l.Lq == x.Lq && l.Lk == x.Lk; }

at::Tensor rows_f32(const Qkv& x) { return at::empty({x.B, x.H, x.Lq}, x.q->options().dtype(at::kFloat).requires_grad(false)); }
at::Tensor scratch(const Qkv& x, size_t bytes)
{
    return at::empty({(int64_t)bytes}, x.q->options().dtype(at::kByte).requires_grad(false));
}
at::Tensor like(const at::Tensor& t)
{
    return at::empty_strided(t.sizes(), t.strides(), t.options().requires_grad(false));
}

PyObject* pack(std::initializer_list<at::Tensor> ts)
{
    PyObject* r = PyTuple_New((Py_ssize_t)ts.size());
    if (!r) return nullptr;
    Py_ssize_t k = 0;
    for (const at::Tensor& t : ts) {
        PyObject* o;
        if (t.defined()) {
            o = THPVariable_Wrap(t);
        } else {
            o = Py_None;
            Py_INCREF(o);
        }
        if (!o) {
            Py_DECREF(r);
            return nullptr;
        }
        PyTuple_SET_ITEM(r, k++, o);
    }
    return r;
}
PyObject* result(ap_status st, std::initializer_list<at::Tensor> ts)
{
    return st == AP_OK ? pack(ts) : PyLong_FromLong((long)st);
}

#define AP_ENTER(count)                                                                              \
    if (nargs != (count)) {                                                                          \
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");                               \
        return nullptr;                                                                              \
    }                                                                                                \
    HANDLE_TH_ERRORS                                                                                 \
    if (!bound || modes_active()) Py_RETURN_NONE

#define AP_QKV_PTRS x.q->data_ptr(), x.k->data_ptr(), x.v->data_ptr()
#define AP_SIZES (int)x.B, (int)x.H, (int)x.Lq, (int)x.Lk, (int)x.D
#define AP_STRIDES(o) x.q->strides().data(), x.k->strides().data(), x.v->strides().data(), (o).strides().data()
#define AP_LAYOUT l.row_ptr, l.col_idx, l.bitmaps

// (Q, K, V, layout, causal, softmax_scale, return_lse, stream, sched, crop)
PyObject* call_fwd(PyObject*, PyObject* const* a, Py_ssize_t nargs)
{
    AP_ENTER(10);
    Qkv x;
    Lay l;
    Common c;
    ap_schedule s;
    const ap_schedule* sp;
    if (!read_qkv(a[0], a[1], a[2], &x) || !read_layout(a[3], &l) || !read_common(a[4], a[5], a[7], &c) ||
        !read_sched(a[8], c.causal, &s, &sp))
        Py_RETURN_NONE;
    if ((a[6] != Py_True && a[6] != Py_False) || (a[9] != Py_True && a[9] != Py_False)) Py_RETURN_NONE;
    const bool crop = a[9] == Py_True;
    const auto type = x.q->scalar_type();
    if (type != at::kBFloat16 && type != at::kFloat) Py_RETURN_NONE;
    if (crop ? (l.H != x.H || x.Lq > l.Lq || x.Lk > l.Lk) : !same_sizes(x, l)) Py_RETURN_NONE;
    const ap_dtype dt = type == at::kFloat ? AP_F32 : AP_BF16;
    const at::Tensor out = at::empty({x.B, x.H, x.Lq, x.D}, x.q->options().requires_grad(false));
    at::Tensor lse;
    if (a[6] == Py_True) lse = rows_f32(x);
    float* lp = lse.defined() ? (float*)lse.data_ptr() : nullptr;
    ap_status st;
    Py_BEGIN_ALLOW_THREADS
    if (crop)
        st = api.fwd_cropped(AP_QKV_PTRS, out.data_ptr(), lp, dt, AP_SIZES, AP_STRIDES(out), AP_LAYOUT, (int)l.bm,
                             (int)l.bn, (int)l.Lq, (int)l.Lk, sp, c.causal, c.scale, c.stream);
    else
        st = api.fwd(AP_QKV_PTRS, out.data_ptr(), lp, dt, AP_SIZES, AP_STRIDES(out), AP_LAYOUT, (int)l.bm, (int)l.bn,
                     sp, c.causal, c.scale, c.stream);
    Py_END_ALLOW_THREADS
    return result(st, {out, lse});
    END_HANDLE_TH_ERRORS
}

// (Q, K, V, layout, splits, causal, softmax_scale, return_lse, stream, sched, decode)
PyObject* call_split(PyObject*, PyObject* const* a, Py_ssize_t nargs)
{
    AP_ENTER(11);
    Qkv x;
    Lay l;
    Common c;
    ap_schedule s;
    const ap_schedule* sp;
    long splits;
    if (!read_qkv(a[0], a[1], a[2], &x) || !read_layout(a[3], &l) || !to_int(a[4], &splits) ||
        !read_common(a[5], a[6], a[8], &c) || !read_sched(a[9], c.causal, &s, &sp))
        Py_RETURN_NONE;
    if (x.q->scalar_type() != at::kBFloat16 || !same_sizes(x, l) || (a[7] != Py_True && a[7] != Py_False)) Py_RETURN_NONE;
    const bool decode = a[10] == Py_True;
    const size_t bytes = decode && splits <= 1 ? 0 : api.split_bytes(x.B, x.H, x.Lq, x.D, splits);
    const at::Tensor out = at::empty({x.B, x.H, x.Lq, x.D}, x.q->options().requires_grad(false));
    at::Tensor lse;
    if (a[7] == Py_True) lse = rows_f32(x);
    float* lp = lse.defined() ? (float*)lse.data_ptr() : nullptr;
    const at::Tensor ws = scratch(x, bytes < 16 ? 16 : bytes);
    ap_status st;
    Py_BEGIN_ALLOW_THREADS
    if (decode)
        st = api.decode(AP_QKV_PTRS, out.data_ptr(), lp, AP_BF16, AP_SIZES, AP_STRIDES(out), AP_LAYOUT, (int)l.bm,
                        (int)l.bn, c.causal, c.scale, (int)splits, ws.data_ptr(), bytes, c.stream);
    else
        st = api.split(AP_QKV_PTRS, out.data_ptr(), lp, AP_BF16, AP_SIZES, AP_STRIDES(out), AP_LAYOUT, (int)l.bm,
                       (int)l.bn, sp, c.causal, c.scale, (int)splits, ws.data_ptr(), bytes, c.stream);
    Py_END_ALLOW_THREADS
    return result(st, {out, lse});
    END_HANDLE_TH_ERRORS
}

// (Q, K, V, layout, causal, softmax_scale, return_tau, stream, sched)
PyObject* call_entmax_fwd(PyObject*, PyObject* const* a, Py_ssize_t nargs)
{
    AP_ENTER(9);
    Qkv x;
    Lay l;
    Common c;
    ap_schedule s;
    const ap_schedule* sp;
    if (!read_qkv(a[0], a[1], a[2], &x) || !read_layout(a[3], &l) || !read_common(a[4], a[5], a[7], &c) ||
        !read_sched(a[8], c.causal, &s, &sp))
        Py_RETURN_NONE;
    if (x.q->scalar_type() != at::kBFloat16 || !same_sizes(x, l) || (a[6] != Py_True && a[6] != Py_False)) Py_RETURN_NONE;
    const at::Tensor out = at::empty({x.B, x.H, x.Lq, x.D}, x.q->options().requires_grad(false));
    at::Tensor tau;
    if (a[6] == Py_True) tau = rows_f32(x);
    float* tp = tau.defined() ? (float*)tau.data_ptr() : nullptr;
    ap_status st;
    Py_BEGIN_ALLOW_THREADS
    st = api.entmax_fwd(AP_QKV_PTRS, out.data_ptr(), tp, AP_BF16, AP_SIZES, AP_STRIDES(out), AP_LAYOUT, (int)l.bm,
                        (int)l.bn, sp, c.causal, c.scale, c.stream);
    Py_END_ALLOW_THREADS
    return result(st, {out, tau});
    END_HANDLE_TH_ERRORS
}

// (Q, K, V, O or None, dO, rows, layout, layout_t, causal, softmax_scale, stream, sched, col_sched): the softmax
// pass with its O and log-sum-exp, or, without O, the 1.5-entmax pass with its tau
PyObject* call_bwd(PyObject*, PyObject* const* a, Py_ssize_t nargs)
{
    AP_ENTER(13);
    Qkv x;
    Lay l;
    Transposed t;
    Common c;
    ap_schedule s, cs;
    const ap_schedule *sp, *csp;
    if (!read_qkv(a[0], a[1], a[2], &x) || !read_layout(a[6], &l) || !read_transposed(a[7], &t) ||
        !read_common(a[8], a[9], a[10], &c) || !read_sched(a[11], c.causal, &s, &sp) ||
        !read_sched(a[12], c.causal, &cs, &csp))
        Py_RETURN_NONE;
    const bool entmax = a[3] == Py_None;
    const at::Tensor* o = entmax ? nullptr : plain(a[3]);
    const at::Tensor* d = plain(a[4]);
    const at::Tensor* rows = plain(a[5]);
    if ((!o && !entmax) || !d || !rows || (entmax && (!sp || !csp))) Py_RETURN_NONE;
    for (const at::Tensor* y : {o ? o : d, d})
        if (y->sizes() != x.q->sizes() || y->scalar_type() != at::kBFloat16 || y->stride(3) != 1 ||
            y->device() != x.q->device())
            Py_RETURN_NONE;
    if (o && o->strides() != d->strides()) Py_RETURN_NONE;   // the general path copies dO
    if (x.q->scalar_type() != at::kBFloat16 || !same_sizes(x, l)) Py_RETURN_NONE;
    if (rows->dim() != 3 || rows->size(0) != x.B || rows->size(1) != x.H || rows->size(2) != x.Lq ||
        rows->scalar_type() != at::kFloat || rows->device() != x.q->device() || !rows->is_contiguous())
        Py_RETURN_NONE;
    const size_t bytes = entmax ? api.entmax_bytes(x.B, x.H, x.Lq) : api.bwd_bytes(x.B, x.H, x.Lq);
    const at::Tensor dQ = like(*x.q), dK = like(*x.k), dV = like(*x.v), ws = scratch(x, bytes);
    const float* rp = (const float*)rows->data_ptr();
    ap_status st;
    Py_BEGIN_ALLOW_THREADS
    if (entmax)
        st = api.entmax_bwd(AP_QKV_PTRS, d->data_ptr(), rp, dQ.data_ptr(), dK.data_ptr(), dV.data_ptr(), AP_BF16,
                            AP_SIZES, AP_STRIDES(*d), AP_LAYOUT, t.ptr[0], t.ptr[1], t.ptr[2], (int)l.bm, (int)l.bn,
                            sp, csp, c.causal, c.scale, ws.data_ptr(), bytes, c.stream);
    else if (sp || csp)
        st = api.bwd_sched(AP_QKV_PTRS, o->data_ptr(), d->data_ptr(), rp, dQ.data_ptr(), dK.data_ptr(),
                           dV.data_ptr(), AP_BF16, AP_SIZES, AP_STRIDES(*o), AP_LAYOUT, t.ptr[0], t.ptr[1], t.ptr[2],
                           (int)l.bm, (int)l.bn, sp, csp, c.causal, c.scale, ws.data_ptr(), bytes, c.stream);
    else
        st = api.bwd(AP_QKV_PTRS, o->data_ptr(), d->data_ptr(), rp, dQ.data_ptr(), dK.data_ptr(), dV.data_ptr(),
                     AP_BF16, AP_SIZES, AP_STRIDES(*o), AP_LAYOUT, t.ptr[0], t.ptr[1], t.ptr[2], (int)l.bm,
                     (int)l.bn, c.causal, c.scale, ws.data_ptr(), bytes, c.stream);
    Py_END_ALLOW_THREADS
    return result(st, {dQ, dK, dV});
    END_HANDLE_TH_ERRORS
}

// bind(addresses in the order of Api, get_device, get_stream)
PyObject* call_bind(PyObject*, PyObject* const* a, Py_ssize_t nargs)
{
    constexpr Py_ssize_t N = sizeof(Api) / sizeof(void*);
    if (nargs != N + 2) {
        PyErr_SetString(PyExc_TypeError, "bind: wrong number of arguments");
        return nullptr;
    }
    void* p[N];
    for (Py_ssize_t k = 0; k < N; ++k) {
        p[k] = PyLong_AsVoidPtr(a[k]);
        if (PyErr_Occurred()) return nullptr;
        if (!p[k]) {
            PyErr_SetString(PyExc_ValueError, "bind: null address");
            return nullptr;
        }
    }
    static_assert(sizeof p == sizeof api, "function pointers only");
    memcpy(&api, p, sizeof api);
    Py_INCREF(a[N]);
    Py_INCREF(a[N + 1]);
    Py_XDECREF(get_device);
    Py_XDECREF(get_stream);
    get_device = a[N];
    get_stream = a[N + 1];
    bound = true;
    Py_RETURN_NONE;
}

#define AP_METHOD(name) {#name, (PyCFunction)(void (*)(void))call_##name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {AP_METHOD(bind), AP_METHOD(fwd), AP_METHOD(split), AP_METHOD(entmax_fwd), AP_METHOD(bwd),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "ap_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_ap_calls(void) { return PyModule_Create(&module); }
