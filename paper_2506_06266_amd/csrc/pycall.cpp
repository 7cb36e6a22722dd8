// The per-call host work of the Python binding's smallest entry points in native code: descriptor, output tensors,
// workspace, the checks on the tensors handed over, the library call.  In Python with ctypes it is a third of a call whose
// kernels take ten microseconds (decode of four requests, us of host time a call: 14.2, of which the two launches are 6.5, now 10.0;
// a forward and backward call of fp32 attention over 2 x 64 tokens 23.8 -> 19.2; decode of one request over three shared
// cartridges 16.7 -> 10.5).  The library is reached through the handle the binding
// opened (no link dependency on it).
//
// Every function takes the arguments of its namesake in binding.py by position and returns the outputs, or the status of
// a call that failed (an int, which the binding turns into its exception).
#include <dlfcn.h>

#include <algorithm>
#include <string>
#include <vector>

#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>

#include "cartridge.h"

namespace {

struct Api {
    decltype(&cart_attn_fwd_workspace) attn_fwd_workspace;
    decltype(&cart_attn_fwd) attn_fwd;
    decltype(&cart_attn_bwd_workspace) attn_bwd_workspace;
    decltype(&cart_attn_bwd) attn_bwd;
    decltype(&cart_kl_workspace) kl_workspace;
    decltype(&cart_distill_kl_fwd_bwd) kl;
    decltype(&cart_teacher_topk) topk;
    decltype(&cart_decode_workspace) decode_workspace;
    decltype(&cart_decode) decode;
    decltype(&cart_decode_composed_workspace) composed_workspace;
    decltype(&cart_decode_composed) composed;
} api;

// a tensor argument (null: None)
const at::Tensor* tensor_or_none(PyObject* o) {
    if (o == Py_None) return nullptr;
    if (!THPVariable_Check(o)) throw torch::TypeError(std::string("expected a tensor, got ") + Py_TYPE(o)->tp_name);
    return &THPVariable_Unpack(o);
}
const at::Tensor& tensor(PyObject* o) {
    const at::Tensor* t = tensor_or_none(o);
    if (!t) throw torch::TypeError("expected a tensor, got None");
    return *t;
}
// what binding.py's _ptr returns (an empty tensor's address is null)
void* address(const at::Tensor* t) {
    if (!t) return nullptr;
    TORCH_CHECK_VALUE(t->is_cuda() && t->is_contiguous(), "tensors handed to libcartridge must be contiguous device tensors");
    return t->mutable_data_ptr();
}
// Numbers as a ctypes field takes them, which the entry points left in Python hand theirs to: an integer is whatever has
// __index__ (numpy's, a tensor of one), cut to its width, a float is none; a real is whatever has __float__ or __index__.
int32_t int32(PyObject* o) {
    if (PyLong_CheckExact(o)) return static_cast<int32_t>(PyLong_AsUnsignedLongLongMask(o));
    PyObject* const i = PyNumber_Index(o);
    if (!i) throw python_error();
    const int32_t r = static_cast<int32_t>(PyLong_AsUnsignedLongLongMask(i));
    Py_DECREF(i);
    return r;
}
float real(PyObject* o) {
    const double x = PyFloat_AsDouble(o);
    if (x == -1.0 && PyErr_Occurred()) throw python_error();
    return static_cast<float>(x);
}
// int(o)
int32_t truncated(PyObject* o) {
    if (PyBool_Check(o)) return o == Py_True;
    PyObject* const i = PyNumber_Long(o);
    if (!i) throw python_error();
    const int32_t r = static_cast<int32_t>(PyLong_AsUnsignedLongLongMask(i));
    Py_DECREF(i);
    return r;
}
PyObject* stream_of = nullptr;      // the binding's _stream: a stream object or None -> its raw handle
void* stream(PyObject* o) {
    PyObject* const r = PyObject_CallOneArg(stream_of, o);
    if (!r) throw python_error();
    void* const p = PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    if (!p && PyErr_Occurred()) throw python_error();
    return p;
}
int dtype_code(const at::Tensor& t) {
    if (t.scalar_type() == at::kFloat) return CART_F32;
    if (t.scalar_type() == at::kBFloat16) return CART_BF16;
    throw torch::TypeError(std::string("unsupported dtype ") + c10::toString(t.scalar_type()));
}
// size i, of a tensor of `dims` dimensions (0: of any number above i)
int32_t size(const at::Tensor& t, int64_t dims, int64_t i) {
    TORCH_CHECK_VALUE(dims ? t.dim() == dims : t.dim() > i, "a tensor of ", t.dim(), " dimensions where ", dims ? "" : "more than ",
                      dims ? dims : i, " are expected");
    return static_cast<int32_t>(t.size(i));
}
int32_t slots(const at::Tensor* z) { return z ? size(*z, 0, 1) : 0; }

at::Tensor like(PyObject* given, const at::Tensor& t) { return given == Py_None ? at::empty_like(t) : tensor(given); }
at::Tensor fresh(PyObject* given, at::IntArrayRef sizes, at::ScalarType type, const at::Tensor& beside) {
    return given == Py_None ? at::empty(sizes, beside.options().dtype(type)) : tensor(given);
}
// the workspace: the caller's, or `need` bytes
struct Workspace {
    at::Tensor own;
    void* p = nullptr;
    size_t bytes = 0;
    Workspace(PyObject* given, size_t need, const at::Tensor& beside) {
        if (given != Py_None) {
            const at::Tensor& t = tensor(given);
            p = address(&t);
            bytes = static_cast<size_t>(t.numel());
        } else if (need > 0) {
            own = at::empty({static_cast<int64_t>(need)}, beside.options().dtype(at::kByte));
            p = own.mutable_data_ptr();
            bytes = need;
        }
    }
};
template <typename F>
int without_gil(F&& f) {
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = f();
    Py_END_ALLOW_THREADS
    return status;
}
PyObject* outputs(int status, std::initializer_list<const at::Tensor*> ts) {
    if (status != CART_OK) return PyLong_FromLong(status);
    PyObject* const r = PyTuple_New(static_cast<Py_ssize_t>(ts.size()));
    if (!r) throw python_error();
    Py_ssize_t i = 0;
    for (const at::Tensor* t : ts) {
        PyObject* v;
        if (t->defined()) v = THPVariable_Wrap(*t);
        else { Py_INCREF(Py_None); v = Py_None; }
        PyTuple_SET_ITEM(r, i++, v);
    }
    return r;
}
void count(Py_ssize_t n, Py_ssize_t want) {
    if (n != want) throw torch::TypeError(std::to_string(want) + " arguments expected, got " + std::to_string(n));
}

cart_attn_desc attn_desc(const at::Tensor& q, const at::Tensor& k, int32_t P, float scale, int32_t n_frozen, int32_t accumulate, int32_t impl) {
    cart_attn_desc d = {};
    d.B = size(q, 4, 0); d.S = size(q, 4, 1); d.Hq = size(q, 4, 2); d.D = size(q, 4, 3);
    d.Hkv = size(k, 0, 2);
    d.P = P;
    d.dtype = static_cast<decltype(d.dtype)>(dtype_code(q));
    d.softmax_scale = scale;
    d.n_frozen = n_frozen;
    d.dz_accumulate = accumulate;
    d.impl = static_cast<decltype(d.impl)>(impl);
    return d;
}

// q, k_own, v_own, z_k, z_v, scale, impl, o, lse, workspace, stream
PyObject* attn_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    count(n, 11);
    const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]), &v = tensor(a[2]);
    const at::Tensor *zk = tensor_or_none(a[3]), *zv = tensor_or_none(a[4]);
    const cart_attn_desc d = attn_desc(q, k, slots(zk), real(a[5]), 0, 0, int32(a[6]));
    const at::Tensor o = like(a[7], q), lse = fresh(a[8], {d.B, d.Hq, d.S}, at::kFloat, q);
    const Workspace ws(a[9], api.attn_fwd_workspace(&d), q);
    void *pq = address(&q), *pk = address(&k), *pv = address(&v), *pzk = address(zk), *pzv = address(zv), *po = address(&o), *pl = address(&lse);
    void* const st = stream(a[10]);
    return outputs(without_gil([&] { return api.attn_fwd(&d, pq, pk, pv, pzk, pzv, po, static_cast<float*>(pl), ws.p, ws.bytes, st); }), {&o, &lse});
    END_HANDLE_TH_ERRORS
}

// q, k_own, v_own, z_k, z_v, o, lse, d_o, scale, n_frozen, d_z_k, d_z_v, dz_accumulate, impl, d_q, d_k_own, d_v_own, workspace, stream
PyObject* attn_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    count(n, 19);
    const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]), &v = tensor(a[2]), &o = tensor(a[5]), &lse = tensor(a[6]), &d_o = tensor(a[7]);
    const at::Tensor *zk = tensor_or_none(a[3]), *zv = tensor_or_none(a[4]);
    const cart_attn_desc d = attn_desc(q, k, slots(zk), real(a[8]), int32(a[9]), truncated(a[12]), int32(a[13]));
    const at::Tensor dq = like(a[14], q), dk = like(a[15], k), dv = like(a[16], v);
    at::Tensor dzk, dzv;
    if (a[10] != Py_None) dzk = tensor(a[10]);
    if (a[11] != Py_None) dzv = tensor(a[11]);
    if (d.P > 0 && !dzk.defined()) {
        const int accumulate = PyObject_IsTrue(a[12]);
        if (accumulate < 0) throw python_error();
        TORCH_CHECK_VALUE(!accumulate, "dz_accumulate needs d_z_k / d_z_v");
        dzk = at::empty(zk->sizes(), q.options().dtype(at::kFloat));
        dzv = at::empty((zv ? zv : zk)->sizes(), q.options().dtype(at::kFloat));
    }
    const Workspace ws(a[17], api.attn_bwd_workspace(&d), q);
    void *pq = address(&q), *pk = address(&k), *pv = address(&v), *pzk = address(zk), *pzv = address(zv), *po = address(&o), *pl = address(&lse),
         *pdo = address(&d_o), *pdq = address(&dq), *pdk = address(&dk), *pdv = address(&dv),
         *pdzk = address(dzk.defined() ? &dzk : nullptr), *pdzv = address(dzv.defined() ? &dzv : nullptr);
    void* const st = stream(a[18]);
    return outputs(without_gil([&] {
        return api.attn_bwd(&d, pq, pk, pv, pzk, pzv, po, static_cast<float*>(pl), pdo, pdq, pdk, pdv, static_cast<float*>(pdzk),
                            static_cast<float*>(pdzv), ws.p, ws.bytes, st);
    }), {&dq, &dk, &dv, &dzk, &dzv});
    END_HANDLE_TH_ERRORS
}

// logits, teacher_idx, teacher_logp, scale, mode, d_logits, loss, row_kl, workspace, stream
PyObject* distill_kl(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    count(n, 10);
    const at::Tensor &x = tensor(a[0]), &idx = tensor(a[1]);
    const at::Tensor *logp = tensor_or_none(a[2]), *row_kl = tensor_or_none(a[7]);
    cart_kl_desc d = {};
    d.N = size(x, 2, 0); d.V = size(x, 2, 1); d.K = size(idx, 0, 1);
    d.logits_dtype = static_cast<decltype(d.logits_dtype)>(dtype_code(x));
    d.scale = real(a[3]);
    d.mode = static_cast<decltype(d.mode)>(int32(a[4]));
    const at::Tensor dx = like(a[5], x), loss = fresh(a[6], {1}, at::kFloat, x);
    const Workspace ws(a[8], api.kl_workspace(&d), x);
    void *px = address(&x), *pi = address(&idx), *pp = address(logp), *pl = address(&loss), *pd = address(&dx), *pr = address(row_kl);
    void* const st = stream(a[9]);
    return outputs(without_gil([&] {
        return api.kl(&d, px, static_cast<int32_t*>(pi), static_cast<float*>(pp), static_cast<float*>(pl), pd, static_cast<float*>(pr), ws.p,
                      ws.bytes, st);
    }), {&loss, &dx});
    END_HANDLE_TH_ERRORS
}

// logits, k, teacher_idx, teacher_logp, stream
PyObject* teacher_topk(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    count(n, 5);
    const at::Tensor& x = tensor(a[0]);
    cart_topk_desc d = {};
    d.N = size(x, 2, 0); d.V = size(x, 2, 1); d.K = int32(a[1]);
    d.logits_dtype = static_cast<decltype(d.logits_dtype)>(dtype_code(x));
    const at::Tensor idx = fresh(a[2], {d.N, d.K}, at::kInt, x), lp = fresh(a[3], {d.N, d.K}, at::kFloat, x);
    void *px = address(&x), *pi = address(&idx), *pp = address(&lp);
    void* const st = stream(a[4]);
    return outputs(without_gil([&] { return api.topk(&d, px, static_cast<int32_t*>(pi), static_cast<float*>(pp), st); }), {&idx, &lp});
    END_HANDLE_TH_ERRORS
}

// q, z_k, z_v, k_own, v_own, cu_lens, max_own_len, scale, impl, o, lse, workspace, stream
PyObject* decode(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    count(n, 13);
    const at::Tensor &q = tensor(a[0]), &k = tensor(a[3]), &v = tensor(a[4]), &cu = tensor(a[5]);
    const at::Tensor *zk = tensor_or_none(a[1]), *zv = tensor_or_none(a[2]);
    cart_decode_desc d = {};
    d.B = size(q, 3, 0); d.Hq = size(q, 3, 1); d.D = size(q, 3, 2);
    d.Hkv = size(k, 0, 1);
    d.P = slots(zk);
    d.total_own_tokens = size(k, 0, 0);
    d.max_own_len = int32(a[6]);
    d.dtype = static_cast<decltype(d.dtype)>(dtype_code(q));
    d.softmax_scale = real(a[7]);
    d.impl = static_cast<decltype(d.impl)>(int32(a[8]));
    const at::Tensor o = like(a[9], q), lse = fresh(a[10], {d.B, d.Hq}, at::kFloat, q);
    const Workspace ws(a[11], api.decode_workspace(&d), q);
    void *pq = address(&q), *pzk = address(zk), *pzv = address(zv), *pk = address(&k), *pv = address(&v), *pc = address(&cu), *po = address(&o),
         *pl = address(&lse);
    void* const st = stream(a[12]);
    return outputs(without_gil([&] {
        return api.decode(&d, pq, pzk, pzv, pk, pv, static_cast<int32_t*>(pc), po, static_cast<float*>(pl), ws.p, ws.bytes, st);
    }), {&o, &lse});
    END_HANDLE_TH_ERRORS
}

// q, shared (a list of pairs), pool_k, pool_v, cart_id, k_own, v_own, cu_lens, max_own_len, scale, o, lse, workspace, stream
PyObject* decode_composed(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    count(n, 14);
    const at::Tensor &q = tensor(a[0]), &k = tensor(a[5]), &v = tensor(a[6]), &cu = tensor(a[7]);
    const at::Tensor *pool_k = tensor_or_none(a[2]), *pool_v = tensor_or_none(a[3]), *cart_id = tensor_or_none(a[4]);
    cart_decode_composed_desc d = {};
    d.B = size(q, 3, 0); d.Hq = size(q, 3, 1); d.D = size(q, 3, 2);
    if (!PyList_Check(a[1]) && !PyTuple_Check(a[1])) throw torch::TypeError("a list of (z_k, z_v) is expected");
    std::vector<cart_segment> segs(static_cast<size_t>(std::max<Py_ssize_t>(PySequence_Fast_GET_SIZE(a[1]), 1)));
    for (Py_ssize_t i = 0; i < PySequence_Fast_GET_SIZE(a[1]); ++i) {
        PyObject* const pair = PySequence_Fast_GET_ITEM(a[1], i);
        if ((!PyList_Check(pair) && !PyTuple_Check(pair)) || PySequence_Fast_GET_SIZE(pair) != 2) throw torch::TypeError("a pair (z_k, z_v) is expected");
        const at::Tensor &zk = tensor(PySequence_Fast_GET_ITEM(pair, 0)), *zv = tensor_or_none(PySequence_Fast_GET_ITEM(pair, 1));
        segs[i].z_k = address(&zk);
        segs[i].z_v = address(zv);
        segs[i].p = size(zk, 0, 1);
    }
    d.Hkv = size(k, 0, 1);
    d.n_shared = static_cast<int32_t>(PySequence_Fast_GET_SIZE(a[1]));
    if (pool_k) { d.n_pool = size(*pool_k, 0, 0); d.pool_p = size(*pool_k, 0, 2); }
    d.total_own_tokens = size(k, 0, 0);
    d.max_own_len = int32(a[8]);
    d.dtype = static_cast<decltype(d.dtype)>(dtype_code(q));
    d.softmax_scale = real(a[9]);
    const at::Tensor o = like(a[10], q), lse = fresh(a[11], {d.B, d.Hq}, at::kFloat, q);
    const Workspace ws(a[12], api.composed_workspace(&d, segs.data()), q);
    void *pq = address(&q), *ppk = address(pool_k), *ppv = address(pool_v), *pid = address(cart_id), *pk = address(&k), *pv = address(&v),
         *pc = address(&cu), *po = address(&o), *pl = address(&lse);
    void* const st = stream(a[13]);
    return outputs(without_gil([&] {
        return api.composed(&d, pq, segs.data(), ppk, ppv, static_cast<int32_t*>(pid), pk, pv, static_cast<int32_t*>(pc), po,
                            static_cast<float*>(pl), ws.p, ws.bytes, st);
    }), {&o, &lse});
    END_HANDLE_TH_ERRORS
}

// the handle of the opened library, the binding's _stream
PyObject* init(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    count(n, 2);
    void* const lib = PyLong_AsVoidPtr(a[0]);
    TORCH_CHECK_VALUE(lib, "no library");
    Py_INCREF(a[1]);
    stream_of = a[1];
    auto get = [&](auto& f, const char* name) {
        f = reinterpret_cast<std::remove_reference_t<decltype(f)>>(dlsym(lib, name));
        TORCH_CHECK_VALUE(f, name, " is missing in the library");
    };
    get(api.attn_fwd_workspace, "cart_attn_fwd_workspace");
    get(api.attn_fwd, "cart_attn_fwd");
    get(api.attn_bwd_workspace, "cart_attn_bwd_workspace");
    get(api.attn_bwd, "cart_attn_bwd");
    get(api.kl_workspace, "cart_kl_workspace");
    get(api.kl, "cart_distill_kl_fwd_bwd");
    get(api.topk, "cart_teacher_topk");
    get(api.decode_workspace, "cart_decode_workspace");
    get(api.decode, "cart_decode");
    get(api.composed_workspace, "cart_decode_composed_workspace");
    get(api.composed, "cart_decode_composed");
    Py_RETURN_NONE;
    END_HANDLE_TH_ERRORS
}

#define FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(attn_fwd), FAST(attn_bwd), FAST(distill_kl), FAST(teacher_topk), FAST(decode), FAST(decode_composed),
                         FAST(init), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pycall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pycall() { return PyModule_Create(&module); }
