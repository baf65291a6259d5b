// Python extension module: the hot path of binding.py's wrappers in native code.
//
// A wrapper in Python spends 5-10 us on attribute lookups, torch.empty and ctypes conversions before the library
// is called -- more than a small kernel takes.  The functions here do the same checks and allocations on the C++ tensors
// and call the C ABI of libsage.so through the addresses that init() is given (one copy of the library, the
// one binding.load() opened).  They handle the calls that are in order: anything else (a wrong type or shape, an argument
// that is not a plain number) returns None, and the Python wrapper then takes its own path, which raises the error.
// Return values: the outputs; an int, the status of a call that the library refused; or None.
// The interpreter lock is released around the library calls, as ctypes does.
#include <Python.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <torch/csrc/autograd/python_variable.h>
#include <cstring>

#include "../../include/sage.h"

#ifndef SAGE_NATIVE_HASH
#define SAGE_NATIVE_HASH "unknown"
#endif

namespace {

const char tagged_hash[] = "SAGE_NATIVE_HASH=" SAGE_NATIVE_HASH;

struct Api {
    decltype(&sage_quant_q) quant_q;
    decltype(&sage_rope_quant_q) rope_quant_q;
    decltype(&sage_smooth_quant_k_workspace) k_workspace;
    decltype(&sage_smooth_quant_k) smooth_quant_k;
    decltype(&sage_rope_smooth_quant_k) rope_smooth_quant_k;
    decltype(&sage_quant_qk) quant_qk;
    decltype(&sage_quant_v_workspace) v_workspace;
    decltype(&sage_quant_v) quant_v;
    decltype(&sage_attn_split_workspace) split_workspace;
    decltype(&sage_attn_cross_fwd) attn_cross;
    decltype(&sage_attn_cross_split_fwd) attn_split;
    decltype(&sage_attn_pv_int8_cross_fwd) pv8_cross;
    decltype(&sage_attn_pv_int8_cross_split_fwd) pv8_split;
    decltype(&sage_attention_workspace) attention_workspace;
    decltype(&sage_attention_fwd) attention;
} api;
PyObject *get_device, *get_stream;          // torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream

constexpr auto F16 = at::kHalf, F32 = at::kFloat, I8 = at::kChar, U8 = at::kByte;

const at::Tensor* tensor(PyObject* o) { return THPVariable_Check(o) ? &THPVariable_Unpack(o) : nullptr; }
bool on_device(const at::Tensor& t) { return t.is_cuda() && t.is_contiguous(); }

// Arguments of one call, read in order; ok turns false where one is not what the fast path handles.
struct Args {
    PyObject* const* a;
    bool ok = true, elsewhere = false;       // elsewhere: a stream was named that is not the current one
    explicit Args(PyObject* const* args) : a(args) {}
    // a contiguous device tensor of this type
    const at::Tensor* in(at::ScalarType type, int dims) {
        const at::Tensor* t = tensor(*a++);
        ok = ok && t && on_device(*t) && t->scalar_type() == type && (dims == 0 || t->dim() == dims);
        return t;
    }
    // the same or None
    PyObject* given(at::ScalarType type) {
        PyObject* o = *a++;
        if (o == Py_None) return nullptr;
        const at::Tensor* t = tensor(o);
        ok = ok && t && on_device(*t) && t->scalar_type() == type;
        return o;
    }
    // any device tensor or None (scratch of unstated type)
    PyObject* scratch() {
        PyObject* o = *a++;
        if (o == Py_None) return nullptr;
        const at::Tensor* t = tensor(o);
        ok = ok && t && on_device(*t);
        return o;
    }
    int integer() {
        PyObject* o = *a++;
        if (!PyLong_Check(o)) { ok = false; return 0; }        // (a bool is an int here too)
        int overflow = 0;
        const long v = PyLong_AsLongAndOverflow(o, &overflow);
        ok = ok && !overflow && v >= -0x7fffffffL && v <= 0x7fffffffL;
        return (int)v;
    }
    float real() {
        PyObject* o = *a++;
        if (!PyFloat_Check(o)) { ok = false; return 0.0f; }
        return (float)PyFloat_AS_DOUBLE(o);
    }
    // the current stream's handle, or null and false where it cannot be told
    static bool current(void*& p) {
        PyObject* dev = PyObject_CallNoArgs(get_device);
        PyObject* s = dev ? PyObject_CallOneArg(get_stream, dev) : nullptr;
        Py_XDECREF(dev);
        p = s ? PyLong_AsVoidPtr(s) : nullptr;
        Py_XDECREF(s);
        const bool told = !PyErr_Occurred();
        PyErr_Clear();
        return told;
    }
    void* stream() {
        PyObject* o = *a++;
        if (!ok) return nullptr;
        void *p = nullptr, *now = nullptr;
        if (o == Py_None) {
            ok = current(p);
            return p;
        }
        p = PyLong_Check(o) ? PyLong_AsVoidPtr(o) : nullptr;
        if (!PyLong_Check(o) || PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        elsewhere = ok && current(now) && p != now;
        return p;
    }
    // Memory allocated here is the current stream's: a call on another one is taken only with every buffer given.
    bool take(bool all_given) const { return ok && (all_given || !elsewhere); }
};

// An output or scratch tensor: the caller's, or a new one on the device of `like`.
struct Buffer {
    at::Tensor own;
    const at::Tensor* t = nullptr;
    PyObject* from = nullptr;
    void take(PyObject* given, const at::Tensor& like, at::IntArrayRef sizes, at::ScalarType type) {
        from = given;
        if (given) { t = &THPVariable_Unpack(given); return; }
        own = at::empty(sizes, at::TensorOptions().device(like.device()).dtype(type));
        t = &own;
    }
    void bytes(PyObject* given, const at::Tensor& like, size_t need) {
        if (given || need > 0) take(given, like, {(int64_t)need}, U8);
    }
    void* p() const { return t ? t->data_ptr() : nullptr; }
    size_t size() const { return t ? (size_t)t->nbytes() : 0; }
    PyObject* out() const { return from ? (Py_INCREF(from), from) : THPVariable_Wrap(own); }
};

PyObject* none() { Py_RETURN_NONE; }
template <class F> int call(F&& f) {
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = f();
    Py_END_ALLOW_THREADS
    return st;
}
// What the interpreter calls.  No C++ exception may pass through it: what throws here -- an allocation that fails, the
// sizes of a tensor that has none in numbers (symbolic, nested) -- the Python path meets again and reports.
using Entry = PyObject* (*)(PyObject* const*, Py_ssize_t);
template <Entry F> PyObject* guarded(PyObject*, PyObject* const* argv, Py_ssize_t n) {
    try {
        return F(argv, n);
    } catch (const std::exception&) {
        PyErr_Clear();
        return none();
    }
}
PyObject* result(int st, std::initializer_list<const Buffer*> outs) {
    if (st != 0) return PyLong_FromLong(st);
    if (outs.size() == 1) return (*outs.begin())->out();
    PyObject* t = PyTuple_New((Py_ssize_t)outs.size());
    Py_ssize_t i = 0;
    for (const Buffer* b : outs) PyTuple_SET_ITEM(t, i++, b->out());
    return t;
}
int64_t blocks(int64_t n, int block) { return block > 0 ? (n + block - 1) / block : 0; }
bool fits(const at::Tensor& t) {
    for (int i = 0; i < 4; ++i)
        if (t.size(i) > 0x7fffffff) return false;
    return true;
}

// (q, cos, sin, sm_scale, block_q, q_i8 | None, q_scale | None, stream | None); the tables both None unless ROPE: the call is
// named by its entry, so that a missing table does not turn it into the other one
template <bool ROPE> PyObject* py_quant_q(PyObject* const* argv, Py_ssize_t n) {
    if (n != 8) return none();
    Args a(argv);
    const at::Tensor* q = a.in(F16, 4);
    PyObject *cs = a.given(F32), *sn = a.given(F32);
    const float sm = a.real();
    const int block = a.integer();
    PyObject *gi = a.given(I8), *gs = a.given(F32);
    void* st = a.stream();
    if (!a.take(gi && gs) || block < 1 || !fits(*q) || ROPE != (cs != nullptr) || ROPE != (sn != nullptr)) return none();
    const int64_t B = q->size(0), H = q->size(1), N = q->size(2), D = q->size(3);
    const at::Tensor *c = cs ? tensor(cs) : nullptr, *s = sn ? tensor(sn) : nullptr;
    if (c && (c->dim() != 2 || c->size(0) != N || c->size(1) != D / 2 || s->dim() != 2 || s->size(0) != N || s->size(1) != D / 2)) return none();
    Buffer i8, sc;
    i8.take(gi, *q, {B, H, N, D}, I8);
    sc.take(gs, *q, {B, H, blocks(N, block)}, F32);
    void *pq = q->data_ptr(), *pi = i8.p(), *ps = sc.p();
    const void *pc = c ? c->data_ptr() : nullptr, *pn = s ? s->data_ptr() : nullptr;
    const int e = call([&] {
        return ROPE ? api.rope_quant_q(pq, (const float*)pc, (const float*)pn, (int8_t*)pi, (float*)ps, B, H, N, D, sm, block, st)
                    : api.quant_q(pq, (int8_t*)pi, (float*)ps, B, H, N, D, sm, block, st);
    });
    return result(e, {&i8, &sc});
}

// (k, cos, sin, block_k, k_i8 | None, k_scale | None, k_mean | None, workspace | None, stream | None); tables as above
template <bool ROPE> PyObject* py_smooth_quant_k(PyObject* const* argv, Py_ssize_t n) {
    if (n != 9) return none();
    Args a(argv);
    const at::Tensor* k = a.in(F16, 4);
    PyObject *cs = a.given(F32), *sn = a.given(F32);
    const int block = a.integer();
    PyObject *gi = a.given(I8), *gs = a.given(F32), *gm = a.given(F32), *gw = a.scratch();
    void* st = a.stream();
    if (!a.take(gi && gs && gm && gw) || block < 1 || !fits(*k) || ROPE != (cs != nullptr) || ROPE != (sn != nullptr)) return none();
    const int64_t B = k->size(0), H = k->size(1), N = k->size(2), D = k->size(3);
    const at::Tensor *c = cs ? tensor(cs) : nullptr, *s = sn ? tensor(sn) : nullptr;
    if (c && (c->dim() != 2 || c->size(0) != N || c->size(1) != D / 2 || s->dim() != 2 || s->size(0) != N || s->size(1) != D / 2)) return none();
    Buffer i8, sc, mean, ws;
    i8.take(gi, *k, {B, H, N, D}, I8);
    sc.take(gs, *k, {B, H, blocks(N, block)}, F32);
    mean.take(gm, *k, {B, H, D}, F32);
    ws.bytes(gw, *k, api.k_workspace(B, H, N, D));
    void *pk = k->data_ptr(), *pi = i8.p(), *ps = sc.p(), *pm = mean.p(), *pw = ws.p();
    const void *pc = c ? c->data_ptr() : nullptr, *pn = s ? s->data_ptr() : nullptr;
    const size_t wb = ws.size();
    const int e = call([&] {
        return ROPE ? api.rope_smooth_quant_k(pk, (const float*)pc, (const float*)pn, (int8_t*)pi, (float*)ps, (float*)pm, pw, wb, B, H, N, D, block, st)
                    : api.smooth_quant_k(pk, (int8_t*)pi, (float*)ps, (float*)pm, pw, wb, B, H, N, D, block, st);
    });
    return result(e, {&i8, &sc, &mean});
}

// (q, k, sm_scale, block_q, block_k, q_i8, q_scale, k_i8, k_scale, k_mean, workspace, stream), the last seven | None
PyObject* py_quant_qk(PyObject* const* argv, Py_ssize_t n) {
    if (n != 12) return none();
    Args a(argv);
    const at::Tensor *q = a.in(F16, 4), *k = a.in(F16, 4);
    const float sm = a.real();
    const int bq = a.integer(), bk = a.integer();
    PyObject *gqi = a.given(I8), *gqs = a.given(F32), *gki = a.given(I8), *gks = a.given(F32), *gm = a.given(F32), *gw = a.scratch();
    void* st = a.stream();
    if (!a.take(gqi && gqs && gki && gks && gm && gw) || bq < 1 || bk < 1 || !fits(*q) || !fits(*k)) return none();
    const int64_t B = q->size(0), H = q->size(1), Nq = q->size(2), D = q->size(3), Nkv = k->size(2);
    if (k->size(0) != B || k->size(1) != H || k->size(3) != D) return none();
    Buffer qi, qs, ki, ks, mean, ws;
    qi.take(gqi, *q, {B, H, Nq, D}, I8);
    qs.take(gqs, *q, {B, H, blocks(Nq, bq)}, F32);
    ki.take(gki, *q, {B, H, Nkv, D}, I8);
    ks.take(gks, *q, {B, H, blocks(Nkv, bk)}, F32);
    mean.take(gm, *q, {B, H, D}, F32);
    ws.bytes(gw, *q, api.k_workspace(B, H, Nkv, D));
    void *pq = q->data_ptr(), *pk = k->data_ptr(), *p0 = qi.p(), *p1 = qs.p(), *p2 = ki.p(), *p3 = ks.p(), *p4 = mean.p(), *pw = ws.p();
    const size_t wb = ws.size();
    const int e = call([&] {
        return api.quant_qk(pq, pk, (int8_t*)p0, (float*)p1, (int8_t*)p2, (float*)p3, (float*)p4, pw, wb, B, H, Nq, Nkv, D, sm, bq, bk, st);
    });
    return result(e, {&qi, &qs, &ki, &ks, &mean});
}

// (v, v_i8t | None, v_scale | None, workspace | None, stream | None)
PyObject* py_quant_v(PyObject* const* argv, Py_ssize_t n) {
    if (n != 5) return none();
    Args a(argv);
    const at::Tensor* v = a.in(F16, 4);
    PyObject *gi = a.given(I8), *gs = a.given(F32), *gw = a.scratch();
    void* st = a.stream();
    if (!a.take(gi && gs && gw) || !fits(*v)) return none();
    const int64_t B = v->size(0), H = v->size(1), N = v->size(2), D = v->size(3), Np = blocks(N, 64) * 64;
    if (gi) {
        const at::Tensor& t = *tensor(gi);
        if (t.dim() != 4 || t.size(0) != B || t.size(1) != H || t.size(2) != D || t.size(3) != Np) return none();
    }
    Buffer i8, sc, ws;
    i8.take(gi, *v, {B, H, D, Np}, I8);
    sc.take(gs, *v, {B, H, D}, F32);
    ws.bytes(gw, *v, api.v_workspace(B, H, N, D));
    void *pv = v->data_ptr(), *pi = i8.p(), *ps = sc.p(), *pw = ws.p();
    const size_t wb = ws.size();
    return result(call([&] { return api.quant_v(pv, (int8_t*)pi, (float*)ps, pw, wb, B, H, N, D, st); }), {&i8, &sc});
}

// (kind, q_i8, q_scale, k_i8, k_scale, v, v_scale, causal, sm_scale, block_q, block_k, n_splits, out | None, workspace | None,
// stream | None); PV8: v the INT8 codes, with their scales, else v fp16 and v_scale None; kind: 0 equal lengths, 1 any lengths,
// 2 keys split
template <bool PV8> PyObject* py_attn(PyObject* const* argv, Py_ssize_t n) {
    if (n != 15) return none();
    Args a(argv);
    const int kind = a.integer();
    const at::Tensor *qi = a.in(I8, 4), *qs = a.in(F32, 0), *ki = a.in(I8, 4), *ks = a.in(F32, 0), *v = a.in(PV8 ? I8 : F16, 4);
    PyObject* gvs = a.given(F32);
    const int causal = a.integer();
    const float sm = a.real();
    const int bq = a.integer(), bk = a.integer(), splits = a.integer();
    PyObject *go = a.given(F16), *gw = a.given(U8);
    void* st = a.stream();
    if (!a.take(go && (gw || kind != 2)) || PV8 != (gvs != nullptr) || !fits(*qi) || !fits(*ki) || !fits(*v)) return none();
    const int64_t B = ki->size(0), H = ki->size(1), Nkv = ki->size(2), D = ki->size(3), Nq = qi->size(2);
    if (qi->size(0) != B || qi->size(1) != H || qi->size(3) != D || v->size(0) != B || v->size(1) != H) return none();
    if (kind == 0 && Nq != Nkv) return none();
    if (PV8 ? v->size(2) != D || v->size(3) != blocks(Nkv, 64) * 64 : v->size(2) != Nkv || v->size(3) != D) return none();
    Buffer o, ws;
    o.take(go, *v, {B, H, Nq, D}, F16);
    if (kind == 2) ws.bytes(gw, *v, api.split_workspace(B, H, Nq, Nkv, D, causal != 0, splits));
    void *p0 = qi->data_ptr(), *p1 = qs->data_ptr(), *p2 = ki->data_ptr(), *p3 = ks->data_ptr(), *p4 = v->data_ptr(), *po = o.p(), *pw = ws.p();
    void* pvs = gvs ? tensor(gvs)->data_ptr() : nullptr;
    const size_t wb = ws.size();
    const int c = causal != 0;
    const int e = call([&] {
        const int8_t *q8 = (const int8_t*)p0, *k8 = (const int8_t*)p2, *v8 = (const int8_t*)p4;
        const float *qsc = (const float*)p1, *ksc = (const float*)p3, *vsc = (const float*)pvs;
        if (PV8)
            return kind != 2 ? api.pv8_cross(q8, qsc, k8, ksc, v8, vsc, po, B, H, Nq, Nkv, D, c, sm, bq, bk, st)
                              : api.pv8_split(q8, qsc, k8, ksc, v8, vsc, po, pw, wb, B, H, Nq, Nkv, D, c, sm, bq, bk, splits, st);
        return kind != 2 ? api.attn_cross(q8, qsc, k8, ksc, p4, po, B, H, Nq, Nkv, D, c, sm, bq, bk, st)
                          : api.attn_split(q8, qsc, k8, ksc, p4, po, pw, wb, B, H, Nq, Nkv, D, c, sm, bq, bk, splits, st);
    });
    return result(e, {&o});
}

// (q, k, v, causal, sm_scale, block_q, block_k, pv_int8, out | None, workspace | None, stream | None)
PyObject* py_attention(PyObject* const* argv, Py_ssize_t n) {
    if (n != 11) return none();
    Args a(argv);
    const at::Tensor *q = a.in(F16, 4), *k = a.in(F16, 4), *v = a.in(F16, 4);
    const int causal = a.integer();
    const float sm = a.real();
    const int bq = a.integer(), bk = a.integer(), pv8 = a.integer();
    PyObject *go = a.given(F16), *gw = a.given(U8);
    void* st = a.stream();
    if (!a.take(go && gw) || !fits(*q) || !fits(*k) || v->sizes() != k->sizes()) return none();
    const int64_t B = q->size(0), H = q->size(1), Nq = q->size(2), D = q->size(3), Nkv = k->size(2);
    if (k->size(0) != B || k->size(1) != H || k->size(3) != D) return none();
    if (go && tensor(go)->sizes() != q->sizes()) return none();
    Buffer o, ws;
    o.take(go, *q, {B, H, Nq, D}, F16);
    ws.bytes(gw, *q, api.attention_workspace(B, H, Nq, Nkv, D, causal != 0, bq, bk, pv8 != 0));
    void *pq = q->data_ptr(), *pk = k->data_ptr(), *pv = v->data_ptr(), *po = o.p(), *pw = ws.p();
    const size_t wb = ws.size();
    return result(call([&] { return api.attention(pq, pk, pv, po, pw, wb, B, H, Nq, Nkv, D, causal != 0, sm, bq, bk, pv8 != 0, st); }), {&o});
}

// (torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream, 15 addresses in Api's order)
PyObject* py_init(PyObject* const* argv, Py_ssize_t n) {
    constexpr int COUNT = sizeof(Api) / sizeof(void*);
    if (n != 2 + COUNT) {
        PyErr_SetString(PyExc_ValueError, "init: wrong number of addresses");
        return nullptr;
    }
    void* p[COUNT];
    for (int i = 0; i < COUNT; ++i) {
        p[i] = PyLong_AsVoidPtr(argv[2 + i]);
        if (PyErr_Occurred()) return nullptr;
    }
    static_assert(sizeof p == sizeof api, "Api is function pointers only");
    memcpy(&api, p, sizeof api);
    Py_INCREF(argv[0]);
    Py_INCREF(argv[1]);
    get_device = argv[0];
    get_stream = argv[1];
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"init", (PyCFunction)(void (*)(void))guarded<py_init>, METH_FASTCALL, nullptr},
    {"quant_q", (PyCFunction)(void (*)(void))guarded<py_quant_q<false>>, METH_FASTCALL, nullptr},
    {"rope_quant_q", (PyCFunction)(void (*)(void))guarded<py_quant_q<true>>, METH_FASTCALL, nullptr},
    {"smooth_quant_k", (PyCFunction)(void (*)(void))guarded<py_smooth_quant_k<false>>, METH_FASTCALL, nullptr},
    {"rope_smooth_quant_k", (PyCFunction)(void (*)(void))guarded<py_smooth_quant_k<true>>, METH_FASTCALL, nullptr},
    {"quant_qk", (PyCFunction)(void (*)(void))guarded<py_quant_qk>, METH_FASTCALL, nullptr},
    {"quant_v", (PyCFunction)(void (*)(void))guarded<py_quant_v>, METH_FASTCALL, nullptr},
    {"attn", (PyCFunction)(void (*)(void))guarded<py_attn<false>>, METH_FASTCALL, nullptr},
    {"attn_pv_int8", (PyCFunction)(void (*)(void))guarded<py_attn<true>>, METH_FASTCALL, nullptr},
    {"attention", (PyCFunction)(void (*)(void))guarded<py_attention>, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_sage_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject* PyInit__sage_native(void) {
    PyObject* m = PyModule_Create(&module);
    if (m) PyModule_AddStringConstant(m, "source_hash", tagged_hash + sizeof("SAGE_NATIVE_HASH=") - 1);
    return m;
}
