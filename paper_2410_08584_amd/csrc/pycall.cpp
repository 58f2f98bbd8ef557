// The calls of a layer and of a decode step, from Python objects to the C ABI without ctypes: reading a tensor's address, shape and
// strides and converting a dozen arguments there takes 3 to 5 us of Python a call, which is what the smallest layers and the decode
// steps over short caches last (a layer of 4 heads, n = 576: four calls, 32.7 us of host time; a decode step: 4.8 us around two
// launches).  A call takes plain torch.Tensor objects and plain numbers; for whatever else (a subclass, another dtype, a shape or
// stride that is not as expected, CUDA not initialised) it returns None before anything is launched, and the caller goes the general way,
// which handles it or says what is wrong.  Otherwise it returns the library's error code.  The GIL is released around the library call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <climits>

#include "zipvl.h"

namespace {

PyObject *s_data_ptr, *s_shape, *s_dtype, *s_stride, *s_numel, *s_is_contiguous, *s_hi_codes, *s_hi_params, *s_lo_codes, *s_lo_params, *s_K, *s_V,
    *s_len_hi, *s_len_lo, *s_cap_hi, *s_cap_lo, *s_d;
PyObject *g_tensor, *g_f32, *g_bf16, *g_is_initialized, *g_get_device, *g_get_stream;

// An owned reference.
struct Ref {
    PyObject* p;
    explicit Ref(PyObject* o) : p(o) {}
    ~Ref() { Py_XDECREF(p); }
    Ref(const Ref&) = delete;
    Ref& operator=(const Ref&) = delete;
};

// The arguments of a call; `ok` falls to false at the first that is not as expected.
struct Args {
    PyObject* const* a;
    bool ok = true;

    PyObject* method(PyObject* self, PyObject* name) { return PyObject_VectorcallMethod(name, &self, 1 | PY_VECTORCALL_ARGUMENTS_OFFSET, nullptr); }
    bool tensor(PyObject* t) { return ok = ok && Py_TYPE(t) == (PyTypeObject*)g_tensor; }
    long long number(PyObject* o) {
        if (!ok || !o || !PyLong_CheckExact(o)) { ok = false; return 0; }
        const long long v = PyLong_AsLongLong(o);
        if (v == -1 && PyErr_Occurred()) ok = false;
        return v;
    }
    int int32(PyObject* o) {
        const long long v = number(o);
        if (v < INT_MIN || v > INT_MAX) ok = false;
        return ok ? (int)v : 0;
    }
    double real(PyObject* o) {
        if (!ok || !(PyFloat_CheckExact(o) || PyLong_CheckExact(o))) { ok = false; return 0; }
        const double v = PyFloat_AsDouble(o);
        if (v == -1 && PyErr_Occurred()) ok = false;
        return v;
    }
    void* address(PyObject* t) {
        if (!tensor(t)) return nullptr;
        Ref r(method(t, s_data_ptr));
        if (!r.p) { ok = false; return nullptr; }
        void* v = PyLong_AsVoidPtr(r.p);
        if (!v && PyErr_Occurred()) ok = false;
        return v;
    }
    void* address_or_null(PyObject* t) { return t == Py_None ? nullptr : address(t); }
    size_t bytes(PyObject* t) {                              // of a workspace: its elements are taken for bytes, as everywhere
        if (!tensor(t)) return 0;
        Ref r(method(t, s_numel));
        if (!r.p) { ok = false; return 0; }
        return (size_t)number(r.p);
    }
    void dense(PyObject* t) {
        if (t == Py_None || !tensor(t)) return;
        Ref r(method(t, s_is_contiguous));
        if (r.p != Py_True) ok = false;
    }
    template <int N> void extents(PyObject* tuple, int64_t (&out)[N]) {
        if (!ok || !tuple || !PyTuple_Check(tuple) || PyTuple_GET_SIZE(tuple) != N) { ok = false; return; }
        for (int i = 0; i < N; ++i) out[i] = number(PyTuple_GET_ITEM(tuple, i));
    }
    template <int N> void shape(PyObject* t, int64_t (&out)[N]) {
        if (!tensor(t)) return;
        Ref r(PyObject_GetAttr(t, s_shape));
        extents(r.p, out);
    }
    void strides(PyObject* t, int64_t (&out)[3]) {           // of a [B, H, n, d] view with contiguous rows
        if (!tensor(t)) return;
        Ref r(method(t, s_stride));
        int64_t st[4] = {};
        extents(r.p, st);
        if (st[3] != 1) ok = false;
        for (int i = 0; i < 3; ++i) out[i] = st[i];
    }
    int dtype(PyObject* t) {
        if (!tensor(t)) return 0;
        Ref r(PyObject_GetAttr(t, s_dtype));
        if (r.p != g_f32 && r.p != g_bf16) ok = false;
        return r.p == g_bf16;
    }
    int32_t narrow(int64_t v) {
        if (v < INT_MIN || v > INT_MAX) ok = false;
        return (int32_t)v;
    }
    // dims of a layer; q may be NULL (its heads are then K's), and v
    zipvl_dims layer(PyObject* q, PyObject* k, PyObject* v) {
        zipvl_dims d = {};
        int64_t sq[4] = {}, sk[4] = {};
        shape(k, sk);
        if (q) shape(q, sq);
        const int64_t* ref = q ? sq : sk;
        d.B = narrow(ref[0]); d.n = narrow(ref[2]); d.d = narrow(ref[3]);
        d.Hq = narrow(ref[1]); d.Hkv = narrow(sk[1]);
        d.dtype = dtype(q ? q : k);
        if (q) strides(q, d.q_strides);
        strides(k, d.k_strides);
        if (v) strides(v, d.v_strides);
        return d;
    }
    zipvl_dims step(PyObject* B, PyObject* Hq, PyObject* Hkv, int64_t n, int64_t dim, int code) {
        zipvl_dims d = {};
        d.B = int32(B); d.Hq = int32(Hq); d.Hkv = int32(Hkv);
        d.n = narrow(n); d.d = narrow(dim); d.dtype = code;
        return d;
    }
    void* stream() {                                         // torch's current one
        if (!ok) return nullptr;
        Ref up(PyObject_CallNoArgs(g_is_initialized));
        if (up.p != Py_True) { ok = false; return nullptr; }
        Ref device(PyObject_CallNoArgs(g_get_device));
        if (!device.p) { ok = false; return nullptr; }
        Ref s(PyObject_CallOneArg(g_get_stream, device.p));
        if (!s.p) { ok = false; return nullptr; }
        void* v = PyLong_AsVoidPtr(s.p);
        if (!v && PyErr_Occurred()) ok = false;
        return v;
    }
};

// What an argument raised the general way raises again; an interrupt (the calls into torch run Python code) would be lost.
PyObject* general_way() {
    if (PyErr_Occurred() && !PyErr_ExceptionMatches(PyExc_Exception)) return nullptr;
    PyErr_Clear();
    Py_RETURN_NONE;
}

// `call` runs without the GIL
template <typename F>
PyObject* finish(const Args& x, F&& call) {
    if (!x.ok) return general_way();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

bool count_is(Py_ssize_t n, Py_ssize_t want) { return n == want; }

// (Q, K, probe_pos, scale, flags, mass, rank, ws)
PyObject* score(PyObject*, PyObject* const* a, Py_ssize_t na) {
    if (!count_is(na, 8)) return general_way();
    Args x{a};
    const zipvl_dims d = x.layer(a[0], a[1], nullptr);
    int32_t probes[ZIPVL_MAX_PROBES];
    const bool list = PyList_CheckExact(a[2]), seq = list || PyTuple_CheckExact(a[2]);
    const Py_ssize_t m = seq ? PySequence_Fast_GET_SIZE(a[2]) : 0;
    if (m < 1 || m > ZIPVL_MAX_PROBES) return general_way();
    for (Py_ssize_t i = 0; i < m; ++i) probes[i] = x.int32(PySequence_Fast_GET_ITEM(a[2], i));
    const float scale = (float)x.real(a[3]);
    const int flags = x.int32(a[4]);
    x.dense(a[5]);
    x.dense(a[6]);
    void *q = x.address(a[0]), *k = x.address(a[1]), *mass = x.address(a[5]), *rank = x.address_or_null(a[6]), *ws = x.address(a[7]);
    const size_t ws_bytes = x.bytes(a[7]);
    void* st = x.stream();
    return finish(x, [&] { return zipvl_score(q, k, &d, probes, (int)m, scale, flags, (float*)mass, (float*)rank, ws, ws_bytes, st); });
}

// (mass, rank, tau, idx, k, status, ws)
PyObject* select(PyObject*, PyObject* const* a, Py_ssize_t na) {
    if (!count_is(na, 7)) return general_way();
    Args x{a};
    int64_t s[2] = {};
    x.shape(a[0], s);
    const int units = x.narrow(s[0]), n = x.narrow(s[1]);
    const double tau = x.real(a[2]);
    x.dense(a[0]);
    x.dense(a[1]);
    x.dense(a[3]);
    x.dense(a[4]);
    void *mass = x.address(a[0]), *rank = x.address_or_null(a[1]), *idx = x.address(a[3]), *k = x.address(a[4]);
    void *status = x.address_or_null(a[5]), *ws = x.address_or_null(a[6]);
    const size_t ws_bytes = a[6] == Py_None ? 0 : x.bytes(a[6]);
    void* st = x.stream();
    return finish(x, [&] { return zipvl_select((float*)mass, (float*)rank, units, n, tau, (int32_t*)idx, (int32_t*)k, (int32_t*)status, ws, ws_bytes, st); });
}

// (K, V, idx, k, cap, flags, Kc, Vc, len)
PyObject* compact_kv(PyObject*, PyObject* const* a, Py_ssize_t na) {
    if (!count_is(na, 9)) return general_way();
    Args x{a};
    const zipvl_dims d = x.layer(nullptr, a[0], a[1]);
    const int cap = x.int32(a[4]), flags = x.int32(a[5]);
    void *K = x.address(a[0]), *V = x.address(a[1]), *idx = x.address_or_null(a[2]), *k = x.address_or_null(a[3]);
    void *Kc = x.address(a[6]), *Vc = x.address(a[7]), *len = x.address(a[8]);
    void* st = x.stream();
    return finish(x, [&] { return zipvl_compact_kv(K, V, &d, (int32_t*)idx, (int32_t*)k, Kc, Vc, cap, (int32_t*)len, flags, st); });
}

// (Q, K, V, idx, k, scale, flags, O, ws)
PyObject* sparse_prefill(PyObject*, PyObject* const* a, Py_ssize_t na) {
    if (!count_is(na, 9)) return general_way();
    Args x{a};
    const zipvl_dims d = x.layer(a[0], a[1], a[2]);
    const float scale = (float)x.real(a[5]);
    const int flags = x.int32(a[6]);
    void *Q = x.address(a[0]), *K = x.address(a[1]), *V = x.address(a[2]), *idx = x.address_or_null(a[3]), *k = x.address_or_null(a[4]);
    void *O = x.address(a[7]), *ws = x.address(a[8]);
    const size_t ws_bytes = x.bytes(a[8]);
    void* st = x.stream();
    return finish(x, [&] { return zipvl_sparse_prefill(Q, K, V, &d, (int32_t*)idx, (int32_t*)k, scale, flags, O, ws, ws_bytes, st); });
}

// (Kc, Vc, len, k_new, v_new, B, Hkv)
PyObject* kv_append(PyObject*, PyObject* const* a, Py_ssize_t na) {
    if (!count_is(na, 7)) return general_way();
    Args x{a};
    int64_t s[3] = {};
    x.shape(a[0], s);
    const zipvl_dims d = x.step(a[5], a[6], a[6], s[1], s[2], x.dtype(a[0]));
    void *Kc = x.address(a[0]), *Vc = x.address(a[1]), *len = x.address(a[2]), *kn = x.address(a[3]), *vn = x.address(a[4]);
    void* st = x.stream();
    return finish(x, [&] { return zipvl_kv_append(Kc, Vc, (int32_t*)len, d.n, kn, vn, &d, st); });
}

// (q, Kc, Vc, len, k_new, v_new, scale, B, Hq, Hkv, ws, o)
PyObject* decode_step(PyObject*, PyObject* const* a, Py_ssize_t na) {
    if (!count_is(na, 12)) return general_way();
    Args x{a};
    int64_t s[3] = {};
    x.shape(a[1], s);
    const zipvl_dims d = x.step(a[7], a[8], a[9], s[1], s[2], x.dtype(a[1]));
    const float scale = (float)x.real(a[6]);
    void *q = x.address(a[0]), *Kc = x.address(a[1]), *Vc = x.address(a[2]), *len = x.address(a[3]), *kn = x.address(a[4]), *vn = x.address(a[5]);
    void *ws = x.address(a[10]), *o = x.address(a[11]);
    const size_t ws_bytes = x.bytes(a[10]);
    void* st = x.stream();
    return finish(x, [&] { return zipvl_decode_step(q, Kc, Vc, (int32_t*)len, d.n, kn, vn, &d, scale, o, ws, ws_bytes, st); });
}

// (q, cache, scale, B, Hq, Hkv, K_tail, V_tail, len_tail, o, ws)
PyObject* decode_attn_q(PyObject*, PyObject* const* a, Py_ssize_t na) {
    if (!count_is(na, 11)) return general_way();
    Args x{a};
    Ref K(PyObject_GetAttr(a[1], s_K)), V(PyObject_GetAttr(a[1], s_V)), lh(PyObject_GetAttr(a[1], s_len_hi)), ll(PyObject_GetAttr(a[1], s_len_lo));
    Ref ch(PyObject_GetAttr(a[1], s_cap_hi)), cl(PyObject_GetAttr(a[1], s_cap_lo)), dd(PyObject_GetAttr(a[1], s_d));
    if (!K.p || !V.p || !lh.p || !ll.p || !ch.p || !cl.p || !dd.p || !PyDict_CheckExact(K.p) || !PyDict_CheckExact(V.p)) return general_way();
    auto parts = [&](PyObject* dict) {
        auto part = [&](PyObject* name) -> void* {
            if (!x.ok) return nullptr;
            PyObject* t = PyDict_GetItemWithError(dict, name);
            if (!t) { x.ok = false; return nullptr; }
            return x.address(t);
        };
        zipvl_qtensor t;
        t.hi_codes = decltype(t.hi_codes)(part(s_hi_codes));
        t.hi_params = decltype(t.hi_params)(part(s_hi_params));
        t.lo_codes = decltype(t.lo_codes)(part(s_lo_codes));
        t.lo_params = decltype(t.lo_params)(part(s_lo_params));
        return t;
    };
    const zipvl_qtensor kq = parts(K.p), vq = parts(V.p);
    const int cap_hi = x.int32(ch.p), cap_lo = x.int32(cl.p);
    int64_t s[3] = {};
    if (a[6] != Py_None) x.shape(a[6], s);
    const zipvl_dims d = x.step(a[3], a[4], a[5], (int64_t)cap_hi + cap_lo + s[1], x.number(dd.p), x.dtype(a[0]));
    const float scale = (float)x.real(a[2]);
    void *q = x.address(a[0]), *hi = x.address(lh.p), *lo = x.address(ll.p), *Kt = x.address_or_null(a[6]), *Vt = x.address_or_null(a[7]);
    void *lt = x.address_or_null(a[8]), *o = x.address(a[9]), *ws = x.address(a[10]);
    const size_t ws_bytes = x.bytes(a[10]);
    const int cap_tail = x.narrow(s[1]);
    void* st = x.stream();
    return finish(x, [&] {
        return zipvl_decode_attn_q(q, &kq, &vq, (int32_t*)hi, (int32_t*)lo, cap_hi, cap_lo, Kt, Vt, (int32_t*)lt, cap_tail, &d, scale, o, ws, ws_bytes, st);
    });
}

#define ZIPVL_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {ZIPVL_METHOD(score), ZIPVL_METHOD(select), ZIPVL_METHOD(compact_kv), ZIPVL_METHOD(sparse_prefill), ZIPVL_METHOD(kv_append),
                         ZIPVL_METHOD(decode_step), ZIPVL_METHOD(decode_attn_q), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pycall", "Calls of libzipvl.so on torch tensors", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pycall(void) {
    struct { PyObject** at; const char* text; } names[] = {
        {&s_data_ptr, "data_ptr"}, {&s_shape, "shape"}, {&s_dtype, "dtype"}, {&s_stride, "stride"}, {&s_numel, "numel"}, {&s_is_contiguous, "is_contiguous"},
        {&s_hi_codes, "hi_codes"}, {&s_hi_params, "hi_params"}, {&s_lo_codes, "lo_codes"}, {&s_lo_params, "lo_params"}, {&s_K, "K"}, {&s_V, "V"},
        {&s_len_hi, "len_hi"}, {&s_len_lo, "len_lo"}, {&s_cap_hi, "cap_hi"}, {&s_cap_lo, "cap_lo"}, {&s_d, "d"}};
    for (auto& n : names)
        if (!(*n.at = PyUnicode_InternFromString(n.text))) return nullptr;
    Ref torch(PyImport_ImportModule("torch"));
    if (!torch.p) return nullptr;
    struct { PyObject** at; const char *in, *name; } objects[] = {
        {&g_tensor, nullptr, "Tensor"}, {&g_f32, nullptr, "float32"}, {&g_bf16, nullptr, "bfloat16"}, {&g_is_initialized, "cuda", "is_initialized"},
        {&g_get_device, "_C", "_cuda_getDevice"}, {&g_get_stream, "_C", "_cuda_getCurrentRawStream"}};
    for (auto& o : objects) {
        Ref in(o.in ? PyObject_GetAttrString(torch.p, o.in) : nullptr);
        if (o.in && !in.p) return nullptr;
        if (!(*o.at = PyObject_GetAttrString(o.in ? in.p : torch.p, o.name))) return nullptr;
    }
    return PyModule_Create(&module);
}
