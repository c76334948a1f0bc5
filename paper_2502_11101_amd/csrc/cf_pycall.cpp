// The marshalling of binding.py in native code (CPython C API): one function per C entry point that takes the
// arguments of its Python namesake in order and returns the cf_status.  A call's arguments are up to 27 pointers and
// integers; ctypes and the stream lookup spent 5.7 us on them, here it is 1.0 us (a decode step's call on the host, with the frequency
// table kept: 13.8 -> 6.8 us, at 12.5 us on the GPU; a 32-layer stack: 469 -> 224 us).
//
// Pointer arguments are None (NULL), an int (an address) or an object with data_ptr() (a tensor); structs come through the
// buffer protocol (the ctypes structures of binding.py); a stream is None (torch's current stream), an int or an object
// with a cuda_stream attribute.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>

#include "cachefocus.h"

namespace {

PyObject *g_data_ptr, *g_cuda_stream;               // interned names
PyObject *g_get_device, *g_get_stream;              // torch._C's raw accessors, once torch has been asked for a stream

// Reads a call's positional arguments one by one; the first failure sticks.
struct Args {
    PyObject* const* v;
    Py_ssize_t n, at = 0;
    bool ok = true;
    Py_buffer held[2];
    int n_held = 0;

    Args(PyObject* const* args, Py_ssize_t count, Py_ssize_t want, const char* name) : v(args), n(count) {
        if (count != want) {
            PyErr_Format(PyExc_TypeError, "%s takes %zd arguments (%zd given)", name, want, count);
            ok = false;
        }
    }
    ~Args() {
        for (int i = 0; i < n_held; ++i) PyBuffer_Release(&held[i]);
    }
    PyObject* next() { return ok ? v[at++] : nullptr; }

    void* ptr() {
        PyObject* o = next();
        if (!o || o == Py_None) return nullptr;
        if (PyLong_Check(o)) return address(o);
        PyObject* p = PyObject_CallMethodNoArgs(o, g_data_ptr);
        if (!p) { ok = false; return nullptr; }
        void* r = address(p);
        Py_DECREF(p);
        return r;
    }
    void* address(PyObject* o) {
        const unsigned long long x = PyLong_AsUnsignedLongLongMask(o);
        if (x == (unsigned long long)-1 && PyErr_Occurred()) ok = false;
        return reinterpret_cast<void*>(static_cast<uintptr_t>(x));
    }
    int64_t i64() {                                  // integers wrap like ctypes'
        PyObject* o = next();
        if (!o) return 0;
        const unsigned long long x = PyLong_AsUnsignedLongLongMask(o);
        if (x == (unsigned long long)-1 && PyErr_Occurred()) ok = false;
        return static_cast<int64_t>(x);
    }
    int32_t i32() { return static_cast<int32_t>(i64()); }
    template <class T> const T* structure() {        // None: NULL
        PyObject* o = next();
        if (!o || o == Py_None) return nullptr;
        if (PyObject_GetBuffer(o, &held[n_held], PyBUF_SIMPLE) != 0) { ok = false; return nullptr; }
        const Py_buffer& b = held[n_held++];
        if (b.len != (Py_ssize_t)sizeof(T)) {
            PyErr_SetString(PyExc_TypeError, "a structure of the wrong size");
            ok = false;
            return nullptr;
        }
        return static_cast<const T*>(b.buf);
    }
    void* stream() {
        PyObject* o = next();
        if (!o) return nullptr;
        if (o == Py_None) return current_stream();
        if (PyLong_Check(o)) return address(o);
        PyObject* s = PyObject_GetAttr(o, g_cuda_stream);
        if (!s) { ok = false; return nullptr; }
        void* r = address(s);
        Py_DECREF(s);
        return r;
    }
    void* current_stream() {
        if (!g_get_stream && !find_accessors()) { ok = false; return nullptr; }
        PyObject* dev = PyObject_CallNoArgs(g_get_device);
        PyObject* s = dev ? PyObject_CallOneArg(g_get_stream, dev) : nullptr;
        Py_XDECREF(dev);
        if (!s) { ok = false; return nullptr; }
        void* r = address(s);
        Py_DECREF(s);
        return r;
    }
    static bool find_accessors() {
        // the first time through the public function, which also initialises torch's side of the device
        PyObject* cuda = PyImport_ImportModule("torch.cuda");
        PyObject* first = cuda ? PyObject_CallMethod(cuda, "current_stream", nullptr) : nullptr;
        PyObject* c = first ? PyImport_ImportModule("torch._C") : nullptr;
        PyObject* dev = c ? PyObject_GetAttrString(c, "_cuda_getDevice") : nullptr;
        PyObject* raw = dev ? PyObject_GetAttrString(c, "_cuda_getCurrentRawStream") : nullptr;
        Py_XDECREF(cuda);
        Py_XDECREF(first);
        Py_XDECREF(c);
        if (!raw) { Py_XDECREF(dev); return false; }
        g_get_device = dev;
        g_get_stream = raw;
        return true;
    }
};

template <class F>
PyObject* finish(const Args& a, F call) {
    if (!a.ok) return nullptr;
    long status;
    Py_BEGIN_ALLOW_THREADS                           // a launch may wait for room in its queue
    status = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

#define CF_PY(NAME) PyObject* NAME(PyObject*, PyObject* const* args, Py_ssize_t nargs)

// (arguments are read into variables first: the order of evaluation inside a call is not defined)
#define CF_ATTENTION_ARGS                                                                                              \
    const cf_layer_desc* desc = a.structure<cf_layer_desc>();                                                          \
    void* q = a.ptr(); void* q_off = a.ptr(); int32_t q_stored = a.i32(); void* q_new = a.ptr();                      \
    void* ks = a.ptr(); void* vs = a.ptr(); int64_t n_store = a.i64(); void* k1 = a.ptr(); void* v1 = a.ptr();        \
    void* segs = a.ptr(); void* n_seg = a.ptr(); int32_t seg_stride = a.i32(); int32_t batch = a.i32();               \
    int32_t max_tq = a.i32(); int64_t max_kv = a.i64(); void* out = a.ptr(); void* mass = a.ptr(); void* score = a.ptr(); \
    int32_t score_stride = a.i32()
#define CF_ATTENTION_PASS                                                                                              \
    desc, q, (const int32_t*)q_off, q_stored, (const int32_t*)q_new, ks, vs, n_store, k1, v1, (const cf_segment*)segs, \
        (const int32_t*)n_seg, seg_stride, batch, max_tq, max_kv, out, (float*)mass, (float*)score, score_stride

CF_PY(prefill_attention) {
    Args a(args, nargs, 24, "prefill_attention");
    CF_ATTENTION_ARGS;
    void* ws = a.ptr(); int64_t ws_bytes = a.i64(); void* flag = a.ptr(); void* stream = a.stream();
    return finish(a, [&] { return cf_prefill_attention(CF_ATTENTION_PASS, ws, (size_t)ws_bytes, (int32_t*)flag, stream); });
}

CF_PY(prefill_attention_static) {
    Args a(args, nargs, 22, "prefill_attention_static");
    CF_ATTENTION_ARGS;
    void* flag = a.ptr(); void* stream = a.stream();
    return finish(a, [&] { return cf_prefill_attention_static(CF_ATTENTION_PASS, (int32_t*)flag, stream); });
}

CF_PY(prefill_layer) {
    Args a(args, nargs, 27, "prefill_layer");
    CF_ATTENTION_ARGS;
    void* ws = a.ptr(); int64_t ws_bytes = a.i64();
    const cf_prune_step* prune = a.structure<cf_prune_step>();
    int32_t n_pending = a.i32(), defer = a.i32(); void* flag = a.ptr(); void* stream = a.stream();
    return finish(a, [&] { return cf_prefill_layer(CF_ATTENTION_PASS, ws, (size_t)ws_bytes, prune, n_pending, defer, (int32_t*)flag, stream); });
}

CF_PY(reposition_keys) {
    Args a(args, nargs, 9, "reposition_keys");
    const cf_layer_desc* desc = a.structure<cf_layer_desc>();
    void* in = a.ptr(); void* out = a.ptr(); void* segs = a.ptr(); int32_t n_seg = a.i32(); int64_t n_store = a.i64();
    int32_t max_len = a.i32(); void* flag = a.ptr(); void* stream = a.stream();
    return finish(a, [&] { return cf_reposition_keys(desc, in, out, (const cf_segment*)segs, n_seg, n_store, max_len, (int32_t*)flag, stream); });
}

CF_PY(assemble_cache) {
    Args a(args, nargs, 23, "assemble_cache");
    const cf_layer_desc* desc = a.structure<cf_layer_desc>();
    void* ks = a.ptr(); void* vs = a.ptr(); int64_t n_store = a.i64(); void* k1 = a.ptr(); void* v1 = a.ptr(); void* q_off = a.ptr();
    void* segs = a.ptr(); void* n_seg = a.ptr(); int32_t seg_stride = a.i32(), batch = a.i32(), max_tq = a.i32(), max_len = a.i32();
    void* off = a.ptr(); int64_t cap = a.i64(), ts = a.i64(), hs = a.i64(); void* kf = a.ptr(); void* vf = a.ptr();
    void* len = a.ptr(); void* pos = a.ptr(); void* flag = a.ptr(); void* stream = a.stream();
    return finish(a, [&] {
        return cf_assemble_cache(desc, ks, vs, n_store, k1, v1, (const int32_t*)q_off, (const cf_segment*)segs, (const int32_t*)n_seg,
                                 seg_stride, batch, max_tq, max_len, (const int64_t*)off, cap, ts, hs, kf, vf, (int32_t*)len,
                                 (int32_t*)pos, (int32_t*)flag, stream);
    });
}

CF_PY(prune_topk) {
    Args a(args, nargs, 11, "prune_topk");
    void* score = a.ptr(); void* len = a.ptr(); void* cand = a.ptr(); void* n_cand = a.ptr();
    int32_t keep = a.i32(), batch = a.i32(), stride = a.i32(); void* idx = a.ptr(); void* n_keep = a.ptr();
    void* flag = a.ptr(); void* stream = a.stream();
    return finish(a, [&] {
        return cf_prune_topk((const float*)score, (const int32_t*)len, (const int32_t*)cand, (const int32_t*)n_cand, keep, batch, stride,
                             (int32_t*)idx, (int32_t*)n_keep, (int32_t*)flag, stream);
    });
}

CF_PY(assign_positions) {
    Args a(args, nargs, 15, "assign_positions");
    void* len = a.ptr(); void* ranked = a.ptr(); void* n_ranked = a.ptr();
    int32_t batch = a.i32(), stride = a.i32(), begin = a.i32(), end = a.i32(), strategy = a.i32(), force = a.i32();
    void* start = a.ptr(); void* q_start = a.ptr(); void* n_reuse = a.ptr(); void* order = a.ptr(); void* flag = a.ptr();
    void* stream = a.stream();
    return finish(a, [&] {
        return cf_assign_positions((const int32_t*)len, (const int32_t*)ranked, (const int32_t*)n_ranked, batch, stride, begin, end, strategy,
                                   force, (int32_t*)start, (int32_t*)q_start, (int32_t*)n_reuse, (int32_t*)order, (int32_t*)flag, stream);
    });
}

CF_PY(gather_segments) {
    Args a(args, nargs, 17, "gather_segments");
    void* off = a.ptr(); void* len = a.ptr(); void* order = a.ptr(); void* n_order = a.ptr(); void* start = a.ptr(); void* q_start = a.ptr();
    void* q_off = a.ptr(); int32_t batch = a.i32(), stride = a.i32(), prefix = a.i32(), doc_start = a.i32(), q_stored = a.i32();
    void* segs = a.ptr(); void* n_seg = a.ptr(); int32_t seg_stride = a.i32(); void* flag = a.ptr(); void* stream = a.stream();
    return finish(a, [&] {
        return cf_gather_segments((const int64_t*)off, (const int32_t*)len, (const int32_t*)order, (const int32_t*)n_order,
                                  (const int32_t*)start, (const int32_t*)q_start, (const int32_t*)q_off, batch, stride, prefix, doc_start,
                                  q_stored, (cf_segment*)segs, (int32_t*)n_seg, seg_stride, (int32_t*)flag, stream);
    });
}

#define CF_METHOD(NAME) {#NAME, (PyCFunction)(void (*)(void))NAME, METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {CF_METHOD(prefill_attention), CF_METHOD(prefill_attention_static), CF_METHOD(prefill_layer),
                           CF_METHOD(reposition_keys), CF_METHOD(assemble_cache), CF_METHOD(prune_topk),
                           CF_METHOD(assign_positions), CF_METHOD(gather_segments), {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_cfcall", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__cfcall(void) {
    g_data_ptr = PyUnicode_InternFromString("data_ptr");
    g_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    return g_data_ptr && g_cuda_stream ? PyModule_Create(&g_module) : nullptr;
}
