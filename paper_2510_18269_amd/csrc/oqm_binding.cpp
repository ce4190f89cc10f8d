// Argument marshalling of the hot-path calls of libtom_oqm.so for the Python binding.
//
// A one-frame append or a small retrieval keeps the GPU busy for 6 to 20 us, less than what
// ctypes, torch.cuda.current_stream() and the per-tensor attribute look-ups in Python cost the
// host around the launches (append 9.3 us, retrieval 19.9 us, the four calls of a tiny stream
// 39 us with a launch at 3.2 us).  Here a tensor costs one data_ptr() call and the stream one
// call of torch's raw-stream getter.  The library is entered without the interpreter lock, as
// ctypes enters it.
//
// Every function takes positional arguments only and returns an int or None; the public
// functions with their names and defaults are in oqm.py.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>

#include "tom_oqm.h"

namespace {

PyObject *g_raise, *g_int32, *g_int64, *g_void_p, *g_is_initialized, *g_get_device, *g_get_raw_stream, *g_slow_stream;
PyObject *s_is_cuda, *s_data_ptr, *s_numel, *s_element_size, *s_stride, *s_cuda_stream;

// What ctypes does with c_int32 / c_int64: a Python int is truncated; `slow`, a callable registered by oqm.py, makes
// one of whatever else ctypes takes (__index__, its own integer objects) or raises its error.
bool to_int(PyObject* o, PyObject* slow, int64_t& out) {
    if (PyLong_Check(o)) {
        out = (int64_t)PyLong_AsUnsignedLongLongMask(o);
        return true;
    }
    PyObject* r = PyObject_CallOneArg(slow, o);
    if (!r) return false;
    const bool ok = PyLong_Check(r);
    if (ok) out = (int64_t)PyLong_AsUnsignedLongLongMask(r);
    else PyErr_SetString(PyExc_SystemError, "the registered conversion did not return an int");
    Py_DECREF(r);
    return ok;
}
bool to_i64(PyObject* o, int64_t& out) { return to_int(o, g_int64, out); }
bool to_i32(PyObject* o, int32_t& out) {
    int64_t v;
    if (!to_int(o, g_int32, v)) return false;
    out = (int32_t)(uint32_t)v;
    return true;
}

bool method_i64(PyObject* o, PyObject* name, int64_t& out) {
    PyObject* r = PyObject_CallMethodNoArgs(o, name);
    if (!r) return false;
    const bool ok = to_i64(r, out);
    Py_DECREF(r);
    return ok;
}

// What ctypes does with c_void_p: None, an int, or (through the registered callable) one of its own pointer
// objects.  A handle is never anything else: a tensor's address must not be taken for one.
bool to_void_p(PyObject* o, void*& out) {
    int64_t v = 0;
    if (o != Py_None && !to_int(o, g_void_p, v)) return false;
    out = reinterpret_cast<void*>((uintptr_t)v);
    return true;
}
bool to_handle(PyObject* o, tom_oqm_t*& out) {
    void* p;
    if (!to_void_p(o, p)) return false;
    out = static_cast<tom_oqm_t*>(p);
    return true;
}

// None, a raw device pointer, or a tensor on the device.
bool to_ptr(PyObject* o, void*& out) {
    if (o == Py_None || PyLong_Check(o)) return to_void_p(o, out);
    PyObject* c = PyObject_GetAttr(o, s_is_cuda);
    if (!c) return false;
    const int on_device = PyObject_IsTrue(c);
    Py_DECREF(c);
    if (on_device < 0) return false;
    if (!on_device) {
        PyErr_SetString(PyExc_AssertionError, "device tensor expected");
        return false;
    }
    PyObject* r = PyObject_CallMethodNoArgs(o, s_data_ptr);
    if (!r) return false;
    const bool ok = to_void_p(r, out);
    Py_DECREF(r);
    return ok;
}

// None: the current stream of the current device; else a raw handle or an object with one.
bool to_stream(PyObject* o, void*& out) {
    if (PyLong_Check(o)) return to_void_p(o, out);
    PyObject* r;
    if (o == Py_None) {
        PyObject* up = PyObject_CallNoArgs(g_is_initialized);
        if (!up) return false;
        const int ready = PyObject_IsTrue(up);
        Py_DECREF(up);
        if (ready < 0) return false;
        if (ready) {
            PyObject* dev = PyObject_CallNoArgs(g_get_device);
            if (!dev) return false;
            r = PyObject_CallOneArg(g_get_raw_stream, dev);
            Py_DECREF(dev);
        } else {
            r = PyObject_CallNoArgs(g_slow_stream);  // initialises the device, or finds that there is none
        }
    } else {
        r = PyObject_GetAttr(o, s_cuda_stream);
    }
    if (!r) return false;
    const bool ok = to_void_p(r, out);
    Py_DECREF(r);
    return ok;
}

// Workspace tensor (or None): pointer and size in bytes.
bool to_workspace(PyObject* o, void*& ptr, size_t& bytes) {
    bytes = 0;
    if (o != Py_None) {
        int64_t n, e;
        if (!method_i64(o, s_numel, n) || !method_i64(o, s_element_size, e)) return false;
        bytes = (size_t)n * (size_t)e;
    }
    return to_ptr(o, ptr);
}

bool arity(Py_ssize_t n, Py_ssize_t want) {
    if (n == want) return true;
    PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", want, n);
    return false;
}

// TOM_OK -> `result`; anything else raises through the callable that oqm.py registered.
PyObject* finish(int status, PyObject* result) {
    if (status == TOM_OK || !result) return result;
    Py_DECREF(result);
    PyObject* st = PyLong_FromLong(status);
    if (!st) return nullptr;
    PyObject* r = PyObject_CallOneArg(g_raise, st);
    Py_DECREF(st);
    if (r) {
        Py_DECREF(r);
        PyErr_SetString(PyExc_SystemError, "the registered error callable returned");
    }
    return nullptr;
}
PyObject* finish_none(int status) {
    Py_INCREF(Py_None);
    return finish(status, Py_None);
}

// The strides of a tensor as a new tuple.
PyObject* strides_of(PyObject* tensor) {
    PyObject* s = PyObject_CallMethodNoArgs(tensor, s_stride);
    if (!s || PyTuple_CheckExact(s)) return s;
    PyObject* t = PySequence_Tuple(s);
    Py_DECREF(s);
    return t;
}

// strides: a tuple of four, or None for 5-d tensors k and v of equal strides with contiguous channels.
bool to_strides(PyObject* o, PyObject* k, PyObject* v, int64_t (&out)[4]) {
    PyObject* t = o;
    if (o == Py_None) {
        t = strides_of(k);
        if (!t) return false;
    } else {
        Py_INCREF(t);
    }
    bool ok = PyTuple_Check(t) && PyTuple_GET_SIZE(t) == (o == Py_None ? 5 : 4);
    if (ok && o == Py_None) {
        int64_t channel = 0;
        ok = to_i64(PyTuple_GET_ITEM(t, 4), channel) && channel == 1;
        if (ok) {
            PyObject* vs = strides_of(v);
            const int same = vs ? PyObject_RichCompareBool(vs, t, Py_EQ) : -1;
            Py_XDECREF(vs);
            if (same == 0) PyErr_SetString(PyExc_AssertionError, "k and v must have the same strides");
            if (same != 1) {
                Py_DECREF(t);
                return false;
            }
        }
    }
    if (!ok) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_AssertionError, "contiguous channel axis expected");
    } else {
        for (int i = 0; i < 4 && ok; ++i) ok = to_i64(PyTuple_GET_ITEM(t, i), out[i]);
    }
    Py_DECREF(t);
    return ok;
}

PyObject* set_num_groups(PyObject*, PyObject* const* a, Py_ssize_t n) {
    tom_oqm_t* h;
    int32_t groups;
    if (!arity(n, 2) || !to_handle(a[0], h) || !to_i32(a[1], groups)) return nullptr;
    return finish_none(tom_oqm_set_num_groups(h, groups));
}

// h, layer0, n_layers, n_frames, k, v, k_for_summary, strides, commit, stream -> first group
PyObject* quantize_append(PyObject*, PyObject* const* a, Py_ssize_t n) {
    tom_oqm_t* h;
    void *k, *v, *ks, *stream;
    int32_t layer0, n_layers, n_frames, first = -1;
    int64_t strides[4];
    if (!arity(n, 10) || !to_strides(a[7], a[4], a[5], strides) || !to_handle(a[0], h) || !to_i32(a[1], layer0) ||
        !to_i32(a[2], n_layers) || !to_i32(a[3], n_frames) || !to_ptr(a[4], k) || !to_ptr(a[5], v) || !to_ptr(a[6], ks))
        return nullptr;
    const int commit = PyObject_IsTrue(a[8]);
    if (commit < 0 || !to_stream(a[9], stream)) return nullptr;
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = tom_oqm_quantize_append(h, layer0, n_layers, n_frames, k, v, ks, strides, commit,
                                 stream, &first);
    Py_END_ALLOW_THREADS
    return finish(st, PyLong_FromLong(first));
}

// h, layer0, n_layers, q, q_dtype, t_q, scores, score_stride, token_scores, path, workspace, stream
PyObject* score_groups(PyObject*, PyObject* const* a, Py_ssize_t n) {
    tom_oqm_t* h;
    void *q, *scores, *tokens, *ws, *stream;
    int32_t layer0, n_layers, q_dtype, t_q, path;
    int64_t stride;
    size_t ws_bytes;
    if (!arity(n, 12) || !to_handle(a[0], h) || !to_i32(a[1], layer0) || !to_i32(a[2], n_layers) || !to_ptr(a[3], q) ||
        !to_i32(a[4], q_dtype) || !to_i32(a[5], t_q) || !to_ptr(a[6], scores) || !to_i64(a[7], stride) ||
        !to_ptr(a[8], tokens) || !to_i32(a[9], path) || !to_workspace(a[10], ws, ws_bytes) || !to_stream(a[11], stream))
        return nullptr;
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = tom_oqm_score_groups(h, layer0, n_layers, q, q_dtype, t_q,
                              static_cast<float*>(scores), stride, static_cast<float*>(tokens), path, ws, ws_bytes,
                              stream);
    Py_END_ALLOW_THREADS
    return finish_none(st);
}

// scores, score_stride, n_rows, n_groups, k, order, idx, stream -> k_eff
PyObject* topk(PyObject*, PyObject* const* a, Py_ssize_t n) {
    void *scores, *idx, *stream;
    int32_t n_rows, n_groups, k, order, k_eff = -1;
    int64_t stride;
    if (!arity(n, 8) || !to_ptr(a[0], scores) || !to_i64(a[1], stride) || !to_i32(a[2], n_rows) ||
        !to_i32(a[3], n_groups) || !to_i32(a[4], k) || !to_i32(a[5], order) || !to_ptr(a[6], idx) ||
        !to_stream(a[7], stream))
        return nullptr;
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = tom_oqm_topk(static_cast<float*>(scores), stride, n_rows, n_groups, k, order, static_cast<int32_t*>(idx),
                      &k_eff, stream);
    Py_END_ALLOW_THREADS
    return finish(st, PyLong_FromLong(k_eff));
}

// h, layer0, n_layers, idx, k, k_eff, k_out, v_out, stream
PyObject* dequant_gather(PyObject*, PyObject* const* a, Py_ssize_t n) {
    tom_oqm_t* h;
    void *idx, *ko, *vo, *stream;
    int32_t layer0, n_layers, k, k_eff;
    if (!arity(n, 9) || !to_handle(a[0], h) || !to_i32(a[1], layer0) || !to_i32(a[2], n_layers) || !to_ptr(a[3], idx) ||
        !to_i32(a[4], k) || !to_i32(a[5], k_eff) || !to_ptr(a[6], ko) || !to_ptr(a[7], vo) || !to_stream(a[8], stream))
        return nullptr;
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = tom_oqm_dequant_gather(h, layer0, n_layers, static_cast<int32_t*>(idx), k, k_eff, ko,
                                vo, stream);
    Py_END_ALLOW_THREADS
    return finish_none(st);
}

// h, layer0, n_layers, idx, k, k_eff, prefix_rows, sys_k, sys_v, k_out, v_out, stream
PyObject* assemble_active(PyObject*, PyObject* const* a, Py_ssize_t n) {
    tom_oqm_t* h;
    void *idx, *sk, *sv, *ko, *vo, *stream;
    int32_t layer0, n_layers, k, k_eff, prefix;
    if (!arity(n, 12) || !to_handle(a[0], h) || !to_i32(a[1], layer0) || !to_i32(a[2], n_layers) || !to_ptr(a[3], idx) ||
        !to_i32(a[4], k) || !to_i32(a[5], k_eff) || !to_i32(a[6], prefix) || !to_ptr(a[7], sk) || !to_ptr(a[8], sv) ||
        !to_ptr(a[9], ko) || !to_ptr(a[10], vo) || !to_stream(a[11], stream))
        return nullptr;
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = tom_oqm_assemble_active(h, layer0, n_layers, static_cast<int32_t*>(idx), k, k_eff,
                                 prefix, sk, sv, ko, vo, stream);
    Py_END_ALLOW_THREADS
    return finish_none(st);
}

// h, layer0, n_layers, q, q_dtype, t_q, k, path, scores, score_stride, idx, prefix_rows, sys_k, sys_v, k_out, v_out,
// [workspace,] stream -> k_eff; without a workspace the library's static scratch array is used
PyObject* retrieve_with(PyObject* const* a, bool own_workspace) {
    tom_oqm_t* h;
    void *q, *scores, *idx, *sk, *sv, *ko, *vo, *ws = nullptr, *stream;
    int32_t layer0, n_layers, q_dtype, t_q, k, path, prefix, k_eff = -1;
    int64_t stride;
    size_t ws_bytes = 0;
    if (!to_handle(a[0], h) || !to_i32(a[1], layer0) || !to_i32(a[2], n_layers) || !to_ptr(a[3], q) ||
        !to_i32(a[4], q_dtype) || !to_i32(a[5], t_q) || !to_i32(a[6], k) || !to_i32(a[7], path) ||
        !to_ptr(a[8], scores) || !to_i64(a[9], stride) || !to_ptr(a[10], idx) || !to_i32(a[11], prefix) ||
        !to_ptr(a[12], sk) || !to_ptr(a[13], sv) || !to_ptr(a[14], ko) || !to_ptr(a[15], vo) ||
        (own_workspace && !to_workspace(a[16], ws, ws_bytes)) || !to_stream(a[own_workspace ? 17 : 16], stream))
        return nullptr;
    int st;
    Py_BEGIN_ALLOW_THREADS
    if (own_workspace)
        st = tom_oqm_retrieve(h, layer0, n_layers, q, q_dtype, t_q, k, path,
                              static_cast<float*>(scores), stride, static_cast<int32_t*>(idx), prefix, sk, sv, ko, vo,
                              ws, ws_bytes, &k_eff, stream);
    else
        st = tom_oqm_retrieve_noalloc(h, layer0, n_layers, q, q_dtype, t_q, k, path,
                                      static_cast<float*>(scores), stride, static_cast<int32_t*>(idx), prefix, sk, sv,
                                      ko, vo, &k_eff, stream);
    Py_END_ALLOW_THREADS
    return finish(st, PyLong_FromLong(k_eff));
}
PyObject* retrieve(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return arity(n, 18) ? retrieve_with(a, true) : nullptr;
}
PyObject* retrieve_noalloc(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return arity(n, 17) ? retrieve_with(a, false) : nullptr;
}

// The Python callables that the functions above need, in the order of the globals.
PyObject* setup(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (!arity(n, 8)) return nullptr;
    PyObject** const slots[8] = {&g_raise, &g_int32, &g_int64, &g_void_p, &g_is_initialized, &g_get_device, &g_get_raw_stream,
                                 &g_slow_stream};
    for (int i = 0; i < 8; ++i) {
        Py_INCREF(a[i]);
        Py_XSETREF(*slots[i], a[i]);
    }
    Py_RETURN_NONE;
}

#define FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(setup), FAST(set_num_groups), FAST(quantize_append), FAST(score_groups), FAST(topk),
                         FAST(dequant_gather), FAST(assemble_active), FAST(retrieve), FAST(retrieve_noalloc),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_oqm_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__oqm_binding(void) {
    s_is_cuda = PyUnicode_InternFromString("is_cuda");
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_numel = PyUnicode_InternFromString("numel");
    s_element_size = PyUnicode_InternFromString("element_size");
    s_stride = PyUnicode_InternFromString("stride");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (!s_is_cuda || !s_data_ptr || !s_numel || !s_element_size || !s_stride || !s_cuda_stream) return nullptr;
    return PyModule_Create(&module);
}
