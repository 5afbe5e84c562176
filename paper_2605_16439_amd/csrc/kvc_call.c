/* Argument marshalling of the per-layer entry points for the Python binding, in C: a decode step calls the library once per
 * layer, and what a caller pays per call beyond the kernel launches is time in which a small call's GPU idles.  Measured on the
 * MI355X host for a call of two launches: 13.7 us with ctypes objects and torch.cuda.current_stream() (2.8 us of it), of which
 * the library itself 6 to 7 us.
 *
 * Each function takes the binding's Python objects as they are: ctypes structures (buffer protocol), tensors (data_ptr()),
 * None, numbers.  The addresses of the library's functions come from the binding (bind()), so there is one copy of the
 * library.  The interpreter lock is released during the call. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include "../../include/kvcapsule.h"

static PyObject *s_data_ptr, *s_numel, *s_stride, *s_size, *k_int[4];

/* address of a ctypes structure of `size` bytes (its owner outlives the call: it is one of the arguments) */
static int address_of(PyObject *o, Py_ssize_t size, const void **out)
{
    Py_buffer v;
    if (PyObject_GetBuffer(o, &v, PyBUF_SIMPLE) != 0) return -1;
    const int ok = v.len == size;
    *out = v.buf;
    PyBuffer_Release(&v);
    if (!ok) PyErr_SetString(PyExc_TypeError, "structure of another size");
    return ok ? 0 : -1;
}
static int method_u64(PyObject *o, PyObject *name, uint64_t *out)
{
    PyObject *r = PyObject_CallMethodNoArgs(o, name);
    if (!r) return -1;
    *out = PyLong_AsUnsignedLongLongMask(r);
    Py_DECREF(r);
    return *out == (uint64_t)-1 && PyErr_Occurred() ? -1 : 0;
}
static int pointer_of(PyObject *o, void **out)          /* a tensor, or None */
{
    uint64_t a = 0;
    if (o != Py_None && method_u64(o, s_data_ptr, &a) != 0) return -1;
    *out = (void *)(uintptr_t)a;
    return 0;
}
static int int_of(PyObject *o, int64_t *out)            /* what int() takes; wider values are cut off as ctypes does */
{
    if (PyLong_CheckExact(o)) {
        *out = (int64_t)PyLong_AsUnsignedLongLongMask(o);
    } else {
        PyObject *r = PyNumber_Long(o);
        if (!r) return -1;
        *out = (int64_t)PyLong_AsUnsignedLongLongMask(r);
        Py_DECREF(r);
    }
    return *out == -1 && PyErr_Occurred() ? -1 : 0;
}
static int workspace_of(PyObject *o, void **p, size_t *bytes)       /* 256-byte aligned part of a byte tensor */
{
    uint64_t base, n;
    if (method_u64(o, s_data_ptr, &base) != 0 || method_u64(o, s_numel, &n) != 0) return -1;
    const uint64_t off = (0 - base) & 255u;
    *p = (void *)(uintptr_t)(base + off);
    *bytes = n - off;
    return 0;
}

static void *g_compress, *g_compress_generic, *g_decode, *g_decode_generic, *g_decode_static, *g_ragged, *g_hidden, *g_static, *g_full;

static PyObject *bind(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    (void)self;
    void **const f[9] = {&g_compress, &g_compress_generic, &g_decode, &g_decode_generic, &g_decode_static, &g_ragged, &g_hidden, &g_static, &g_full};
    if (n != 9) { PyErr_SetString(PyExc_TypeError, "nine function addresses"); return NULL; }
    for (int i = 0; i < 9; ++i) {
        *f[i] = PyLong_AsVoidPtr(a[i]);
        if (!*f[i]) { if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address"); return NULL; }
    }
    Py_RETURN_NONE;
}

#define ARGS(N) do { (void)self; if (n != (N)) { PyErr_SetString(PyExc_TypeError, "number of arguments"); return NULL; } \
                     if (!g_full) { PyErr_SetString(PyExc_RuntimeError, "bind() first"); return NULL; } } while (0)
#define SHAPE(i, v) const void *v; if (address_of(a[i], sizeof(kvc_shape), &v)) return NULL
#define PARAMS(i, v) const void *v; if (address_of(a[i], sizeof(kvc_params), &v)) return NULL
#define PTR(i, v) void *v; if (pointer_of(a[i], &v)) return NULL
#define INT(i, v) int64_t v; if (int_of(a[i], &v)) return NULL
#define FLT(i, v) const double v = PyFloat_AsDouble(a[i]); if (v == -1.0 && PyErr_Occurred()) return NULL
#define WS(i, v, b) void *v; size_t b; if (workspace_of(a[i], &v, &b)) return NULL
#define STREAM(i, v) int64_t v##_; if (int_of(a[i], &v##_)) return NULL; void *v = (void *)(uintptr_t)v##_
#define RETURN_STATUS(call) do { int st_; Py_BEGIN_ALLOW_THREADS st_ = (int)(call); Py_END_ALLOW_THREADS return PyLong_FromLong(st_); } while (0)

/* shape, params, K, V, vis_start, Kc, Vc, workspace, stream, generic: K and V strided alike, d contiguous (checked by the caller) */
static PyObject *compress(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    ARGS(10);
    SHAPE(0, s); PARAMS(1, p); PTR(2, K); PTR(3, V); INT(4, vis); PTR(5, Kc); PTR(6, Vc); WS(7, w, wb); STREAM(8, st);
    PyObject *sk = PyObject_CallMethodNoArgs(a[2], s_stride), *sv = sk ? PyObject_CallMethodNoArgs(a[3], s_stride) : NULL;
    int64_t x[4] = {0, 0, 0, 0}, len = 0;
    int ok = 0;
    if (sv) {
        ok = PyObject_RichCompareBool(sk, sv, Py_EQ);
        if (ok == 1 && PyTuple_Check(sk) && PyTuple_GET_SIZE(sk) == 4) {
            for (int i = 0; i < 4 && ok == 1; ++i) ok = int_of(PyTuple_GET_ITEM(sk, i), &x[i]) == 0 ? 1 : -1;
            if (ok == 1 && x[3] != 1) ok = 0;
        } else if (ok == 1) {
            ok = 0;
        }
        if (ok == 0) PyErr_SetString(PyExc_AssertionError, "K and V have four dimensions, the same strides and contiguous channels");
    }
    Py_XDECREF(sk);
    Py_XDECREF(sv);
    if (ok != 1) return NULL;
    PyObject *r = PyObject_CallMethodOneArg(a[2], s_size, k_int[2]);
    if (!r) return NULL;
    ok = int_of(r, &len);
    Py_DECREF(r);
    if (ok != 0) return NULL;
    const int gen = PyObject_IsTrue(a[9]);
    if (gen < 0) return NULL;
    kvc_status (*f)(const kvc_shape *, const kvc_params *, const void *, const void *, int64_t, int64_t, int64_t, int32_t, int32_t, void *,
                    void *, void *, size_t, void *) = gen ? g_compress_generic : g_compress;
    RETURN_STATUS(f(s, p, K, V, x[0], x[1], x[2], (int32_t)vis, (int32_t)len, Kc, Vc, w, wb, st));
}

/* shape, params, q, Kc, Vc, Kt, Vt, text_len, text_cap, k_new, v_new, scale, out, lse, workspace, stream, generic */
static PyObject *decode(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    ARGS(17);
    SHAPE(0, s); PARAMS(1, p); PTR(2, q); PTR(3, Kc); PTR(4, Vc); PTR(5, Kt); PTR(6, Vt); INT(7, t); INT(8, cap); PTR(9, kn); PTR(10, vn);
    FLT(11, sc); PTR(12, out); PTR(13, lse); WS(14, w, wb); STREAM(15, st);
    const int gen = PyObject_IsTrue(a[16]);
    if (gen < 0) return NULL;
    kvc_status (*f)(const kvc_shape *, const kvc_params *, const void *, const void *, const void *, void *, void *, int32_t, int32_t,
                    const void *, const void *, float, void *, float *, void *, size_t, void *) = gen ? g_decode_generic : g_decode;
    RETURN_STATUS(f(s, p, q, Kc, Vc, Kt, Vt, (int32_t)t, (int32_t)cap, kn, vn, (float)sc, out, lse, w, wb, st));
}

/* shape, params, q, Kc, Vc, Kt, Vt, text_len, text_cap, k_new, v_new, scale, out, lse, stream */
static PyObject *decode_static(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    ARGS(15);
    SHAPE(0, s); PARAMS(1, p); PTR(2, q); PTR(3, Kc); PTR(4, Vc); PTR(5, Kt); PTR(6, Vt); INT(7, t); INT(8, cap); PTR(9, kn); PTR(10, vn);
    FLT(11, sc); PTR(12, out); PTR(13, lse); STREAM(14, st);
    kvc_status (*f)(const kvc_shape *, const kvc_params *, const void *, const void *, const void *, void *, void *, int32_t, int32_t,
                    const void *, const void *, float, void *, float *, void *) = g_decode_static;
    RETURN_STATUS(f(s, p, q, Kc, Vc, Kt, Vt, (int32_t)t, (int32_t)cap, kn, vn, (float)sc, out, lse, st));
}

/* shape, params, q, Kc, Vc, Kt, Vt, n_images, text_len, text_cap, k_new, v_new, scale, out, lse, workspace, stream */
static PyObject *ragged(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    ARGS(17);
    SHAPE(0, s); PARAMS(1, p); PTR(2, q); PTR(3, Kc); PTR(4, Vc); PTR(5, Kt); PTR(6, Vt); PTR(7, ni); PTR(8, tl); INT(9, cap); PTR(10, kn); PTR(11, vn);
    FLT(12, sc); PTR(13, out); PTR(14, lse); WS(15, w, wb); STREAM(16, st);
    kvc_status (*f)(const kvc_shape *, const kvc_params *, const void *, const void *, const void *, void *, void *, const int32_t *,
                    const int32_t *, int32_t, const void *, const void *, float, void *, float *, void *, size_t, void *) = g_ragged;
    RETURN_STATUS(f(s, p, q, Kc, Vc, Kt, Vt, ni, tl, (int32_t)cap, kn, vn, (float)sc, out, lse, w, wb, st));
}

/* shape, W1, activation, Kc, H, stream */
static PyObject *hidden(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    ARGS(6);
    SHAPE(0, s); PTR(1, w); INT(2, act); PTR(3, Kc); PTR(4, H); STREAM(5, st);
    kvc_status (*f)(const kvc_shape *, const void *, int32_t, const void *, void *, void *) = g_hidden;
    RETURN_STATUS(f(s, w, (int32_t)act, Kc, H, st));
}

/* shape, q, Kc, Vc, Kt, Vt, text_len, text_cap, k_new, v_new, scale, out, lse, workspace, stream */
static PyObject *static_decode(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    ARGS(15);
    SHAPE(0, s); PTR(1, q); PTR(2, Kc); PTR(3, Vc); PTR(4, Kt); PTR(5, Vt); INT(6, t); INT(7, cap); PTR(8, kn); PTR(9, vn);
    FLT(10, sc); PTR(11, out); PTR(12, lse); WS(13, w, wb); STREAM(14, st);
    kvc_status (*f)(const kvc_shape *, const void *, const void *, const void *, void *, void *, int32_t, int32_t, const void *, const void *,
                    float, void *, float *, void *, size_t, void *) = g_static;
    RETURN_STATUS(f(s, q, Kc, Vc, Kt, Vt, (int32_t)t, (int32_t)cap, kn, vn, (float)sc, out, lse, w, wb, st));
}

/* B, Hq, Hkv, d, dtype, q, K, V, stride_b, stride_h, stride_s, kv_len, kv_cap, k_new, v_new, scale, out, lse, workspace, stream */
static PyObject *full(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    ARGS(20);
    INT(0, B); INT(1, Hq); INT(2, Hkv); INT(3, d); INT(4, dt); PTR(5, q); PTR(6, K); PTR(7, V); INT(8, sb); INT(9, sh); INT(10, ss);
    INT(11, len); INT(12, cap); PTR(13, kn); PTR(14, vn); FLT(15, sc); PTR(16, out); PTR(17, lse); WS(18, w, wb); STREAM(19, st);
    kvc_status (*f)(int32_t, int32_t, int32_t, int32_t, int32_t, const void *, void *, void *, int64_t, int64_t, int64_t, int32_t, int32_t,
                    const void *, const void *, float, void *, float *, void *, size_t, void *) = g_full;
    RETURN_STATUS(f((int32_t)B, (int32_t)Hq, (int32_t)Hkv, (int32_t)d, (int32_t)dt, q, K, V, sb, sh, ss, (int32_t)len, (int32_t)cap, kn, vn,
                    (float)sc, out, lse, w, wb, st));
}

#define ENTRY(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, NULL}
static PyMethodDef methods[] = {ENTRY(bind), ENTRY(compress), ENTRY(decode), ENTRY(decode_static), ENTRY(ragged), ENTRY(hidden),
                                ENTRY(static_decode), ENTRY(full), {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_kvc_call", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__kvc_call(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_numel = PyUnicode_InternFromString("numel");
    s_stride = PyUnicode_InternFromString("stride");
    s_size = PyUnicode_InternFromString("size");
    for (int i = 0; i < 4; ++i) k_int[i] = PyLong_FromLong(i);
    if (!s_data_ptr || !s_numel || !s_stride || !s_size || !k_int[3]) return NULL;
    return PyModule_Create(&module);
}
