// The Python binding's calls into libfb4.so without ctypes: the entry points that a program calls per layer, with the
// addresses, sizes and strides read from the tensor objects here.  Bound by the interpreter: a call of fb4_quantize on 300 x
// 1152 spent 1.6 us of 5.1 in Python and ctypes; 4.1 so, what the launches take one behind the other.
// Only the ordinary argument types are read here.  Whatever else comes -- other types, other shapes, an error on the way -- goes
// to the same call through ctypes, which converts or refuses it by ctypes' own rules: which arguments are taken and what is
// raised for the others is decided in one place.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>
#include <string.h>

#include "../../include/fb4.h"

static PyObject *s_data_ptr, *s_shape, *s_stride, *s_numel, *zero;
static PyTypeObject *options_type, *handle_type;   // fb4_opts and ctypes.c_void_p (bind)

// The readers return 0, or -1 for what they do not read.

static int bytes_of(PyObject* o, PyTypeObject* type, void* out, Py_ssize_t size)
{
    Py_buffer b;
    if (!type || !PyObject_TypeCheck(o, type) || PyObject_GetBuffer(o, &b, PyBUF_SIMPLE)) return -1;
    const int ok = b.len >= size;   // (a subclass may have more fields)
    if (ok) memcpy(out, b.buf, (size_t)size);
    PyBuffer_Release(&b);
    return ok ? 0 : -1;
}

// Address held by None (null), an integer, or a c_void_p.
static int address(PyObject* o, void** out)
{
    *out = NULL;
    if (o == Py_None) return 0;
    if (!PyLong_Check(o)) return bytes_of(o, handle_type, out, (Py_ssize_t)sizeof *out);
    *out = (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(o);
    return 0;
}

static int options(PyObject* o, fb4_opts* out) { return bytes_of(o, options_type, out, (Py_ssize_t)sizeof *out); }

static int integer(PyObject* o, int64_t* out)
{
    if (!PyLong_Check(o)) return -1;
    *out = (int64_t)PyLong_AsUnsignedLongLongMask(o);
    return 0;
}

// Data pointer of a tensor, null for None.
static int tensor(PyObject* t, void** out)
{
    *out = NULL;
    if (t == Py_None) return 0;
    PyObject* r = PyObject_CallMethodNoArgs(t, s_data_ptr);
    if (!r) return -1;
    const int rc = PyLong_Check(r) ? address(r, out) : -1;
    Py_DECREF(r);
    return rc;
}

static int shape(PyObject* t, Py_ssize_t n, int64_t* d)
{
    PyObject* s = PyObject_GetAttr(t, s_shape);
    if (!s) return -1;
    int rc = PyTuple_Check(s) && PyTuple_GET_SIZE(s) == n ? 0 : -1;
    for (Py_ssize_t i = 0; i < n && rc == 0; ++i) rc = integer(PyTuple_GET_ITEM(s, i), d + i);
    Py_DECREF(s);
    return rc;
}

// Row stride in elements of a matrix with d = its sizes (a single row's own stride says nothing).
static int row_stride(PyObject* t, const int64_t* d, int64_t* out)
{
    *out = d[1];
    if (d[0] <= 1) return 0;
    PyObject* r = PyObject_CallMethodOneArg(t, s_stride, zero);
    if (!r) return -1;
    const int rc = integer(r, out);
    Py_DECREF(r);
    return rc;
}

static int numel(PyObject* t, int64_t* out)
{
    PyObject* r = PyObject_CallMethodNoArgs(t, s_numel);
    if (!r) return -1;
    const int rc = integer(r, out);
    Py_DECREF(r);
    return rc;
}

// Number of groups of a [groups][8] tensor.
static int groups_of(PyObject* t, int64_t* out)
{
    PyObject* s = PyObject_GetAttr(t, s_shape);
    if (!s) return -1;
    PyObject* r = PySequence_GetItem(s, 0);
    Py_DECREF(s);
    if (!r) return -1;
    const int rc = integer(r, out);
    Py_DECREF(r);
    return rc;
}

// The same for arguments that may be None: 0.
static int count_or_none(PyObject* t, int (*count)(PyObject*, int64_t*), int64_t* out)
{
    *out = 0;
    return t == Py_None ? 0 : count(t, out);
}

// The same calls through ctypes (bind).
enum { k_quantize, k_quantize_seda, k_quantize_decompose, k_dequantize, k_repack_mxfp8, k_layernorm_quantize, k_gelu_quantize, k_attention_scores, kCalls };
static const char* const call_names[kCalls] = {"quantize", "quantize_seda", "quantize_decompose", "dequantize", "repack_mxfp8",
                                               "layernorm_quantize", "gelu_quantize", "attention_scores"};
static PyObject* through_ctypes[kCalls];

static PyObject* elsewhere(int call, PyObject* const* a, Py_ssize_t n)
{
    PyErr_Clear();   // (what cannot be read is raised there)
    if (!through_ctypes[call]) {
        PyErr_SetString(PyExc_RuntimeError, "bind has not been called");
        return NULL;
    }
    return PyObject_Vectorcall(through_ctypes[call], a, (size_t)n, NULL);
}

#define ARGS PyObject *self, PyObject *const *a, Py_ssize_t n
// the library call with other Python threads running, as ctypes does it
#define RETURN_CALL(call)        \
    int rc;                      \
    Py_BEGIN_ALLOW_THREADS       \
    rc = call;                   \
    Py_END_ALLOW_THREADS         \
    return PyLong_FromLong(rc)

// (luts, opts, x, codes, meta, stream)
static PyObject* py_quantize(ARGS)
{
    void *h, *x, *c, *m, *s;
    fb4_opts o;
    int64_t d[2], st;
    if (n != 6 || address(a[0], &h) || options(a[1], &o) || shape(a[2], 2, d) || row_stride(a[2], d, &st) || tensor(a[2], &x) ||
        tensor(a[3], &c) || tensor(a[4], &m) || address(a[5], &s))
        return elsewhere(k_quantize, a, n);
    RETURN_CALL(fb4_quantize(h, &o, x, d[0], d[1], st, c, m, s));
}

// (luts, opts, x, token_group, sub_formatbooks, codes, meta, stream)
static PyObject* py_quantize_seda(ARGS)
{
    void *h, *x, *tg, *sub, *c, *m, *s;
    fb4_opts o;
    int64_t d[2], st, g;
    if (n != 8 || address(a[0], &h) || options(a[1], &o) || shape(a[2], 2, d) || row_stride(a[2], d, &st) || tensor(a[2], &x) ||
        tensor(a[3], &tg) || tensor(a[4], &sub) || groups_of(a[4], &g) || tensor(a[5], &c) || tensor(a[6], &m) || address(a[7], &s))
        return elsewhere(k_quantize_seda, a, n);
    RETURN_CALL(fb4_quantize_seda(h, &o, x, d[0], d[1], st, tg, sub, (int)g, c, m, s));
}

// (luts, opts, x, salient_rows, token_group, sub_formatbooks, codes1, meta1, codes2, meta2, stream)
static PyObject* py_quantize_decompose(ARGS)
{
    void *h, *x, *sal, *tg, *sub, *c1, *m1, *c2, *m2, *s;
    fb4_opts o;
    int64_t d[2], st, g, n_sal;
    if (n != 11 || address(a[0], &h) || options(a[1], &o) || shape(a[2], 2, d) || row_stride(a[2], d, &st) || tensor(a[2], &x) ||
        tensor(a[3], &sal) || numel(a[3], &n_sal) || tensor(a[4], &tg) || tensor(a[5], &sub) || count_or_none(a[5], groups_of, &g) || tensor(a[6], &c1) ||
        tensor(a[7], &m1) || tensor(a[8], &c2) || tensor(a[9], &m2) || address(a[10], &s))
        return elsewhere(k_quantize_decompose, a, n);
    RETURN_CALL(fb4_quantize_decompose(h, &o, x, d[0], d[1], st, tg, sub, (int)g, sal, n_sal, c1, m1, c2, m2, s));
}

// (luts, codes1, meta1, block, codes2, meta2, salient_rows, out, out_dtype, stream)
static PyObject* py_dequantize(ARGS)
{
    void *h, *c1, *m1, *c2, *m2, *sal, *out, *s;
    int64_t d[2], block, n_sal, dtype, st;
    if (n != 10 || address(a[0], &h) || shape(a[1], 2, d) || tensor(a[1], &c1) || tensor(a[2], &m1) || integer(a[3], &block) ||
        tensor(a[4], &c2) || tensor(a[5], &m2) || tensor(a[6], &sal) || count_or_none(a[6], numel, &n_sal) || tensor(a[7], &out) || integer(a[8], &dtype) ||
        address(a[9], &s))
        return elsewhere(k_dequantize, a, n);
    d[1] *= 2;
    if (row_stride(a[7], d, &st)) return elsewhere(k_dequantize, a, n);
    RETURN_CALL(fb4_dequantize(h, c1, m1, d[0], d[1], (int)block, c2, m2, sal, n_sal, out, (int)dtype, st, s));
}

// (luts, codes, meta, block, elems, scales, stream)
static PyObject* py_repack_mxfp8(ARGS)
{
    void *h, *c, *m, *e, *sc, *s;
    int64_t d[2], block, st;
    if (n != 7 || address(a[0], &h) || shape(a[1], 2, d) || tensor(a[1], &c) || tensor(a[2], &m) || integer(a[3], &block) ||
        tensor(a[4], &e) || tensor(a[5], &sc) || address(a[6], &s))
        return elsewhere(k_repack_mxfp8, a, n);
    d[1] *= 2;
    if (row_stride(a[4], d, &st)) return elsewhere(k_repack_mxfp8, a, n);
    RETURN_CALL(fb4_repack_mxfp8(h, c, m, d[0], d[1], (int)block, e, st, sc, s));
}

// (luts, opts, x, gamma, beta, eps, token_group, sub_formatbooks, codes, meta, y_out, stream)
static PyObject* py_layernorm_quantize(ARGS)
{
    void *h, *x, *ga, *be, *tg, *sub, *c, *m, *y, *s;
    fb4_opts o;
    int64_t d[2], st, g;
    if (n != 12 || !PyFloat_Check(a[5]) || address(a[0], &h) || options(a[1], &o) || shape(a[2], 2, d) || row_stride(a[2], d, &st) || tensor(a[2], &x) ||
        tensor(a[3], &ga) || tensor(a[4], &be) || tensor(a[6], &tg) || tensor(a[7], &sub) || count_or_none(a[7], groups_of, &g) || tensor(a[8], &c) ||
        tensor(a[9], &m) || tensor(a[10], &y) || address(a[11], &s))
        return elsewhere(k_layernorm_quantize, a, n);
    const double eps = PyFloat_Check(a[5]) ? PyFloat_AS_DOUBLE(a[5]) : 0.0;
    RETURN_CALL(fb4_layernorm_quantize(h, &o, x, d[0], d[1], st, ga, be, (float)eps, tg, sub, (int)g, c, m, y, s));
}

// (luts, opts, x, approximate, token_group, sub_formatbooks, codes, meta, stream)
static PyObject* py_gelu_quantize(ARGS)
{
    void *h, *x, *tg, *sub, *c, *m, *s;
    fb4_opts o;
    int64_t d[2], st, g, approximate;
    if (n != 9 || address(a[0], &h) || options(a[1], &o) || shape(a[2], 2, d) || row_stride(a[2], d, &st) || tensor(a[2], &x) ||
        integer(a[3], &approximate) || tensor(a[4], &tg) || tensor(a[5], &sub) || count_or_none(a[5], groups_of, &g) || tensor(a[6], &c) || tensor(a[7], &m) ||
        address(a[8], &s))
        return elsewhere(k_gelu_quantize, a, n);
    RETURN_CALL(fb4_gelu_quantize(h, &o, x, d[0], d[1], st, (int)approximate, tg, sub, (int)g, c, m, s));
}

// (q, k, mode, scores, stream)
static PyObject* py_attention_scores(ARGS)
{
    void *q, *k, *out, *s;
    int64_t d[3], mode;
    if (n != 5 || shape(a[0], 3, d) || tensor(a[0], &q) || tensor(a[1], &k) || integer(a[2], &mode) || tensor(a[3], &out) || address(a[4], &s))
        return elsewhere(k_attention_scores, a, n);
    RETURN_CALL(fb4_attention_scores(q, k, d[0], d[1], d[2], (int)mode, out, s));
}

// (fb4_opts, c_void_p, object with the same calls through ctypes)
static PyObject* py_bind(ARGS)
{
    if (n != 3 || !PyType_Check(a[0]) || !PyType_Check(a[1])) {
        PyErr_SetString(PyExc_TypeError, "bind(options type, handle type, calls through ctypes)");
        return NULL;
    }
    PyObject* found[kCalls];
    for (int i = 0; i < kCalls; ++i) {
        found[i] = PyObject_GetAttrString(a[2], call_names[i]);
        if (!found[i]) {
            while (i > 0) Py_DECREF(found[--i]);
            return NULL;
        }
    }
    for (int i = 0; i < kCalls; ++i) Py_XSETREF(through_ctypes[i], found[i]);
    Py_INCREF(a[0]);
    Py_XSETREF(options_type, (PyTypeObject*)a[0]);
    Py_INCREF(a[1]);
    Py_XSETREF(handle_type, (PyTypeObject*)a[1]);
    Py_RETURN_NONE;
}

#define METHOD(name) {#name, (PyCFunction)(void (*)(void))py_##name, METH_FASTCALL, NULL}
static PyMethodDef methods[] = {METHOD(quantize), METHOD(quantize_seda), METHOD(quantize_decompose), METHOD(dequantize), METHOD(repack_mxfp8),
                                METHOD(layernorm_quantize), METHOD(gelu_quantize), METHOD(attention_scores), METHOD(bind), {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fb4call", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__fb4call(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_shape = PyUnicode_InternFromString("shape");
    s_stride = PyUnicode_InternFromString("stride");
    s_numel = PyUnicode_InternFromString("numel");
    zero = PyLong_FromLong(0);
    if (!s_data_ptr || !s_shape || !s_stride || !s_numel || !zero) return NULL;
    return PyModule_Create(&module);
}
