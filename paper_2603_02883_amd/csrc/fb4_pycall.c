// The Python binding's calls into libfb4.so without ctypes: the entry points that a program calls per layer and every few
// steps, with the addresses, sizes and strides read from the tensor objects here.  Bound by the interpreter: a call of fb4_quantize on 300 x
// 1152 spent 1.6 us of 5.1 in Python and ctypes, 0.9 so, 0.3 where the tensors' own reader answers (look): 4.35 to 3.75-4.05 a call.
// A refresh of 4 frames of 25 x 55 tokens, four calls: 25.1 us through ctypes, 21.3 so.
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

// What a tensor type lends to C code, by the DLPack C exchange protocol (data layout of its major version 1): a reader of address,
// sizes and strides that makes no Python objects.  us: the three matrices of fb4_quantize by their methods 0.54, so 0.09.
typedef struct {
    void* data;
    struct { int32_t type, id; } device;
    int32_t ndim;
    struct { uint8_t code, bits; uint16_t lanes; } dtype;
    int64_t *shape, *strides;   // the tensor's own
    uint64_t byte_offset;
} dl_tensor;
typedef struct {
    struct { uint32_t major, minor; } version;
    void *previous, *allocator, *from_object, *to_object;
    int (*read)(void* object, dl_tensor* out);
    void* current_stream;
} dl_exchange;
static PyTypeObject* tensor_type;   // of exactly this type are the objects that `read_tensor` takes
static int (*read_tensor)(void*, dl_tensor*);

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

// 1 and the tensor's fields, or 0 for what its type's reader does not take (no storage, say, whose methods will say so).
static int look(PyObject* t, dl_tensor* d)
{
    if (!read_tensor || Py_TYPE(t) != tensor_type) return 0;
    if (read_tensor(t, d) == 0) return 1;
    PyErr_Clear();
    return 0;
}
static void* data_of(const dl_tensor* d) { return d->data ? (char*)d->data + d->byte_offset : NULL; }

// Data pointer of a tensor, null for None.
static int tensor(PyObject* t, void** out)
{
    *out = NULL;
    if (t == Py_None) return 0;
    dl_tensor v;
    if (look(t, &v)) {
        *out = data_of(&v);
        return 0;
    }
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
    dl_tensor v;
    if (look(t, &v) && v.ndim > 0) {
        *out = v.strides[0];
        return 0;
    }
    PyObject* r = PyObject_CallMethodOneArg(t, s_stride, zero);
    if (!r) return -1;
    const int rc = integer(r, out);
    Py_DECREF(r);
    return rc;
}

// Sizes and address of a tensor of n dimensions that its type's reader takes.  (Copied at once, as everywhere here: the reader's
// sizes are the tensor's own, which a later argument's methods, or another thread during the call, may change.)
static int plain(PyObject* t, Py_ssize_t n, int64_t* d, void** out)
{
    dl_tensor v;
    if (!look(t, &v) || v.ndim != n) return -1;
    for (Py_ssize_t i = 0; i < n; ++i) d[i] = v.shape[i];
    *out = data_of(&v);
    return 0;
}

// ... of any tensor of n dimensions.
static int sized(PyObject* t, Py_ssize_t n, int64_t* d, void** out)
{
    if (plain(t, n, d, out) == 0) return 0;
    return shape(t, n, d) || tensor(t, out) ? -1 : 0;
}

// Sizes, row stride and address of a matrix.
static int matrix(PyObject* t, int64_t* d, int64_t* st, void** out)
{
    dl_tensor v;
    if (look(t, &v) && v.ndim == 2) {
        d[0] = v.shape[0];
        d[1] = v.shape[1];
        *st = d[0] > 1 ? v.strides[0] : d[1];
        *out = data_of(&v);
        return 0;
    }
    return shape(t, 2, d) || row_stride(t, d, st) || tensor(t, out) ? -1 : 0;
}

static int numel(PyObject* t, int64_t* out)
{
    dl_tensor v;
    if (look(t, &v)) {
        *out = 1;
        for (int32_t i = 0; i < v.ndim; ++i) *out *= v.shape[i];
        return 0;
    }
    PyObject* r = PyObject_CallMethodNoArgs(t, s_numel);
    if (!r) return -1;
    const int rc = integer(r, out);
    Py_DECREF(r);
    return rc;
}

// Number of groups of a [groups][8] tensor.
static int groups_of(PyObject* t, int64_t* out)
{
    dl_tensor v;
    if (look(t, &v) && v.ndim > 0) {
        *out = v.shape[0];
        return 0;
    }
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
enum { k_quantize, k_quantize_seda, k_quantize_decompose, k_dequantize, k_repack_mxfp8, k_layernorm_quantize, k_gelu_quantize, k_attention_scores,
       k_select_salient_tokens, k_seda_assign, k_seda_main_anchor, k_seda_profile, kCalls };
static const char* const call_names[kCalls] = {"quantize", "quantize_seda", "quantize_decompose", "dequantize", "repack_mxfp8",
                                               "layernorm_quantize", "gelu_quantize", "attention_scores",
                                               "select_salient_tokens", "seda_assign", "seda_main_anchor", "seda_profile"};
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
    if (n != 6 || address(a[0], &h) || options(a[1], &o) || matrix(a[2], d, &st, &x) ||
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
    if (n != 8 || address(a[0], &h) || options(a[1], &o) || matrix(a[2], d, &st, &x) ||
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
    if (n != 11 || address(a[0], &h) || options(a[1], &o) || matrix(a[2], d, &st, &x) ||
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
    if (n != 10 || address(a[0], &h) || sized(a[1], 2, d, &c1) || tensor(a[2], &m1) || integer(a[3], &block) ||
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
    if (n != 7 || address(a[0], &h) || sized(a[1], 2, d, &c) || tensor(a[2], &m) || integer(a[3], &block) ||
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
    if (n != 12 || !PyFloat_Check(a[5]) || address(a[0], &h) || options(a[1], &o) || matrix(a[2], d, &st, &x) ||
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
    if (n != 9 || address(a[0], &h) || options(a[1], &o) || matrix(a[2], d, &st, &x) ||
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
    if (n != 5 || sized(a[0], 3, d, &q) || tensor(a[1], &k) || integer(a[2], &mode) || tensor(a[3], &out) || address(a[4], &s))
        return elsewhere(k_attention_scores, a, n);
    RETURN_CALL(fb4_attention_scores(q, k, d[0], d[1], d[2], (int)mode, out, s));
}

// The refresh of the attention-guided choices, from tensors that their type's reader takes (the others: by ctypes).

// (scores, grid_h, grid_w, tile_h, tile_w, rows_out, stream)
static PyObject* py_select_salient_tokens(ARGS)
{
    void *sc, *out, *s;
    int64_t d[3], gh, gw, th, tw;
    if (n != 7 || plain(a[0], 3, d, &sc) || integer(a[1], &gh) || integer(a[2], &gw) || integer(a[3], &th) || integer(a[4], &tw) ||
        tensor(a[5], &out) || address(a[6], &s) || d[2] != gh * gw || th == 0 || tw == 0)
        return elsewhere(k_select_salient_tokens, a, n);
    RETURN_CALL(fb4_select_salient_tokens(sc, d[0], (int)d[1], (int)gh, (int)gw, (int)th, (int)tw, out, s));
}

// (q, k, joint, frames, grid_h, grid_w, anchors, tile_h, tile_w, window, window_t, threshold, token_group, anchor_group, scores, stream)
static PyObject* py_seda_assign(ARGS)
{
    void *q, *k, *anchors, *tg, *ag, *sc, *s;
    int64_t d[4], frames, gh, gw, th, tw, w, wt, n_anchors;
    if (n != 16 || !PyBool_Check(a[2]) || !PyFloat_Check(a[11]) || plain(a[0], a[2] == Py_True ? 3 : 4, d, &q) || tensor(a[1], &k) ||
        integer(a[3], &frames) || integer(a[4], &gh) || integer(a[5], &gw) || tensor(a[6], &anchors) || numel(a[6], &n_anchors) || integer(a[7], &th) ||
        integer(a[8], &tw) || integer(a[9], &w) || integer(a[10], &wt) || tensor(a[12], &tg) || tensor(a[13], &ag) || tensor(a[14], &sc) ||
        address(a[15], &s))
        return elsewhere(k_seda_assign, a, n);
    const int joint = a[2] == Py_True;
    const float threshold = (float)PyFloat_AS_DOUBLE(a[11]);
    RETURN_CALL(fb4_seda_assign(q, k, joint, frames, (int)d[joint ? 0 : 1], (int)gh, (int)gw, d[joint ? 2 : 3], anchors, n_anchors, (int)th, (int)tw,
                                (int)w, (int)wt, threshold, tg, ag, sc, s));
}

// (temporal_scores, qt, kt, candidates, grid_h, grid_w, tile_h, tile_w, prune_threshold, main_anchor, kept, prune_scores, stream)
static PyObject* py_seda_main_anchor(ARGS)
{
    void *ts, *q, *k, *c, *main, *kept, *ps, *s;
    int64_t d[4], dc[2], gh, gw, th, tw;
    if (n != 13 || !PyFloat_Check(a[8]) || tensor(a[0], &ts) || plain(a[1], 4, d, &q) || tensor(a[2], &k) || plain(a[3], 2, dc, &c) ||
        integer(a[4], &gh) || integer(a[5], &gw) || integer(a[6], &th) || integer(a[7], &tw) || tensor(a[9], &main) || tensor(a[10], &kept) ||
        tensor(a[11], &ps) || address(a[12], &s) || d[0] != gh * gw || dc[0] != d[2] || th == 0 || tw == 0)
        return elsewhere(k_seda_main_anchor, a, n);
    const float threshold = (float)PyFloat_AS_DOUBLE(a[8]);
    RETURN_CALL(fb4_seda_main_anchor(ts, q, k, d[2], (int)d[1], (int)gh, (int)gw, d[3], c, (int)dc[1], (int)th, (int)tw, threshold, main, kept, ps, s));
}

// (luts, meta, anchor_group, n_groups, counts, sub_formatbooks, stream)
static PyObject* py_seda_profile(ARGS)
{
    void *h, *m, *ag, *counts, *sub, *s;
    int64_t d[2], g;
    if (n != 7 || address(a[0], &h) || plain(a[1], 2, d, &m) || tensor(a[2], &ag) || integer(a[3], &g) || tensor(a[4], &counts) ||
        tensor(a[5], &sub) || address(a[6], &s))
        return elsewhere(k_seda_profile, a, n);
    RETURN_CALL(fb4_seda_profile(h, m, d[0], d[1], ag, (int)g, counts, sub, s));
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

// (tensor type, its exchange capsule): True if tensors of exactly this type are read through it from now on
static PyObject* py_read_through(ARGS)
{
    const dl_exchange* lent = NULL;
    if (n == 2 && PyType_Check(a[0]) && PyCapsule_IsValid(a[1], "dlpack_exchange_api"))
        lent = (const dl_exchange*)PyCapsule_GetPointer(a[1], "dlpack_exchange_api");
    read_tensor = lent && lent->version.major == 1 ? lent->read : NULL;   // (a type need not have one)
    if (read_tensor) {
        Py_INCREF(a[0]);
        Py_XSETREF(tensor_type, (PyTypeObject*)a[0]);
    }
    return PyBool_FromLong(read_tensor != NULL);
}

#define METHOD(name) {#name, (PyCFunction)(void (*)(void))py_##name, METH_FASTCALL, NULL}
static PyMethodDef methods[] = {METHOD(quantize), METHOD(quantize_seda), METHOD(quantize_decompose), METHOD(dequantize), METHOD(repack_mxfp8),
                                METHOD(layernorm_quantize), METHOD(gelu_quantize), METHOD(attention_scores), METHOD(select_salient_tokens),
                                METHOD(seda_assign), METHOD(seda_main_anchor), METHOD(seda_profile), METHOD(bind),
                                METHOD(read_through), {NULL, NULL, 0, NULL}};
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
