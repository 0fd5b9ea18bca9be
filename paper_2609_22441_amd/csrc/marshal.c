/*
 * Argument marshalling of the hot entry points in native code: the checks of binding.py on plain
 * torch tensors, then the C call. Each function returns the call's status, or None when an
 * argument is anything but the plain case (another type, dtype, device or layout, too short, a
 * subclass, a raw pointer): nothing was called then, and binding.py's own checks either raise or
 * make the call. Python's attribute protocol is used throughout, so the module depends on no
 * torch header or ABI. An AttributeError, a TypeError or an OverflowError on the way means "not
 * plain"; any other exception (a KeyboardInterrupt, a MemoryError) is the caller's and is raised.
 *
 * A cc_join through binding.py's checks costs the host about 8 us, more than the kernel of a
 * request of 10,000 candidates takes (5.6 us): such requests in a row took 9.1 us each, through
 * this module 6.2.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

typedef struct cc_store cc_store;
typedef int (*info_fn)(const cc_store *, int64_t *, int32_t *);
typedef int (*join_fn)(const cc_store *, const int64_t *, int64_t, const int64_t *, int64_t,
                       const void *, int32_t, const void *, void *, int64_t, int8_t *, void *);
typedef int (*batched_fn)(const cc_store *, int32_t, const int64_t *, const int64_t *, int64_t,
                          const int64_t *, const int64_t *, int64_t, const void *, int32_t,
                          const void *, int32_t, const int64_t *const *, void *, int64_t, int8_t *,
                          void *);
typedef int (*authors_fn)(const cc_store *, int32_t, const int64_t *, const int64_t *,
                          const int64_t *, int64_t, const int64_t *, const int64_t *, int64_t,
                          const void *, int32_t, const void *, int32_t, const int64_t *const *,
                          void *, int64_t, int8_t *, void *);
typedef int (*padded_fn)(const cc_store *, int32_t, const int64_t *, const int64_t *, int64_t,
                         const int64_t *, const int64_t *, int64_t, const void *, int32_t,
                         const void *, int32_t, const int64_t *const *, int64_t, void *, int64_t,
                         int8_t *, int8_t *, void *);
typedef int (*resolve_fn)(const cc_store *, const int64_t *, int64_t, int64_t *, void *);
typedef int (*upsert_fn)(cc_store *, int64_t, const int64_t *, const int64_t *, const void *, void *,
                         int64_t, int64_t *, int64_t *, void *);
typedef int (*sort_fn)(int32_t, int32_t, int32_t, const int64_t *, const int64_t *, const void *,
                       int32_t, int64_t, int64_t, int64_t *, void *, void *, int64_t, void *);

static PyObject *t_type, *t_i64, *t_i8;       /* torch.Tensor, torch.int64, torch.int8 */
static PyObject *current_stream;              /* () -> handle of torch's current stream */
static PyObject *n_dtype, *n_is_cuda, *n_numel, *n_contiguous, *n_data_ptr, *n_shape, *n_stride,
    *n_element_size, *n_cuda_stream;

/* What a check that failed returns: 0, with no exception set if what came up (if anything) means
 * that an argument is not plain. */
static int not_plain(void) {
    if (PyErr_ExceptionMatches(PyExc_AttributeError) || PyErr_ExceptionMatches(PyExc_TypeError) ||
        PyErr_ExceptionMatches(PyExc_OverflowError))
        PyErr_Clear();
    return 0;
}

/* What a function returns after a check that failed. */
static PyObject *no_call(void) {
    if (PyErr_Occurred())
        return NULL;
    Py_RETURN_NONE;
}

/* Arguments of the plain case read as numbers; -1 when x is not that. */
static int64_t call_int(PyObject *x, PyObject *name) {
    PyObject *r = PyObject_CallMethodNoArgs(x, name);
    const int64_t v = r && PyLong_Check(r) ? PyLong_AsLongLong(r) : -1;
    Py_XDECREF(r);
    if (v == -1 && PyErr_Occurred())
        not_plain();
    return v;
}

static int is_true(PyObject *r) {             /* steals r */
    if (!r)
        return not_plain();
    const int t = r == Py_True;
    Py_DECREF(r);
    return t;
}

/* A plain tensor in GPU memory, of `dtype` unless it is NULL. */
static int plain(PyObject *x, PyObject *dtype) {
    if ((PyObject *)Py_TYPE(x) != t_type || !is_true(PyObject_GetAttr(x, n_is_cuda)))
        return 0;
    if (!dtype)
        return 1;
    PyObject *d = PyObject_GetAttr(x, n_dtype);
    if (!d)
        return not_plain();
    const int same = d == dtype;
    Py_DECREF(d);
    return same;
}

static int pointer(PyObject *x, void **p) {
    PyObject *r = PyObject_CallMethodNoArgs(x, n_data_ptr);
    if (!r)
        return not_plain();
    *p = PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    return PyErr_Occurred() ? not_plain() : 1;
}

/* Dense array of at least `need` elements; *numel gets the element count. */
static int array_of(PyObject *x, PyObject *dtype, int64_t need, void **p, int64_t *numel) {
    if (!plain(x, dtype) || !is_true(PyObject_CallMethodNoArgs(x, n_contiguous)))
        return 0;
    const int64_t n = call_int(x, n_numel);
    if (n < 0 || n < need)
        return 0;
    if (numel)
        *numel = n;
    return pointer(x, p);
}

/* Sizes a tuple of two integers holds. */
static int pair_of(PyObject *t, int64_t *a, int64_t *b) {     /* steals t */
    if (!t)
        return not_plain();
    const int pair = PyTuple_Check(t) && PyTuple_GET_SIZE(t) == 2;
    if (pair) {
        *a = PyLong_AsLongLong(PyTuple_GET_ITEM(t, 0));
        if (!PyErr_Occurred())
            *b = PyLong_AsLongLong(PyTuple_GET_ITEM(t, 1));
    }
    Py_DECREF(t);
    return PyErr_Occurred() ? not_plain() : pair;
}

/* Dense [>= n, columns] array of rows; *row_bytes gets the bytes per row. */
static int rows_of(PyObject *x, int64_t n, void **p, int64_t *row_bytes) {
    int64_t r, c, e;
    if (!plain(x, NULL) || !pair_of(PyObject_GetAttr(x, n_shape), &r, &c) || r < n ||
        !is_true(PyObject_CallMethodNoArgs(x, n_contiguous)) ||
        (e = call_int(x, n_element_size)) <= 0)
        return 0;
    *row_bytes = c * e;
    return *row_bytes > 0 && *row_bytes <= INT32_MAX && pointer(x, p);
}

/* Output rows [>= n, >= width bytes] with dense rows and any row stride. */
static int out_of(PyObject *x, int64_t n, int64_t width, void **p, int64_t *stride) {
    int64_t r, c, sr, sc, e;
    if (!plain(x, NULL) || !pair_of(PyObject_GetAttr(x, n_shape), &r, &c) || r < n ||
        !pair_of(PyObject_CallMethodNoArgs(x, n_stride), &sr, &sc) || sc != 1 ||
        (e = call_int(x, n_element_size)) <= 0 || c * e < width)
        return 0;
    *stride = sr * e;
    return pointer(x, p);
}

/* NULL for None, else a dense buffer of at least `bytes` bytes. */
static int bytes_of(PyObject *x, int64_t bytes, void **p, int64_t *size) {
    int64_t n, e;
    if (x == Py_None) {
        *p = NULL;
        return size == NULL;
    }
    if (!array_of(x, NULL, 0, p, &n) || (e = call_int(x, n_element_size)) <= 0 || n * e < bytes)
        return 0;
    if (size)
        *size = n * e;
    return 1;
}

static int number(PyObject *x, int64_t *v) {  /* a plain int */
    if (!PyLong_CheckExact(x))
        return 0;
    *v = PyLong_AsLongLong(x);
    return PyErr_Occurred() ? not_plain() : 1;
}

static int address(PyObject *x, void **p) {   /* a store handle or a function: an int */
    if (!PyLong_CheckExact(x))
        return 0;
    *p = PyLong_AsVoidPtr(x);
    return PyErr_Occurred() ? not_plain() : 1;
}

/* The stream argument: None (torch's current one), a handle or a stream object. */
static int stream_of(PyObject *x, void **p) {
    if (PyLong_CheckExact(x))
        return address(x, p);
    PyObject *r = x == Py_None ? PyObject_CallNoArgs(current_stream)
                               : PyObject_GetAttr(x, n_cuda_stream);
    if (!r)
        return not_plain();
    const int ok = address(r, p);
    Py_DECREF(r);
    return ok;
}

/* Reads the store, which the library itself only compares against 0: asked when every argument has
 * passed that needs no row width, so a call that is refused for one of them reads no handle. */
static int doc_row_bytes(PyObject *info, const cc_store *s, int64_t *bytes) {
    void *f;
    int32_t w = 0;
    if (!s || !address(info, &f) || ((info_fn)f)(s, NULL, &w) != 0)
        return 0;
    *bytes = w;
    return 1;
}

#define CALL(...)                  \
    int st;                        \
    Py_BEGIN_ALLOW_THREADS         \
    st = __VA_ARGS__;              \
    Py_END_ALLOW_THREADS           \
    return PyLong_FromLong(st)

/* join(cc_join, cc_store_info, store, cand_idx, keys, feats, out, hit, default_row, stream) */
static PyObject *m_join(PyObject *self, PyObject *const *a, Py_ssize_t n_args) {
    (void)self;
    void *fn, *store, *cand, *keys, *feats, *out, *hit, *def, *stream;
    int64_t n, k, ew, stride, dw;
    if (n_args != 10 || !address(a[0], &fn) || !address(a[2], &store) ||
        !array_of(a[3], t_i64, 0, &cand, &n) || !array_of(a[4], t_i64, 0, &keys, &k) ||
        !rows_of(a[5], k, &feats, &ew) || !array_of(a[7], t_i8, n, &hit, NULL) ||
        !bytes_of(a[8], ew, &def, NULL) || !stream_of(a[9], &stream) ||
        !doc_row_bytes(a[1], store, &dw) || !out_of(a[6], n, dw + ew, &out, &stride))
        return no_call();
    CALL(((join_fn)fn)(store, cand, n, keys, k, feats, (int32_t)ew, def, out, stride, hit, stream));
}

/* Inputs that the batched forms share. */
typedef struct {
    void *store, *co, *cand, *ko, *keys, *feats, *def, *extra[1], *stream;
    int64_t B, tc, tk, ew, L;
} Batch;

/* a: store, cand_offsets, cand_idx, key_offsets, keys, feats, default_row, extra, stream
 * (extra: None, or the second lookup's keys). */
static int batch_of(PyObject *const *a, Batch *b) {
    int64_t nb;
    if (!address(a[0], &b->store) || !array_of(a[1], t_i64, 1, &b->co, &nb) || nb - 1 > INT32_MAX ||
        !array_of(a[2], t_i64, 0, &b->cand, &b->tc) || !array_of(a[3], t_i64, nb, &b->ko, NULL) ||
        !array_of(a[4], t_i64, 0, &b->keys, &b->tk) || !rows_of(a[5], b->tk, &b->feats, &b->ew) ||
        !bytes_of(a[6], b->ew, &b->def, NULL) || !stream_of(a[8], &b->stream))
        return 0;
    b->B = nb - 1;
    b->L = a[7] == Py_None ? 1 : 2;
    return b->L == 1 || array_of(a[7], t_i64, b->tc, &b->extra[0], NULL);
}

/* batched(cc_join_batched, cc_join_batched_authors, cc_store_info, <batch>, out, hit, author_ids) */
static PyObject *m_batched(PyObject *self, PyObject *const *a, Py_ssize_t n_args) {
    (void)self;
    Batch b;
    void *fn, *fn_authors, *out, *hit, *authors = NULL;
    int64_t stride, dw;
    if (n_args != 15 || !address(a[0], &fn) || !address(a[1], &fn_authors) || !batch_of(a + 3, &b) ||
        !array_of(a[13], t_i8, b.tc * b.L, &hit, NULL) ||
        (a[14] != Py_None && !array_of(a[14], t_i64, b.tc, &authors, NULL)) ||
        !doc_row_bytes(a[2], b.store, &dw) || !out_of(a[12], b.tc, dw + b.L * b.ew, &out, &stride))
        return no_call();
    const int64_t *const *ex = b.L == 2 ? (const int64_t *const *)b.extra : NULL;
    if (a[14] != Py_None) {
        CALL(((authors_fn)fn_authors)(b.store, (int32_t)b.B, b.co, b.cand, authors, b.tc, b.ko,
                                      b.keys, b.tk, b.feats, (int32_t)b.ew, b.def, (int32_t)b.L, ex,
                                      out, stride, hit, b.stream));
    }
    CALL(((batched_fn)fn)(b.store, (int32_t)b.B, b.co, b.cand, b.tc, b.ko, b.keys, b.tk, b.feats,
                          (int32_t)b.ew, b.def, (int32_t)b.L, ex, out, stride, hit, b.stream));
}

/* padded(cc_join_batched_padded, cc_store_info, <batch>, n_max, out, hit, valid) */
static PyObject *m_padded(PyObject *self, PyObject *const *a, Py_ssize_t n_args) {
    (void)self;
    Batch b;
    void *fn, *out, *hit, *valid;
    int64_t n_max, stride, dw;
    if (n_args != 15 || !address(a[0], &fn) || !batch_of(a + 2, &b) || !number(a[11], &n_max) ||
        n_max < 1 || n_max > INT32_MAX || !array_of(a[13], t_i8, b.B * n_max * b.L, &hit, NULL) ||
        !array_of(a[14], t_i8, b.B * n_max, &valid, NULL) || !doc_row_bytes(a[1], b.store, &dw) ||
        !out_of(a[12], b.B * n_max, dw + b.L * b.ew, &out, &stride))
        return no_call();
    const int64_t *const *ex = b.L == 2 ? (const int64_t *const *)b.extra : NULL;
    CALL(((padded_fn)fn)(b.store, (int32_t)b.B, b.co, b.cand, b.tc, b.ko, b.keys, b.tk, b.feats,
                         (int32_t)b.ew, b.def, (int32_t)b.L, ex, n_max, out, stride, hit, valid,
                         b.stream));
}

/* resolve(cc_resolve_ids, store, doc_ids, positions, stream) */
static PyObject *m_resolve(PyObject *self, PyObject *const *a, Py_ssize_t n_args) {
    (void)self;
    void *fn, *store, *ids, *pos, *stream;
    int64_t n;
    if (n_args != 5 || !address(a[0], &fn) || !address(a[1], &store) ||
        !array_of(a[2], t_i64, 0, &ids, &n) || !array_of(a[3], t_i64, n, &pos, NULL) ||
        !stream_of(a[4], &stream))
        return no_call();
    CALL(((resolve_fn)fn)(store, ids, n, pos, stream));
}

/* upsert(cc_store_upsert, cc_store_info, store, doc_ids, author_ids, doc_rows, workspace, stream):
 * (status, new ids, rejected records) */
static PyObject *m_upsert(PyObject *self, PyObject *const *a, Py_ssize_t n_args) {
    (void)self;
    void *fn, *store, *ids, *authors, *rows, *ws, *stream;
    int64_t n, dw, rb, ws_bytes, n_new = 0, n_rejected = 0;
    if (n_args != 8 || !address(a[0], &fn) || !address(a[2], &store) ||
        !array_of(a[3], t_i64, 0, &ids, &n) || !array_of(a[4], t_i64, n, &authors, NULL) ||
        !rows_of(a[5], n, &rows, &rb) || a[6] == Py_None || !bytes_of(a[6], 0, &ws, &ws_bytes) ||
        !stream_of(a[7], &stream) || !doc_row_bytes(a[1], store, &dw) || rb != dw)
        return no_call();
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = ((upsert_fn)fn)(store, n, ids, authors, rows, ws, ws_bytes, &n_new, &n_rejected, stream);
    Py_END_ALLOW_THREADS
    return Py_BuildValue("iLL", st, (long long)n_new, (long long)n_rejected);
}

/* sort(cc_sort_affinity_method, method, key_bits, key_offsets, keys_in, rows_in, keys_out, rows_out,
 * workspace, max_keys, stream) */
static PyObject *m_sort(PyObject *self, PyObject *const *a, Py_ssize_t n_args) {
    (void)self;
    void *fn, *ko, *ki, *ri, *k, *r, *ws, *stream;
    int64_t method, bits, nb, tk, rb, rb_out, ws_bytes, max_keys;
    if (n_args != 11 || !address(a[0], &fn) || !number(a[1], &method) || !number(a[2], &bits) ||
        method != (int32_t)method || bits != (int32_t)bits ||
        !array_of(a[3], t_i64, 1, &ko, &nb) || nb - 1 > INT32_MAX ||
        !array_of(a[4], t_i64, 0, &ki, &tk) || !rows_of(a[5], tk, &ri, &rb) ||
        !array_of(a[6], t_i64, tk, &k, NULL) || !rows_of(a[7], tk, &r, &rb_out) || rb_out != rb ||
        a[8] == Py_None || !bytes_of(a[8], 0, &ws, &ws_bytes) || !number(a[9], &max_keys) ||
        !stream_of(a[10], &stream))
        return no_call();
    CALL(((sort_fn)fn)((int32_t)method, (int32_t)bits, (int32_t)(nb - 1), ko, ki, ri, (int32_t)rb, tk,
                       max_keys, k, r, ws, ws_bytes, stream));
}

/* init(torch.Tensor, torch.int64, torch.int8, current_stream) */
static PyObject *m_init(PyObject *self, PyObject *args) {
    (void)self;
    PyObject *t, *i64, *i8, *cs;
    if (!PyArg_ParseTuple(args, "OOOO", &t, &i64, &i8, &cs))
        return NULL;
    Py_INCREF(t);
    Py_INCREF(i64);
    Py_INCREF(i8);
    Py_INCREF(cs);
    Py_XSETREF(current_stream, cs);
    Py_XSETREF(t_type, t);
    Py_XSETREF(t_i64, i64);
    Py_XSETREF(t_i8, i8);
    Py_RETURN_NONE;
}

static PyMethodDef methods[] = {
    {"init", m_init, METH_VARARGS, "The types the other functions accept, and the query of the current stream."},
    {"join", (PyCFunction)(void (*)(void))m_join, METH_FASTCALL, "cc_join"},
    {"batched", (PyCFunction)(void (*)(void))m_batched, METH_FASTCALL, "cc_join_batched"},
    {"padded", (PyCFunction)(void (*)(void))m_padded, METH_FASTCALL, "cc_join_batched_padded"},
    {"resolve", (PyCFunction)(void (*)(void))m_resolve, METH_FASTCALL, "cc_resolve_ids"},
    {"upsert", (PyCFunction)(void (*)(void))m_upsert, METH_FASTCALL, "cc_store_upsert"},
    {"sort", (PyCFunction)(void (*)(void))m_sort, METH_FASTCALL, "cc_sort_affinity_method"},
    {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal",
                                    "Native argument marshalling of the hot entry points.", -1,
                                    methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__marshal(void) {
    n_dtype = PyUnicode_InternFromString("dtype");
    n_is_cuda = PyUnicode_InternFromString("is_cuda");
    n_numel = PyUnicode_InternFromString("numel");
    n_contiguous = PyUnicode_InternFromString("is_contiguous");
    n_data_ptr = PyUnicode_InternFromString("data_ptr");
    n_shape = PyUnicode_InternFromString("shape");
    n_stride = PyUnicode_InternFromString("stride");
    n_element_size = PyUnicode_InternFromString("element_size");
    n_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (!n_cuda_stream || !n_dtype || !n_is_cuda || !n_numel || !n_contiguous || !n_data_ptr || !n_shape ||
        !n_stride || !n_element_size)
        return NULL;
    return PyModule_Create(&module);
}
