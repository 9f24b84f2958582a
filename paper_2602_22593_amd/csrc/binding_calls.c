/* The calls of binding.py whose argument marshalling costs more than their launch, in C.
 *
 * Each function takes the arguments of the binding's function of that name, makes the same checks by asking the tensors
 * the same questions, and calls the library with the GIL released, as ctypes does.  What any check would refuse, and
 * anything out of the ordinary (a tensor subclass, an integer that is none, a workspace still to be made), is answered
 * with None before anything is called: the Python code then answers it as it always did.
 *
 * What a call from Python took with the arguments marshalled there, and takes now (us): decode of four short sequences 6.9,
 * 5.5 (the kernel 4.5); kv_linear_view of 100 rows of 4096 x 1024 8.2, 5.9 (the kernel 5.8).
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include "flying_kv.h"

typedef int (*decode_fn)(const void*, void*, const void*, int64_t, const int32_t*, int64_t, const int32_t*, int, int,
                         const kv_view*, float, void*, size_t, void*);
typedef int (*prefill_fn)(const void*, void*, const void*, int64_t, const int32_t*, int64_t, const int32_t*, const int32_t*,
                          int, int64_t, int, int, const kv_view*, float, void*, size_t, void*);
typedef size_t (*prefill_bytes_fn)(const kv_view*, int, int64_t, int, int);
typedef int (*linear_fn)(const void*, int64_t, const void*, int64_t, int64_t, const kv_weight_view*, void*, int64_t, int, void*,
                         size_t, void*);
typedef size_t (*linear_bytes_fn)(const kv_weight_view*, int);
typedef int (*append_fn)(void*, int64_t, const kv_view*, const void*, const void*, const int32_t*, int64_t, const int32_t*, int,
                         void*);
typedef int (*repack_fn)(void*, int64_t, const kv_view*, const kv_view*, const int32_t*, int64_t, const int32_t*, int64_t,
                         const int32_t*, int, int, void*);

static decode_fn f_decode;
static prefill_fn f_prefill;
static prefill_bytes_fn f_prefill_bytes;
static linear_fn f_linear;
static linear_bytes_fn f_linear_bytes;
static append_fn f_append;
static repack_fn f_repack;

static PyObject *tensor_type, *parameter_type, *weight_view_type;   /* exact types only */
static PyObject *bf16_types, *int32_type, *uint8_type;              /* dtypes: a tuple, and two */
static PyObject *get_device, *raw_stream, *workspaces;              /* of torch._C; the binding's dict */
static PyObject *n_is_cuda, *n_dtype, *n_is_contiguous, *n_data_ptr, *n_shape, *n_stride, *n_numel, *n_element_size,
    *n_get_device, *n_cuda_stream, *n_handle, *n_value, *n_block_bytes, *n_n_q_local, *n_n_kv_local, *n_head_dim, *n_scratch,
    *n_zero, *n_one;

/* All helpers return 1, or 0 where the Python code is to answer (an exception may be set then: `answer` clears it). */

static int is_tensor(PyObject* t)
{
    return (PyObject*)Py_TYPE(t) == tensor_type || (PyObject*)Py_TYPE(t) == parameter_type;
}

static int true_attr(PyObject* t, PyObject* name)
{
    PyObject* v = PyObject_GetAttr(t, name);
    const int yes = v == Py_True;
    Py_XDECREF(v);
    return yes;
}

static PyObject* ask(PyObject* t, PyObject* name, PyObject* arg)
{
    PyObject* args[3] = {NULL, t, arg};   /* (the first is the callee's to use) */
    return PyObject_VectorcallMethod(name, args + 1, (arg ? 2 : 1) | PY_VECTORCALL_ARGUMENTS_OFFSET, NULL);
}

static int to_int64(PyObject* v, int64_t* out)   /* steals v */
{
    int ok = v && PyLong_CheckExact(v);
    if (ok) {
        *out = PyLong_AsLongLong(v);
        ok = !(*out == -1 && PyErr_Occurred());
    }
    Py_XDECREF(v);
    return ok;
}

static int ask_int(PyObject* t, PyObject* name, PyObject* arg, int64_t* out) { return to_int64(ask(t, name, arg), out); }

static int int_attr(PyObject* o, PyObject* name, int64_t* out) { return to_int64(PyObject_GetAttr(o, name), out); }

static int int_arg(PyObject* v, int64_t* out)   /* that fits a C int */
{
    Py_INCREF(v);
    return to_int64(v, out) && *out >= INT32_MIN && *out <= INT32_MAX;
}

static int float_arg(PyObject* v, float* out)
{
    if (!PyFloat_CheckExact(v) && !PyLong_CheckExact(v)) return 0;
    const double d = PyFloat_AsDouble(v);
    *out = (float)d;
    return !(d == -1.0 && PyErr_Occurred());
}

static int dtype_is(PyObject* t, PyObject* want)
{
    PyObject* d = PyObject_GetAttr(t, n_dtype);
    int yes = d && d == want;
    if (d && PyTuple_CheckExact(want))
        for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(want); ++i) yes |= PyTuple_GET_ITEM(want, i) == d;
    Py_XDECREF(d);
    return yes;
}

static int address(PyObject* t, void** out)
{
    int64_t p;
    if (!ask_int(t, n_data_ptr, NULL, &p)) return 0;
    *out = (void*)(uintptr_t)p;
    return 1;
}

/* binding._dev */
static int dev(PyObject* t, PyObject* dtype, void** out)
{
    if (!is_tensor(t) || !true_attr(t, n_is_cuda) || !dtype_is(t, dtype)) return 0;
    PyObject* c = ask(t, n_is_contiguous, NULL);
    const int yes = c == Py_True;
    Py_XDECREF(c);
    return yes && address(t, out);
}

/* The sizes of a tensor with exactly n dimensions. */
static int sizes(PyObject* t, int n, int64_t* out)
{
    PyObject* s = is_tensor(t) ? PyObject_GetAttr(t, n_shape) : NULL;
    int ok = s && PyTuple_Check(s) && PyTuple_GET_SIZE(s) == n;
    for (int i = 0; ok && i < n; ++i) {
        PyObject* v = PyTuple_GET_ITEM(s, i);
        Py_INCREF(v);
        ok = to_int64(v, out + i);
    }
    Py_XDECREF(s);
    return ok;
}

/* binding._dev_rows, with the sizes and the row stride */
static int dev_rows(PyObject* t, PyObject* dtype, void** out, int64_t size[2], int64_t* row)
{
    int64_t s1;
    if (!sizes(t, 2, size) || !true_attr(t, n_is_cuda) || !dtype_is(t, dtype)) return 0;
    if (size[1] > 1 && !(ask_int(t, n_stride, n_one, &s1) && s1 == 1)) return 0;
    return ask_int(t, n_stride, n_zero, row) && address(t, out);
}

static int pool_blocks(PyObject* pool, int64_t block_bytes, int whole, int64_t* out)
{
    int64_t n, e;
    if (block_bytes <= 0 || !ask_int(pool, n_numel, NULL, &n) || !ask_int(pool, n_element_size, NULL, &e)) return 0;
    *out = n * e / block_bytes;
    return !whole || n * e % block_bytes == 0;
}

static int view_handle(PyObject* view, const kv_view** out)
{
    int64_t p;
    PyObject* h = PyObject_GetAttr(view, n_handle);
    const int ok = h && int_attr(h, n_value, &p);
    Py_XDECREF(h);
    if (!ok) return 0;
    *out = (const kv_view*)(uintptr_t)p;
    return p != 0;
}

/* The stream's handle: as given, or torch's current one of `device`, a new reference (the current device's: NULL). */
static int stream_handle(PyObject* stream, PyObject* device, int64_t* out)
{
    if (stream != Py_None) return int_attr(stream, n_cuda_stream, out);
    PyObject* d = device ? device : PyObject_CallNoArgs(get_device);
    PyObject* h = d ? PyObject_CallOneArg(raw_stream, d) : NULL;
    if (!device) Py_XDECREF(d);
    return to_int64(h, out);
}

/* The workspace: as given, or the binding's own of that device and stream where it is large enough.  A new reference. */
static int workspace(PyObject* ws, PyObject* on, PyObject* stream, size_t need, PyObject** keep, void** out, size_t* bytes)
{
    int64_t n;
    *keep = NULL;
    if (ws == Py_None) {
        PyObject *device = ask(on, n_get_device, NULL), *h = NULL, *key = NULL;
        int64_t handle;
        if (device && stream_handle(stream, device, &handle)) h = PyLong_FromLongLong(handle);
        if (h) key = PyTuple_Pack(3, device, h, n_scratch);
        ws = key ? PyDict_GetItemWithError(workspaces, key) : NULL;
        Py_XINCREF(ws);
        Py_XDECREF(key);
        Py_XDECREF(h);
        Py_XDECREF(device);
        *keep = ws;
        if (!ws || !ask_int(ws, n_numel, NULL, &n) || n < 0 || (size_t)n < need) return 0;
    } else {
        Py_INCREF(ws);
        *keep = ws;
        if (!is_tensor(ws) || !ask_int(ws, n_numel, NULL, &n)) return 0;
    }
    *bytes = (size_t)n;
    return dev(ws, uint8_type, out);
}

static PyObject* answer(int made, int rc)
{
    if (made) return PyLong_FromLong(rc);
    PyErr_Clear();
    Py_RETURN_NONE;
}

#define ARGS(n) \
    if (nargs != (n)) { PyErr_SetString(PyExc_TypeError, "wrong number of arguments"); return NULL; }

/* decode(q, kv_pool, block_table, ctx_lens, view, max_ctx_len, out, scale, workspace, stream) */
static PyObject* call_decode(PyObject* self, PyObject* const* a, Py_ssize_t nargs)
{
    ARGS(10)
    int64_t batch, q[3], table[2], row, hq, d, bb, blocks, max_ctx, ws_n, stream;
    void *pq, *pout, *ppool, *ptable, *pctx, *pws;
    const kv_view* view;
    float scale;
    int rc = 0;
    const int ok = sizes(a[3], 1, &batch) && sizes(a[0], 3, q) && int_attr(a[4], n_n_q_local, &hq) &&
                   int_attr(a[4], n_head_dim, &d) && q[0] == batch && q[1] == hq && q[2] == d && sizes(a[2], 2, table) &&
                   table[0] == batch && int_attr(a[4], n_block_bytes, &bb) && dev(a[0], bf16_types, &pq) &&
                   dev(a[6], bf16_types, &pout) && dev(a[1], bf16_types, &ppool) && pool_blocks(a[1], bb, 1, &blocks) &&
                   dev(a[2], int32_type, &ptable) && ask_int(a[2], n_stride, n_zero, &row) && dev(a[3], int32_type, &pctx) &&
                   int_arg(a[5], &max_ctx) && view_handle(a[4], &view) && float_arg(a[7], &scale) &&
                   dev(a[8], uint8_type, &pws) && ask_int(a[8], n_numel, NULL, &ws_n) && stream_handle(a[9], NULL, &stream) &&
                   batch <= INT32_MAX;
    if (ok) {
        Py_BEGIN_ALLOW_THREADS
        rc = f_decode(pq, pout, ppool, blocks, ptable, row, pctx, (int)batch, (int)max_ctx, view, scale, pws, (size_t)ws_n,
                      (void*)(uintptr_t)stream);
        Py_END_ALLOW_THREADS
    }
    return answer(ok, rc);
}

/* prefill(q, kv_pool, block_table, ctx_lens, q_offsets, view, max_ctx_len, max_q_len, out, scale, workspace, stream) */
static PyObject* call_prefill(PyObject* self, PyObject* const* a, Py_ssize_t nargs)
{
    ARGS(12)
    int64_t batch, q[3], off, table[2], row, hq, d, bb, blocks, max_ctx, max_q, stream;
    void *pq, *pout, *ppool, *ptable, *pctx, *poff, *pws;
    size_t ws_n = 0;
    const kv_view* view;
    PyObject* keep = NULL;
    float scale;
    int rc = 0;
    const int ok = sizes(a[3], 1, &batch) && sizes(a[0], 3, q) && int_attr(a[5], n_n_q_local, &hq) &&
                   int_attr(a[5], n_head_dim, &d) && q[1] == hq && q[2] == d && sizes(a[4], 1, &off) && off == batch + 1 &&
                   sizes(a[2], 2, table) && table[0] == batch && int_attr(a[5], n_block_bytes, &bb) &&
                   dev(a[0], bf16_types, &pq) && dev(a[8], bf16_types, &pout) && dev(a[1], bf16_types, &ppool) &&
                   pool_blocks(a[1], bb, 0, &blocks) && dev(a[2], int32_type, &ptable) &&
                   ask_int(a[2], n_stride, n_zero, &row) && dev(a[3], int32_type, &pctx) && dev(a[4], int32_type, &poff) &&
                   int_arg(a[6], &max_ctx) && int_arg(a[7], &max_q) && view_handle(a[5], &view) && float_arg(a[9], &scale) &&
                   batch <= INT32_MAX && stream_handle(a[11], NULL, &stream) &&
                   workspace(a[10], a[0], a[11],
                             a[10] == Py_None ? f_prefill_bytes(view, (int)batch, q[0], (int)max_ctx, (int)max_q) : 0, &keep,
                             &pws, &ws_n);
    if (ok) {
        Py_BEGIN_ALLOW_THREADS
        rc = f_prefill(pq, pout, ppool, blocks, ptable, row, pctx, poff, (int)batch, q[0], (int)max_ctx, (int)max_q, view, scale,
                       pws, ws_n, (void*)(uintptr_t)stream);
        Py_END_ALLOW_THREADS
    }
    Py_XDECREF(keep);
    return answer(ok, rc);
}

/* linear(x, w_full, view, out, workspace, stream) */
static PyObject* call_linear(PyObject* self, PyObject* const* a, Py_ssize_t nargs)
{
    ARGS(6)
    int64_t x[2], w[2], y[2], ldx, ldw, ldy, stream;
    void *px, *pw, *py, *pws;
    size_t ws_n = 0;
    PyObject* keep = NULL;
    Py_buffer view;
    int rc = 0;
    if ((PyObject*)Py_TYPE(a[2]) != weight_view_type || PyObject_GetBuffer(a[2], &view, PyBUF_SIMPLE) != 0) return answer(0, 0);
    const kv_weight_view* v = (const kv_weight_view*)view.buf;
    const int ok = view.len == (Py_ssize_t)sizeof(kv_weight_view) && dev_rows(a[0], bf16_types, &px, x, &ldx) &&
                   x[1] == v->col_count && dev_rows(a[1], bf16_types, &pw, w, &ldw) && dev_rows(a[3], bf16_types, &py, y, &ldy) &&
                   x[0] <= INT32_MAX && stream_handle(a[5], NULL, &stream) &&
                   workspace(a[4], a[0], a[5], a[4] == Py_None ? f_linear_bytes(v, (int)x[0]) : 0, &keep, &pws, &ws_n);
    if (ok) {
        Py_BEGIN_ALLOW_THREADS
        rc = f_linear(px, ldx, pw, w[0], ldw, v, py, ldy, (int)x[0], pws, ws_n, (void*)(uintptr_t)stream);
        Py_END_ALLOW_THREADS
    }
    PyBuffer_Release(&view);
    Py_XDECREF(keep);
    return answer(ok, rc);
}

/* append(kv_pool, view, k_new, v_new, block_table, positions, stream) */
static PyObject* call_append(PyObject* self, PyObject* const* a, Py_ssize_t nargs)
{
    ARGS(7)
    int64_t n, k[3], v[3], hkv, d, bb, blocks, row, stream;
    void *ppool, *pk, *pv, *ptable, *ppos;
    const kv_view* view;
    int rc = 0;
    const int ok = sizes(a[5], 1, &n) && int_attr(a[1], n_n_kv_local, &hkv) && int_attr(a[1], n_head_dim, &d) &&
                   sizes(a[2], 3, k) && sizes(a[3], 3, v) && k[0] == n && k[1] == hkv && k[2] == d && v[0] == n && v[1] == hkv &&
                   v[2] == d && int_attr(a[1], n_block_bytes, &bb) && dev(a[0], bf16_types, &ppool) &&
                   pool_blocks(a[0], bb, 0, &blocks) && view_handle(a[1], &view) && dev(a[2], bf16_types, &pk) &&
                   dev(a[3], bf16_types, &pv) && dev(a[4], int32_type, &ptable) && ask_int(a[4], n_stride, n_zero, &row) &&
                   dev(a[5], int32_type, &ppos) && n <= INT32_MAX && stream_handle(a[6], NULL, &stream);
    if (ok) {
        Py_BEGIN_ALLOW_THREADS
        rc = f_append(ppool, blocks, view, pk, pv, ptable, row, ppos, (int)n, (void*)(uintptr_t)stream);
        Py_END_ALLOW_THREADS
    }
    return answer(ok, rc);
}

/* repack(kv_pool, src_view, dst_view, src_block_table, dst_block_table, n_tokens, max_tokens, stream) */
static PyObject* call_repack(PyObject* self, PyObject* const* a, Py_ssize_t nargs)
{
    ARGS(8)
    int64_t n, bb, blocks, src_row, dst_row, most, stream;
    void *ppool, *psrc, *pdst, *pn;
    const kv_view *src, *dst;
    int rc = 0;
    const int ok = sizes(a[5], 1, &n) && int_attr(a[1], n_block_bytes, &bb) && dev(a[0], bf16_types, &ppool) &&
                   pool_blocks(a[0], bb, 0, &blocks) && view_handle(a[1], &src) && view_handle(a[2], &dst) &&
                   dev(a[3], int32_type, &psrc) && ask_int(a[3], n_stride, n_zero, &src_row) && dev(a[4], int32_type, &pdst) &&
                   ask_int(a[4], n_stride, n_zero, &dst_row) && dev(a[5], int32_type, &pn) && int_arg(a[6], &most) &&
                   n <= INT32_MAX && stream_handle(a[7], NULL, &stream);
    if (ok) {
        Py_BEGIN_ALLOW_THREADS
        rc = f_repack(ppool, blocks, src, dst, psrc, src_row, pdst, dst_row, pn, (int)n, (int)most, (void*)(uintptr_t)stream);
        Py_END_ALLOW_THREADS
    }
    return answer(ok, rc);
}

/* setup((addresses of the seven functions), (types), (dtypes), (torch._C functions), dict) */
static PyObject* setup(PyObject* self, PyObject* args)
{
    unsigned long long f[7];
    PyObject *t0, *t1, *t2, *bf, *i32, *u8, *gd, *rs, *ws;
    if (!PyArg_ParseTuple(args, "(KKKKKKK)(OOO)(OOO)(OO)O!", f, f + 1, f + 2, f + 3, f + 4, f + 5, f + 6, &t0, &t1, &t2, &bf, &i32,
                          &u8, &gd, &rs, &PyDict_Type, &ws))
        return NULL;
    f_decode = (decode_fn)(uintptr_t)f[0];
    f_prefill = (prefill_fn)(uintptr_t)f[1];
    f_prefill_bytes = (prefill_bytes_fn)(uintptr_t)f[2];
    f_linear = (linear_fn)(uintptr_t)f[3];
    f_linear_bytes = (linear_bytes_fn)(uintptr_t)f[4];
    f_append = (append_fn)(uintptr_t)f[5];
    f_repack = (repack_fn)(uintptr_t)f[6];
    PyObject** const to[] = {&tensor_type, &parameter_type, &weight_view_type, &bf16_types, &int32_type, &uint8_type,
                             &get_device,  &raw_stream,     &workspaces};
    PyObject* const from[] = {t0, t1, t2, bf, i32, u8, gd, rs, ws};
    for (int i = 0; i < 9; ++i) {
        Py_INCREF(from[i]);
        Py_XSETREF(*to[i], from[i]);
    }
    Py_RETURN_NONE;
}

static PyMethodDef methods[] = {
    {"setup", setup, METH_VARARGS, NULL},
    {"decode", (PyCFunction)(void (*)(void))call_decode, METH_FASTCALL, NULL},
    {"prefill", (PyCFunction)(void (*)(void))call_prefill, METH_FASTCALL, NULL},
    {"linear", (PyCFunction)(void (*)(void))call_linear, METH_FASTCALL, NULL},
    {"append", (PyCFunction)(void (*)(void))call_append, METH_FASTCALL, NULL},
    {"repack", (PyCFunction)(void (*)(void))call_repack, METH_FASTCALL, NULL},
    {NULL, NULL, 0, NULL},
};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__calls(void)
{
    struct {
        PyObject** to;
        const char* text;
    } const names[] = {
        {&n_is_cuda, "is_cuda"}, {&n_dtype, "dtype"}, {&n_is_contiguous, "is_contiguous"}, {&n_data_ptr, "data_ptr"},
        {&n_shape, "shape"}, {&n_stride, "stride"}, {&n_numel, "numel"}, {&n_element_size, "element_size"},
        {&n_get_device, "get_device"}, {&n_cuda_stream, "cuda_stream"}, {&n_handle, "handle"}, {&n_value, "value"},
        {&n_block_bytes, "block_bytes"}, {&n_n_q_local, "n_q_local"}, {&n_n_kv_local, "n_kv_local"},
        {&n_head_dim, "head_dim"}, {&n_scratch, "scratch"},
    };
    for (size_t i = 0; i < sizeof(names) / sizeof(names[0]); ++i)
        if (!*names[i].to && !(*names[i].to = PyUnicode_InternFromString(names[i].text))) return NULL;
    if (!(n_zero = PyLong_FromLong(0)) || !(n_one = PyLong_FromLong(1))) return NULL;
    return PyModule_Create(&module);
}
