/* Argument marshalling of the hot entry points for Python, as an extension module.
 *
 * A small call is bound by the host: on a graph of 4,096 vertices the aggregation kernel runs for 6 us and a call through
 * ctypes took 10.3, of which 4.3 were the library and the launch, 2.7 torch.cuda.current_stream() and the rest Python
 * statements per argument.  Here each argument costs one method call on the tensor and the stream two calls into torch._C.
 *
 * The functions take the arguments of the C entry points as Python objects, in the order of the functions of binding.py of
 * the same names, check what those documented (types, contiguity, column stride) and return the status. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include "gnnagg.h"

static PyObject *dtype_f32, *dtype_bf16, *dtype_i32, *dtype_i64, *get_device, *get_raw_stream, *stream_type;
static PyObject *s_data_ptr, *s_stride, *s_dtype, *s_handle, *s_cuda_stream, *s_is_contiguous, *s_nbytes, *s_shape;

static __typeof__(&gnn_aggregate_fwd) fn_aggregate_fwd;
static __typeof__(&gnn_aggregate_bwd) fn_aggregate_bwd;
static __typeof__(&gnn_ap_fwd) fn_ap_fwd;
static __typeof__(&gnn_ap_bwd_vertex) fn_ap_bwd_vertex;
static __typeof__(&gnn_ap_bwd_vertex_arg_edges) fn_ap_bwd_vertex_arg;
static __typeof__(&gnn_ap_bwd_edge) fn_ap_bwd_edge;
static __typeof__(&gnn_sage_layer_fwd) fn_sage_layer_fwd;
static __typeof__(&gnn_sage_layer_bwd) fn_sage_layer_bwd;

/* ---- scalars: 0 on success, -1 with an exception set */

static int to_i64(PyObject *o, int64_t *out) {
    if (PyLong_CheckExact(o)) {
        *out = PyLong_AsLongLong(o);
    } else {
        PyObject *n = PyNumber_Long(o);
        if (!n) return -1;
        *out = PyLong_AsLongLong(n);
        Py_DECREF(n);
    }
    return *out == -1 && PyErr_Occurred() ? -1 : 0;
}

static int to_int(PyObject *o, int *out) {
    int64_t v;
    if (to_i64(o, &v)) return -1;
    *out = (int)v;
    return 0;
}

static int attr_ptr(PyObject *o, PyObject *name, void **out) {
    PyObject *v = PyObject_GetAttr(o, name);
    if (!v) return -1;
    *out = v == Py_None ? NULL : PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    return *out == NULL && PyErr_Occurred() ? -1 : 0;
}

static int plan_ptr(PyObject *plan, gnn_plan **out) {
    *out = NULL;
    return plan == Py_None ? 0 : attr_ptr(plan, s_handle, (void **)out);
}

/* None: torch's current stream of the current device; a torch stream; or a stream handle as a number */
static int stream_ptr(PyObject *stream, void **out) {
    if (stream == Py_None) {
        PyObject *dev = PyObject_CallNoArgs(get_device);
        if (!dev) return -1;
        PyObject *raw = PyObject_CallOneArg(get_raw_stream, dev);
        Py_DECREF(dev);
        if (!raw) return -1;
        *out = PyLong_AsVoidPtr(raw);
        Py_DECREF(raw);
        return *out == NULL && PyErr_Occurred() ? -1 : 0;
    }
    const int is_stream = PyObject_IsInstance(stream, stream_type);
    if (is_stream < 0) return -1;
    if (is_stream) return attr_ptr(stream, s_cuda_stream, out);
    int64_t v;
    if (to_i64(stream, &v)) return -1;
    *out = (void *)(intptr_t)v;
    return 0;
}

/* ---- tensors */

/* new reference, or NULL with an exception set */
static PyObject *dtype_of(PyObject *t) { return PyObject_GetAttr(t, s_dtype); }

static int index_width(PyObject *indptr, int32_t *is_64) {
    PyObject *d = dtype_of(indptr);
    if (!d) return -1;
    const int ok = d == dtype_i64 || d == dtype_i32;
    *is_64 = d == dtype_i64;
    Py_DECREF(d);
    if (!ok) PyErr_SetString(PyExc_TypeError, "indptr must be int32 or int64");
    return ok ? 0 : -1;
}

/* a tensor's sizes, the first two (a tensor has no len() that is cheap) */
static int size_of(PyObject *t, int64_t size[2]) {
    PyObject *shape = PyObject_GetAttr(t, s_shape);
    if (!shape) return -1;
    const Py_ssize_t dims = PyTuple_Check(shape) ? PyTuple_GET_SIZE(shape) : 0;
    for (int i = 0; i < 2; ++i) size[i] = i < dims ? PyLong_AsLongLong(PyTuple_GET_ITEM(shape, i)) : 0;
    Py_DECREF(shape);
    return PyErr_Occurred() ? -1 : 0;
}

/* dimensions and the strides of the first two */
static int strides_of(PyObject *t, int *dims, int64_t stride[2]) {
    PyObject *s = PyObject_CallMethodNoArgs(t, s_stride);
    if (!s) return -1;
    if (!PyTuple_Check(s)) {
        Py_DECREF(s);
        PyErr_SetString(PyExc_TypeError, "tensor expected");
        return -1;
    }
    *dims = (int)PyTuple_GET_SIZE(s);
    for (int i = 0; i < 2; ++i) stride[i] = i < *dims ? PyLong_AsLongLong(PyTuple_GET_ITEM(s, i)) : 1;
    Py_DECREF(s);
    return PyErr_Occurred() ? -1 : 0;
}

/* one-dimensional arguments have to be contiguous */
static int check_vector(PyObject *t, int dims, const int64_t stride[2]) {
    if (dims != 1 || stride[0] == 1) return 0;
    int64_t size[2];
    if (size_of(t, size)) return -1;
    if (size[0] <= 1) return 0;
    PyErr_SetString(PyExc_ValueError, "1-D arguments must be contiguous");
    return -1;
}

static int data_ptr(PyObject *t, void **out) {
    PyObject *p = PyObject_CallMethodNoArgs(t, s_data_ptr);
    if (!p) return -1;
    *out = PyLong_AsVoidPtr(p);
    Py_DECREF(p);
    return *out == NULL && PyErr_Occurred() ? -1 : 0;
}

/* Pointer of an argument of any shape (None: NULL) */
static int any_ptr(PyObject *t, void **out) {
    *out = NULL;
    if (t == Py_None) return 0;
    int dims;
    int64_t stride[2];
    return strides_of(t, &dims, stride) || check_vector(t, dims, stride) || data_ptr(t, out) ? -1 : 0;
}

/* Pointer of a feature argument and its row stride; 0 where there is none to speak of (None, not two-dimensional, one row).
 * unit_columns: two-dimensional ones of more rows need a column stride of 1. */
static int matrix(PyObject *t, int unit_columns, void **out, int64_t *row_stride, int *dims_out) {
    *out = NULL;
    *row_stride = 0;
    if (dims_out) *dims_out = 0;
    if (t == Py_None) return 0;
    int dims;
    int64_t stride[2];
    if (strides_of(t, &dims, stride) || check_vector(t, dims, stride)) return -1;
    if (dims_out) *dims_out = dims;
    if (dims == 2) {
        int64_t size[2];
        if (size_of(t, size)) return -1;
        if (size[0] > 1) {
            if (unit_columns && stride[1] != 1) {
                PyErr_SetString(PyExc_ValueError, "feature matrices must have unit column stride");
                return -1;
            }
            *row_stride = stride[0];
        }
    }
    return data_ptr(t, out);
}

static int is_f32(PyObject *t, const char *what) {
    if (t == Py_None) return 0;
    PyObject *d = dtype_of(t);
    if (!d) return -1;
    const int ok = d == dtype_f32;
    Py_DECREF(d);
    if (!ok) PyErr_SetString(PyExc_TypeError, what);
    return ok ? 0 : -1;
}
static const char *const kOnlyF32 = "the general primitive takes float32 features";

static int is_contiguous(PyObject *t) {
    PyObject *r = PyObject_CallMethodNoArgs(t, s_is_contiguous);
    if (!r) return -1;
    const int yes = PyObject_IsTrue(r);
    Py_DECREF(r);
    return yes;
}

static int workspace_of(PyObject *t, void **out, int64_t *bytes) {
    *out = NULL;
    *bytes = 0;
    if (t == Py_None) return 0;
    PyObject *n = PyObject_GetAttr(t, s_nbytes);
    if (!n) return -1;
    *bytes = PyLong_AsLongLong(n);
    Py_DECREF(n);
    if (*bytes == -1 && PyErr_Occurred()) return -1;
    return data_ptr(t, out);
}

static int expect(Py_ssize_t have, Py_ssize_t want) {
    if (have == want) return 0;
    PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", want, have);
    return -1;
}

/* ---- entry points */

/* backward, indptr, indices, edge_w, X, Y, N, F, op, plan, stream, workspace, ldx, ldy, flags, max_slices */
static PyObject *aggregate(PyObject *self, PyObject *const *a, Py_ssize_t n) {
    (void)self;
    if (expect(n, 16)) return NULL;
    if (!fn_aggregate_fwd) { PyErr_SetString(PyExc_RuntimeError, "connect() first"); return NULL; }
    PyObject *X = a[4], *Y = a[5];
    PyObject *dx = dtype_of(X), *dy = dx ? dtype_of(Y) : NULL;
    const int same = dx && dx == dy;
    gnn_opts o = {0};
    o.dtype = dx == dtype_bf16 ? GNN_BF16 : GNN_F32;
    const int known = dx == dtype_bf16 || dx == dtype_f32;
    Py_XDECREF(dx);
    Py_XDECREF(dy);
    if (!dy) return NULL;
    if (!same) { PyErr_SetString(PyExc_TypeError, "input and output features must have the same dtype"); return NULL; }
    if (!known) { PyErr_SetString(PyExc_TypeError, "features must be float32 or bfloat16"); return NULL; }
    void *indptr, *indices, *w, *x, *y;
    int64_t N, F;
    int op;
    if (index_width(a[1], &o.indptr_is_64) || any_ptr(a[1], &indptr) || any_ptr(a[2], &indices) || any_ptr(a[3], &w) ||
        matrix(X, 0, &x, &o.ldx, NULL) || matrix(Y, 0, &y, &o.ldy, NULL) || to_i64(a[6], &N) || to_i64(a[7], &F) ||
        to_int(a[8], &op) || plan_ptr(a[9], &o.plan) || stream_ptr(a[10], &o.stream) ||
        workspace_of(a[11], &o.workspace, &o.workspace_bytes) || (a[12] != Py_None && to_i64(a[12], &o.ldx)) ||
        (a[13] != Py_None && to_i64(a[13], &o.ldy)) || to_int(a[14], &o.flags) || to_int(a[15], &o.max_slices))
        return NULL;
    const int backward = a[0] == Py_True;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = (backward ? fn_aggregate_bwd : fn_aggregate_fwd)(indptr, indices, w, x, y, N, F, op, &o);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

/* common options of the operator table; e: the tensor that tells the edge operand's width */
static int ap_options(gnn_ap_opts *o, PyObject *indptr, PyObject *plan, PyObject *stream, PyObject *edge_ids, PyObject *e,
                      int e_dims, int64_t d) {
    if (indptr && index_width(indptr, &o->indptr_is_64)) return -1;
    if (e != Py_None && d != 1) {
        if (e_dims == 1) {
            o->edge_width = 1;
        } else {
            int64_t size[2];
            if (size_of(e, size)) return -1;
            o->edge_width = size[1] == 1;
        }
    }
    if (edge_ids != Py_None) {
        PyObject *dt = dtype_of(edge_ids);
        if (!dt) return -1;
        Py_DECREF(dt);
        if (dt != dtype_i64) { PyErr_SetString(PyExc_TypeError, "edge_ids must be int64"); return -1; }
        if (any_ptr(edge_ids, (void **)&o->edge_ids)) return -1;
    }
    return plan_ptr(plan, &o->plan) || stream_ptr(stream, &o->stream) ? -1 : 0;
}

/* indptr, indices, fV, fE, fO, arg_e, N, d, binop, reduce, plan, edge_ids, stream, flags, max_slices */
static PyObject *ap_fwd(PyObject *self, PyObject *const *a, Py_ssize_t n) {
    (void)self;
    if (expect(n, 15)) return NULL;
    if (!fn_ap_fwd) { PyErr_SetString(PyExc_RuntimeError, "connect() first"); return NULL; }
    if (is_f32(a[2], kOnlyF32) || is_f32(a[3], kOnlyF32) || is_f32(a[4], kOnlyF32)) return NULL;
    if (a[5] != Py_None) {
        PyObject *dt = dtype_of(a[5]);
        if (!dt) return NULL;
        Py_DECREF(dt);
        const int dense = dt == dtype_i32 ? is_contiguous(a[5]) : 0;
        if (dense < 0) return NULL;
        if (!dense) { PyErr_SetString(PyExc_TypeError, "arg_e must be a contiguous int32 tensor"); return NULL; }
    }
    gnn_ap_opts o = {0};
    void *indptr, *indices, *fV, *fE, *fO, *arg;
    int64_t N, d;
    int binop, reduce, e_dims;
    if (to_i64(a[6], &N) || to_i64(a[7], &d) || to_int(a[8], &binop) || to_int(a[9], &reduce) || matrix(a[2], 1, &fV, &o.ldv, NULL) ||
        matrix(a[3], 1, &fE, &o.lde, &e_dims) || matrix(a[4], 1, &fO, &o.ldo, NULL) || any_ptr(a[0], &indptr) ||
        any_ptr(a[1], &indices) || any_ptr(a[5], &arg) || ap_options(&o, a[0], a[10], a[12], a[11], a[3], e_dims, d) ||
        to_int(a[13], &o.flags) || to_int(a[14], &o.max_slices))
        return NULL;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = fn_ap_fwd(indptr, indices, fV, fE, fO, arg, N, d, binop, reduce, &o);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

/* indptr_t, indices_t, dO, fE, dfV, N, d, binop, plan, edge_ids, stream */
static PyObject *ap_bwd_vertex(PyObject *self, PyObject *const *a, Py_ssize_t n) {
    (void)self;
    if (expect(n, 11)) return NULL;
    if (!fn_ap_bwd_vertex) { PyErr_SetString(PyExc_RuntimeError, "connect() first"); return NULL; }
    if (is_f32(a[2], kOnlyF32) || is_f32(a[3], kOnlyF32) || is_f32(a[4], kOnlyF32)) return NULL;
    gnn_ap_opts o = {0};
    void *indptr, *indices, *dO, *fE, *dfV;
    int64_t N, d;
    int binop, e_dims;
    if (to_i64(a[5], &N) || to_i64(a[6], &d) || to_int(a[7], &binop) || matrix(a[2], 1, &dO, &o.ldo, NULL) ||
        matrix(a[3], 1, &fE, &o.lde, &e_dims) || matrix(a[4], 1, &dfV, &o.ldv, NULL) || any_ptr(a[0], &indptr) ||
        any_ptr(a[1], &indices) || ap_options(&o, a[0], a[8], a[10], a[9], a[3], e_dims, d))
        return NULL;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = fn_ap_bwd_vertex(indptr, indices, dO, fE, dfV, N, d, binop, &o);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

/* indices, arg_e, dO, fE, dfV, n_vertex_rows, N, d, binop, edge_ids, stream */
static PyObject *ap_bwd_vertex_arg(PyObject *self, PyObject *const *a, Py_ssize_t n) {
    (void)self;
    if (expect(n, 11)) return NULL;
    if (!fn_ap_bwd_vertex_arg) { PyErr_SetString(PyExc_RuntimeError, "connect() first"); return NULL; }
    if (is_f32(a[2], kOnlyF32) || is_f32(a[3], kOnlyF32) || is_f32(a[4], kOnlyF32)) return NULL;
    gnn_ap_opts o = {0};
    void *indices, *arg, *dO, *fE, *dfV;
    int64_t rows, N, d;
    int binop, e_dims;
    if (to_i64(a[5], &rows) || to_i64(a[6], &N) || to_i64(a[7], &d) || to_int(a[8], &binop) || matrix(a[2], 1, &dO, &o.ldo, NULL) ||
        matrix(a[3], 1, &fE, &o.lde, &e_dims) || matrix(a[4], 1, &dfV, &o.ldv, NULL) || any_ptr(a[0], &indices) ||
        any_ptr(a[1], &arg) || ap_options(&o, NULL, Py_None, a[10], a[9], a[3], e_dims, d))
        return NULL;
    int64_t edges[2] = {0, 0}; /* a hint: unknown where the argument is no tensor */
    if (a[0] != Py_None && size_of(a[0], edges)) { PyErr_Clear(); edges[0] = 0; }
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = fn_ap_bwd_vertex_arg(indices, arg, dO, fE, dfV, rows, N, d, binop, edges[0], &o);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

/* indptr, indices, arg_e, fV, fE, dO, dfE, N, d, binop, plan, edge_ids, stream */
static PyObject *ap_bwd_edge(PyObject *self, PyObject *const *a, Py_ssize_t n) {
    (void)self;
    if (expect(n, 13)) return NULL;
    if (!fn_ap_bwd_edge) { PyErr_SetString(PyExc_RuntimeError, "connect() first"); return NULL; }
    if (is_f32(a[3], kOnlyF32) || is_f32(a[4], kOnlyF32) || is_f32(a[5], kOnlyF32) || is_f32(a[6], kOnlyF32)) return NULL;
    gnn_ap_opts o = {0};
    void *indptr, *indices, *arg, *fV, *fE, *dO, *dfE;
    int64_t N, d;
    int binop, e_dims;
    if (to_i64(a[7], &N) || to_i64(a[8], &d) || to_int(a[9], &binop) || matrix(a[3], 1, &fV, &o.ldv, NULL) || any_ptr(a[4], &fE) ||
        matrix(a[5], 1, &dO, &o.ldo, NULL) || matrix(a[6], 1, &dfE, &o.lde, &e_dims) || any_ptr(a[0], &indptr) ||
        any_ptr(a[1], &indices) || any_ptr(a[2], &arg) || ap_options(&o, a[0], a[10], a[12], a[11], a[6], e_dims, d))
        return NULL;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = fn_ap_bwd_edge(indptr, indices, arg, fV, fE, dO, dfE, N, d, binop, &o);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

/* fp32, dense, or None */
static int dense_f32(PyObject *t, void **out) {
    *out = NULL;
    if (t == Py_None) return 0;
    if (is_f32(t, kOnlyF32)) return -1;
    const int dense = is_contiguous(t);
    if (dense < 0) return -1;
    if (!dense) { PyErr_SetString(PyExc_ValueError, "the layer calls take dense (contiguous) tensors"); return -1; }
    return data_ptr(t, out);
}

/* indptr, indices, X, W, bias, saved, H, plan, relu, order, stream, flags */
static PyObject *sage_layer_fwd(PyObject *self, PyObject *const *a, Py_ssize_t n) {
    (void)self;
    if (expect(n, 12)) return NULL;
    if (!fn_sage_layer_fwd) { PyErr_SetString(PyExc_RuntimeError, "connect() first"); return NULL; }
    gnn_layer_opts o = {0};
    void *indptr, *indices, *X, *W, *bias, *saved, *H;
    int64_t xshape[2], wshape[2];
    if (dense_f32(a[2], &X) || dense_f32(a[3], &W) || dense_f32(a[4], &bias) || dense_f32(a[5], &saved) || dense_f32(a[6], &H) ||
        index_width(a[0], &o.indptr_is_64) || any_ptr(a[0], &indptr) || any_ptr(a[1], &indices) || plan_ptr(a[7], &o.plan) ||
        to_int(a[9], &o.order) || stream_ptr(a[10], &o.stream) || to_int(a[11], &o.flags) || size_of(a[2], xshape) ||
        size_of(a[3], wshape) || (o.relu = PyObject_IsTrue(a[8])) < 0)
        return NULL;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = fn_sage_layer_fwd(indptr, indices, X, W, bias, saved, H, xshape[0], wshape[0], wshape[1], &o);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

/* indptr_t, indices_t, X, W, saved, H, dH, dX, dW, db, plan, workspace, relu, order, stream, flags */
static PyObject *sage_layer_bwd(PyObject *self, PyObject *const *a, Py_ssize_t n) {
    (void)self;
    if (expect(n, 16)) return NULL;
    if (!fn_sage_layer_bwd) { PyErr_SetString(PyExc_RuntimeError, "connect() first"); return NULL; }
    gnn_layer_opts o = {0};
    void *indptr, *indices, *p[8];
    int64_t xshape[2], wshape[2];
    for (int i = 0; i < 8; ++i)
        if (dense_f32(a[2 + i], &p[i])) return NULL;
    if (index_width(a[0], &o.indptr_is_64) || any_ptr(a[0], &indptr) || any_ptr(a[1], &indices) || plan_ptr(a[10], &o.plan) ||
        workspace_of(a[11], &o.workspace, &o.workspace_bytes) || to_int(a[13], &o.order) || stream_ptr(a[14], &o.stream) ||
        to_int(a[15], &o.flags) || size_of(a[2], xshape) || size_of(a[3], wshape) || (o.relu = PyObject_IsTrue(a[12])) < 0)
        return NULL;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = fn_sage_layer_bwd(indptr, indices, p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7], xshape[0], wshape[0], wshape[1], &o);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

/* connect({name: address}, torch): the library's entry points and torch's types */
static PyObject *connect(PyObject *self, PyObject *args) {
    (void)self;
    PyObject *addresses, *torch;
    if (!PyArg_ParseTuple(args, "O!O", &PyDict_Type, &addresses, &torch)) return NULL;
    const struct { const char *name; void **fn; } fns[] = {
        {"gnn_aggregate_fwd", (void **)&fn_aggregate_fwd}, {"gnn_aggregate_bwd", (void **)&fn_aggregate_bwd},
        {"gnn_ap_fwd", (void **)&fn_ap_fwd}, {"gnn_ap_bwd_vertex", (void **)&fn_ap_bwd_vertex},
        {"gnn_ap_bwd_vertex_arg_edges", (void **)&fn_ap_bwd_vertex_arg}, {"gnn_ap_bwd_edge", (void **)&fn_ap_bwd_edge},
        {"gnn_sage_layer_fwd", (void **)&fn_sage_layer_fwd}, {"gnn_sage_layer_bwd", (void **)&fn_sage_layer_bwd}};
    const struct { const char *name; PyObject **slot; } attrs[] = {
        {"float32", &dtype_f32}, {"bfloat16", &dtype_bf16}, {"int32", &dtype_i32}, {"int64", &dtype_i64}};
    for (size_t i = 0; i < sizeof(attrs) / sizeof(attrs[0]); ++i)
        if (!*attrs[i].slot && !(*attrs[i].slot = PyObject_GetAttrString(torch, attrs[i].name))) return NULL;
    if (!get_raw_stream) {
        PyObject *C = PyObject_GetAttrString(torch, "_C");
        get_device = C ? PyObject_GetAttrString(C, "_cuda_getDevice") : NULL;
        get_raw_stream = get_device ? PyObject_GetAttrString(C, "_cuda_getCurrentRawStream") : NULL;
        Py_XDECREF(C);
        if (!get_raw_stream) return NULL;
    }
    if (!stream_type) {
        PyObject *cuda = PyObject_GetAttrString(torch, "cuda");
        stream_type = cuda ? PyObject_GetAttrString(cuda, "Stream") : NULL;
        Py_XDECREF(cuda);
        if (!stream_type) return NULL;
    }
    for (size_t i = 0; i < sizeof(fns) / sizeof(fns[0]); ++i) {
        PyObject *v = PyDict_GetItemString(addresses, fns[i].name);
        if (!v) { PyErr_SetString(PyExc_KeyError, fns[i].name); return NULL; }
        *fns[i].fn = PyLong_AsVoidPtr(v);
        if (!*fns[i].fn) { if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, fns[i].name); return NULL; }
    }
    Py_RETURN_NONE;
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, NULL}
static PyMethodDef methods[] = {FAST(aggregate), FAST(ap_fwd), FAST(ap_bwd_vertex), FAST(ap_bwd_vertex_arg), FAST(ap_bwd_edge),
                                FAST(sage_layer_fwd), FAST(sage_layer_bwd), {"connect", connect, METH_VARARGS, NULL},
                                {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pycall", "Argument marshalling of the hot entry points.", -1, methods,
                                    NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__pycall(void) {
    const struct { const char *text; PyObject **slot; } names[] = {
        {"data_ptr", &s_data_ptr}, {"stride", &s_stride}, {"dtype", &s_dtype}, {"handle", &s_handle},
        {"cuda_stream", &s_cuda_stream}, {"is_contiguous", &s_is_contiguous}, {"nbytes", &s_nbytes}, {"shape", &s_shape}};
    for (size_t i = 0; i < sizeof(names) / sizeof(names[0]); ++i)
        if (!(*names[i].slot = PyUnicode_InternFromString(names[i].text))) return NULL;
    return PyModule_Create(&module);
}
