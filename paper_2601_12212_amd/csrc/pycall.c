/*
 * Argument marshalling between the Python binding and the C ABI: tensors -> device pointers, sizes and strides, the
 * current torch stream -> hipStream_t.  One native call per entry point: an eager step at batch 1 is six kernel launches
 * of about 3 us of host time each, and marshalling its three calls through ctypes and torch's Python-level stream
 * object cost another 5.5 us per call (2.8 of them the stream); here it is about 1 us.
 *
 * Every function takes the positional arguments of its namesake in binding.py and returns the dt_status as an int.
 * Tensors are anything with data_ptr(), shape, stride(), dtype and nbytes.  This module knows the interpreter and no torch; what
 * can be read without the interpreter goes through a reader that was built for the torch that is running (tensor_reader.cpp), if
 * set_reader() was given one.  The interpreter lock is released during the library call.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "../../include/dt.h"
#include "tensor_reader.h"

static PyObject *g_f32, *g_bf16, *g_get_device, *g_get_stream;  /* set by setup() */
static PyObject *s_data_ptr, *s_shape, *s_stride, *s_dtype, *s_nbytes;
static PyObject *g_capsule;                                     /* set by set_reader(); holds the reader */
static const dt_tensor_reader *g_reader;

/* the reader, unless the tensors' functions are overridden now; asked once a call (15 times was 0.2 us of 0.65) */
static const dt_tensor_reader *reader_now(void) { return g_reader && !g_reader->overridden() ? g_reader : NULL; }

/* Each helper does nothing once an error is set, so a call's arguments are converted in a row and checked once. */
static void *ptr(const dt_tensor_reader *rd, PyObject *t) {
    void *p = NULL;
    PyObject *r;
    if (t == Py_None || PyErr_Occurred()) return NULL;
    if (rd && rd->data_ptr(t, &p)) return p;
    r = PyObject_CallMethodNoArgs(t, s_data_ptr);
    if (r) {
        p = PyLong_AsVoidPtr(r);
        Py_DECREF(r);
    }
    return p;
}
static long long num(PyObject *o) { return PyErr_Occurred() ? 0 : PyLong_AsLongLong(o); }
static int inum(PyObject *o) {
    const long long v = num(o);
    if (!PyErr_Occurred() && (v > INT32_MAX || v < INT32_MIN)) PyErr_SetString(PyExc_OverflowError, "argument does not fit an int");
    return (int)v;
}
static uint64_t unum(PyObject *o) { return PyErr_Occurred() ? 0 : PyLong_AsUnsignedLongLongMask(o); }
static float fnum(PyObject *o) { return PyErr_Occurred() ? 0.f : (float)PyFloat_AsDouble(o); }
/* the first n sizes of a tensor that has at least (exactly, if `exact`) n dimensions */
static void shape(const dt_tensor_reader *rd, PyObject *t, int n, int exact, long long *out) {
    PyObject *s;
    int i;
    for (i = 0; i < n; ++i) out[i] = 0;
    if (PyErr_Occurred()) return;
    if (rd && rd->sizes(t, n, exact, out)) return;
    s = PyObject_GetAttr(t, s_shape);
    if (!s) return;
    if (!PyTuple_Check(s) || (exact ? PyTuple_GET_SIZE(s) != n : PyTuple_GET_SIZE(s) < n))
        PyErr_Format(PyExc_ValueError, "dt: expected a tensor of %d dimensions", n);
    else
        for (i = 0; i < n; ++i) out[i] = num(PyTuple_GET_ITEM(s, i));
    Py_DECREF(s);
}
static long long stride(const dt_tensor_reader *rd, PyObject *t, long dim) {
    PyObject *d, *r;
    long long v = 0;
    if (PyErr_Occurred()) return 0;
    if (rd && rd->stride(t, dim, &v)) return v;
    d = PyLong_FromLong(dim);
    r = d ? PyObject_CallMethodOneArg(t, s_stride, d) : NULL;
    if (r) v = num(r);
    Py_XDECREF(d);
    Py_XDECREF(r);
    return v;
}
static dt_dtype dtype(const dt_tensor_reader *rd, PyObject *t) {
    dt_dtype v = DT_F32;
    PyObject *d;
    int bf16;
    if (PyErr_Occurred()) return v;
    if (rd && rd->dtype(t, &bf16)) return bf16 ? DT_BF16 : DT_F32;
    d = PyObject_GetAttr(t, s_dtype);
    if (!d) return v;
    if (d == g_bf16) v = DT_BF16;
    else if (d != g_f32) PyErr_Format(PyExc_TypeError, "dt: tensors are float32 or bfloat16, got %S", d);
    Py_DECREF(d);
    return v;
}
static size_t nbytes(const dt_tensor_reader *rd, PyObject *t) {
    PyObject *r;
    size_t v = 0;
    if (t == Py_None || PyErr_Occurred()) return 0;
    if (rd && rd->nbytes(t, &v)) return v;
    r = PyObject_GetAttr(t, s_nbytes);
    if (r) {
        v = (size_t)num(r);
        Py_DECREF(r);
    }
    return v;
}
/* torch's current stream on the current device */
static void *stream(void) {
    void *p = NULL;
    PyObject *dev, *st;
    if (PyErr_Occurred()) return NULL;
    if (!g_get_stream) {
        PyErr_SetString(PyExc_RuntimeError, "setup() has not been called");
        return NULL;
    }
    dev = PyObject_CallNoArgs(g_get_device);
    st = dev ? PyObject_CallOneArg(g_get_stream, dev) : NULL;
    if (st) p = PyLong_AsVoidPtr(st);
    Py_XDECREF(dev);
    Py_XDECREF(st);
    return p;
}

#define NEED(n)                                                                                      \
    if (nargs != (n)) {                                                                              \
        PyErr_Format(PyExc_TypeError, "expected %d arguments, got %d", (int)(n), (int)nargs);        \
        return NULL;                                                                                 \
    }
#define NEED_TENSORS(n)                                                                              \
    NEED(n)                                                                                          \
    const dt_tensor_reader *const rd = reader_now();
#define CALL(expr)                                                                                   \
    do {                                                                                             \
        int rc_;                                                                                     \
        if (PyErr_Occurred()) return NULL;                                                           \
        Py_BEGIN_ALLOW_THREADS rc_ = (expr);                                                         \
        Py_END_ALLOW_THREADS return PyLong_FromLong(rc_);                                            \
    } while (0)
#define FN(name) static PyObject *name(PyObject *self, PyObject *const *a, Py_ssize_t nargs)

/* logits, k, top_val, top_id, lse, ws */
FN(topk_rows) {
    NEED_TENSORS(6)
    void *const st = stream(), *const x = ptr(rd, a[0]), *const v = ptr(rd, a[2]), *const i = ptr(rd, a[3]), *const l = ptr(rd, a[4]), *const w = ptr(rd, a[5]);
    const dt_dtype t = dtype(rd, a[0]);
    const long long row = stride(rd, a[0], 0);
    const int k = inum(a[1]);
    const size_t wb = nbytes(rd, a[5]);
    long long s[2];
    shape(rd, a[0], 2, 1, s);
    CALL(dt_topk_rows(st, x, t, s[0], (int)s[1], row, k, v, i, l, w, wb));
}
/* logits, k, top_val, top_id, lse */
FN(topk_rows_static) {
    NEED_TENSORS(5)
    void *const st = stream(), *const x = ptr(rd, a[0]), *const v = ptr(rd, a[2]), *const i = ptr(rd, a[3]), *const l = ptr(rd, a[4]);
    const dt_dtype t = dtype(rd, a[0]);
    const long long row = stride(rd, a[0], 0);
    const int k = inum(a[1]);
    long long s[2];
    shape(rd, a[0], 2, 1, s);
    CALL(dt_topk_rows_static(st, x, t, s[0], (int)s[1], row, k, v, i, l));
}
/* params, draft_logits, row_off, total_rows, root_token, TT_cap, n_nodes, tokens, parents, depth, score, logp, src_row,
   anc_mask, ws, flags */
FN(build_tree) {
    NEED_TENSORS(16)
    void *const st = stream(), *const prm = ptr(rd, a[0]), *const x = ptr(rd, a[1]), *const off = ptr(rd, a[2]), *const root = ptr(rd, a[4]);
    void *o[8];
    void *const w = ptr(rd, a[14]);
    const dt_dtype t = dtype(rd, a[1]);
    const long long row = stride(rd, a[1], 0), rows = num(a[3]);
    const int cap = inum(a[5]), flags = inum(a[15]);
    const size_t wb = nbytes(rd, a[14]);
    long long b[1], s[2];
    int i;
    for (i = 0; i < 8; ++i) o[i] = ptr(rd, a[6 + i]);
    shape(rd, a[0], 1, 0, b);
    shape(rd, a[1], 2, 0, s);
    CALL(dt_build_tree(st, (int)b[0], prm, x, t, (int)s[1], row, off, rows, root, cap, o[0], o[1], o[2], o[3], o[4], o[5], o[6],
                       o[7], w, wb, flags));
}
/* q, k_tree, v_tree, n_nodes, k_prefix_ptrs, v_prefix_ptrs, prefix_len, max_prefix_len, kv_stride_tok, kv_stride_head,
   anc_mask, scale, out, ws */
FN(tree_attention) {
    NEED_TENSORS(14)
    void *const st = stream();
    void *p[7];
    void *const mask = ptr(rd, a[10]), *const out = ptr(rd, a[12]), *const w = ptr(rd, a[13]);
    const dt_dtype t = dtype(rd, a[0]);
    const int maxlen = inum(a[7]);
    const long long stok = num(a[8]), shead = num(a[9]);
    const float scale = fnum(a[11]);
    const size_t wb = nbytes(rd, a[13]);
    long long s[4], kv[3];
    int i;
    for (i = 0; i < 7; ++i) p[i] = ptr(rd, a[i]);
    shape(rd, a[0], 4, 1, s);
    shape(rd, a[1], 3, 0, kv);
    CALL(dt_tree_attention(st, (int)s[0], t, (int)s[2], (int)kv[2], (int)s[3], scale, p[0], p[1], p[2], p[3],
                           (const void *const *)p[4], (const void *const *)p[5], p[6], maxlen, stok, shead, mask, (int)s[1], out, w,
                           wb));
}
/* mode, temperature, target_logits, n_nodes, tokens, parents, depth, logp, anc_mask, philox_seed, philox_step, accept_len,
   best_node, path_nodes, out_tokens, node_argmax, ws */
FN(accept_tree) {
    NEED_TENSORS(17)
    void *const st = stream(), *const x = ptr(rd, a[2]);
    void *p[6], *o[5];
    void *const w = ptr(rd, a[16]);
    const int mode = inum(a[0]);
    const float temp = fnum(a[1]);
    const dt_dtype t = dtype(rd, a[2]);
    const long long row = stride(rd, a[2], 1);
    const uint64_t seed = unum(a[9]), step = unum(a[10]);
    const size_t wb = nbytes(rd, a[16]);
    long long s[3];
    int i;
    for (i = 0; i < 6; ++i) p[i] = ptr(rd, a[3 + i]);
    for (i = 0; i < 5; ++i) o[i] = ptr(rd, a[11 + i]);
    shape(rd, a[2], 3, 1, s);
    CALL(dt_accept(st, (int)s[0], (dt_accept_mode)mode, temp, x, t, (int)s[2], row, p[0], p[1], p[2], p[3], p[4], p[5], (int)s[1],
                   seed, step, o[0], o[1], o[2], o[3], o[4], w, wb));
}
/* level, params, level_logits, rows_per_seq, prefix_len, TT_cap, state, n_expand, exp_token, exp_parent_slot, exp_row,
   exp_pos, exp_mask, ws, flags */
FN(expand_level) {
    NEED_TENSORS(15)
    void *const st = stream(), *const prm = ptr(rd, a[1]), *const x = ptr(rd, a[2]), *const len = ptr(rd, a[4]), *const state = ptr(rd, a[6]);
    void *o[6];
    void *const w = ptr(rd, a[13]);
    const dt_dtype t = dtype(rd, a[2]);
    const long long row = stride(rd, a[2], 0);
    const int level = inum(a[0]), R = inum(a[3]), cap = inum(a[5]), flags = inum(a[14]);
    const size_t wb = nbytes(rd, a[13]);
    long long b[1], s[2];
    int i;
    for (i = 0; i < 6; ++i) o[i] = ptr(rd, a[7 + i]);
    shape(rd, a[1], 1, 0, b);
    shape(rd, a[2], 2, 0, s);
    CALL(dt_expand_level(st, (int)b[0], level, prm, x, t, (int)s[1], row, R, len, cap, state, o[0], o[1], o[2], o[3], o[4], o[5], w,
                         wb, flags));
}
/* params, V, root_token, TT_cap, state, n_nodes, tokens, parents, depth, score, logp, src_row, anc_mask, flags */
FN(finish_tree) {
    NEED_TENSORS(14)
    void *const st = stream(), *const prm = ptr(rd, a[0]), *const root = ptr(rd, a[2]), *const state = ptr(rd, a[4]);
    void *o[8];
    const int V = inum(a[1]), cap = inum(a[3]), flags = inum(a[13]);
    long long b[1];
    int i;
    for (i = 0; i < 8; ++i) o[i] = ptr(rd, a[5 + i]);
    shape(rd, a[0], 1, 0, b);
    CALL(dt_finish_tree(st, (int)b[0], prm, V, root, cap, state, o[0], o[1], o[2], o[3], o[4], o[5], o[6], o[7], flags));
}
/* features, W1, b1, W2, b2, W3, b3, action_table, cache_interval, sample, philox_seed, philox_step, cache_step,
   cached_action, params_out, action_out, queried_out, logits_out, ws */
FN(policy_step) {
    NEED_TENSORS(19)
    void *const st = stream();
    void *p[8], *o[6];
    void *const w = ptr(rd, a[18]);
    const dt_dtype t = dtype(rd, a[0]);
    const long long row = stride(rd, a[0], 0);
    const int interval = inum(a[8]), sample = inum(a[9]);
    const uint64_t seed = unum(a[10]), step = unum(a[11]);
    const size_t wb = nbytes(rd, a[18]);
    long long f[2], h[2];
    int i;
    for (i = 0; i < 8; ++i) p[i] = ptr(rd, a[i]);
    for (i = 0; i < 6; ++i) o[i] = ptr(rd, a[12 + i]);
    shape(rd, a[0], 2, 1, f);
    shape(rd, a[5], 2, 1, h);
    CALL(dt_policy_step(st, (int)f[0], t, p[0], row, (int)f[1], (int)h[0], (int)h[1], p[1], p[2], p[3], p[4], p[5], p[6], p[7],
                        interval, sample, seed, step, o[0], o[1], o[2], o[3], o[4], o[5], w, wb));
}
/* dtype_of, Hkv, D, k_tree_ptrs, v_tree_ptrs, k_prefix_ptrs, v_prefix_ptrs, prefix_len, prefix_cap, kv_stride_tok,
   kv_stride_head, n_nodes, path_nodes, accept_len, out_tokens, TT_cap, new_prefix_len, next_root_token */
FN(commit) {
    NEED_TENSORS(18)
    void *const st = stream();
    void *p[6], *q[4];
    void *const len = ptr(rd, a[16]), *const root = ptr(rd, a[17]);
    const dt_dtype t = dtype(rd, a[0]);
    const int Hkv = inum(a[1]), D = inum(a[2]), cap = inum(a[15]);
    const long long stok = num(a[9]), shead = num(a[10]);
    long long s[2];
    int i;
    for (i = 0; i < 6; ++i) p[i] = ptr(rd, a[3 + i]);
    for (i = 0; i < 4; ++i) q[i] = ptr(rd, a[11 + i]);
    shape(rd, a[5], 2, 1, s);
    CALL(dt_commit(st, (int)s[1], (int)s[0], t, Hkv, D, (const void *const *)p[0], (const void *const *)p[1], (void *const *)p[2],
                   (void *const *)p[3], p[4], p[5], stok, shead, q[0], q[1], q[2], q[3], cap, len, root));
}
/* accept_len, count_bonus, elapsed_seconds, cache_step, reward_sum, reward_steps, reward_avg, interval_done,
   elapsed_per_seq */
FN(reward_step) {
    NEED_TENSORS(9)
    void *const st = stream(), *const len = ptr(rd, a[0]), *const per = ptr(rd, a[8]);
    void *p[5];
    const int bonus = inum(a[1]);
    const float secs = fnum(a[2]);
    long long b[1];
    int i;
    for (i = 0; i < 5; ++i) p[i] = ptr(rd, a[3 + i]);
    shape(rd, a[0], 1, 0, b);
    CALL(dt_reward_step(st, (int)b[0], len, bonus, secs, per, p[0], p[1], p[2], p[3], p[4]));
}
/* torch.float32, torch.bfloat16, callable -> current device, callable(device) -> its current raw stream */
FN(setup) {
    NEED(4)
    Py_INCREF(a[0]); Py_INCREF(a[1]); Py_INCREF(a[2]); Py_INCREF(a[3]);
    Py_XSETREF(g_f32, a[0]);
    Py_XSETREF(g_bf16, a[1]);
    Py_XSETREF(g_get_device, a[2]);
    Py_XSETREF(g_get_stream, a[3]);
    Py_RETURN_NONE;
}
/* the `reader` of a tensor reader's module, or None: through the tensors' methods only */
FN(set_reader) {
    const dt_tensor_reader *r = NULL;
    NEED(1)
    if (a[0] != Py_None && !(r = (const dt_tensor_reader *)PyCapsule_GetPointer(a[0], DT_TENSOR_READER))) return NULL;
    Py_INCREF(a[0]);
    Py_XSETREF(g_capsule, a[0]);
    g_reader = r;
    Py_RETURN_NONE;
}

#define ENTRY(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, NULL}
static PyMethodDef methods[] = {ENTRY(topk_rows), ENTRY(topk_rows_static), ENTRY(build_tree), ENTRY(tree_attention),
                                ENTRY(accept_tree), ENTRY(expand_level), ENTRY(finish_tree), ENTRY(policy_step),
                                ENTRY(commit), ENTRY(reward_step), ENTRY(setup), ENTRY(set_reader),
                                {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_dtcall", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__dtcall(void) {
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_shape = PyUnicode_InternFromString("shape");
    s_stride = PyUnicode_InternFromString("stride");
    s_dtype = PyUnicode_InternFromString("dtype");
    s_nbytes = PyUnicode_InternFromString("nbytes");
    if (!s_data_ptr || !s_shape || !s_stride || !s_dtype || !s_nbytes) return NULL;
    return PyModule_Create(&module);
}
