/* Marshalling of the entry points that a serving loop calls per layer and token: tensors and scalars in, the C ABI
 * call out.  The Python side of a call was the bound of the small ones (ls_decode_attend on one sequence: 12.4 us of
 * host time a call, of which 3 us the lookup of the stream through torch.cuda and about 5 us ctypes objects, for two
 * launches of 2 us each); here an argument costs two or three interned attribute or method calls. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include "../../include/loopserve.h"

static PyObject *s_data_ptr, *s_is_cuda, *s_is_contiguous, *s_size;   /* interned names */
static PyObject *get_device, *get_raw_stream;                         /* torch._C functions */

/* Device address of a contiguous GPU tensor; None is NULL.  0 on success. */
static int dev_ptr(PyObject* t, void** out) {
    if (t == Py_None) { *out = NULL; return 0; }
    PyObject* r = PyObject_GetAttr(t, s_is_cuda);
    if (!r) return -1;
    int ok = r == Py_True;
    Py_DECREF(r);
    if (ok) {
        if (!(r = PyObject_CallMethodNoArgs(t, s_is_contiguous))) return -1;
        ok = r == Py_True;
        Py_DECREF(r);
    }
    if (!ok) { PyErr_SetString(PyExc_AssertionError, "tensors must be contiguous device tensors"); return -1; }
    if (!(r = PyObject_CallMethodNoArgs(t, s_data_ptr))) return -1;
    *out = PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    return *out == NULL && PyErr_Occurred() ? -1 : 0;
}

/* t.size(dim) */
static int dim_of(PyObject* t, long dim, int32_t* out) {
    PyObject* d = PyLong_FromLong(dim);
    PyObject* r = d ? PyObject_CallMethodOneArg(t, s_size, d) : NULL;
    Py_XDECREF(d);
    if (!r) return -1;
    const long v = PyLong_AsLong(r);
    Py_DECREF(r);
    if (v == -1 && PyErr_Occurred()) return -1;
    *out = (int32_t)v;
    return 0;
}

/* The stream PyTorch currently issues to on the current device. */
static int cur_stream(void** out) {
    PyObject* dev = PyObject_CallNoArgs(get_device);
    PyObject* r = dev ? PyObject_CallOneArg(get_raw_stream, dev) : NULL;
    Py_XDECREF(dev);
    if (!r) return -1;
    *out = PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    return *out == NULL && PyErr_Occurred() ? -1 : 0;
}

/* An LsShape (a ctypes structure: exports its bytes as a buffer), copied. */
static int shape_of(PyObject* o, ls_shape* s) {
    Py_buffer b;
    if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) return -1;
    const int ok = b.len == (Py_ssize_t)sizeof(ls_shape);
    if (ok) memcpy(s, b.buf, sizeof(ls_shape));
    PyBuffer_Release(&b);
    if (!ok) PyErr_SetString(PyExc_TypeError, "shape must be an LsShape");
    return ok ? 0 : -1;
}

#define ARGS(count) if (nargs != (count)) { PyErr_Format(PyExc_TypeError, "%s takes %d arguments", __func__, (int)(count)); return NULL; }
#define CTX(i) ls_ctx* ctx = (ls_ctx*)PyLong_AsVoidPtr(a[i]); if (!ctx && PyErr_Occurred()) return NULL
#define SHAPE(i) ls_shape sh; if (shape_of(a[i], &sh)) return NULL
#define PTR(name, i) void* name; if (dev_ptr(a[i], &name)) return NULL
#define DIM(name, i, d) int32_t name; if (dim_of(a[i], d, &name)) return NULL
#define STREAM void* st; if (cur_stream(&st)) return NULL
#define RETURN(expr) int rc; Py_BEGIN_ALLOW_THREADS rc = (expr); Py_END_ALLOW_THREADS return PyLong_FromLong(rc)
#define DEF(name) static PyObject* name(PyObject* self, PyObject* const* a, Py_ssize_t nargs)

DEF(score) {          /* ctx, shape, q_win, q_pos, k, vert, slash, vmax, smax, total */
    (void)self; ARGS(10) CTX(0); SHAPE(1);
    PTR(q, 2); PTR(qp, 3); PTR(k, 4); PTR(ve, 5); PTR(sl, 6); PTR(vm, 7); PTR(sm, 8); PTR(to, 9); STREAM;
    RETURN(ls_score(ctx, &sh, q, qp, k, ve, sl, vm, sm, to, st));
}
DEF(score_window) {   /* ctx, shape, q_win, q_pos, k, a_win */
    (void)self; ARGS(6) CTX(0); SHAPE(1); PTR(q, 2); PTR(qp, 3); PTR(k, 4); PTR(aw, 5); STREAM;
    RETURN(ls_score_window(ctx, &sh, q, qp, k, aw, st));
}
DEF(select_lines) {   /* ctx, shape, alpha, vert, slash, vmax, smax, total, v_idx, v_cnt, s_idx, s_cnt, accounted */
    (void)self; ARGS(13) CTX(0); SHAPE(1);
    const float alpha = (float)PyFloat_AsDouble(a[2]); if (PyErr_Occurred()) return NULL;
    PTR(ve, 3); PTR(sl, 4); PTR(vm, 5); PTR(sm, 6); PTR(to, 7); PTR(vi, 8); DIM(cv, 8, -1); PTR(vc, 9); PTR(si, 10);
    DIM(cs, 10, -1); PTR(sc, 11); PTR(ac, 12); STREAM;
    RETURN(ls_select(ctx, &sh, alpha, ve, sl, vm, sm, to, vi, vc, cv, si, sc, cs, ac, st));
}
DEF(select_exact) {   /* ctx, shape, alpha, a_win, q_pos, vert, slash, total, v_idx, v_cnt, s_idx, s_cnt, accounted */
    (void)self; ARGS(13) CTX(0); SHAPE(1);
    const float alpha = (float)PyFloat_AsDouble(a[2]); if (PyErr_Occurred()) return NULL;
    PTR(aw, 3); PTR(qp, 4); PTR(ve, 5); PTR(sl, 6); PTR(to, 7); PTR(vi, 8); DIM(cv, 8, -1); PTR(vc, 9); PTR(si, 10);
    DIM(cs, 10, -1); PTR(sc, 11); PTR(ac, 12); STREAM;
    RETURN(ls_select_exact(ctx, &sh, alpha, aw, qp, ve, sl, to, vi, vc, cv, si, sc, cs, ac, st));
}
DEF(merge_lines) {    /* ctx, shape, then v_idx, v_cnt, s_idx, s_cnt of a, b and the result */
    (void)self; ARGS(14) CTX(0); SHAPE(1);
    PTR(va, 2); DIM(cva, 2, -1); PTR(vca, 3); PTR(sa, 4); DIM(csa, 4, -1); PTR(sca, 5);
    PTR(vb, 6); DIM(cvb, 6, -1); PTR(vcb, 7); PTR(sb, 8); DIM(csb, 8, -1); PTR(scb, 9);
    PTR(vo, 10); DIM(cvo, 10, -1); PTR(vco, 11); PTR(so, 12); DIM(cso, 12, -1); PTR(sco, 13); STREAM;
    RETURN(ls_merge_lines(ctx, &sh, va, vca, cva, sa, sca, csa, vb, vcb, cvb, sb, scb, csb, vo, vco, cvo, so, sco, cso, st));
}
DEF(sparse_prefill) { /* ctx, shape, q, k, v, v_idx, v_cnt, s_idx, s_cnt, out, lse */
    (void)self; ARGS(11) CTX(0); SHAPE(1);
    PTR(q, 2); PTR(k, 3); PTR(v, 4); PTR(vi, 5); DIM(cv, 5, -1); PTR(vc, 6); PTR(si, 7); DIM(cs, 7, -1); PTR(sc, 8);
    PTR(out, 9); PTR(lse, 10); STREAM;
    RETURN(ls_sparse_prefill(ctx, &sh, q, k, v, vi, vc, cv, si, sc, cs, out, lse, st));
}
DEF(kv_compress) {    /* ctx, shape, budget, q_obs, k, v, keep_idx, keep_cnt, k_out, v_out */
    (void)self; ARGS(10) CTX(0); SHAPE(1);
    const long budget = PyLong_AsLong(a[2]); if (PyErr_Occurred()) return NULL;
    PTR(q, 3); PTR(k, 4); PTR(v, 5); PTR(ki, 6); PTR(kc, 7); PTR(ko, 8); PTR(vo, 9); STREAM;
    RETURN(ls_kv_compress(ctx, &sh, (int32_t)budget, q, k, v, ki, kc, ko, vo, st));
}
DEF(decode_attend) {  /* ctx, shape, q, k_c, v_c, cnt, k_t, v_t, out, lse */
    (void)self; ARGS(10) CTX(0); SHAPE(1);
    PTR(q, 2); PTR(kc, 3); DIM(cap, 3, 2); PTR(vc, 4); PTR(cnt, 5); PTR(kt, 6); PTR(vt, 7); PTR(out, 8); PTR(lse, 9); STREAM;
    int32_t T = 0;
    if (a[6] != Py_None && dim_of(a[6], 2, &T)) return NULL;
    RETURN(ls_decode_attend(ctx, &sh, cap, T, q, kc, vc, cnt, kt, vt, out, lse, st));
}

static PyMethodDef methods[] = {
#define M(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, NULL}
    M(score), M(score_window), M(select_lines), M(select_exact), M(merge_lines), M(sparse_prefill), M(kv_compress),
    M(decode_attend), {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_lsnative", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__lsnative(void) {
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_is_cuda = PyUnicode_InternFromString("is_cuda");
    s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
    s_size = PyUnicode_InternFromString("size");
    PyObject* c = PyImport_ImportModule("torch._C");
    if (!c) return NULL;
    get_device = PyObject_GetAttrString(c, "_cuda_getDevice");
    get_raw_stream = PyObject_GetAttrString(c, "_cuda_getCurrentRawStream");
    Py_DECREF(c);
    if (!get_device || !get_raw_stream) return NULL;
    return PyModule_Create(&module);
}
