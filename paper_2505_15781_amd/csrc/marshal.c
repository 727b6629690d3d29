/* Argument marshalling of the calls that a program makes once per layer and step, where ctypes is a large part of the
 * call: a cache update + attention of two rows takes the device 7.0 us, and its nineteen arguments cost 7.3 us through
 * ctypes (conversions and temporary pointer objects) against 0.8-2.8 us here (two hosts). Together with attribute
 * lookups that no longer import, the call went from 16.4 us (host-bound) to 8.0 us (device-bound). Plain CPython C API; the library's functions
 * are handed over as addresses at import, so this module links against nothing.
 *
 * Tensors are asked for data_ptr(), shape and nbytes by name: no dependence on torch's headers or layout. */
/* Only the stable ABI (Python 3.10 and later): the module's file name says nothing about the interpreter it was built
 * with, so nothing of that interpreter's object layout may be compiled in. */
#define Py_LIMITED_API 0x030A0000
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stddef.h>
#include <stdint.h>

typedef int (*attn_update_fn)(void *, void *, const void *, const void *, const void *, const int32_t *, const int32_t *, void *,
                              int32_t, int32_t, int32_t, int32_t, int32_t, int32_t, int32_t, int32_t, void *, size_t, void *);
typedef int (*attn_update_static_fn)(void *, void *, const void *, const void *, const void *, const int32_t *, const int32_t *,
                                     void *, int32_t, int32_t, int32_t, int32_t, int32_t, int32_t, int32_t, int32_t, void *);

static attn_update_fn f_attn_update;
static attn_update_static_fn f_attn_update_static;
static PyObject *s_data_ptr, *s_shape, *s_nbytes, *s_value;
static PyObject *c_int_type;      /* ctypes.c_int32 */

/* address of a tensor's first element, NULL for None; -1 with an exception set on failure */
static int get_ptr(PyObject *t, void **p) {
    *p = NULL;
    if (t == Py_None) return 0;
    PyObject *v = PyObject_CallMethodObjArgs(t, s_data_ptr, NULL);
    if (!v) return -1;
    *p = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    return PyErr_Occurred() ? -1 : 0;
}

/* a whole number of 32 bits, as ctypes takes it for an int32 argument: int, anything with __index__, or a ctypes int; a
 * number that does not fit is an error (it would name other sizes than the caller's) */
static int get_i32(PyObject *o, int32_t *v) {
    PyObject *held = NULL;
    if (!PyLong_Check(o) && c_int_type) {
        const int is_c_int = PyObject_IsInstance(o, c_int_type);
        if (is_c_int < 0) return -1;
        if (is_c_int) {
            if (!(held = PyObject_GetAttr(o, s_value))) return -1;
            o = held;
        }
    }
    const long x = PyLong_AsLong(o);
    Py_XDECREF(held);
    if (x == -1 && PyErr_Occurred()) return -1;
    if (x < INT32_MIN || x > INT32_MAX) {
        PyErr_SetString(PyExc_OverflowError, "argument does not fit 32 bits");
        return -1;
    }
    *v = (int32_t)x;
    return 0;
}

/* up to `max` sizes of a tensor; returns the number of dimensions, -1 with an exception set on failure */
static Py_ssize_t get_shape(PyObject *t, int32_t *dims, Py_ssize_t max) {
    PyObject *s = PyObject_GetAttr(t, s_shape);
    if (!s) return -1;
    if (!PyTuple_Check(s)) {
        PyObject *seq = PySequence_Tuple(s);
        Py_DECREF(s);
        if (!(s = seq)) return -1;
    }
    Py_ssize_t n = PyTuple_Size(s);
    for (Py_ssize_t i = 0; i < n && i < max; ++i)
        if (get_i32(PyTuple_GetItem(s, i), &dims[i])) {
            n = -1;
            break;
        }
    Py_DECREF(s);
    return n;
}

/* (k_cache, v_cache, q, k_new, v_new, active_idx, active_off, out, rows, max_rows_per_seq, dtype, workspace, stream) for
 * `with_workspace`, without `workspace` else: the status code of the library call */
static PyObject *call_attn_update(PyObject *const *a, Py_ssize_t n, int with_workspace) {
    if (n != (with_workspace ? 13 : 12)) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return NULL;
    }
    if (!f_attn_update) {
        PyErr_SetString(PyExc_RuntimeError, "bind() has not been called");
        return NULL;
    }
    void *p[8], *ws = NULL, *stream;
    int32_t c[4], h[4], rows, max_rows, dtype;
    size_t ws_bytes = 0;
    Py_ssize_t d = get_shape(a[0], c, 4);
    if (d < 0) return NULL;
    if (d != 4) {
        PyErr_SetString(PyExc_ValueError, "the cache has four dimensions: batch, kv heads, positions, head_dim");
        return NULL;
    }
    /* query heads: from q, or from the output when there is no q of three dimensions */
    d = a[2] == Py_None ? 0 : get_shape(a[2], h, 4);
    if (d < 0) return NULL;
    if (d != 3) {
        d = get_shape(a[7], h, 4);
        if (d < 0) return NULL;
        if (d < 2) {
            PyErr_SetString(PyExc_IndexError, "out has too few dimensions");
            return NULL;
        }
    }
    for (int i = 0; i < 8; ++i)
        if (get_ptr(a[i], &p[i])) return NULL;
    if (get_i32(a[8], &rows) || get_i32(a[9], &max_rows) || get_i32(a[10], &dtype)) return NULL;
    if (with_workspace && a[11] != Py_None) {
        if (get_ptr(a[11], &ws)) return NULL;
        PyObject *b = PyObject_GetAttr(a[11], s_nbytes);
        if (!b) return NULL;
        ws_bytes = PyLong_AsSize_t(b);
        Py_DECREF(b);
    }
    stream = PyLong_AsVoidPtr(a[n - 1]);
    if (PyErr_Occurred()) return NULL;
    int rc;
    Py_BEGIN_ALLOW_THREADS      /* as ctypes does: other threads may run while a launch is enqueued */
    rc = with_workspace ? f_attn_update(p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7], rows, max_rows, c[0], h[1], c[1], c[2], c[3],
                                        dtype, ws, ws_bytes, stream)
                        : f_attn_update_static(p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7], rows, max_rows, c[0], h[1], c[1], c[2],
                                               c[3], dtype, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

static PyObject *py_attn_update(PyObject *self, PyObject *const *a, Py_ssize_t n) { return call_attn_update(a, n, 1); }
static PyObject *py_attn_update_static(PyObject *self, PyObject *const *a, Py_ssize_t n) { return call_attn_update(a, n, 0); }

/* bind(address of dkv_attn_update, address of dkv_attn_update_static, ctypes.c_int32) */
static PyObject *py_bind(PyObject *self, PyObject *const *a, Py_ssize_t n) {
    if (n != 3) {
        PyErr_SetString(PyExc_TypeError, "two addresses and the integer type are expected");
        return NULL;
    }
    void *x = PyLong_AsVoidPtr(a[0]), *y = PyLong_AsVoidPtr(a[1]);
    if (PyErr_Occurred()) return NULL;
    f_attn_update = (attn_update_fn)x;
    f_attn_update_static = (attn_update_static_fn)y;
    PyObject *old = c_int_type;
    Py_INCREF(a[2]);
    c_int_type = a[2];
    Py_XDECREF(old);
    Py_RETURN_NONE;
}

static PyMethodDef methods[] = {
    {"attn_update", (PyCFunction)(void (*)(void))py_attn_update, METH_FASTCALL, NULL},
    {"attn_update_static", (PyCFunction)(void (*)(void))py_attn_update_static, METH_FASTCALL, NULL},
    {"bind", (PyCFunction)(void (*)(void))py_bind, METH_FASTCALL, NULL},
    {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__marshal(void) {
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_shape = PyUnicode_InternFromString("shape");
    s_nbytes = PyUnicode_InternFromString("nbytes");
    s_value = PyUnicode_InternFromString("value");
    return s_data_ptr && s_shape && s_nbytes && s_value ? PyModule_Create(&module) : NULL;
}
