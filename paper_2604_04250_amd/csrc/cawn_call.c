/*
 * Argument marshalling of the Python binding: one function that takes a descriptor, tensors and a stream and calls an
 * entry point of libcawn (include/cawn.h).  It computes nothing and keeps nothing but the names it looks up.
 *
 * A one-token call takes 3 us on the GPU; its dozen tensors, each wrapped and checked in Python and converted again by
 * ctypes, took 9.7 us on the host, which was the whole price of a decoding step.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stddef.h>
#include <stdint.h>

#include "cawn.h"

static PyObject *s_data_ptr, *s_is_cuda, *s_nbytes, *s_cuda_stream;
static PyObject *get_stream, *get_device;      /* raw handle of a device's current stream; the current device */
static PyObject *desc_type;                    /* the binding's cawn_desc */

/* device pointer of a tensor, or NULL for None; -1 with an exception set when it is neither */
static int pointer(PyObject *t, void **out)
{
    *out = NULL;
    if (t == Py_None) return 0;
    PyObject *c = PyObject_GetAttr(t, s_is_cuda);
    if (!c) return -1;
    const int cuda = PyObject_IsTrue(c);
    Py_DECREF(c);
    if (cuda < 0) return -1;
    if (!cuda) {
        PyErr_SetString(PyExc_AssertionError, "libcawn takes device pointers");
        return -1;
    }
    PyObject *p = PyObject_CallMethodNoArgs(t, s_data_ptr);
    if (!p) return -1;
    *out = PyLong_AsVoidPtr(p);
    Py_DECREF(p);
    return *out || !PyErr_Occurred() ? 0 : -1;
}

static int stream_of(PyObject *s, void **out)
{
    PyObject *v;
    if (s == Py_None) {
        PyObject *d = PyObject_CallNoArgs(get_device);
        if (!d) return -1;
        v = PyObject_CallOneArg(get_stream, d);
        Py_DECREF(d);
    } else {
        v = PyObject_GetAttr(s, s_cuda_stream);
        if (!v) {
            if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return -1;
            PyErr_Clear();
            v = PyNumber_Long(s);
        }
    }
    if (!v) return -1;
    *out = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    return *out || !PyErr_Occurred() ? 0 : -1;
}

#define MAX_P 28
#define P1 p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7], p[8], p[9], p[10], p[11], p[12]
#define V1 void *, void *, void *, void *, void *, void *, void *, void *, void *, void *, void *, void *, void *
#define P14 P1, p[13]
#define V14 V1, void *
#define P15 P14, p[14]
#define V15 V14, void *
#define P16 P15, p[15]
#define V16 V15, void *
#define P18 P16, p[16], p[17]
#define V18 V16, void *, void *
#define P19 P18, p[18]
#define V19 V18, void *
#define P21 P19, p[19], p[20]
#define V21 V19, void *, void *
#define P22 P21, p[21]
#define V22 V21, void *
#define P24 P22, p[22], p[23]
#define V24 V22, void *, void *
#define P28 P24, p[24], p[25], p[26], p[27]
#define V28 V24, void *, void *, void *, void *
#define WS(n, PP, VV) case n: r = ((int (*)(const cawn_desc *, VV, size_t, void *))fn)(d, PP, bytes, st); break;
#define WSB(n, PP, VV) case n: r = ((int (*)(const cawn_desc *, VV, size_t, int32_t, void *))fn)(d, PP, bytes, bf16, st); break;

/*
 * call(address, form, desc, tensor, ..., stream): form 0 no workspace; 1 the last tensor is the workspace and its size
 * follows it; 2 like 1, and the argument after the workspace is activations_bf16.
 */
static PyObject *call(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    (void)self;
    const Py_ssize_t first = 3;
    if (n < first + 2) return PyErr_Format(PyExc_TypeError, "call: too few arguments");
    void *fn = PyLong_AsVoidPtr(args[0]);
    if (!fn) return PyErr_Occurred() ? NULL : PyErr_Format(PyExc_ValueError, "call: no function");
    const long form = PyLong_AsLong(args[1]);
    if (form == -1 && PyErr_Occurred()) return NULL;
    const Py_ssize_t np = n - first - 1 - (form == 2 ? 1 : 0);
    if (np < 1 || np > MAX_P) return PyErr_Format(PyExc_TypeError, "call: wrong number of tensors");
    void *p[MAX_P], *st;
    for (Py_ssize_t i = 0; i < np; ++i)
        if (pointer(args[first + i], &p[i]) < 0) return NULL;
    size_t bytes = 0;
    int32_t bf16 = 0;
    if (form > 0 && args[first + np - 1] != Py_None) {
        PyObject *b = PyObject_GetAttr(args[first + np - 1], s_nbytes);
        if (!b) return NULL;
        bytes = PyLong_AsSize_t(b);
        Py_DECREF(b);
        if (bytes == (size_t)-1 && PyErr_Occurred()) return NULL;
    }
    if (form == 2) {
        bf16 = (int32_t)PyLong_AsLong(args[first + np]);
        if (bf16 == -1 && PyErr_Occurred()) return NULL;
    }
    if (stream_of(args[n - 1], &st) < 0) return NULL;
    const int is_desc = desc_type ? PyObject_IsInstance(args[2], desc_type) : 0;
    if (is_desc < 0) return NULL;
    if (!is_desc) return PyErr_Format(PyExc_TypeError, "call: not a cawn_desc");
    Py_buffer view;
    if (PyObject_GetBuffer(args[2], &view, PyBUF_SIMPLE) < 0) return NULL;
    if (view.len < (Py_ssize_t)sizeof(cawn_desc)) {      /* (a subclass may be longer) */
        PyBuffer_Release(&view);
        return PyErr_Format(PyExc_TypeError, "call: cawn_desc has another layout than include/cawn.h");
    }
    const cawn_desc *d = (const cawn_desc *)view.buf;
    int r = 0, known = 1;
    Py_BEGIN_ALLOW_THREADS
    if (form == 0) {
        if (np == 12)
            r = ((int (*)(const cawn_desc *, void *, void *, void *, void *, void *, void *, void *, void *, void *, void *,
                          void *, void *, void *))fn)(d, p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7], p[8], p[9], p[10],
                                                      p[11], st);
        else known = 0;
    } else if (form == 1) {
        switch (np) {
            WS(13, P1, V1) WS(14, P14, V14) WS(15, P15, V15) WS(16, P16, V16) WS(19, P19, V19) WS(21, P21, V21)
            WS(22, P22, V22) WS(24, P24, V24)
        default: known = 0;
        }
    } else {
        switch (np) {
            WSB(18, P18, V18) WSB(28, P28, V28)
        default: known = 0;
        }
    }
    Py_END_ALLOW_THREADS
    PyBuffer_Release(&view);
    if (!known) return PyErr_Format(PyExc_TypeError, "call: no entry point takes %zd tensors", np);
    return PyLong_FromLong(r);
}

static PyObject *setup(PyObject *self, PyObject *args)
{
    (void)self;
    PyObject *d, *a, *b;
    if (!PyArg_ParseTuple(args, "OOO", &d, &a, &b)) return NULL;
    Py_INCREF(d);
    Py_INCREF(a);
    Py_INCREF(b);
    Py_XSETREF(desc_type, d);
    Py_XSETREF(get_device, a);
    Py_XSETREF(get_stream, b);
    Py_RETURN_NONE;
}

static PyMethodDef methods[] = {{"call", (PyCFunction)(void (*)(void))call, METH_FASTCALL, "call an entry point of libcawn"},
                                {"setup", setup, METH_VARARGS, "descriptor type, current device, current raw stream of a device"},
                                {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_cawn_call", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__cawn_call(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_is_cuda = PyUnicode_InternFromString("is_cuda");
    s_nbytes = PyUnicode_InternFromString("nbytes");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (!s_data_ptr || !s_is_cuda || !s_nbytes || !s_cuda_stream) return NULL;
    return PyModule_Create(&module);
}
