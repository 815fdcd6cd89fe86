/*
 * The Python side of gspc_conv2d_grouped: argument marshalling in C.
 *
 * A call of the library for a small layer is a launch of 3-4 us on the GPU; through ctypes, which converts
 * thirteen arguments by type and builds an object for each pointer, the call took 4.6 us of host time, 2.5-2.8 of them
 * in Python (64 -> 64 on 32x32, g = 4, N = 1).  Here they are 0.4, and the call takes 3.8 in all.  The library is not
 * linked: binding.py hands over the address of the function that it loaded.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>

typedef int (*conv_fn)(const void *, const void *, int, int, int, int, int, int, int, int, int, int, void *);

static conv_fn g_conv = NULL;
static PyObject *s_data_ptr, *s_value;

static PyObject *bind(PyObject *self, PyObject *arg) {
    (void)self;
    void *p = PyLong_AsVoidPtr(arg);
    if (!p && PyErr_Occurred()) return NULL;
    g_conv = (conv_fn)p;
    Py_RETURN_NONE;
}

/* tensor.data_ptr(), NULL for None.  0: done, -1: exception. */
static int tensor_ptr(PyObject *t, void **out) {
    if (t == Py_None) {
        *out = NULL;
        return 0;
    }
    PyObject *v = PyObject_CallMethodNoArgs(t, s_data_ptr);
    if (!v) return -1;
    *out = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    return !*out && PyErr_Occurred() ? -1 : 0;
}

/* conv(input, handle, N, Cin, H, W, Cout, KH, KW, stride, pad, groups, output) -> status code, or NotImplemented where an
 * argument is of a kind that only the general route converts (a number that is not a plain int, or does not fit one). */
static PyObject *conv(PyObject *self, PyObject *const *a, Py_ssize_t n) {
    (void)self;
    if (n != 13 || !g_conv) Py_RETURN_NOTIMPLEMENTED;
    int v[10];
    for (int i = 0; i < 10; ++i) {
        if (!PyLong_CheckExact(a[2 + i])) Py_RETURN_NOTIMPLEMENTED;
        int over;
        const long x = PyLong_AsLongAndOverflow(a[2 + i], &over);
        if (over || x != (int)x) Py_RETURN_NOTIMPLEMENTED;
        v[i] = (int)x;
    }
    void *in, *w = NULL, *out;
    if (a[1] != Py_None) {
        PyObject *h = PyObject_GetAttr(a[1], s_value);     /* a ctypes.c_void_p */
        if (!h) {
            PyErr_Clear();
            Py_RETURN_NOTIMPLEMENTED;
        }
        const int plain = h == Py_None || PyLong_CheckExact(h);
        if (plain && h != Py_None) w = PyLong_AsVoidPtr(h);
        Py_DECREF(h);
        if (!plain) Py_RETURN_NOTIMPLEMENTED;
        if (!w && PyErr_Occurred()) return NULL;
    }
    if (tensor_ptr(a[0], &in) || tensor_ptr(a[12], &out)) return NULL;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_conv(in, w, v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], v[8], v[9], out);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

static PyMethodDef methods[] = {
    {"bind", bind, METH_O, "bind(address of gspc_conv2d_grouped)"},
    {"conv", (PyCFunction)(void (*)(void))conv, METH_FASTCALL, "one grouped convolution"},
    {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_gspc_call", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__gspc_call(void) {
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_value = PyUnicode_InternFromString("value");
    return s_data_ptr && s_value ? PyModule_Create(&module) : NULL;
}
