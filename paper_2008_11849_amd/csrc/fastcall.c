/*
 * The two executor calls of the Python binding as C functions.  A small product takes little longer
 * on the GPU than its launch does on the host, and marshalling four arguments through ctypes is a
 * seventh of that: sp.spmm on a 1024 x 512 x 49 layer keeps the host for 2.95 us through ctypes and
 * for 2.55 us through here, and takes 3.15 and 2.65 to 2.85 us per call back to back.
 *
 * Arguments that are not plain integers (or None) go to the ctypes functions handed over by
 * bind(), which accept everything ctypes does; so does the raising of errors.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

typedef int (*execute_fn)(const void *, const void *, void *, void *);

static execute_fn g_run[2];
static PyObject *g_general[2], *g_check, *g_handle;

/* 1: *out is the address an int or None stands for; 0: something else */
static int address(PyObject *o, void **out) {
    if (o == Py_None) { *out = NULL; return 1; }
    if (!PyLong_CheckExact(o)) return 0;
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);
    if (v == (unsigned long long)-1 && PyErr_Occurred()) { PyErr_Clear(); return 0; }
    *out = (void *)(uintptr_t)v;
    return 1;
}

static PyObject *execute(int which, PyObject *self, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames) {
    (void)self;
    if (g_check == NULL) {
        PyErr_SetString(PyExc_RuntimeError, "bind() has not been called: import the sparsert module");
        return NULL;
    }
    if (kwnames == NULL && (nargs == 3 || nargs == 4)) {
        PyObject *handle = PyObject_GetAttr(args[0], g_handle);
        if (handle == NULL) return NULL;
        void *p[4] = {NULL, NULL, NULL, NULL};
        const int plain = address(handle, &p[0]) && address(args[1], &p[1]) && address(args[2], &p[2]) && (nargs < 4 || address(args[3], &p[3]));
        Py_DECREF(handle);
        if (plain) {
            int rc;
            Py_BEGIN_ALLOW_THREADS   /* as ctypes does: the runtime may wait for room in its queue */
            rc = g_run[which](p[0], p[1], p[2], p[3]);
            Py_END_ALLOW_THREADS
            if (rc == 0) Py_RETURN_NONE;
            return PyObject_CallFunction(g_check, "i", rc);
        }
    }
    return PyObject_Vectorcall(g_general[which], args, (size_t)nargs, kwnames);
}

static PyObject *spmm(PyObject *self, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames) { return execute(0, self, args, nargs, kwnames); }
static PyObject *conv3x3(PyObject *self, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames) { return execute(1, self, args, nargs, kwnames); }

static PyObject *bind(PyObject *self, PyObject *args) {
    unsigned long long spmm_at, conv_at;
    PyObject *general_spmm, *general_conv, *check;
    (void)self;
    if (!PyArg_ParseTuple(args, "KKOOO", &spmm_at, &conv_at, &general_spmm, &general_conv, &check)) return NULL;
    g_run[0] = (execute_fn)(uintptr_t)spmm_at;
    g_run[1] = (execute_fn)(uintptr_t)conv_at;
    Py_INCREF(general_spmm); Py_INCREF(general_conv); Py_INCREF(check);
    Py_XSETREF(g_general[0], general_spmm);
    Py_XSETREF(g_general[1], general_conv);
    Py_XSETREF(g_check, check);
    Py_RETURN_NONE;
}

static PyMethodDef methods[] = {
    {"spmm", (PyCFunction)(void (*)(void))spmm, METH_FASTCALL | METH_KEYWORDS,
     "spmm(plan, B_dev, C_dev, stream=0)\n--\n\nsparsert_spmm: device addresses and a hipStream_t as integers."},
    {"conv3x3", (PyCFunction)(void (*)(void))conv3x3, METH_FASTCALL | METH_KEYWORDS,
     "conv3x3(plan, X_dev, Y_dev, stream=0)\n--\n\nsparsert_conv3x3: device addresses and a hipStream_t as integers."},
    {"bind", bind, METH_VARARGS, "bind(spmm address, conv3x3 address, general spmm, general conv3x3, check): set up by the binding."},
    {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__fastcall(void) {
    g_handle = PyUnicode_InternFromString("handle");
    return g_handle ? PyModule_Create(&module) : NULL;
}
