/* Calls of the library's entry points with integers and device addresses for arguments, as the Python binding makes them on every pass:
 * call(address, arguments...) -> return code, without the conversions that ctypes makes of each argument (a call of nine, with
 * the kernel's launch: 3.5 us through ctypes, 3.2 so).  The GIL is released around the call, as ctypes does. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

typedef int64_t i;

static PyObject *call(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    i a[11] = {0};
    int rc = 0;
    (void)self;
    if (n < 1) {
        PyErr_SetString(PyExc_TypeError, "call(address, ...)");
        return NULL;
    }
    void *const f = PyLong_AsVoidPtr(args[0]);
    if (!f) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "call: no address");
        return NULL;
    }
    --n;
    if (n != 5 && n != 9 && n != 10 && n != 11) {
        PyErr_Format(PyExc_TypeError, "call: no entry point takes %zd arguments", n);
        return NULL;
    }
    for (Py_ssize_t j = 0; j < n; ++j) {
        PyObject *const o = args[j + 1];
        a[j] = o == Py_None ? 0 : (i)PyLong_AsLongLong(o);
        if (a[j] == -1 && PyErr_Occurred()) return NULL;
    }
    Py_BEGIN_ALLOW_THREADS
    switch (n) {
    case 5: rc = ((int (*)(i, i, i, i, i))f)(a[0], a[1], a[2], a[3], a[4]); break;
    case 9: rc = ((int (*)(i, i, i, i, i, i, i, i, i))f)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8]); break;
    case 10: rc = ((int (*)(i, i, i, i, i, i, i, i, i, i))f)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9]); break;
    default:
        rc = ((int (*)(i, i, i, i, i, i, i, i, i, i, i))f)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10]);
    }
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

static PyMethodDef methods[] = {{"call", (PyCFunction)(void (*)(void))call, METH_FASTCALL, NULL}, {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__fastcall(void) { return PyModule_Create(&module); }
