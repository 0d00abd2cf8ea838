/* The binding's ttc_execute as a CPython function: four integers unpacked, one call through a pointer, None returned.
   What bounds a small problem is the host: 70 x 33 x 45 fp32 (2,0,1) takes 2.45 us a launch from a C loop, 3.32 us from a Python
   loop through ctypes, whose argument conversions are most of the difference, and 2.99 us through this.  Anything but the plain case (three or four positional arguments that are
   ints, the library loaded) goes to the Python function `slow`, which does what it always did. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>

typedef int (*execute_fn)(void*, const void*, void*, void*);
static execute_fn entry = NULL;          /* set once, by bind() */
static PyObject* slow = NULL;            /* (plan, A, B, stream=None), through ctypes */
static PyObject* fail = NULL;            /* (status): raises */

static PyObject* execute(PyObject* self, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames)
{
    (void)self;
    int plain = entry != NULL && kwnames == NULL && (nargs == 3 || nargs == 4);
    for (Py_ssize_t i = 0; plain && i < nargs; ++i) plain = PyLong_CheckExact(args[i]) || (i == 3 && args[i] == Py_None);
    if (!plain) {
        if (slow == NULL) {
            PyErr_SetString(PyExc_RuntimeError, "ttc_execute is not bound");
            return NULL;
        }
        return PyObject_Vectorcall(slow, args, (size_t)nargs, kwnames);
    }
    void* p[4] = {NULL, NULL, NULL, NULL};
    for (Py_ssize_t i = 0; i < nargs; ++i)           /* as ctypes takes an int for a pointer: its low 64 bits */
        if (args[i] != Py_None) p[i] = (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(args[i]);
    if (PyErr_Occurred()) return NULL;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = entry(p[0], p[1], p[2], p[3]);
    Py_END_ALLOW_THREADS
    if (status == 0) Py_RETURN_NONE;
    return PyObject_CallFunction(fail, "i", status);
}

/* bind(slow, fail): the Python side; bind(address): the library's entry point. */
static PyObject* bind(PyObject* self, PyObject* const* args, Py_ssize_t nargs)
{
    (void)self;
    if (nargs == 2) {
        Py_INCREF(args[0]);
        Py_INCREF(args[1]);
        Py_XSETREF(slow, args[0]);
        Py_XSETREF(fail, args[1]);
    } else if (nargs == 1) {
        void* address = PyLong_AsVoidPtr(args[0]);
        if (address == NULL && PyErr_Occurred()) return NULL;
        entry = (execute_fn)address;
    } else {
        PyErr_SetString(PyExc_TypeError, "bind() takes one or two arguments");
        return NULL;
    }
    Py_RETURN_NONE;
}

static PyMethodDef methods[] = {
    {"ttc_execute", (PyCFunction)(void (*)(void))execute, METH_FASTCALL | METH_KEYWORDS,
     "ttc_execute(plan, A, B, stream=None)\n--\n\nA, B: device addresses (tensor.data_ptr()); stream: hipStream_t as an integer or None."},
    {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, NULL},
    {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__call(void) { return PyModule_Create(&module); }
