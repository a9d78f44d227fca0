/* Calls an entry point of libluvc from Python: call(address, arg, ...) with integers and None (a null pointer), returning the
 * status.  Every argument of these functions is an integer or a pointer, which the x86-64 calling convention passes in
 * 64-bit slots the caller cleans up, so one function type with the largest number of slots serves them all.  ctypes
 * converts an argument list of this length in about 3 us, as long as the launch behind it takes; this takes 0.3. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#if !defined(__x86_64__)
#error "pycall.c relies on the x86-64 System V calling convention"
#endif

#define SLOTS 26
typedef uint64_t u;
typedef int (*entry_t)(u, u, u, u, u, u, u, u, u, u, u, u, u, u, u, u, u, u, u, u, u, u, u, u, u, u);

static PyObject *call(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    (void)self;
    if (n < 1 || n > SLOTS + 1) {
        PyErr_Format(PyExc_TypeError, "call() takes an address and at most %d arguments", SLOTS);
        return NULL;
    }
    u a[SLOTS + 1] = {0};
    for (Py_ssize_t i = 0; i < n; ++i) {
        if (args[i] == Py_None) continue;
        a[i] = PyLong_AsUnsignedLongLongMask(args[i]);
        if (a[i] == (u)-1 && PyErr_Occurred()) return NULL;
    }
    const entry_t f = (entry_t)(uintptr_t)a[0];
    if (!f) {
        PyErr_SetString(PyExc_ValueError, "call() needs an address");
        return NULL;
    }
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f(a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10], a[11], a[12], a[13], a[14], a[15], a[16], a[17], a[18], a[19], a[20], a[21],
           a[22], a[23], a[24], a[25], a[26]);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

static PyMethodDef methods[] = {{"call", (PyCFunction)(void (*)(void))call, METH_FASTCALL, "call(address, *integers) -> status"}, {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_luvc_call", NULL, -1, methods, NULL, NULL, NULL, NULL};
PyMODINIT_FUNC PyInit__luvc_call(void) { return PyModule_Create(&module); }
