/* One collective call from Python: what binding.py would do with ctypes, in the usual case of a list of
 * tensors and plain integers.  A small payload takes the GPU 2 to 4 us and the C call 3; marshalling eight
 * tensors through ctypes took 1.1 us more (calls one after the other, 8 ranks x 16 KiB 4.6 us, 3.5 like this).
 *
 *   call(function, bufs, n_elems, dtype, schedule, stream[, redop]) -> status, or None where an argument is of
 *   another kind: the caller then goes through ctypes, which takes them all and reports what it does not take.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "../../include/blink.h"

typedef blink_status_t (*plain_fn)(void* const*, int, size_t, blink_dtype_t, blink_schedule_t*, void*);
typedef blink_status_t (*redop_fn)(void* const*, int, size_t, blink_dtype_t, blink_redop_t, blink_schedule_t*, void*);

static PyObject *data_ptr_name, *address_name;

/* A non-negative int of at most 64 bits; 0 if it is something else. */
static int word(PyObject* o, unsigned long long* out) {
    if (!PyLong_CheckExact(o)) return 0;
    *out = PyLong_AsUnsignedLongLong(o);
    if (*out == (unsigned long long)-1 && PyErr_Occurred()) {
        PyErr_Clear();
        return 0;
    }
    return 1;
}

static PyObject* call(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
    void* bufs[BLINK_MAX_RANKS];
    unsigned long long fn, n, dtype, schedule, stream, redop = 0;
    (void)self;
    if (nargs < 6 || nargs > 7) {
        PyErr_SetString(PyExc_TypeError, "call takes 6 or 7 arguments");
        return NULL;
    }
    PyObject* const list = args[1];
    const int is_list = PyList_CheckExact(list);
    if (!(is_list || PyTuple_CheckExact(list)) || !word(args[0], &fn) || fn == 0 || !word(args[2], &n) || !word(args[3], &dtype) ||
        dtype > 0x7fffffff || !word(args[5], &stream) || (nargs == 7 && (!word(args[6], &redop) || redop > 0x7fffffff)))
        Py_RETURN_NONE;
    const Py_ssize_t k = Py_SIZE(list);
    if (k > BLINK_MAX_RANKS) Py_RETURN_NONE;
    for (Py_ssize_t i = 0; i < k; ++i) {
        if (Py_SIZE(list) != k) Py_RETURN_NONE; /* (data_ptr may be anybody's code) */
        PyObject* const b = is_list ? PyList_GET_ITEM(list, i) : PyTuple_GET_ITEM(list, i);
        unsigned long long at;
        Py_INCREF(b);
        PyObject* const p = PyLong_CheckExact(b) ? Py_NewRef(b) : PyObject_CallMethodNoArgs(b, data_ptr_name);
        Py_DECREF(b);
        if (!p) {
            if (!PyErr_ExceptionMatches(PyExc_AttributeError) && !PyErr_ExceptionMatches(PyExc_TypeError)) return NULL;
            PyErr_Clear();
            Py_RETURN_NONE;
        }
        const int ok = word(p, &at);
        Py_DECREF(p);
        if (!ok) Py_RETURN_NONE;
        bufs[i] = (void*)at;
    }
    PyObject* const handle = PyObject_GetAttr(args[4], address_name);
    if (!handle) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    const int ok = word(handle, &schedule);
    Py_DECREF(handle);
    if (!ok) Py_RETURN_NONE;
    blink_status_t status;
    Py_BEGIN_ALLOW_THREADS /* as ctypes does: a call may wait (a schedule's first one, a timed choice) */
    if (nargs == 7)
        status = ((redop_fn)fn)(bufs, (int)k, (size_t)n, (blink_dtype_t)dtype, (blink_redop_t)redop, (blink_schedule_t*)schedule,
                                (void*)stream);
    else
        status = ((plain_fn)fn)(bufs, (int)k, (size_t)n, (blink_dtype_t)dtype, (blink_schedule_t*)schedule, (void*)stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong((long)status);
}

static PyMethodDef methods[] = {
    {"call", (PyCFunction)(void (*)(void))call, METH_FASTCALL, NULL},
    {NULL, NULL, 0, NULL},
};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_blinkcall", NULL, 0, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__blinkcall(void) {
    data_ptr_name = PyUnicode_InternFromString("data_ptr");
    address_name = PyUnicode_InternFromString("_address");
    if (!data_ptr_name || !address_name) return NULL;
    return PyModule_Create(&module);
}
