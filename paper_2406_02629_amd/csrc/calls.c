/* Python callables for the C entry points of include/ssnet.h whose arguments are integers and pointers and whose result is an int.
 * With ctypes the conversion is 0.3 to 1 us of a call, of the 3 us that a launch costs the host, and layers of a few thousand elements wait for
 * the host: share, product and reduction of a dense layer are enqueued in 14.4 us instead of 15.9, a network of 11 small layers runs in 72.8 instead of 80.4.
 * bind(address, count, pointers, general) -> callable of `count` ints; bit i of `pointers`: argument i is a pointer, and None is a null one.
 * As with ctypes, integers are taken modulo 2^64, a narrower parameter sees its low bits, and the interpreter is released during the call.
 * Arguments of any other kind or number go to `general`, the ctypes function of the same entry point: it takes what has __index__ (integers of
 * numpy, tensors of one element), objects of ctypes' own types and what their from_param takes, and refuses the rest.  Without `general` they are errors. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stddef.h>
#include <stdint.h>

enum { MOST = 16 };

typedef uint64_t W;
typedef int (*entry6)(W, W, W, W, W, W);
typedef int (*entry11)(W, W, W, W, W, W, W, W, W, W, W);
typedef int (*entry16)(W, W, W, W, W, W, W, W, W, W, W, W, W, W, W, W);

typedef struct {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    void *entry;
    Py_ssize_t count;
    unsigned long pointers;
    PyObject *general;
} Call;

static PyObject *argument_error;

/* (x86-64 System V: integers and pointers go one to a register or stack slot of 64 bits, and the caller clears the stack, so that further
 * arguments than the entry point has do no harm) */
static PyObject *call(PyObject *self, PyObject *const *args, size_t nargsf, PyObject *names)
{
    const Call *c = (const Call *)self;
    W a[MOST] = {0};
    if (PyVectorcall_NARGS(nargsf) != c->count || (names && PyTuple_GET_SIZE(names))) {
        if (c->general) return PyObject_Vectorcall(c->general, args, nargsf, names);
        PyErr_Format(PyExc_TypeError, "expected %zd arguments", c->count);
        return NULL;
    }
    for (Py_ssize_t i = 0; i < c->count; i++) {
        if (args[i] == Py_None && c->pointers >> i & 1) continue;
        if (!PyLong_Check(args[i])) {
            if (c->general) return PyObject_Vectorcall(c->general, args, nargsf, names);
            PyErr_Format(argument_error, "argument %zd: an int is needed, not %s", i + 1, Py_TYPE(args[i])->tp_name);
            return NULL;
        }
        a[i] = PyLong_AsUnsignedLongLongMask(args[i]);
        if (a[i] == (W)-1 && PyErr_Occurred()) return NULL;
    }
    int rc;
    Py_BEGIN_ALLOW_THREADS
    if (c->count <= 6)
        rc = ((entry6)c->entry)(a[0], a[1], a[2], a[3], a[4], a[5]);
    else if (c->count <= 11)
        rc = ((entry11)c->entry)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10]);
    else
        rc = ((entry16)c->entry)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10], a[11], a[12], a[13], a[14], a[15]);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

static void release(PyObject *self)
{
    Py_XDECREF(((Call *)self)->general);
    PyObject_Free(self);
}

static PyTypeObject CallType = {
    PyVarObject_HEAD_INIT(NULL, 0)
    .tp_name = "_calls.Call",
    .tp_basicsize = sizeof(Call),
    .tp_dealloc = release,
    .tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL,
    .tp_vectorcall_offset = offsetof(Call, vectorcall),
    .tp_call = PyVectorcall_Call,
    .tp_doc = "an entry point of the library",
};

static PyObject *bind(PyObject *self, PyObject *args)
{
    unsigned long long address;
    unsigned long pointers;
    Py_ssize_t count;
    PyObject *general = NULL;
    if (!PyArg_ParseTuple(args, "Knk|O", &address, &count, &pointers, &general)) return NULL;
    if (!address || count < 0 || count > MOST) {
        PyErr_SetString(PyExc_ValueError, "an address and at most 16 arguments");
        return NULL;
    }
    Call *c = PyObject_New(Call, &CallType);
    if (!c) return NULL;
    c->vectorcall = call;
    c->entry = (void *)(uintptr_t)address;
    c->count = count;
    c->pointers = pointers;
    Py_XINCREF(general);
    c->general = general;
    return (PyObject *)c;
}

static PyMethodDef methods[] = {{"bind", bind, METH_VARARGS, "bind(address, count, pointers[, general]) -> callable"}, {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__calls(void)
{
    PyObject *ctypes = PyImport_ImportModule("ctypes");
    if (!ctypes || PyType_Ready(&CallType) < 0) return NULL;
    argument_error = PyObject_GetAttrString(ctypes, "ArgumentError");
    Py_DECREF(ctypes);
    if (!argument_error) return NULL;
    return PyModule_Create(&module);
}
