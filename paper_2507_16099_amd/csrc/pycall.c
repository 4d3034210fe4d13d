/* Calls of the C ABI from Python, and the look at a matrix that precedes them, without ctypes.
 *
 * A decode linear takes 4.5 us on the GPU; its call cost 5.9 us on the host, of which 2.3 are the launch, 1.0 ctypes' conversion of
 * seventeen arguments, 1.0 the shapes and strides of three matrices and 0.4 five addresses.  With this module 3.7 us in all.
 *
 *   Call(address, signature[, other])
 *                                  callable; signature: one letter per argument, 't' = tensor (None or an object with data_ptr(): a
 *                                  number in its place is refused), 'l' = integer (an int, passed in 64 bits); returns the C
 *                                  function's int.  The interpreter lock is released during the call.  Where an integer is not
 *                                  an int (NumPy's, a 0-d tensor, what else ctypes takes or refuses) the call is left to
 *                                  other(*arguments); without one it is refused.
 *   Mat(other)                     callable: (tensor, itemsize) -> (rows, cols, ld) of a 2-D tensor on the GPU that is not empty, with
 *                                  elements of that size and a contiguous last dimension; anything else is left to
 *                                  other(tensor, itemsize).
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stddef.h>
#include <stdint.h>

enum { MAX_ARGS = 18 };
typedef int64_t L;

static PyObject *s_data_ptr, *s_shape, *s_is_cuda, *s_element_size, *s_stride;

typedef struct {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    void* address;
    PyObject* other; /* NULL: none */
    int n;
    char kind[MAX_ARGS];
} Call;

/* all integers and pointers: the first six travel in registers, the others in eight bytes of stack each */
static int call_n(void* f, int n, const L* a) {
#define A1 a[0]
#define A2 A1, a[1]
#define A3 A2, a[2]
#define A4 A3, a[3]
#define A5 A4, a[4]
#define A6 A5, a[5]
#define A7 A6, a[6]
#define A8 A7, a[7]
#define A9 A8, a[8]
#define A10 A9, a[9]
#define A11 A10, a[10]
#define A12 A11, a[11]
#define A13 A12, a[12]
#define A14 A13, a[13]
#define A15 A14, a[14]
#define A16 A15, a[15]
#define A17 A16, a[16]
#define A18 A17, a[17]
#define T1 L
#define T2 T1, L
#define T3 T2, L
#define T4 T3, L
#define T5 T4, L
#define T6 T5, L
#define T7 T6, L
#define T8 T7, L
#define T9 T8, L
#define T10 T9, L
#define T11 T10, L
#define T12 T11, L
#define T13 T12, L
#define T14 T13, L
#define T15 T14, L
#define T16 T15, L
#define T17 T16, L
#define T18 T17, L
#define CASE(N) case N: return ((int (*)(T##N))f)(A##N);
    switch (n) {
        CASE(1) CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8) CASE(9) CASE(10) CASE(11) CASE(12) CASE(13) CASE(14) CASE(15)
        CASE(16) CASE(17) CASE(18)
    }
    return -1; /* not reached: Call() checks n */
}

static PyObject* call_vectorcall(PyObject* self, PyObject* const* args, size_t nargsf, PyObject* kwnames) {
    Call* c = (Call*)self;
    L a[MAX_ARGS];
    int rc;
    if (PyVectorcall_NARGS(nargsf) != c->n || (kwnames && PyTuple_GET_SIZE(kwnames) != 0))
        return PyErr_Format(PyExc_TypeError, "this function takes %d positional arguments", c->n);
    for (int i = 0; i < c->n; ++i) {
        PyObject* o = args[i];
        if (c->kind[i] == 't' && o == Py_None) {
            a[i] = 0;
        } else if (c->kind[i] == 'l' && PyLong_Check(o)) {
            a[i] = (L)PyLong_AsUnsignedLongLongMask(o);
        } else if (c->kind[i] == 't') {
            PyObject* p = PyObject_CallMethodNoArgs(o, s_data_ptr);
            if (!p) return NULL;
            a[i] = (L)PyLong_AsUnsignedLongLongMask(p);
            Py_DECREF(p);
        } else if (c->other) {
            return PyObject_Vectorcall(c->other, args, (size_t)c->n, NULL);
        } else {
            return PyErr_Format(PyExc_TypeError, "argument %d: an int is required, not %.100s", i + 1, Py_TYPE(o)->tp_name);
        }
        if (a[i] == -1 && PyErr_Occurred()) return NULL;
    }
    Py_BEGIN_ALLOW_THREADS
    rc = call_n(c->address, c->n, a);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

static PyObject* call_new(PyTypeObject* type, PyObject* args, PyObject* kw) {
    unsigned long long address;
    const char* kinds;
    Py_ssize_t n;
    PyObject* other = NULL;
    if (kw && PyDict_GET_SIZE(kw) != 0) return PyErr_Format(PyExc_TypeError, "Call() takes no keyword arguments");
    if (!PyArg_ParseTuple(args, "Ks#|O", &address, &kinds, &n, &other)) return NULL;
    if (other && !PyCallable_Check(other)) return PyErr_Format(PyExc_TypeError, "a callable is required");
    if (address == 0 || n < 1 || n > MAX_ARGS) return PyErr_Format(PyExc_ValueError, "an address and 1 to %d arguments", MAX_ARGS);
    for (Py_ssize_t i = 0; i < n; ++i)
        if (kinds[i] != 't' && kinds[i] != 'l') return PyErr_Format(PyExc_ValueError, "argument kinds are 't' and 'l'");
    Call* c = (Call*)type->tp_alloc(type, 0);
    if (!c) return NULL;
    c->vectorcall = call_vectorcall;
    c->address = (void*)(uintptr_t)address;
    Py_XINCREF(other);
    c->other = other;
    c->n = (int)n;
    for (Py_ssize_t i = 0; i < n; ++i) c->kind[i] = kinds[i];
    return (PyObject*)c;
}

static void call_dealloc(PyObject* self) {
    Py_XDECREF(((Call*)self)->other);
    Py_TYPE(self)->tp_free(self);
}

static PyTypeObject CallType = {
    PyVarObject_HEAD_INIT(NULL, 0).tp_name = "_pycall.Call",
    .tp_basicsize = sizeof(Call),
    .tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL,
    .tp_vectorcall_offset = offsetof(Call, vectorcall),
    .tp_call = PyVectorcall_Call,
    .tp_new = call_new,
    .tp_dealloc = call_dealloc,
};

/* the two entries of a tuple of two ints */
static int pair_of(PyObject* t, L* x, L* y) {
    if (!t || !PyTuple_Check(t) || PyTuple_GET_SIZE(t) != 2) return 0;
    PyObject *a = PyTuple_GET_ITEM(t, 0), *b = PyTuple_GET_ITEM(t, 1);
    if (!PyLong_Check(a) || !PyLong_Check(b)) return 0;
    *x = PyLong_AsLongLong(a);
    *y = PyLong_AsLongLong(b);
    return 1;
}

typedef struct {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    PyObject* other;
} Mat;

static PyObject* mat_vectorcall(PyObject* self, PyObject* const* args, size_t nargsf, PyObject* kwnames) {
    if (PyVectorcall_NARGS(nargsf) != 2 || (kwnames && PyTuple_GET_SIZE(kwnames) != 0)) return PyErr_Format(PyExc_TypeError, "a tensor and an item size");
    PyObject* t = args[0];
    L rows = 0, cols = 0, ld = 0, inner = 0;
    int ok = 0;
    PyObject *cuda = NULL, *shape = NULL, *size = NULL, *stride = NULL;
    if ((cuda = PyObject_GetAttr(t, s_is_cuda)) && cuda == Py_True && (shape = PyObject_GetAttr(t, s_shape)) && pair_of(shape, &rows, &cols) &&
        (size = PyObject_CallMethodNoArgs(t, s_element_size)) && PyLong_Check(size) && PyLong_Check(args[1]) &&
        PyLong_AsLongLong(size) == PyLong_AsLongLong(args[1]) && (stride = PyObject_CallMethodNoArgs(t, s_stride)) && pair_of(stride, &ld, &inner))
        ok = rows > 0 && cols > 0 && (cols <= 1 || inner == 1) && !PyErr_Occurred();
    if (ok && rows == 1 && ld < cols) ld = cols;
    Py_XDECREF(cuda);
    Py_XDECREF(shape);
    Py_XDECREF(size);
    Py_XDECREF(stride);
    if (!ok) {
        PyErr_Clear();
        PyObject* two[3] = {NULL, t, args[1]};
        return PyObject_Vectorcall(((Mat*)self)->other, two + 1, 2 | PY_VECTORCALL_ARGUMENTS_OFFSET, NULL);
    }
    PyObject* r = PyTuple_New(3);
    PyObject *a = PyLong_FromLongLong(rows), *b = PyLong_FromLongLong(cols), *c = PyLong_FromLongLong(ld);
    if (!r || !a || !b || !c) {
        Py_XDECREF(r);
        Py_XDECREF(a);
        Py_XDECREF(b);
        Py_XDECREF(c);
        return NULL;
    }
    PyTuple_SET_ITEM(r, 0, a);
    PyTuple_SET_ITEM(r, 1, b);
    PyTuple_SET_ITEM(r, 2, c);
    return r;
}

static PyObject* mat_new(PyTypeObject* type, PyObject* args, PyObject* kw) {
    PyObject* other;
    if (kw && PyDict_GET_SIZE(kw) != 0) return PyErr_Format(PyExc_TypeError, "Mat() takes no keyword arguments");
    if (!PyArg_ParseTuple(args, "O", &other)) return NULL;
    if (!PyCallable_Check(other)) return PyErr_Format(PyExc_TypeError, "a callable is required");
    Mat* m = (Mat*)type->tp_alloc(type, 0);
    if (!m) return NULL;
    m->vectorcall = mat_vectorcall;
    Py_INCREF(other);
    m->other = other;
    return (PyObject*)m;
}

static void mat_dealloc(PyObject* self) {
    Py_XDECREF(((Mat*)self)->other);
    Py_TYPE(self)->tp_free(self);
}

static PyTypeObject MatType = {
    PyVarObject_HEAD_INIT(NULL, 0).tp_name = "_pycall.Mat",
    .tp_basicsize = sizeof(Mat),
    .tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL,
    .tp_vectorcall_offset = offsetof(Mat, vectorcall),
    .tp_call = PyVectorcall_Call,
    .tp_new = mat_new,
    .tp_dealloc = mat_dealloc,
};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pycall", NULL, -1, NULL, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__pycall(void) {
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_shape = PyUnicode_InternFromString("shape");
    s_is_cuda = PyUnicode_InternFromString("is_cuda");
    s_element_size = PyUnicode_InternFromString("element_size");
    s_stride = PyUnicode_InternFromString("stride");
    if (!s_data_ptr || !s_shape || !s_is_cuda || !s_element_size || !s_stride || PyType_Ready(&CallType) < 0 || PyType_Ready(&MatType) < 0) return NULL;
    PyObject* m = PyModule_Create(&module);
    if (!m) return NULL;
    if (PyModule_AddObjectRef(m, "Call", (PyObject*)&CallType) < 0 || PyModule_AddObjectRef(m, "Mat", (PyObject*)&MatType) < 0) {
        Py_DECREF(m);
        return NULL;
    }
    return m;
}
