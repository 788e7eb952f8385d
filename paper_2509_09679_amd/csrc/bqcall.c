/* Calls of the library's entry points from Python without ctypes: a Caller holds a function's address and the kinds of its arguments and
 * turns the Python objects of a call into them.  A call through ctypes took 4.2 us of host time, 2 of them in the library: three
 * calls on 1024 float32 rows of 128 took 12.5 us where the GPU needs 8.6.
 *
 *   p  device pointer: None, or an object with data_ptr() (a tensor)
 *   i  int32, u  size_t: Python integers; a call with anything else there goes to `general`, which takes what a ctypes prototype takes
 *      (numpy's integers, objects with __index__) and refuses the rest
 *   s  stream handle: a Python integer
 *   r, q  host descriptors: instances of the two ctypes structures the module is given, passed by address
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

#include "bq.h"

enum { kMaxArgs = 9 };
typedef union {
    void *p;
    uint64_t u;
} Arg;

/* kinds of the entry points' arguments, one per prototype */
static const char *const kKinds[] = {"piipus", "ppprs", "ppppqrs", "pppiprs", "ppppppurs"};
enum { kPrototypes = 5 };

typedef struct {
    PyObject_HEAD
    void *fn;
    int prototype; /* of kKinds */
    int count;
    char kinds[kMaxArgs + 1];
    PyObject *types[2]; /* of 'r' and 'q' */
    PyObject *general;
    vectorcallfunc vectorcall;
} Caller;

static PyObject *name_data_ptr;

static bq_status invoke(void *f, int prototype, const Arg *a)
{
    switch (prototype) {
        case 0: return ((__typeof__(&bq_plan_build))f)(a[0].p, (int32_t)a[1].u, (int32_t)a[2].u, a[3].p, (size_t)a[4].u, a[5].p);
        case 1: return ((__typeof__(&bq_butterfly_fwd))f)(a[0].p, a[1].p, a[2].p, a[3].p, a[4].p);
        case 2: return ((__typeof__(&bq_butterfly_fwd_quant))f)(a[0].p, a[1].p, a[2].p, a[3].p, a[4].p, a[5].p, a[6].p);
        case 3: return ((__typeof__(&bq_kron_fwd))f)(a[0].p, a[1].p, a[2].p, (int32_t)a[3].u, a[4].p, a[5].p, a[6].p);
        default: return ((__typeof__(&bq_butterfly_bwd))f)(a[0].p, a[1].p, a[2].p, a[3].p, a[4].p, a[5].p, (size_t)a[6].u, a[7].p, a[8].p);
    }
}

static PyObject *caller_call(PyObject *self, PyObject *const *args, size_t nargsf, PyObject *kwnames)
{
    Caller *c = (Caller *)self;
    if (PyVectorcall_NARGS(nargsf) != c->count || (kwnames && PyTuple_GET_SIZE(kwnames))) {
        PyErr_Format(PyExc_TypeError, "%d positional arguments expected", c->count);
        return NULL;
    }
    Arg a[kMaxArgs];
    Py_buffer views[2];
    int held = 0, ok = 1, general = 0;
    for (int i = 0; i < c->count && ok; ++i) {
        PyObject *o = args[i];
        switch (c->kinds[i]) {
            case 'p':
                if (o == Py_None) {
                    a[i].p = NULL;
                } else {
                    PyObject *p = PyObject_CallMethodNoArgs(o, name_data_ptr);
                    if (p && !PyLong_Check(p)) {
                        PyObject *q = PyNumber_Long(p);
                        Py_DECREF(p);
                        p = q;
                    }
                    ok = p != NULL;
                    if (ok) {
                        a[i].p = (void *)(uintptr_t)PyLong_AsUnsignedLongLongMask(p);
                        Py_DECREF(p);
                    }
                }
                break;
            case 'r':
            case 'q':
                if (!PyObject_TypeCheck(o, (PyTypeObject *)c->types[c->kinds[i] == 'q'])) {
                    PyErr_Format(PyExc_TypeError, "argument %d must be a %s", i + 1, ((PyTypeObject *)c->types[c->kinds[i] == 'q'])->tp_name);
                    ok = 0;
                } else if (PyObject_GetBuffer(o, &views[held], PyBUF_SIMPLE) != 0) {
                    ok = 0;
                } else {
                    a[i].p = views[held++].buf;
                }
                break;
            default:
                if (c->kinds[i] != 's' && !PyLong_Check(o)) {
                    general = 1;
                } else if (!PyLong_Check(o)) {
                    PyErr_Format(PyExc_TypeError, "argument %d must be an integer", i + 1);
                    ok = 0;
                } else if (c->kinds[i] == 's') {
                    a[i].p = (void *)(uintptr_t)PyLong_AsUnsignedLongLongMask(o);
                } else {
                    a[i].u = PyLong_AsUnsignedLongLongMask(o);
                }
        }
    }
    bq_status status = BQ_OK;
    if (ok && !general) {
        Py_BEGIN_ALLOW_THREADS
        status = invoke(c->fn, c->prototype, a);
        Py_END_ALLOW_THREADS
    }
    while (held) PyBuffer_Release(&views[--held]);
    if (ok && general) return PyObject_Vectorcall(c->general, args, c->count, NULL);
    return ok ? PyLong_FromLong((long)status) : NULL;
}

static PyObject *caller_new(PyTypeObject *type, PyObject *args, PyObject *kw)
{
    unsigned long long fn;
    const char *kinds;
    PyObject *rows, *quant, *general;
    (void)kw;
    if (!PyArg_ParseTuple(args, "KsOOO", &fn, &kinds, &rows, &quant, &general)) return NULL;
    int prototype = 0;
    while (prototype < kPrototypes && strcmp(kinds, kKinds[prototype]) != 0) ++prototype;
    if (!fn || prototype == kPrototypes || !PyType_Check(rows) || !PyType_Check(quant) || !PyCallable_Check(general)) {
        PyErr_SetString(PyExc_ValueError, "Caller(address, kinds, rows type, quant type, general)");
        return NULL;
    }
    Caller *c = (Caller *)type->tp_alloc(type, 0);
    if (!c) return NULL;
    c->fn = (void *)(uintptr_t)fn;
    c->prototype = prototype;
    c->count = (int)strlen(kinds);
    memcpy(c->kinds, kinds, (size_t)c->count + 1);
    Py_INCREF(rows);
    Py_INCREF(quant);
    Py_INCREF(general);
    c->general = general;
    c->types[0] = rows;
    c->types[1] = quant;
    c->vectorcall = caller_call;
    return (PyObject *)c;
}

static void caller_dealloc(PyObject *self)
{
    Py_XDECREF(((Caller *)self)->types[0]);
    Py_XDECREF(((Caller *)self)->types[1]);
    Py_XDECREF(((Caller *)self)->general);
    Py_TYPE(self)->tp_free(self);
}

static PyTypeObject CallerType = {
    PyVarObject_HEAD_INIT(NULL, 0).tp_name = "bqcall.Caller",
    .tp_basicsize = sizeof(Caller),
    .tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL,
    .tp_new = caller_new,
    .tp_dealloc = caller_dealloc,
    .tp_call = PyVectorcall_Call,
    .tp_vectorcall_offset = offsetof(Caller, vectorcall),
};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "bqcall", NULL, -1, NULL, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit_bqcall(void)
{
    name_data_ptr = PyUnicode_InternFromString("data_ptr");
    if (!name_data_ptr || PyType_Ready(&CallerType) < 0) return NULL;
    PyObject *m = PyModule_Create(&module);
    if (!m) return NULL;
    Py_INCREF(&CallerType);
    if (PyModule_AddObject(m, "Caller", (PyObject *)&CallerType) < 0) {
        Py_DECREF(&CallerType);
        Py_DECREF(m);
        return NULL;
    }
    return m;
}
