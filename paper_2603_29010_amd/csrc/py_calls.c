/* The launching entry points as Python calls them: a callable per entry that converts its arguments and calls the C function.
 *
 * A small problem takes the GPU less time than its call takes the host, and of that ctypes (a conversion object per argument) and the
 * Python function in front of it were 1.0 of 5.2 us.  Only what programs really pass is converted here -- int, dtype names, the binding's own
 * Epilogue and Tuning, None, all by position; anything else, and any call before the library is loaded, goes to the Python function that the callable was made
 * from, which accepts and refuses what it always did. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stddef.h>
#include <string.h>
#include <stdint.h>

#include "../../include/ucl.h"

enum { MAX_ARGS = 24 };

typedef struct {
    PyObject_HEAD
    PyObject *dict, *weak, *python;     /* python: the function it was made from */
    PyObject *dtypes, *epilogue, *tuning, *check;
    void *entry;                        /* address of the C function, NULL until the library is loaded */
    const char *kinds;                  /* one letter per argument: i integer, p pointer, d dtype, e epilogue, t tuning, s stream */
    int n_args, n_required;
    vectorcallfunc vectorcall;
} Call;

typedef union {
    int64_t i;
    void *p;
} Arg;

static PyObject *name_c;

/* 1: converted, 0: not for us */
static int convert(Call *self, char kind, PyObject *o, Arg *a, Py_buffer *view, int *held) {
    int overflow = 0;
    switch (kind) {
    case 'i':
        if (!PyLong_CheckExact(o)) return 0;
        a->i = PyLong_AsLongLongAndOverflow(o, &overflow);
        return !overflow;
    case 'p':
    case 's':
        a->p = NULL;
        if (o == Py_None) return 1;
        if (!PyLong_CheckExact(o)) return 0;
        a->i = PyLong_AsLongLongAndOverflow(o, &overflow);
        return !overflow && a->i >= 0;
    case 'd': {
        if (PyUnicode_CheckExact(o)) {
            o = PyDict_GetItemWithError(self->dtypes, o);
            if (!o) {
                PyErr_Clear();
                return 0;
            }
        }
        if (!PyLong_CheckExact(o)) return 0;
        a->i = PyLong_AsLongLongAndOverflow(o, &overflow);
        return !overflow && a->i >= INT32_MIN && a->i <= INT32_MAX;
    }
    default: {                          /* the structure behind an Epilogue's or a Tuning's attribute c */
        PyObject *c;
        a->p = NULL;
        if (o == Py_None) return 1;
        if ((PyObject *)Py_TYPE(o) != (kind == 'e' ? self->epilogue : self->tuning)) return 0;
        c = PyObject_GetAttr(o, name_c);
        if (!c || PyObject_GetBuffer(c, view, PyBUF_SIMPLE) < 0) {
            Py_XDECREF(c);
            PyErr_Clear();
            return 0;
        }
        Py_DECREF(c);                   /* (the buffer holds it) */
        *held = 1;
        if (view->len < (Py_ssize_t)(kind == 'e' ? sizeof(ucl_epilogue) : sizeof(ucl_tuning))) return 0;
        a->p = view->buf;
        return 1;
    }
    }
}

typedef ucl_status (*gemm_fn)(int64_t, int64_t, int64_t, const void *, int32_t, int64_t, int64_t, const void *, int32_t, int64_t, int64_t, void *, int32_t,
                              int64_t, int64_t, const ucl_epilogue *, const ucl_tuning *, void *);
typedef ucl_status (*batched_fn)(int64_t, int64_t, int64_t, int64_t, const void *, int32_t, int64_t, int64_t, int64_t, const void *, int32_t, int64_t, int64_t,
                                 int64_t, void *, int32_t, int64_t, int64_t, int64_t, const ucl_epilogue *, const ucl_tuning *, void *);
typedef ucl_status (*conv_fn)(int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, const void *,
                              int32_t, const void *, int32_t, void *, int32_t, const ucl_epilogue *, const ucl_tuning *, void *);
typedef ucl_status (*transpose_fn)(int64_t, int64_t, int64_t, const void *, int32_t, void *, int32_t, void *);
static const char GEMM[] = "iiipdiipdiipdiiets", BATCHED[] = "iiiipdiiipdiiipdiiiets", CONV[] = "iiiiiiiiiiiiipdpdpdets", TRANSPOSE[] = "iiipdpds";

static PyObject *call(PyObject *callable, PyObject *const *args, size_t nargsf, PyObject *kwnames) {
    Call *self = (Call *)callable;
    const Py_ssize_t n = PyVectorcall_NARGS(nargsf);
    Arg a[MAX_ARGS];
    Py_buffer view[2];
    int held[2] = {0, 0}, ok = 1, k;
    ucl_status st = UCL_OK;
    if (!self->entry || (kwnames && PyTuple_GET_SIZE(kwnames)) || n < self->n_required || n > self->n_args)
        return PyObject_Vectorcall(self->python, args, nargsf, kwnames);
    for (k = 0; k < self->n_args && ok; ++k) {
        const int second = self->kinds[k] == 't';
        a[k].p = NULL;
        if (k < n) ok = convert(self, self->kinds[k], args[k], &a[k], &view[second], &held[second]);
    }
    if (ok) {
        void *f = self->entry;
        const char *kinds = self->kinds;
        Py_BEGIN_ALLOW_THREADS
        if (kinds == GEMM)
            st = ((gemm_fn)f)(a[0].i, a[1].i, a[2].i, a[3].p, (int32_t)a[4].i, a[5].i, a[6].i, a[7].p, (int32_t)a[8].i, a[9].i, a[10].i, a[11].p,
                              (int32_t)a[12].i, a[13].i, a[14].i, a[15].p, a[16].p, a[17].p);
        else if (kinds == BATCHED)
            st = ((batched_fn)f)(a[0].i, a[1].i, a[2].i, a[3].i, a[4].p, (int32_t)a[5].i, a[6].i, a[7].i, a[8].i, a[9].p, (int32_t)a[10].i, a[11].i, a[12].i,
                                 a[13].i, a[14].p, (int32_t)a[15].i, a[16].i, a[17].i, a[18].i, a[19].p, a[20].p, a[21].p);
        else if (kinds == CONV)
            st = ((conv_fn)f)(a[0].i, a[1].i, a[2].i, a[3].i, a[4].i, a[5].i, a[6].i, a[7].i, a[8].i, a[9].i, a[10].i, a[11].i, a[12].i, a[13].p,
                              (int32_t)a[14].i, a[15].p, (int32_t)a[16].i, a[17].p, (int32_t)a[18].i, a[19].p, a[20].p, a[21].p);
        else
            st = ((transpose_fn)f)(a[0].i, a[1].i, a[2].i, a[3].p, (int32_t)a[4].i, a[5].p, (int32_t)a[6].i, a[7].p);
        Py_END_ALLOW_THREADS
    }
    if (held[0]) PyBuffer_Release(&view[0]);
    if (held[1]) PyBuffer_Release(&view[1]);
    if (!ok) return PyObject_Vectorcall(self->python, args, nargsf, kwnames);
    if (st != UCL_OK) return PyObject_CallFunction(self->check, "i", (int)st);         /* raises, with the message of this thread's last error */
    Py_RETURN_NONE;
}

static PyObject *call_new(PyTypeObject *type, PyObject *args, PyObject *kw) {
    const char *kind;
    PyObject *python, *dtypes, *epilogue, *tuning, *check;
    Call *self;
    (void)kw;
    if (!PyArg_ParseTuple(args, "sOO!OOO", &kind, &python, &PyDict_Type, &dtypes, &epilogue, &tuning, &check)) return NULL;
    if (!(self = (Call *)type->tp_alloc(type, 0))) return NULL;
    self->kinds = !strcmp(kind, "gemm") ? GEMM : !strcmp(kind, "batched") ? BATCHED : !strcmp(kind, "conv") ? CONV : TRANSPOSE;
    self->n_args = (int)strlen(self->kinds);
    self->n_required = self->n_args - (self->kinds == TRANSPOSE ? 1 : 3);
    Py_INCREF(self->python = python);
    Py_INCREF(self->dtypes = dtypes);
    Py_INCREF(self->epilogue = epilogue);
    Py_INCREF(self->tuning = tuning);
    Py_INCREF(self->check = check);
    self->vectorcall = call;
    return (PyObject *)self;
}

static int call_traverse(Call *self, visitproc visit, void *arg) {
    Py_VISIT(self->dict); Py_VISIT(self->python); Py_VISIT(self->dtypes); Py_VISIT(self->epilogue); Py_VISIT(self->tuning); Py_VISIT(self->check);
    return 0;
}
static int call_clear(Call *self) {
    Py_CLEAR(self->dict); Py_CLEAR(self->python); Py_CLEAR(self->dtypes); Py_CLEAR(self->epilogue); Py_CLEAR(self->tuning); Py_CLEAR(self->check);
    return 0;
}
static void call_dealloc(Call *self) {
    PyObject_GC_UnTrack(self);
    if (self->weak) PyObject_ClearWeakRefs((PyObject *)self);
    call_clear(self);
    Py_TYPE(self)->tp_free((PyObject *)self);
}

static PyObject *call_bind(Call *self, PyObject *address) {
    void *p = PyLong_AsVoidPtr(address);
    if (!p && PyErr_Occurred()) return NULL;
    self->entry = p;
    Py_RETURN_NONE;
}

/* It stands where a function stood: what one answers, it answers (pickled and copied as the name of its module that it is, bound as a method of a class that
 * holds it, attributes that it has not those of the function it was made from). */
static PyObject *call_reduce(Call *self, PyObject *none) {
    (void)none;
    return PyObject_GetAttrString(self->python, "__qualname__");
}
static PyObject *call_getattro(PyObject *self, PyObject *name) {
    PyObject *v = PyObject_GenericGetAttr(self, name);
    if (v || !PyErr_ExceptionMatches(PyExc_AttributeError) || !((Call *)self)->python) return v;
    PyErr_Clear();
    return PyObject_GetAttr(((Call *)self)->python, name);
}
static PyObject *call_get(PyObject *self, PyObject *of, PyObject *type) {
    (void)type;
    if (of && of != Py_None) return PyMethod_New(self, of);
    Py_INCREF(self);
    return self;
}

static PyMethodDef methods[] = {{"__reduce__", (PyCFunction)call_reduce, METH_NOARGS, "The name under which its module holds it."}, {"bind", (PyCFunction)call_bind, METH_O, "Sets the address of the C function."}, {NULL, NULL, 0, NULL}};
static PyGetSetDef getset[] = {{"__dict__", PyObject_GenericGetDict, PyObject_GenericSetDict, NULL, NULL}, {NULL, NULL, NULL, NULL, NULL}};
static PyTypeObject CallType = {
    PyVarObject_HEAD_INIT(NULL, 0).tp_name = "paper_2603_29010_amd._calls.Call",
    .tp_basicsize = sizeof(Call),
    .tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_GC | Py_TPFLAGS_HAVE_VECTORCALL,
    .tp_new = call_new,
    .tp_dealloc = (destructor)call_dealloc,
    .tp_traverse = (traverseproc)call_traverse,
    .tp_clear = (inquiry)call_clear,
    .tp_call = PyVectorcall_Call,
    .tp_getattro = call_getattro,
    .tp_descr_get = call_get,
    .tp_weaklistoffset = offsetof(Call, weak),
    .tp_vectorcall_offset = offsetof(Call, vectorcall),
    .tp_dictoffset = offsetof(Call, dict),
    .tp_methods = methods,
    .tp_getset = getset,
};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", NULL, -1, NULL, NULL, NULL, NULL, NULL};
PyMODINIT_FUNC PyInit__calls(void) {
    PyObject *m;
    if (!(name_c = PyUnicode_InternFromString("c")) || PyType_Ready(&CallType) < 0 || !(m = PyModule_Create(&module))) return NULL;
    Py_INCREF(&CallType);
    if (PyModule_AddObject(m, "Call", (PyObject *)&CallType) < 0) return NULL;
    return m;
}
