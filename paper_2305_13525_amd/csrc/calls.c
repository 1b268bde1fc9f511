/* The calls of a training loop, from Python into libaxo.so without ctypes: argument marshalling only.
 *
 * A small product takes 3 us of GPU time and its HIP launch 2.6 us on the host, so what a call costs around the launch shows: axo_fc_fwd
 * with nothing to launch takes 2.1 us through ctypes and 0.2 us through here, a 256 x 256 x 256 forward called in a loop 5.3 and 4.6 us.
 *
 * Each function takes what the ctypes wrapper of its name in binding.py takes and returns what that returns.  Arguments
 * of the plain kinds are converted here: a Problem, integers in the range of their C type, None for a pointer.  For
 * anything else (keywords, other types, values out of range, a library that is not loaded yet) the wrapper itself is called,
 * so that every conversion, error and default is its own. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "../../include/axo.h"

typedef union {
    const void *ptr;
    int64_t i64;
    size_t size;
    int i32;
} value;

/* Kinds of arguments: p problem, v pointer, l int64_t, i int, z size_t.  The last three of a product are its workspace, the
 * workspace's bytes and the stream. */
typedef struct {
    const char *name, *kinds;
    Py_ssize_t required; /* arguments without a default */
    value defaults[4];   /* of the others */
    int (*call)(void *address, const value *a);
    void *address;
    PyObject *wrapper;
} entry;

#define MOST_ARGUMENTS 14

static PyObject *problem_type, *raise_if;

static int call_fwd(void *f, const value *a) {
    return ((int (*)(const axo_problem_t *, const void *, int64_t, const void *, int64_t, const void *, int, void *, int64_t, void *, size_t,
                     void *))f)(a[0].ptr, a[1].ptr, a[2].i64, a[3].ptr, a[4].i64, a[5].ptr, a[6].i32, (void *)a[7].ptr, a[8].i64,
                                (void *)a[9].ptr, a[10].size, (void *)a[11].ptr);
}
static int call_grad(void *f, const value *a) {
    return ((int (*)(const axo_problem_t *, const void *, int64_t, const void *, int64_t, void *, int64_t, void *, size_t, void *))f)(
        a[0].ptr, a[1].ptr, a[2].i64, a[3].ptr, a[4].i64, (void *)a[5].ptr, a[6].i64, (void *)a[7].ptr, a[8].size, (void *)a[9].ptr);
}
static int call_dgrad_act(void *f, const value *a) {
    return ((int (*)(const axo_problem_t *, const void *, int64_t, const void *, int64_t, const void *, int64_t, int, void *, int64_t, void *,
                     size_t, void *))f)(a[0].ptr, a[1].ptr, a[2].i64, a[3].ptr, a[4].i64, a[5].ptr, a[6].i64, a[7].i32, (void *)a[8].ptr,
                                        a[9].i64, (void *)a[10].ptr, a[11].size, (void *)a[12].ptr);
}
static int call_bias_grad(void *f, const value *a) {
    return ((int (*)(const axo_problem_t *, const void *, int64_t, float *, int, void *))f)(a[0].ptr, a[1].ptr, a[2].i64,
                                                                                            (float *)a[3].ptr, a[4].i32, (void *)a[5].ptr);
}
static int call_bias_grad_ws(void *f, const value *a) {
    return ((int (*)(const axo_problem_t *, const void *, int64_t, float *, int, void *, size_t, void *))f)(
        a[0].ptr, a[1].ptr, a[2].i64, (float *)a[3].ptr, a[4].i32, (void *)a[5].ptr, a[6].size, (void *)a[7].ptr);
}

enum { FWD, DGRAD, WGRAD, DGRAD_ACT, WGRAD_ACC, BIAS_GRAD, BIAS_GRAD_WS, BIAS_GRAD_STATIC, ENTRIES };
static entry entries[ENTRIES] = {
    {"axo_fc_fwd", "pvlvlvivlvzv", 9, {{0}}, call_fwd, 0, 0},
    {"axo_fc_dgrad", "pvlvlvlvzv", 7, {{0}}, call_grad, 0, 0},
    {"axo_fc_wgrad", "pvlvlvlvzv", 7, {{0}}, call_grad, 0, 0},
    {"axo_fc_dgrad_act", "pvlvlvlivlvzv", 10, {{0}}, call_dgrad_act, 0, 0},
    {"axo_fc_wgrad_acc", "pvlvlvlvzv", 7, {{0}}, call_grad, 0, 0},
    {"axo_bias_grad", "pvlviv", 4, {{0}}, call_bias_grad, 0, 0},
    {"axo_bias_grad_ws", "pvlvivzv", 4, {{0}}, call_bias_grad_ws, 0, 0},
    {"axo_bias_grad_static", "pvlviv", 4, {{0}}, call_bias_grad, 0, 0},
};

/* One argument other than the problem; 0 if it is not of a plain kind. */
static int convert(PyObject *o, char kind, value *out) {
    int overflow;
    long long n;
    if (kind == 'v' && o == Py_None) {
        out->ptr = NULL;
        return 1;
    }
    if (!PyLong_CheckExact(o)) return 0;
    n = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow || (n == -1 && PyErr_Occurred())) {
        PyErr_Clear();
        return 0;
    }
    switch (kind) {
        case 'l': out->i64 = n; return 1;
        case 'i': out->i32 = (int)n; return n == (int)n;
        case 'z': out->size = (size_t)n; return n >= 0;
        default: out->ptr = (const void *)(uintptr_t)n; return n >= 0;
    }
}

static PyObject *call(entry *e, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames) {
    const Py_ssize_t n = (Py_ssize_t)strlen(e->kinds);
    value a[MOST_ARGUMENTS];
    Py_buffer problem;
    PyObject *result, *rc;
    void *const address = e->address;
    int status, check = 1;
    if (!address || kwnames || nargs < e->required || nargs > n + 1 || (PyObject *)Py_TYPE(args[0]) != problem_type) goto wrapper;
    for (Py_ssize_t i = 1; i < n; ++i)
        if (i >= nargs) a[i] = e->defaults[i - e->required];
        else if (!convert(args[i], e->kinds[i], &a[i])) goto wrapper;
    if (nargs == n + 1) {
        if (args[n] != Py_True && args[n] != Py_False) goto wrapper;
        check = args[n] == Py_True;
    }
    if (PyObject_GetBuffer(args[0], &problem, PyBUF_SIMPLE) != 0) return NULL;
    a[0].ptr = problem.buf;
    Py_BEGIN_ALLOW_THREADS;  /* as ctypes does */
    status = e->call(address, a);
    Py_END_ALLOW_THREADS;
    PyBuffer_Release(&problem);
    rc = PyLong_FromLong(status);
    if (!rc || status == 0 || !check) return rc;
    result = PyObject_CallFunction(raise_if, "OsO", rc, e->name, Py_True);
    Py_DECREF(rc);
    return result;
wrapper:
    if (!e->wrapper) {
        PyErr_SetString(PyExc_RuntimeError, "set_up has not been called");
        return NULL;
    }
    return PyObject_Vectorcall(e->wrapper, args, (size_t)nargs, kwnames);
}

#define ENTRY(ID) \
    static PyObject *py_##ID(PyObject *self, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames) { \
        (void)self; \
        return call(&entries[ID], args, nargs, kwnames); \
    }
ENTRY(FWD)
ENTRY(DGRAD)
ENTRY(WGRAD)
ENTRY(DGRAD_ACT)
ENTRY(WGRAD_ACC)
ENTRY(BIAS_GRAD)
ENTRY(BIAS_GRAD_WS)
ENTRY(BIAS_GRAD_STATIC)

/* set_up(Problem, {name: wrapper}, raise_if): once, when binding.py is imported. */
static PyObject *set_up(PyObject *self, PyObject *args) {
    PyObject *type, *wrappers, *raise;
    (void)self;
    if (!PyArg_ParseTuple(args, "OO!O", &type, &PyDict_Type, &wrappers, &raise)) return NULL;
    for (int i = 0; i < ENTRIES; ++i) {
        PyObject *w = PyDict_GetItemString(wrappers, entries[i].name);
        if (!w) return PyErr_Format(PyExc_KeyError, "%s", entries[i].name);
        Py_INCREF(w);
        Py_XSETREF(entries[i].wrapper, w);
    }
    Py_INCREF(type);
    Py_XSETREF(problem_type, type);
    Py_INCREF(raise);
    Py_XSETREF(raise_if, raise);
    Py_RETURN_NONE;
}

/* bind({name: address of the C function}, axo_version() of the library): whenever the library has been loaded.  Functions of another version
 * than the one that this was compiled for may take other arguments: they are left to the wrappers, and False is returned. */
static PyObject *bind(PyObject *self, PyObject *args) {
    void *found[ENTRIES];
    PyObject *addresses;
    int version;
    (void)self;
    for (int i = 0; i < ENTRIES; ++i) entries[i].address = NULL;
    if (!PyArg_ParseTuple(args, "O!i", &PyDict_Type, &addresses, &version)) return NULL;
    if (version != AXO_VERSION) Py_RETURN_FALSE;
    for (int i = 0; i < ENTRIES; ++i) {
        PyObject *o = PyDict_GetItemString(addresses, entries[i].name);
        if (!o) return PyErr_Format(PyExc_KeyError, "%s", entries[i].name);
        found[i] = PyLong_AsVoidPtr(o);
        if (PyErr_Occurred()) return NULL;
    }
    for (int i = 0; i < ENTRIES; ++i) entries[i].address = found[i];
    Py_RETURN_TRUE;
}

#define METHOD(ID, NAME, SIGNATURE) {NAME, (PyCFunction)(void (*)(void))py_##ID, METH_FASTCALL | METH_KEYWORDS, NAME SIGNATURE "\n--\n\n"}
static PyMethodDef methods[] = {
    METHOD(FWD, "axo_fc_fwd", "($module, p, X, ldx, W, ldw, bias, epilogue, Y, ldy, ws=None, ws_bytes=0, stream=None, check=True)"),
    METHOD(DGRAD, "axo_fc_dgrad", "($module, p, dY, lddy, W, ldw, dX, lddx, ws=None, ws_bytes=0, stream=None, check=True)"),
    METHOD(WGRAD, "axo_fc_wgrad", "($module, p, X, ldx, dY, lddy, dW, lddw, ws=None, ws_bytes=0, stream=None, check=True)"),
    METHOD(DGRAD_ACT, "axo_fc_dgrad_act", "($module, p, dY, lddy, W, ldw, pre, ldpre, act, dX, lddx, ws=None, ws_bytes=0, stream=None, check=True)"),
    METHOD(WGRAD_ACC, "axo_fc_wgrad_acc", "($module, p, X, ldx, dY, lddy, dW, lddw, ws=None, ws_bytes=0, stream=None, check=True)"),
    METHOD(BIAS_GRAD, "axo_bias_grad", "($module, p, dY, lddy, db, accumulate=0, stream=None, check=True)"),
    METHOD(BIAS_GRAD_WS, "axo_bias_grad_ws", "($module, p, dY, lddy, db, accumulate=0, ws=None, ws_bytes=0, stream=None, check=True)"),
    METHOD(BIAS_GRAD_STATIC, "axo_bias_grad_static", "($module, p, dY, lddy, db, accumulate=0, stream=None, check=True)"),
    {"set_up", set_up, METH_VARARGS, "set_up(Problem, wrappers, raise_if)"},
    {"bind", bind, METH_VARARGS, "bind(addresses, version)"},
    {NULL, NULL, 0, NULL},
};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", "Calls into libaxo.so without ctypes.", -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__calls(void) { return PyModule_Create(&module); }
