/* CPython marshalling for the calls that a backward pass makes once per
 * parameter (Algorithm 1's autograd_hook fires per gradient): ddp_mark_ready,
 * ddp_mark_ready_local, ddp_finalize_backward.  Through ctypes such a call costs
 * about a microsecond of interpreter time, which for a model with hundreds of
 * parameters is as long as the synchronization itself; here it is an integer
 * conversion and an indirect call.  No arithmetic of the method happens here:
 * the functions receive the addresses of the library's C entry points from the
 * Python binding and pass their arguments through.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

typedef int32_t (*mark_fn)(void*, int32_t);
typedef int32_t (*mark_local_fn)(void*, int32_t, const uint8_t*);
typedef int32_t (*finalize_fn)(void*);

static mark_fn g_mark = NULL;
static mark_local_fn g_mark_local = NULL;
static finalize_fn g_finalize = NULL;
static PyObject* g_c_int32 = NULL;      /* ctypes.c_int32 */

static PyObject* bind_entry_points(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
    if (nargs != 4 || !PyType_Check(args[3])) {
        PyErr_SetString(PyExc_TypeError, "bind(mark_ready_address, finalize_backward_address, mark_ready_local_address, c_int32)");
        return NULL;
    }
    void* a = PyLong_AsVoidPtr(args[0]);
    if (a == NULL && PyErr_Occurred()) return NULL;
    void* b = PyLong_AsVoidPtr(args[1]);
    if (b == NULL && PyErr_Occurred()) return NULL;
    void* l = PyLong_AsVoidPtr(args[2]);
    if (l == NULL && PyErr_Occurred()) return NULL;
    Py_INCREF(args[3]);
    Py_XDECREF(g_c_int32);
    g_c_int32 = args[3];
    g_mark_local = (mark_local_fn)l;
    g_mark = (mark_fn)a;
    g_finalize = (finalize_fn)b;
    Py_RETURN_NONE;
}

/* mark_ready(ctx_address, param_id) -> status */
static PyObject* mark_ready(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
    if (nargs != 2 || g_mark == NULL) {
        PyErr_SetString(PyExc_TypeError, "mark_ready(ctx_address, param_id) after bind()");
        return NULL;
    }
    void* ctx = PyLong_AsVoidPtr(args[0]);
    if (ctx == NULL && PyErr_Occurred()) return NULL;
    const long p = PyLong_AsLong(args[1]);
    if (p == -1 && PyErr_Occurred()) return NULL;
    if (p < INT32_MIN || p > INT32_MAX) {
        PyErr_SetString(PyExc_OverflowError, "param_id does not fit int32");
        return NULL;
    }
    return PyLong_FromLong((long)g_mark(ctx, (int32_t)p));
}

/* A parameter id as a ctypes int32_t argument takes it: an int, whatever converts to one without loss
 * (__index__: numpy integers, one-element integer tensors) or a c_int32, modulo 2^32.  0 on success. */
static int param_id_of(PyObject* o, int32_t* id) {
    PyObject* v = PyLong_Check(o) ? (Py_INCREF(o), o)
                  : PyObject_TypeCheck(o, (PyTypeObject*)g_c_int32) ? PyObject_GetAttrString(o, "value")
                                                                    : PyNumber_Index(o);
    if (v == NULL) return -1;
    *id = (int32_t)PyLong_AsUnsignedLongMask(v);
    Py_DECREF(v);
    return 0;
}

/* mark_ready_local(ctx_address, param_id, flags, replicas) -> status.  ctx_address None = no context (the
 * library's own error).  replicas: dict, ctx_address -> R.  flags: any iterable of R truth values (of any
 * number for a context that is not in the dict).  As a numpy array through ctypes a call took 2.5 us, as
 * long for the 161 marks of ResNet-50 together as the bucket launches of an iteration; 0.29 us so. */
static PyObject* mark_ready_local(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
    if (nargs != 4 || !PyDict_Check(args[3]) || g_mark_local == NULL) {
        PyErr_SetString(PyExc_TypeError, "mark_ready_local(ctx_address, param_id, flags, replicas) after bind()");
        return NULL;
    }
    void* ctx = args[0] == Py_None ? NULL : PyLong_AsVoidPtr(args[0]);
    if (ctx == NULL && PyErr_Occurred()) return NULL;
    int32_t p;
    if (param_id_of(args[1], &p) != 0) return NULL;
    PyObject* replicas = PyDict_GetItemWithError(args[3], args[0]);
    const Py_ssize_t want = replicas != NULL ? PyLong_AsSsize_t(replicas) : -1;
    if (want == -1 && PyErr_Occurred()) return NULL;
    PyObject* seq = PySequence_Fast(args[2], "flags must be iterable");
    if (seq == NULL) return NULL;
    Py_ssize_t n = PySequence_Fast_GET_SIZE(seq);
    uint8_t few[64];
    uint8_t* used = n > 64 ? (uint8_t*)PyMem_Malloc((size_t)n) : few;
    if (used == NULL) {
        Py_DECREF(seq);
        return PyErr_NoMemory();
    }
    int ok = 1;
    /* (a truth value is asked for through Python code where an element has some: the list may change) */
    for (Py_ssize_t i = 0; ok && i < n; ++i) {
        if (i >= PySequence_Fast_GET_SIZE(seq)) { n = i; break; }
        PyObject* item = PySequence_Fast_GET_ITEM(seq, i);
        if (PyLong_CheckExact(item)) {
            used[i] = Py_SIZE(item) != 0;
            continue;
        }
        Py_INCREF(item);
        const int t = PyObject_IsTrue(item);
        Py_DECREF(item);
        if (t < 0) ok = 0;
        else used[i] = (uint8_t)t;
    }
    Py_DECREF(seq);
    if (ok && want >= 0 && n != want) {      /* the library reads exactly R bytes */
        PyErr_Format(PyExc_ValueError, "used has %zd flags, the context has %zd replicas", n, want);
        ok = 0;
    }
    int32_t status = 0;
    if (ok) {
        /* the call may wait for the GPU: other Python threads run meanwhile, as in a call through ctypes */
        Py_BEGIN_ALLOW_THREADS
        status = g_mark_local(ctx, p, used);
        Py_END_ALLOW_THREADS
    }
    if (used != few) PyMem_Free(used);
    return ok ? PyLong_FromLong((long)status) : NULL;
}

/* finalize_backward(ctx_address) -> status */
static PyObject* finalize_backward(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
    if (nargs != 1 || g_finalize == NULL) {
        PyErr_SetString(PyExc_TypeError, "finalize_backward(ctx_address) after bind()");
        return NULL;
    }
    void* ctx = PyLong_AsVoidPtr(args[0]);
    if (ctx == NULL && PyErr_Occurred()) return NULL;
    return PyLong_FromLong((long)g_finalize(ctx));
}

static PyMethodDef methods[] = {
    {"bind", (PyCFunction)(void (*)(void))bind_entry_points, METH_FASTCALL, "set the C entry points"},
    {"mark_ready", (PyCFunction)(void (*)(void))mark_ready, METH_FASTCALL, "ddp_mark_ready"},
    {"mark_ready_local", (PyCFunction)(void (*)(void))mark_ready_local, METH_FASTCALL, "ddp_mark_ready_local"},
    {"finalize_backward", (PyCFunction)(void (*)(void))finalize_backward, METH_FASTCALL, "ddp_finalize_backward"},
    {NULL, NULL, 0, NULL},
};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_ddp_fastcall", NULL, -1, methods};

PyMODINIT_FUNC PyInit__ddp_fastcall(void) { return PyModule_Create(&module); }
