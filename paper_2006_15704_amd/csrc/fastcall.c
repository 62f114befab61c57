/* CPython marshalling for the calls that a backward pass makes once per
 * parameter (Algorithm 1's autograd_hook fires per gradient), ddp_mark_ready,
 * ddp_mark_ready_local, ddp_finalize_backward, and for those that take a list with
 * an entry per parameter or per tensor, ddp_mark_ready_many,
 * ddp_no_sync_accumulate, ddp_sync_static.  Through ctypes such a call costs
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
typedef int32_t (*many_fn)(void*, const int32_t*, int32_t);
typedef int32_t (*accumulate_fn)(void*, void* const*);
typedef int32_t (*static_fn)(int32_t, int32_t, void*, int32_t, const int64_t*, const int32_t*, void* const*, uint64_t);

static mark_fn g_mark = NULL;
static mark_local_fn g_mark_local = NULL;
static finalize_fn g_finalize = NULL;
static many_fn g_many = NULL;
static accumulate_fn g_accumulate = NULL;
static static_fn g_static = NULL;
static PyObject* g_c_int32 = NULL;      /* ctypes.c_int32 */

/* bind(mark_ready, finalize_backward, mark_ready_local, c_int32[, mark_ready_many, no_sync_accumulate, sync_static]):
 * the addresses of the C entry points */
static PyObject* bind_entry_points(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
    if ((nargs != 4 && nargs != 7) || !PyType_Check(args[3])) {
        PyErr_SetString(PyExc_TypeError, "bind(mark_ready, finalize_backward, mark_ready_local, c_int32[, mark_ready_many, no_sync_accumulate, sync_static])");
        return NULL;
    }
    void* a[7] = {NULL, NULL, NULL, NULL, NULL, NULL, NULL};
    for (Py_ssize_t i = 0; i < nargs; ++i) {
        if (i == 3) continue;
        a[i] = PyLong_AsVoidPtr(args[i]);
        if (a[i] == NULL && PyErr_Occurred()) return NULL;
    }
    Py_INCREF(args[3]);
    Py_XDECREF(g_c_int32);
    g_c_int32 = args[3];
    g_mark = (mark_fn)a[0];
    g_finalize = (finalize_fn)a[1];
    g_mark_local = (mark_local_fn)a[2];
    g_many = (many_fn)a[4];
    g_accumulate = (accumulate_fn)a[5];
    g_static = (static_fn)a[6];
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

/* Bits per digit of an int's magnitude in this interpreter, 0 = not known here.  (From 3.11 on the layout comes with Python.h, and
 * there is no header of this name; 3.12 has another layout.) */
#if PY_VERSION_HEX < 0x030B0000
#include <longintrepr.h>
#endif
#if PY_VERSION_HEX < 0x030C0000
#define DIGIT_BITS PyLong_SHIFT
#else
#define DIGIT_BITS 0
#endif

/* The value of an int that is not negative and takes at most two digits (60 bits: every address and size); 0: it is
 * another one.  The interpreter's own conversion checks and copies byte by byte: 1632 pointers in a list took 29 us,
 * 3.3 so (on the CPU of the build machine). */
static inline int small_value(PyObject* o, uint64_t* v) {
#if DIGIT_BITS
    const Py_ssize_t size = Py_SIZE(o);
    const digit* const d = ((PyLongObject*)o)->ob_digit;
    if (size < 0 || size > 2) return 0;
    *v = size == 0 ? 0 : size == 1 ? (uint64_t)d[0] : (uint64_t)d[0] | (uint64_t)d[1] << DIGIT_BITS;
    return 1;
#else
    (void)o;
    (void)v;
    return 0;
#endif
}

/* A list or tuple of plain ints as a C array of `size`-byte elements (8: unsigned when `pointers`, else signed; 4: signed);
 * pointers may be None (NULL).  Returns the array, or NULL without an exception where the sequence is anything
 * else or a value does not fit: the caller then converts it as before, with numpy, which also has the errors.
 * No Python code runs meanwhile, so the sequence stays as it is. */
static void* plain_ints(PyObject* seq, size_t size, int pointers, Py_ssize_t* count) {
    const int list = PyList_CheckExact(seq);
    if (!list && !PyTuple_CheckExact(seq)) return NULL;
    const Py_ssize_t n = list ? PyList_GET_SIZE(seq) : PyTuple_GET_SIZE(seq);
    char* out = (char*)PyMem_RawMalloc((size_t)(n > 0 ? n : 1) * size);
    if (out == NULL) return NULL;
    for (Py_ssize_t i = 0; i < n; ++i) {
        PyObject* o = list ? PyList_GET_ITEM(seq, i) : PyTuple_GET_ITEM(seq, i);
        int ok = PyLong_CheckExact(o);
        uint64_t small;
        if (ok && small_value(o, &small) && (size == 8 || small <= INT32_MAX)) {
            if (size == 8) ((uint64_t*)out)[i] = small;
            else ((int32_t*)out)[i] = (int32_t)small;
            continue;
        }
        if (pointers) {
            uint64_t v = 0;
            if (ok) {
                v = PyLong_AsUnsignedLongLong(o);
                ok = !(v == (uint64_t)-1 && PyErr_Occurred());
            } else {
                ok = o == Py_None;
            }
            ((uint64_t*)out)[i] = v;
        } else if (ok) {
            int over = 0;
            const long long v = PyLong_AsLongLongAndOverflow(o, &over);
            ok = !over && (size == 8 || (v >= INT32_MIN && v <= INT32_MAX));
            if (size == 8) ((int64_t*)out)[i] = v;
            else ((int32_t*)out)[i] = (int32_t)v;
        }
        if (!ok) {
            PyErr_Clear();
            PyMem_RawFree(out);
            return NULL;
        }
    }
    *count = n;
    return out;
}

static int plain_int(PyObject* o, long long lo, long long hi, long long* v) {
    if (!PyLong_CheckExact(o)) return 0;
    int over = 0;
    *v = PyLong_AsLongLongAndOverflow(o, &over);
    return !over && *v >= lo && *v <= hi;
}

/* mark_ready_many(ctx_address, ids) -> status, or None: the caller converts the arguments itself.
 * (130 ids in a list, a whole synchronization of 1.5 million elements, R = 2: 8.6 us through numpy and ctypes, 5.8 so.) */
static PyObject* mark_ready_many(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
    if (nargs != 2 || g_many == NULL) {
        PyErr_SetString(PyExc_TypeError, "mark_ready_many(ctx_address, ids) after bind()");
        return NULL;
    }
    Py_ssize_t n = 0;
    if (!PyLong_CheckExact(args[0])) Py_RETURN_NONE;
    int32_t* ids = (int32_t*)plain_ints(args[1], 4, 0, &n);
    if (ids == NULL || n > INT32_MAX) {
        PyMem_RawFree(ids);
        Py_RETURN_NONE;
    }
    void* ctx = PyLong_AsVoidPtr(args[0]);
    int32_t status;
    Py_BEGIN_ALLOW_THREADS
    status = g_many(ctx, ids, (int32_t)n);
    Py_END_ALLOW_THREADS
    PyMem_RawFree(ids);
    return PyLong_FromLong((long)status);
}

/* no_sync_accumulate(ctx_address, pointers, need) -> status or None, as above; a list of fewer than `need` pointers, which the
 * library would read, is left to the caller too.
 * (1170 pointers: 50 us a call through numpy and ctypes, 22 so, 9 since small_value.) */
static PyObject* no_sync_accumulate(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
    if (nargs != 3 || g_accumulate == NULL) {
        PyErr_SetString(PyExc_TypeError, "no_sync_accumulate(ctx_address, pointers, need) after bind()");
        return NULL;
    }
    Py_ssize_t n = 0;
    const Py_ssize_t need = PyLong_AsSsize_t(args[2]);
    if (need == -1 && PyErr_Occurred()) return NULL;
    if (!PyLong_CheckExact(args[0])) Py_RETURN_NONE;
    void** ptrs = (void**)plain_ints(args[1], 8, 1, &n);
    if (ptrs == NULL || n < need) {
        PyMem_RawFree(ptrs);
        Py_RETURN_NONE;
    }
    void* ctx = PyLong_AsVoidPtr(args[0]);
    int32_t status;
    Py_BEGIN_ALLOW_THREADS
    status = g_accumulate(ctx, ptrs);
    Py_END_ALLOW_THREADS
    PyMem_RawFree(ptrs);
    return PyLong_FromLong((long)status);
}

/* sync_static(R, device, stream, numel, dtype, pointers, cap_bytes) -> status or None, as above.
 * (48 tensors, R = 4: 25 us a call through numpy and ctypes, 15 so; 7.3 with the tables in the launch's arguments, 5.5 since small_value.) */
static PyObject* sync_static(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
    if (nargs != 7 || g_static == NULL) {
        PyErr_SetString(PyExc_TypeError, "sync_static(R, device, stream, numel, dtype, pointers, cap_bytes) after bind()");
        return NULL;
    }
    long long R, device;
    if (!plain_int(args[0], 0, INT32_MAX, &R) || !plain_int(args[1], INT32_MIN, INT32_MAX, &device) ||
        !PyLong_CheckExact(args[2]) || !PyLong_CheckExact(args[6])) Py_RETURN_NONE;
    const unsigned long long stream = PyLong_AsUnsignedLongLong(args[2]);
    const unsigned long long cap = PyErr_Occurred() ? 0 : PyLong_AsUnsignedLongLong(args[6]);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    Py_ssize_t n = 0, nd = 0, np = 0;
    int64_t* numel = (int64_t*)plain_ints(args[3], 8, 0, &n);
    int32_t* dtype = numel != NULL ? (int32_t*)plain_ints(args[4], 4, 0, &nd) : NULL;
    void** ptrs = dtype != NULL ? (void**)plain_ints(args[5], 8, 1, &np) : NULL;
    int32_t status = 0;
    const int ok = ptrs != NULL && n <= INT32_MAX && nd == n && np == R * n;      /* the library reads n, n and R n entries */
    if (ok) {
        Py_BEGIN_ALLOW_THREADS
        status = g_static((int32_t)R, (int32_t)device, (void*)(uintptr_t)stream, (int32_t)n, numel, dtype, ptrs, cap);
        Py_END_ALLOW_THREADS
    }
    PyMem_RawFree(numel);
    PyMem_RawFree(dtype);
    PyMem_RawFree(ptrs);
    if (!ok) Py_RETURN_NONE;
    return PyLong_FromLong((long)status);
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
    {"mark_ready_many", (PyCFunction)(void (*)(void))mark_ready_many, METH_FASTCALL, "ddp_mark_ready_many"},
    {"no_sync_accumulate", (PyCFunction)(void (*)(void))no_sync_accumulate, METH_FASTCALL, "ddp_no_sync_accumulate"},
    {"sync_static", (PyCFunction)(void (*)(void))sync_static, METH_FASTCALL, "ddp_sync_static"},
    {"finalize_backward", (PyCFunction)(void (*)(void))finalize_backward, METH_FASTCALL, "ddp_finalize_backward"},
    {NULL, NULL, 0, NULL},
};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_ddp_fastcall", NULL, -1, methods};

PyMODINIT_FUNC PyInit__ddp_fastcall(void) { return PyModule_Create(&module); }
