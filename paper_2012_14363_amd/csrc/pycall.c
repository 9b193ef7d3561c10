/*
 * pycall.c - the Python side of the pack/unpack calls as a CPython extension: turns arguments into
 * the C types of include/tp_pack.h, calls the library and returns the new position.
 *
 * What bounds a small request is the host's time until its kernel is on the queue.  Of the 7.9 us an
 * enqueue-only call took from Python, 2.6 were torch.cuda.current_stream() (which builds a Stream
 * object) and 1.2 ctypes; here both together take 0.5 us.  Measured from Python, before -> now: an
 * enqueue-only call 7.9 -> 4.7 us, a synchronous pack of 512 bytes 15.4 -> 11.9 us, the two batched
 * calls of a 64^3 halo exchange 26.6 -> 19.9 us.  The library is loaded by binding.lib(), which hands
 * over the addresses of its entry points; nothing of the pack/unpack path lives here.
 *
 * The GIL is released while the library runs.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <pthread.h>
#include <stdint.h>

#include "tp_pack.h"

typedef int (*pack_fn)(const void *, int, tp_type, void *, int64_t, int64_t *, void *);
typedef int (*unpack_fn)(const void *, int64_t, int64_t *, void *, int, tp_type, void *);
typedef int (*pack_batch_fn)(int, const void *const *, const int *, const tp_type *, void *, int64_t, int64_t *, void *);
typedef int (*unpack_batch_fn)(int, const void *, int64_t, int64_t *, void *const *, const int *, const tp_type *, void *);
typedef int (*pack_host_fn)(const void *, int, tp_type, void *, int64_t, int64_t *, void *, int64_t, int, void *, int *);
typedef int (*unpack_host_fn)(const void *, int64_t, int64_t *, void *, int, tp_type, void *, int64_t, int, void *, int *);

enum { PACK, PACK_ASYNC, UNPACK, UNPACK_ASYNC, PACK_BATCH, PACK_BATCH_ASYNC, UNPACK_BATCH, UNPACK_BATCH_ASYNC, PACK_HOST,
       UNPACK_HOST, PACK_HOST_STATIC, ENTRIES };
static const char *const entry_names[ENTRIES] = {
    "tp_pack", "tp_pack_async", "tp_unpack", "tp_unpack_async", "tp_pack_batch", "tp_pack_batch_async", "tp_unpack_batch",
    "tp_unpack_batch_async", "tp_pack_host", "tp_unpack_host", "tp_pack_host_static"};
static void *entries[ENTRIES];   /* all NULL until setup() */

static PyObject *load_library, *raise_error;    /* binding.lib; raises TpError(code, where) */
static PyObject *plain_number, *marshal_batch;  /* binding._scalar, binding._marshal */
static PyObject *first_stream, *get_device, *get_stream;
static int torch_ready;                         /* torch's GPU state exists in this process */
static PyObject *s_data_ptr, *s_cuda_stream, *s_raw;

static void forget_torch(void) { torch_ready = 0; }   /* a forked child has to ask torch anew */

static int ready(void) {
    if (entries[0]) return 1;
    if (!load_library) {
        PyErr_SetString(PyExc_RuntimeError, "binding.lib() has not been set");
        return 0;
    }
    PyObject *r = PyObject_CallNoArgs(load_library);
    if (!r) return 0;
    Py_DECREF(r);
    if (!entries[0]) PyErr_SetString(PyExc_RuntimeError, "the library's entry points are not known");
    return entries[0] != NULL;
}

/* Whole numbers wrap into the C type, as ctypes has it. */
static int as_i64(PyObject *o, int64_t *v) {
    const unsigned long long u = PyLong_AsUnsignedLongLongMask(o);
    if (u == (unsigned long long)-1 && PyErr_Occurred()) return 0;
    *v = (int64_t)u;
    return 1;
}

/* An argument of the C call: a whole number, or the ctypes object that stands for one (wide: c_int64, else c_int). */
static int as_argument(PyObject *o, int wide, int64_t *v) {
    if (PyIndex_Check(o)) return as_i64(o, v);
    PyObject *r = PyObject_CallFunction(plain_number, "Oi", o, wide);
    if (!r) return 0;
    const int ok = as_i64(r, v);
    Py_DECREF(r);
    return ok;
}

static int as_int(PyObject *o, int *v) {
    int64_t w;
    if (!as_argument(o, 0, &w)) return 0;
    *v = (int)(uint32_t)(uint64_t)w;
    return 1;
}

static int as_size(PyObject *o, int64_t *v) { return as_argument(o, 1, v); }

/* A raw address, or anything with data_ptr(). */
static int as_address(PyObject *o, void **p) {
    int64_t v;
    if (PyLong_Check(o)) {
        if (!as_i64(o, &v)) return 0;
    } else {
        PyObject *r = PyObject_CallMethodNoArgs(o, s_data_ptr);
        if (!r) return 0;
        const int ok = as_i64(r, &v);
        Py_DECREF(r);
        if (!ok) return 0;
    }
    *p = (void *)(uintptr_t)v;
    return 1;
}

/* None: the current stream of the current device; a raw handle; or anything with .cuda_stream. */
static int as_stream(PyObject *o, void **stream) {
    int64_t v = 0;
    PyObject *r;
    if (o == NULL || o == Py_None) {
        if (!torch_ready) {
            r = PyObject_CallNoArgs(first_stream);
            torch_ready = r != NULL;
        } else {
            PyObject *device = PyObject_CallNoArgs(get_device);
            if (!device) return 0;
            r = PyObject_CallOneArg(get_stream, device);
            Py_DECREF(device);
        }
    } else if (PyLong_Check(o)) {
        r = o;
        Py_INCREF(r);
    } else {
        r = PyObject_GetAttr(o, s_cuda_stream);
    }
    if (!r) return 0;
    const int ok = as_i64(r, &v);
    Py_DECREF(r);
    *stream = (void *)(uintptr_t)v;
    return ok;
}

static PyObject *outcome(int rc, int entry, int64_t position) {
    if (rc == TP_SUCCESS) return PyLong_FromLongLong(position);
    PyObject *r = PyObject_CallFunction(raise_error, "is", rc, entry_names[entry]);
    Py_XDECREF(r);
    return NULL;
}

/* Positional and keyword arguments of a call into out[0..n); the first `needed` must be given. */
static int collect(const char *name, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames, const char *const *names,
                   int n, int needed, PyObject **out) {
    if (nargs > n) {
        PyErr_Format(PyExc_TypeError, "%s() takes at most %d arguments (%zd given)", name, n, nargs);
        return 0;
    }
    for (int i = 0; i < n; ++i) out[i] = i < nargs ? args[i] : NULL;
    const Py_ssize_t nkw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    for (Py_ssize_t k = 0; k < nkw; ++k) {
        PyObject *key = PyTuple_GET_ITEM(kwnames, k);
        int i = 0;
        while (i < n && PyUnicode_CompareWithASCIIString(key, names[i]) != 0) ++i;
        if (i == n) {
            PyErr_Format(PyExc_TypeError, "%s() got an unexpected keyword argument '%U'", name, key);
            return 0;
        }
        if (out[i]) {
            PyErr_Format(PyExc_TypeError, "%s() got multiple values for argument '%s'", name, names[i]);
            return 0;
        }
        out[i] = args[nargs + k];
    }
    for (int i = 0; i < needed; ++i) {
        if (!out[i]) {
            PyErr_Format(PyExc_TypeError, "%s() missing required argument: '%s'", name, names[i]);
            return 0;
        }
    }
    return 1;
}

/* ---------------------------------------------------------------- one request */
static PyObject *pack_call(int entry, const char *name, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames) {
    static const char *const names[] = {"inbuf", "incount", "t", "outbuf", "outsize", "position", "stream"};
    PyObject *a[7];
    void *in, *out, *stream;
    int count, type, rc;
    int64_t size, position;
    if (!collect(name, args, nargs, kwnames, names, 7, 6, a) || !ready()) return NULL;
    if (!as_address(a[0], &in) || !as_int(a[1], &count) || !as_int(a[2], &type) || !as_address(a[3], &out) ||
        !as_size(a[4], &size) || !as_i64(a[5], &position) || !as_stream(a[6], &stream))
        return NULL;
    Py_BEGIN_ALLOW_THREADS
    rc = ((pack_fn)entries[entry])(in, count, type, out, size, &position, stream);
    Py_END_ALLOW_THREADS
    return outcome(rc, entry, position);
}

static PyObject *unpack_call(int entry, const char *name, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames) {
    static const char *const names[] = {"inbuf", "insize", "position", "outbuf", "outcount", "t", "stream"};
    PyObject *a[7];
    void *in, *out, *stream;
    int count, type, rc;
    int64_t size, position;
    if (!collect(name, args, nargs, kwnames, names, 7, 6, a) || !ready()) return NULL;
    if (!as_address(a[0], &in) || !as_size(a[1], &size) || !as_i64(a[2], &position) || !as_address(a[3], &out) ||
        !as_int(a[4], &count) || !as_int(a[5], &type) || !as_stream(a[6], &stream))
        return NULL;
    Py_BEGIN_ALLOW_THREADS
    rc = ((unpack_fn)entries[entry])(in, size, &position, out, count, type, stream);
    Py_END_ALLOW_THREADS
    return outcome(rc, entry, position);
}

/* ---------------------------------------------------------------- batches */
/* Batch.raw: (n, address of the pointers, of the counts, of the types, the objects these are of); None once one of
 * them has been replaced, and then made anew.  *held is the tuple, whose objects live as long as the caller keeps it. */
static int as_batch(PyObject *o, PyObject **held, int *n, void **ptrs, void **counts, void **types) {
    PyObject *raw = PyObject_GetAttr(o, s_raw);
    if (!raw) {
        if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return 0;
        PyErr_Clear();   /* another class with a Batch's attributes */
    }
    if (!raw || raw == Py_None) {
        Py_XDECREF(raw);
        raw = PyObject_CallOneArg(marshal_batch, o);
        if (!raw) return 0;
    }
    int ok = PyTuple_Check(raw) && PyTuple_GET_SIZE(raw) == 5;
    if (!ok) PyErr_SetString(PyExc_TypeError, "not a Batch");
    ok = ok && as_int(PyTuple_GET_ITEM(raw, 0), n) && as_address(PyTuple_GET_ITEM(raw, 1), ptrs) &&
         as_address(PyTuple_GET_ITEM(raw, 2), counts) && as_address(PyTuple_GET_ITEM(raw, 3), types);
    if (ok) *held = raw;
    else Py_DECREF(raw);
    return ok;
}

static PyObject *pack_batch_call(int entry, const char *name, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames) {
    static const char *const names[] = {"batch", "outbuf", "outsize", "position", "stream"};
    PyObject *a[5], *held;
    void *ptrs, *counts, *types, *out, *stream;
    int n, rc;
    int64_t size, position;
    if (!collect(name, args, nargs, kwnames, names, 5, 4, a) || !ready()) return NULL;
    if (!as_address(a[1], &out) || !as_size(a[2], &size) || !as_i64(a[3], &position) || !as_stream(a[4], &stream) ||
        !as_batch(a[0], &held, &n, &ptrs, &counts, &types))
        return NULL;
    Py_BEGIN_ALLOW_THREADS
    rc = ((pack_batch_fn)entries[entry])(n, ptrs, counts, types, out, size, &position, stream);
    Py_END_ALLOW_THREADS
    Py_DECREF(held);
    return outcome(rc, entry, position);
}

static PyObject *unpack_batch_call(int entry, const char *name, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames) {
    static const char *const names[] = {"inbuf", "insize", "position", "batch", "stream"};
    PyObject *a[5], *held;
    void *ptrs, *counts, *types, *in, *stream;
    int n, rc;
    int64_t size, position;
    if (!collect(name, args, nargs, kwnames, names, 5, 4, a) || !ready()) return NULL;
    if (!as_address(a[0], &in) || !as_size(a[1], &size) || !as_i64(a[2], &position) || !as_stream(a[4], &stream) ||
        !as_batch(a[3], &held, &n, &ptrs, &counts, &types))
        return NULL;
    Py_BEGIN_ALLOW_THREADS
    rc = ((unpack_batch_fn)entries[entry])(n, in, size, &position, ptrs, counts, types, stream);
    Py_END_ALLOW_THREADS
    Py_DECREF(held);
    return outcome(rc, entry, position);
}

/* ---------------------------------------------------------------- host delivery */
static PyObject *host_outcome(int rc, int entry, int64_t position, int used) {
    PyObject *p = outcome(rc, entry, position);
    return p ? Py_BuildValue("(Ni)", p, used) : NULL;
}

/* staging, staging_size, method, stream: the optional tail both host calls share */
static int as_host_tail(PyObject **a, void **staging, int64_t *staging_size, int *method, void **stream) {
    *staging = NULL;
    *staging_size = 0;
    *method = TP_METHOD_AUTO;
    return (!a[0] || a[0] == Py_None || as_address(a[0], staging)) && (!a[1] || as_size(a[1], staging_size)) &&
           (!a[2] || as_int(a[2], method)) && as_stream(a[3], stream);
}

static PyObject *py_pack_host(PyObject *self, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames) {
    static const char *const names[] = {"inbuf", "incount", "t", "host_outbuf", "outsize", "position", "staging", "staging_size",
                                        "method", "stream"};
    PyObject *a[10];
    void *in, *out, *staging, *stream;
    int count, type, method, used = -9, rc;
    int64_t size, position, staging_size;
    (void)self;
    if (!collect("pack_host", args, nargs, kwnames, names, 10, 6, a) || !ready()) return NULL;
    if (!as_address(a[0], &in) || !as_int(a[1], &count) || !as_int(a[2], &type) || !as_address(a[3], &out) ||
        !as_size(a[4], &size) || !as_i64(a[5], &position) || !as_host_tail(a + 6, &staging, &staging_size, &method, &stream))
        return NULL;
    Py_BEGIN_ALLOW_THREADS
    rc = ((pack_host_fn)entries[PACK_HOST])(in, count, type, out, size, &position, staging, staging_size, method, stream, &used);
    Py_END_ALLOW_THREADS
    return host_outcome(rc, PACK_HOST, position, used);
}

static PyObject *py_unpack_host(PyObject *self, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames) {
    static const char *const names[] = {"host_inbuf", "insize", "position", "outbuf", "outcount", "t", "staging", "staging_size",
                                        "method", "stream"};
    PyObject *a[10];
    void *in, *out, *staging, *stream;
    int count, type, method, used = -9, rc;
    int64_t size, position, staging_size;
    (void)self;
    if (!collect("unpack_host", args, nargs, kwnames, names, 10, 6, a) || !ready()) return NULL;
    if (!as_address(a[0], &in) || !as_size(a[1], &size) || !as_i64(a[2], &position) || !as_address(a[3], &out) ||
        !as_int(a[4], &count) || !as_int(a[5], &type) || !as_host_tail(a + 6, &staging, &staging_size, &method, &stream))
        return NULL;
    Py_BEGIN_ALLOW_THREADS
    rc = ((unpack_host_fn)entries[UNPACK_HOST])(in, size, &position, out, count, type, staging, staging_size, method, stream, &used);
    Py_END_ALLOW_THREADS
    return host_outcome(rc, UNPACK_HOST, position, used);
}

/* ---------------------------------------------------------------- module */
#define DEFINE_CALL(kind, entry, name)                                                                               \
    static PyObject *py_##name(PyObject *self, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames) {           \
        (void)self;                                                                                                   \
        return kind(entry, #name, args, nargs, kwnames);                                                              \
    }
DEFINE_CALL(pack_call, PACK, pack)
DEFINE_CALL(pack_call, PACK_ASYNC, pack_async)
DEFINE_CALL(unpack_call, UNPACK, unpack)
DEFINE_CALL(unpack_call, UNPACK_ASYNC, unpack_async)
DEFINE_CALL(pack_batch_call, PACK_BATCH, pack_batch)
DEFINE_CALL(pack_batch_call, PACK_BATCH_ASYNC, pack_batch_async)
DEFINE_CALL(unpack_batch_call, UNPACK_BATCH, unpack_batch)
DEFINE_CALL(unpack_batch_call, UNPACK_BATCH_ASYNC, unpack_batch_async)

static PyObject *py_pack_host_static(PyObject *self, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames) {
    static const char *const names[] = {"inbuf", "incount", "t", "host_outbuf", "outsize", "position", "stream"};
    PyObject *a[7];
    (void)self;
    if (!collect("pack_host_static", args, nargs, kwnames, names, 7, 6, a)) return NULL;
    return pack_call(PACK_HOST_STATIC, "pack_host_static", a, a[6] ? 7 : 6, NULL);   /* pack's arguments under another name */
}

/* setup(addresses, raise_error, scalar, marshal, first_stream, get_device, get_stream): called by binding.lib() */
static PyObject *py_setup(PyObject *self, PyObject *args) {
    PyObject *addresses, *err, *number, *batch, *first, *dev, *str;
    void *found[ENTRIES];
    (void)self;
    if (!PyArg_ParseTuple(args, "O!OOOOOO", &PyDict_Type, &addresses, &err, &number, &batch, &first, &dev, &str)) return NULL;
    for (int i = 0; i < ENTRIES; ++i) {
        PyObject *v = PyDict_GetItemString(addresses, entry_names[i]);
        if (!v) {
            PyErr_SetString(PyExc_KeyError, entry_names[i]);
            return NULL;
        }
        if (!as_address(v, &found[i])) return NULL;
    }
    Py_INCREF(err), Py_INCREF(number), Py_INCREF(batch), Py_INCREF(first), Py_INCREF(dev), Py_INCREF(str);
    Py_XDECREF(raise_error), Py_XDECREF(plain_number), Py_XDECREF(marshal_batch);
    Py_XDECREF(first_stream), Py_XDECREF(get_device), Py_XDECREF(get_stream);
    raise_error = err, plain_number = number, marshal_batch = batch, first_stream = first, get_device = dev, get_stream = str;
    torch_ready = 0;
    for (int i = 0; i < ENTRIES; ++i) entries[i] = found[i];
    Py_RETURN_NONE;
}

static PyObject *py_on_first_use(PyObject *self, PyObject *loader) {
    (void)self;
    Py_INCREF(loader);
    Py_XDECREF(load_library);
    load_library = loader;
    Py_RETURN_NONE;
}

#define FAST(name, doc) {#name, (PyCFunction)(void (*)(void))py_##name, METH_FASTCALL | METH_KEYWORDS, doc}
static PyMethodDef methods[] = {
    FAST(pack, "pack($module, inbuf, incount, t, outbuf, outsize, position, stream=None)\n--\n\n"
               "tp_pack; returns the new position."),
    FAST(pack_async, "pack_async($module, inbuf, incount, t, outbuf, outsize, position, stream=None)\n--\n\n"
                     "tp_pack_async (enqueue only); returns the new position."),
    FAST(unpack, "unpack($module, inbuf, insize, position, outbuf, outcount, t, stream=None)\n--\n\n"
                 "tp_unpack; returns the new position."),
    FAST(unpack_async, "unpack_async($module, inbuf, insize, position, outbuf, outcount, t, stream=None)\n--\n\n"
                       "tp_unpack_async (enqueue only); returns the new position."),
    FAST(pack_batch, "pack_batch($module, batch, outbuf, outsize, position, stream=None)\n--\n\n"
                     "tp_pack_batch; returns the new position."),
    FAST(pack_batch_async, "pack_batch_async($module, batch, outbuf, outsize, position, stream=None)\n--\n\n"
                           "tp_pack_batch_async (enqueue only); returns the new position."),
    FAST(unpack_batch, "unpack_batch($module, inbuf, insize, position, batch, stream=None)\n--\n\n"
                       "tp_unpack_batch; returns the new position."),
    FAST(unpack_batch_async, "unpack_batch_async($module, inbuf, insize, position, batch, stream=None)\n--\n\n"
                             "tp_unpack_batch_async (enqueue only); returns the new position."),
    FAST(pack_host, "pack_host($module, inbuf, incount, t, host_outbuf, outsize, position, staging=None, staging_size=0, "
                    "method=-1, stream=None)\n--\n\ntp_pack_host; returns (new position, method used)."),
    FAST(unpack_host, "unpack_host($module, host_inbuf, insize, position, outbuf, outcount, t, staging=None, staging_size=0, "
                      "method=-1, stream=None)\n--\n\ntp_unpack_host; returns (new position, method used)."),
    FAST(pack_host_static, "pack_host_static($module, inbuf, incount, t, host_outbuf, outsize, position, stream=None)\n--\n\n"
                           "tp_pack_host_static (staged through the library's fixed device array; allocates nothing); "
                           "returns the new position."),
    {"setup", py_setup, METH_VARARGS, "setup(addresses, raise_error, scalar, marshal, first_stream, get_device, get_stream)"},
    {"on_first_use", py_on_first_use, METH_O, "on_first_use(loader): what loads the library when the first call needs it"},
    {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pycall", "Argument marshalling of the pack/unpack calls.", -1, methods,
                                    NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__pycall(void) {
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    s_raw = PyUnicode_InternFromString("raw");
    if (!s_data_ptr || !s_cuda_stream || !s_raw) return NULL;
    pthread_atfork(NULL, NULL, forget_torch);
    return PyModule_Create(&module);
}
