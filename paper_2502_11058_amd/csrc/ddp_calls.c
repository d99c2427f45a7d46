/* The per-iteration calls of the binding with their arguments marshalled in C: what a worker of a small model waits for is the
 * host time of its calls (2.7 us of it the launch).  Each function takes the arguments of the binding's method of that name, behind
 * the context's address, in the forms that programs pass every iteration: exact ints, objects with data_ptr(), a host array of
 * pointers or a list or tuple of tensors, a stream handle, an object with cuda_stream, or None for torch's current stream.  It
 * returns the library's status, or None where an argument has any other form; the binding then takes its general path, which
 * accepts or refuses it.  Nothing is kept from one call for the next. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "dreamddp.h"

/* given once by the binding: the library's entry points, and the Python objects that arguments are told by */
static struct {
    int (*pack)(ddp_ctx *, int, float *, void *);
    int (*unpack)(ddp_ctx *, int, const float *, void *);
    int (*pack16)(ddp_ctx *, int, uint16_t *, void *);
    int (*average)(ddp_ctx *, int, const float *, const float *const *, int, int, float *, double *, void *);
    int (*average16)(ddp_ctx *, int, const uint16_t *, const uint16_t *const *, int, int, float *, double *, void *);
    int (*update)(ddp_ctx *, const ddp_opt *, void *);
    int (*update_layers)(ddp_ctx *, int, int, const ddp_opt *, void *);
    int (*fused)(ddp_ctx *, int, const float *const *, int, int, double *, const ddp_opt *, void *);
    int (*fused16)(ddp_ctx *, int, const uint16_t *const *, int, int, double *, const ddp_opt *, void *);
    int (*fused_layers)(ddp_ctx *, int, int, int, const void *const *, int, int, int, int, double *, const ddp_opt *, void *);
} lib;
static PyObject *array_type, *opt_type;                /* ctypes.Array, the binding's ddp_opt */
static PyObject *bad_fork, *get_device, *raw_stream;   /* torch's raw queries of the current stream */
static PyObject *s_data_ptr, *s_cuda_stream;

/* Each returns 1, or 0 for a form it does not take, without an exception, and where the argument's own code raised one, with it:
 * arguments are looked at in the order of the general path, which would raise the same.  Then the call returns general(). */
static int no(void) {
    PyErr_Clear();
    return 0;
}
static PyObject *general(void) {
    if (PyErr_Occurred()) return NULL;
    Py_RETURN_NONE;
}
static int get_int(PyObject *o, int *out) {
    int over;
    long v;
    if (!PyLong_CheckExact(o)) return 0;
    v = PyLong_AsLongAndOverflow(o, &over);
    if (over || v < INT32_MIN || v > INT32_MAX) return 0;
    *out = (int)v;
    return 1;
}
static int get_address(PyObject *o, void **out) { /* an exact int; a new reference is not taken */
    if (!o || !PyLong_CheckExact(o)) return 0;
    *out = PyLong_AsVoidPtr(o);
    return *out || !PyErr_Occurred() ? 1 : no();
}
static int get_tensor(PyObject *o, void **out) {
    PyObject *p = PyObject_CallMethodNoArgs(o, s_data_ptr);
    int ok = get_address(p, out);
    Py_XDECREF(p);
    return ok;
}
static int get_optional(PyObject *o, void **out) {
    *out = NULL;
    return o == Py_None || get_tensor(o, out);
}
static int get_stream(PyObject *o, void **out) {
    PyObject *p, *dev;
    int ok;
    if (PyLong_Check(o)) return get_address(o, out);
    if (o == Py_None) {
        if (!raw_stream) return 0;
        p = PyObject_CallNoArgs(bad_fork);
        ok = p == Py_False;
        Py_XDECREF(p);
        if (!ok) return 0;
        if (!(dev = PyObject_CallNoArgs(get_device))) return 0;
        p = PyObject_CallOneArg(raw_stream, dev);
        Py_DECREF(dev);
    } else {
        p = PyObject_GetAttr(o, s_cuda_stream);
    }
    ok = get_address(p, out);
    Py_XDECREF(p);
    return ok;
}

typedef struct {
    void *own[DDP_MAX_REPLICAS];
    Py_buffer view;
    void *at;
} Peers;
static void peers_done(Peers *p) {
    if (p->view.obj) PyBuffer_Release(&p->view);
}
/* The library reads N - 1 pointers: those that a list leaves out are null, which it refuses; a shorter array is not taken. */
static int get_peers(PyObject *o, int N, Peers *p) {
    const int need = N > 1 && N <= DDP_MAX_REPLICAS ? N - 1 : 0;  /* (more replicas are refused before any peer is looked at) */
    p->view.obj = NULL;
    p->at = NULL;
    if (o == Py_None) return 1;
    if (PyList_CheckExact(o) || PyTuple_CheckExact(o)) {
        Py_ssize_t n = PySequence_Fast_GET_SIZE(o), i;
        if (n > DDP_MAX_REPLICAS) return 0;
        for (i = 0; i < n && i < PySequence_Fast_GET_SIZE(o); ++i) {  /* (data_ptr is the caller's code: the list may change) */
            PyObject *x = PySequence_Fast_GET_ITEM(o, i);
            int ok;
            Py_INCREF(x);
            p->own[i] = NULL;
            ok = x == Py_None || (PyLong_Check(x) ? get_address(x, &p->own[i]) : get_tensor(x, &p->own[i]));
            Py_DECREF(x);
            if (!ok) return 0;
        }
        if (i < n) return 0;
        for (; i < need; ++i) p->own[i] = NULL;
        if (n) p->at = p->own;
        return 1;
    }
    if (PyObject_IsInstance(o, array_type) != 1 || PyObject_GetBuffer(o, &p->view, PyBUF_SIMPLE) != 0) {
        p->view.obj = NULL;
        return no();
    }
    if (p->view.len && p->view.len < need * (Py_ssize_t)sizeof(void *)) {
        peers_done(p);
        return 0;
    }
    if (p->view.len) p->at = p->view.buf;
    return 1;
}
static void opt_done(Py_buffer *view) {
    if (view->obj) PyBuffer_Release(view);
}
static int get_opt(PyObject *o, Py_buffer *view) {
    view->obj = NULL;
    if ((PyObject *)Py_TYPE(o) != opt_type) return 0;
    if (PyObject_GetBuffer(o, view, PyBUF_SIMPLE) != 0 || view->len < (Py_ssize_t)sizeof(ddp_opt)) {
        opt_done(view);
        view->obj = NULL;
        return no();
    }
    return 1;
}

#define CALL(expr)              \
    do {                        \
        Py_BEGIN_ALLOW_THREADS; \
        rc = (expr);            \
        Py_END_ALLOW_THREADS;   \
    } while (0)
#define CTX ((ddp_ctx *)ctx)
#define FN(name) static PyObject *name(PyObject *self, PyObject *const *a, Py_ssize_t n)

/* (ctx, slot, buffer, stream) */
#define COPY_CALL(name, type)                                                                                                   \
    FN(name) {                                                                                                                  \
        void *ctx, *buf, *stream;                                                                                               \
        int slot, rc;                                                                                                           \
        (void)self;                                                                                                             \
        if (!lib.name || n != 4 || !get_address(a[0], &ctx) || !get_int(a[1], &slot) || !get_tensor(a[2], &buf) || !get_stream(a[3], &stream)) \
            return general();                                                                                                   \
        CALL(lib.name(CTX, slot, (type)buf, stream));                                                                           \
        return PyLong_FromLong(rc);                                                                                             \
    }
COPY_CALL(pack, float *)
COPY_CALL(unpack, const float *)
COPY_CALL(pack16, uint16_t *)

/* (ctx, slot, flat_local, peers, N, local_rank, flat_out, layer_stats, stream) */
#define AVERAGE_CALL(name, type)                                                                                                \
    FN(name) {                                                                                                                  \
        void *ctx, *local, *out, *stats, *stream;                                                                               \
        int slot, N, rank, rc;                                                                                                  \
        Peers p;                                                                                                                \
        (void)self;                                                                                                             \
        if (!lib.name || n != 9 || !get_int(a[4], &N) || !get_peers(a[3], N, &p)) return general();                             \
        if (!get_address(a[0], &ctx) || !get_int(a[1], &slot) || !get_int(a[5], &rank) || !get_tensor(a[2], &local) ||          \
            !get_tensor(a[6], &out) || !get_optional(a[7], &stats) || !get_stream(a[8], &stream)) {                             \
            peers_done(&p);                                                                                                     \
            return general();                                                                                                   \
        }                                                                                                                       \
        CALL(lib.name(CTX, slot, (const type *)local, (const type *const *)p.at, N, rank, (float *)out, (double *)stats, stream)); \
        peers_done(&p);                                                                                                         \
        return PyLong_FromLong(rc);                                                                                             \
    }
AVERAGE_CALL(average, float)
AVERAGE_CALL(average16, uint16_t)

/* (ctx, opt, stream) and (ctx, layer_first, layer_count, opt, stream) */
FN(update) {
    void *ctx, *stream;
    Py_buffer opt;
    int rc;
    (void)self;
    if (!lib.update || n != 3 || !get_address(a[0], &ctx) || !get_opt(a[1], &opt)) return general();
    if (!get_stream(a[2], &stream)) {
        opt_done(&opt);
        return general();
    }
    CALL(lib.update(CTX, (const ddp_opt *)opt.buf, stream));
    opt_done(&opt);
    return PyLong_FromLong(rc);
}
FN(update_layers) {
    void *ctx, *stream;
    Py_buffer opt;
    int first, count, rc;
    (void)self;
    if (!lib.update_layers || n != 5 || !get_address(a[0], &ctx) || !get_int(a[1], &first) || !get_int(a[2], &count) || !get_opt(a[3], &opt))
        return general();
    if (!get_stream(a[4], &stream)) {
        opt_done(&opt);
        return general();
    }
    CALL(lib.update_layers(CTX, first, count, (const ddp_opt *)opt.buf, stream));
    opt_done(&opt);
    return PyLong_FromLong(rc);
}

/* (ctx, slot, peers, N, local_rank, layer_stats, opt, stream) */
#define FUSED_CALL(name, type)                                                                                           \
    FN(name) {                                                                                                           \
        void *ctx, *stats, *stream;                                                                                      \
        int slot, N, rank, rc;                                                                                           \
        Py_buffer opt;                                                                                                   \
        Peers p;                                                                                                         \
        (void)self;                                                                                                      \
        opt.obj = NULL;                                                                                                  \
        if (!lib.name || n != 8 || !get_int(a[3], &N) || !get_peers(a[2], N, &p)) return general();                      \
        if (!get_address(a[0], &ctx) || !get_int(a[1], &slot) || !get_int(a[4], &rank) || !get_optional(a[5], &stats) || \
            !get_opt(a[6], &opt) || !get_stream(a[7], &stream)) {                                                        \
            opt_done(&opt);                                                                                               \
            peers_done(&p);                                                                                               \
            return general();                                                                                             \
        }                                                                                                                 \
        CALL(lib.name(CTX, slot, (const type *const *)p.at, N, rank, (double *)stats, (const ddp_opt *)opt.buf, stream)); \
        opt_done(&opt);                                                                                                   \
        peers_done(&p);                                                                                                   \
        return PyLong_FromLong(rc);                                                                                       \
    }
FUSED_CALL(fused, float)
FUSED_CALL(fused16, uint16_t)

/* (ctx, slot, layer_first, layer_count, peers, wire_dtype, order, N, local_rank, layer_stats, opt, stream) */
FN(fused_layers) {
    void *ctx, *stats, *stream;
    int v[3], w[4], rc, i, ok = 1;
    Py_buffer opt;
    Peers p;
    (void)self;
    opt.obj = NULL;
    if (!lib.fused_layers || n != 12) return general();
    for (i = 0; i < 3 && ok; ++i) ok = get_int(a[1 + i], &v[i]);
    for (i = 0; i < 4 && ok; ++i) ok = get_int(a[5 + i], &w[i]);
    if (!ok || !get_peers(a[4], w[2], &p)) return general();
    if (!get_address(a[0], &ctx) || !get_optional(a[9], &stats) || !get_opt(a[10], &opt) || !get_stream(a[11], &stream)) {
        opt_done(&opt);
        peers_done(&p);
        return general();
    }
    CALL(lib.fused_layers(CTX, v[0], v[1], v[2], (const void *const *)p.at, w[0], w[1], w[2], w[3], (double *)stats, (const ddp_opt *)opt.buf, stream));
    opt_done(&opt);
    peers_done(&p);
    return PyLong_FromLong(rc);
}

/* setup(addresses of the ten entry points in the order of `lib`, ctypes.Array, ddp_opt) */
FN(setup) {
    void *f[10];
    int i;
    (void)self;
    if (n != 3 || !PyTuple_CheckExact(a[0]) || PyTuple_GET_SIZE(a[0]) != 10) return PyErr_Format(PyExc_TypeError, "setup(addresses, array type, options type)");
    for (i = 0; i < 10; ++i)
        if (!get_address(PyTuple_GET_ITEM(a[0], i), &f[i])) return PyErr_Format(PyExc_TypeError, "setup: an address is not an int");
    memcpy(&lib, f, sizeof lib);
    Py_INCREF(a[1]);
    Py_XSETREF(array_type, a[1]);
    Py_INCREF(a[2]);
    Py_XSETREF(opt_type, a[2]);
    Py_RETURN_NONE;
}
/* set_stream_query(is bad fork, current device, raw handle of a device's current stream), or three times None: not known (again) */
FN(set_stream_query) {
    (void)self;
    if (n != 3) return PyErr_Format(PyExc_TypeError, "set_stream_query takes three callables");
    if (a[2] == Py_None) {
        Py_CLEAR(bad_fork);
        Py_CLEAR(get_device);
        Py_CLEAR(raw_stream);
        Py_RETURN_NONE;
    }
    Py_INCREF(a[0]);
    Py_XSETREF(bad_fork, a[0]);
    Py_INCREF(a[1]);
    Py_XSETREF(get_device, a[1]);
    Py_INCREF(a[2]);
    Py_XSETREF(raw_stream, a[2]);
    Py_RETURN_NONE;
}

#define DEF(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, NULL}
static PyMethodDef methods[] = {DEF(pack), DEF(unpack), DEF(pack16), DEF(average), DEF(average16), DEF(update), DEF(update_layers), DEF(fused), DEF(fused16),
                                DEF(fused_layers), DEF(setup), DEF(set_stream_query), {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__calls(void) {
    _Static_assert(sizeof lib == 10 * sizeof(void *), "ten entry points");
    if (!(s_data_ptr = PyUnicode_InternFromString("data_ptr")) || !(s_cuda_stream = PyUnicode_InternFromString("cuda_stream"))) return NULL;
    return PyModule_Create(&module);
}
