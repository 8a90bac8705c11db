/* The launches a training program makes once per operator -- lagom_gemm, lagom_comm_kernel, lagom_comm_steps -- with their
 * arguments taken from Python objects here instead of one ctypes object per pointer.
 *
 * A HIP launch costs the host 2.4 us; through ctypes the arguments of a product cost 2.0 us more, those of an eight-source
 * gather 3.6 and those of a ring share of fourteen steps 33, which is what bounded every call whose kernel is shorter than that.
 *
 * The calls take what such a program passes: tensors (anything with data_ptr()) or ints as addresses, lists or tuples of them, ints
 * as sizes, a tuple, list or lagom_cfg as parameters, None, an int or an object with cuda_stream as the stream.  They return the library's code, or
 * None, having called nothing, for anything else: the caller then goes through ctypes, whose conversions and errors are the definition. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>
#include <string.h>
#include "lagom.h"

typedef int (*gemm_fn)(const void*, const void*, void*, int64_t, int64_t, int64_t, int, lagom_dtype, void*);
typedef int (*comm_fn)(lagom_op, lagom_dtype, const void* const*, int, void* const*, int, int64_t, const lagom_cfg*, void*);
typedef int (*steps_fn)(lagom_dtype, const lagom_comm_step*, int, int64_t, const lagom_cfg*, void*);
static gemm_fn gemm_call;
static comm_fn comm_call;
static steps_fn steps_call;
static PyObject *cfg_type, *data_ptr_name, *cuda_stream_name;

/* Each: 1 if the object is one of the above, else 0, with no exception set but what ends the program (KeyboardInterrupt and its like, from
 * an object's own code). */
static int take_int(PyObject* o, long long lo, long long hi, long long* out) {
    int overflow;
    if (!PyLong_Check(o)) return 0;
    *out = PyLong_AsLongLongAndOverflow(o, &overflow);
    return !overflow && *out >= lo && *out <= hi;
}
static int take_int32(PyObject* o, int* out) {
    long long v;
    if (!take_int(o, INT32_MIN, INT32_MAX, &v)) return 0;
    *out = (int)v;
    return 1;
}
static int take_int64(PyObject* o, int64_t* out) {
    long long v;
    if (!take_int(o, INT64_MIN, INT64_MAX, &v)) return 0;
    *out = v;
    return 1;
}
static int take_address(PyObject* o, void** out) {
    unsigned long long v;
    if (!PyLong_Check(o)) return 0;
    v = PyLong_AsUnsignedLongLong(o);
    if (v == (unsigned long long)-1 && PyErr_Occurred()) { PyErr_Clear(); return 0; }
    *out = (void*)(uintptr_t)v;
    return 1;
}
static int take_owned_address(PyObject* v, void** out) {         /* a new reference, or null with an exception */
    int ok;
    if (!v) {
        if (PyErr_ExceptionMatches(PyExc_Exception)) PyErr_Clear();
        return 0;
    }
    ok = take_address(v, out);
    Py_DECREF(v);
    return ok;
}
static int take_pointer(PyObject* o, void** out) {
    if (PyLong_CheckExact(o)) return take_address(o, out);
    return take_owned_address(PyObject_CallMethodNoArgs(o, data_ptr_name), out);
}
static int take_stream(PyObject* o, void** out) {
    if (o == Py_None) { *out = NULL; return 1; }
    if (PyLong_CheckExact(o)) return take_address(o, out);
    return take_owned_address(PyObject_GetAttr(o, cuda_stream_name), out);
}
static int take_cfg(PyObject* o, lagom_cfg* out) {
    if (PyTuple_CheckExact(o) || PyList_CheckExact(o)) {
        if (PySequence_Fast_GET_SIZE(o) < 3) return 0;
        return take_int32(PySequence_Fast_GET_ITEM(o, 0), &out->nc) && take_int32(PySequence_Fast_GET_ITEM(o, 1), &out->nt) &&
               take_int64(PySequence_Fast_GET_ITEM(o, 2), &out->chunk_bytes);
    }
    if ((PyObject*)Py_TYPE(o) == cfg_type) {
        Py_buffer view;
        int ok;
        if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE)) { PyErr_Clear(); return 0; }
        ok = view.len == (Py_ssize_t)sizeof *out;
        if (ok) memcpy(out, view.buf, sizeof *out);
        PyBuffer_Release(&view);
        return ok;
    }
    return 0;
}
/* `room` addresses at most (the library refuses more than LAGOM_MAX_SRCS of its own accord).  The list is read by index and its
 * length again each time: an object's data_ptr() is anybody's code. */
static int take_pointers(PyObject* o, void** out, int room, int* n) {
    Py_ssize_t i;
    if (!PyList_CheckExact(o) && !PyTuple_CheckExact(o)) return 0;
    for (i = 0; i < PySequence_Fast_GET_SIZE(o); ++i) {
        PyObject* item;
        int ok;
        if (i >= room) return 0;
        item = PySequence_Fast_GET_ITEM(o, i);
        Py_INCREF(item);
        ok = take_pointer(item, &out[i]);
        Py_DECREF(item);
        if (!ok) return 0;
    }
    *n = (int)i;
    return 1;
}

static PyObject* leave(void) {
    if (PyErr_Occurred()) return NULL;
    Py_RETURN_NONE;
}

static PyObject* gemm(PyObject* self, PyObject* const* a, Py_ssize_t n) {
    void *A, *B, *C, *stream;
    int64_t M, N, K;
    int nk, dt, rc;
    (void)self;
    if (n != 9 || !gemm_call) return leave();
    if (!take_pointer(a[0], &A) || !take_pointer(a[1], &B) || !take_pointer(a[2], &C) || !take_int64(a[3], &M) || !take_int64(a[4], &N) ||
        !take_int64(a[5], &K) || !take_int32(a[7], &dt) || !take_stream(a[8], &stream)) return leave();
    nk = PyObject_IsTrue(a[6]);
    if (nk < 0) return NULL;
    Py_BEGIN_ALLOW_THREADS
    rc = gemm_call(A, B, C, M, N, K, nk, (lagom_dtype)dt, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

#define ROOM 64
static PyObject* comm_kernel(PyObject* self, PyObject* const* a, Py_ssize_t n) {
    void *srcs[ROOM], *dsts[ROOM], *stream;
    int op, dt, nsrc, ndst, rc;
    int64_t count;
    lagom_cfg cfg;
    (void)self;
    if (n != 7 || !comm_call) return leave();
    if (!take_int32(a[0], &op) || !take_int32(a[1], &dt) || !take_pointers(a[2], srcs, ROOM, &nsrc) || !take_pointers(a[3], dsts, ROOM, &ndst) ||
        !take_int64(a[4], &count) || !take_cfg(a[5], &cfg) || !take_stream(a[6], &stream)) return leave();
    Py_BEGIN_ALLOW_THREADS
    rc = comm_call((lagom_op)op, (lagom_dtype)dt, (const void* const*)srcs, nsrc, dsts, ndst, count, &cfg, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

#define STEPS_ROOM 1024         /* addresses of all steps */
static PyObject* comm_steps(PyObject* self, PyObject* const* a, Py_ssize_t n) {
    void *ptr[STEPS_ROOM], *stream;
    lagom_comm_step steps[ROOM];
    int dt, rc, used = 0, nsteps = 0;
    int64_t count;
    lagom_cfg cfg;
    (void)self;
    if (n != 5 || !steps_call) return leave();
    if (!take_int32(a[0], &dt) || (!PyList_CheckExact(a[1]) && !PyTuple_CheckExact(a[1]))) return leave();
    for (; nsteps < PySequence_Fast_GET_SIZE(a[1]); ++nsteps) {
        PyObject* s;
        lagom_comm_step* t = &steps[nsteps];
        int op = 0, ok;
        if (nsteps >= ROOM) return leave();
        s = PySequence_Fast_GET_ITEM(a[1], nsteps);
        if (!PyTuple_CheckExact(s) || PyTuple_GET_SIZE(s) != 3) return leave();
        Py_INCREF(s);
        ok = take_int32(PyTuple_GET_ITEM(s, 0), &op);
        t->op = op;
        t->srcs = (const void* const*)&ptr[used];
        ok = ok && take_pointers(PyTuple_GET_ITEM(s, 1), &ptr[used], STEPS_ROOM - used, &t->nsrc);
        if (ok) used += t->nsrc;
        t->dsts = &ptr[used];
        ok = ok && take_pointers(PyTuple_GET_ITEM(s, 2), &ptr[used], STEPS_ROOM - used, &t->ndst);
        if (ok) used += t->ndst;
        Py_DECREF(s);
        if (!ok) return leave();
    }
    if (!take_int64(a[2], &count) || !take_cfg(a[3], &cfg) || !take_stream(a[4], &stream)) return leave();
    Py_BEGIN_ALLOW_THREADS
    rc = steps_call((lagom_dtype)dt, steps, nsteps, count, &cfg, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

/* bind(lagom_gemm, lagom_comm_kernel, lagom_comm_steps, lagom_cfg): the loaded library's functions, as addresses, and the ctypes
 * structure that a configuration may be */
static PyObject* bind(PyObject* self, PyObject* const* a, Py_ssize_t n) {
    void* fn[3];
    int i;
    (void)self;
    if (n != 4) { PyErr_SetString(PyExc_TypeError, "bind() takes three addresses and a type"); return NULL; }
    for (i = 0; i < 3; ++i)
        if (!take_address(a[i], &fn[i])) { PyErr_SetString(PyExc_TypeError, "an address is an int"); return NULL; }
    gemm_call = (gemm_fn)fn[0];
    comm_call = (comm_fn)fn[1];
    steps_call = (steps_fn)fn[2];
    Py_INCREF(a[3]);
    Py_XSETREF(cfg_type, a[3]);
    Py_RETURN_NONE;
}

static PyMethodDef methods[] = {
    {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, NULL},
    {"gemm", (PyCFunction)(void (*)(void))gemm, METH_FASTCALL, NULL},
    {"comm_kernel", (PyCFunction)(void (*)(void))comm_kernel, METH_FASTCALL, NULL},
    {"comm_steps", (PyCFunction)(void (*)(void))comm_steps, METH_FASTCALL, NULL},
    {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__marshal(void) {
    data_ptr_name = PyUnicode_InternFromString("data_ptr");
    cuda_stream_name = PyUnicode_InternFromString("cuda_stream");
    if (!data_ptr_name || !cuda_stream_name) return NULL;
    return PyModule_Create(&module);
}
