/* The calls of the Python binding that a launch goes through (binding.py), against the C API of the Python interpreter.  Through ctypes they took
 * 4 to 12 us of host time each, most of it building argument arrays, around 0.4 to 1.4 us in the library: an encode 5.1 us and 2.4 here, a stack
 * of five 12 and 3, the whole call of a 32-layer step of 4 tokens 62 and 31 us, RoPE of 134 tokens 16.1 and 9.7.
 * Argument marshalling only; nothing is kept from one call for the next.  The library is the one that binding.py loaded (`bind` takes the addresses
 * of its functions).  A negative status of the library is returned as an int, for binding.py to raise. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>
#include <string.h>

#include "../../include/dvm.h"

#define ENC_CAP 8192

static PyObject *s_shape, *s_stride, *s_data_ptr, *s_untyped_storage, *s_nbytes, *s_storage_offset, *s_element_size, *s_numel, *s_value;

static struct {
    int (*encode)(const dvm_ctx *, const dvm_prog *, const dvm_shape *, int, const dvm_shape *, void *, size_t, size_t *, dvm_shape *);
    int (*stack)(const void *const *, const size_t *, int, void *, size_t, size_t *);
    int (*stack_spatial)(const void *const *, const size_t *, int, void *, size_t, size_t *);
    int (*run)(const dvm_ctx *, const void *, size_t, void *const *, int, void *);
    int (*run_batched)(const dvm_ctx *, const void *, size_t, void *const *, int, int, void *, size_t, void *);
    int (*min_bytes)(const void *, size_t, int64_t *, int);
    int (*info)(const void *, size_t, dvm_code_info *);
    int (*tensor)(const void *, size_t, int, int64_t *, int *, int *, int *);
} lib;

/* bind(encode, stack, stack_spatial, run, run_batched, code_min_bytes, code_info_get, code_tensor): addresses */
static PyObject *py_bind(PyObject *self, PyObject *const *a, Py_ssize_t na) {
    (void)self;
    void *p[8];
    if (na != 8) return PyErr_Format(PyExc_TypeError, "bind takes 8 addresses");
    for (int i = 0; i < 8; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (PyErr_Occurred()) return NULL;
    }
    memcpy(&lib, p, sizeof(lib));
    Py_RETURN_NONE;
}

/* An address: an int (or what counts as one), None for 0, or an object with a `value` (c_void_p). */
static int address_of(PyObject *o, void **out) {
    if (PyLong_Check(o)) {
        *out = (void *)(uintptr_t)PyLong_AsUnsignedLongLongMask(o);
    } else if (o == Py_None) {
        *out = NULL;
    } else {
        PyObject *v = PyIndex_Check(o) ? PyNumber_Index(o) : PyObject_GetAttr(o, s_value);
        if (!v) return -1;
        *out = v == Py_None ? NULL : (void *)(uintptr_t)PyLong_AsUnsignedLongLongMask(v);
        Py_DECREF(v);
    }
    return PyErr_Occurred() ? -1 : 0;
}

/* One dvm_shape from a torch tensor.  0, or -1 with an exception; *rank_error is set where the rank exceeds DVM_MAX_RANK. */
static int shape_from_tensor(PyObject *t, dvm_shape *s, int *rank_error) {
    int rc = -1;
    PyObject *dims = PyObject_GetAttr(t, s_shape), *strides = NULL, *ptr = NULL;
    if (!dims) goto done;
    strides = PyObject_CallMethodNoArgs(t, s_stride);
    if (!strides) goto done;
    ptr = PyObject_CallMethodNoArgs(t, s_data_ptr);
    if (!ptr) goto done;
    if (!PyTuple_Check(dims) || !PyTuple_Check(strides)) {
        PyErr_SetString(PyExc_TypeError, "shape and stride of a tensor");
        goto done;
    }
    const Py_ssize_t r = PyTuple_GET_SIZE(dims);
    if (r > DVM_MAX_RANK || PyTuple_GET_SIZE(strides) != r) {
        *rank_error = 1;
        rc = 0;
        goto done;
    }
    memset(s, 0, sizeof(*s));
    s->rank = (int32_t)r;
    for (Py_ssize_t k = 0; k < r; ++k) {
        s->dim[k] = PyLong_AsLongLong(PyTuple_GET_ITEM(dims, k));
        s->stride[k] = PyLong_AsLongLong(PyTuple_GET_ITEM(strides, k));
    }
    const unsigned long long p = PyLong_AsUnsignedLongLong(ptr);
    if (PyErr_Occurred()) goto done;
    s->align_bytes = (p & 15) != 0 ? (int32_t)(p & (0 - p)) : 16;
    rc = 0;
done:
    Py_XDECREF(dims);
    Py_XDECREF(strides);
    Py_XDECREF(ptr);
    return rc;
}

/* Shapes of a sequence: torch tensors, or (with_shapes) objects that expose a dvm_shape through the buffer protocol.  The count, or -1. */
static Py_ssize_t shapes_from(PyObject *seq, dvm_shape *out, int with_shapes, int *rank_error) {
    PyObject *fast = PySequence_Fast(seq, "a sequence of tensors or shapes");
    if (!fast) return -1;
    Py_ssize_t n = PySequence_Fast_GET_SIZE(fast);
    for (Py_ssize_t i = 0; i < n && i < DVM_MAX_TENSORS; ++i) {      /* (the caller looks at the count) */
        PyObject *o = PySequence_Fast_GET_ITEM(fast, i);
        if (with_shapes) {
            Py_buffer b;
            if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) { n = -1; break; }
            const int ok = b.len == (Py_ssize_t)sizeof(dvm_shape);
            if (ok) memcpy(&out[i], b.buf, sizeof(dvm_shape));
            PyBuffer_Release(&b);
            if (!ok) { PyErr_SetString(PyExc_TypeError, "a dvm_shape"); n = -1; break; }
        } else if (shape_from_tensor(o, &out[i], rank_error) != 0) {
            n = -1;
            break;
        }
        if (*rank_error) break;
    }
    Py_DECREF(fast);
    return n;
}

/* encode(ctx, prog, inputs, outputs or None, n_out, with_shapes) -> (bytes, [output dims]), or a status; a rank beyond the limit: None */
static PyObject *py_encode(PyObject *self, PyObject *const *a, Py_ssize_t na) {
    (void)self;
    if (na != 6) return PyErr_Format(PyExc_TypeError, "encode takes 6 arguments");
    void *ctx, *prog;
    if (address_of(a[0], &ctx) != 0 || address_of(a[1], &prog) != 0) return NULL;
    const long n_out = PyLong_AsLong(a[4]), with_shapes = PyLong_AsLong(a[5]);
    if (PyErr_Occurred()) return NULL;
    dvm_shape in[DVM_MAX_TENSORS], lay[DVM_MAX_TENSORS], outs[DVM_MAX_TENSORS];
    int rank_error = 0;
    const Py_ssize_t n_in = shapes_from(a[2], in, (int)with_shapes, &rank_error);
    if (n_in < 0) return NULL;
    const int have = a[3] != Py_None;
    Py_ssize_t n_lay = 0;
    if (have && !rank_error && (n_lay = shapes_from(a[3], lay, (int)with_shapes, &rank_error)) < 0) return NULL;
    if (rank_error) Py_RETURN_NONE;
    if (n_in > DVM_MAX_TENSORS || n_lay > DVM_MAX_TENSORS || n_out > DVM_MAX_TENSORS || (have && n_lay < n_out)) return PyLong_FromLong(DVM_E_ARGS);
    unsigned char buf[ENC_CAP];
    size_t len = 0;
    const int st = lib.encode(ctx, prog, in, (int)n_in, have ? lay : NULL, buf, sizeof(buf), &len, outs);
    if (st != DVM_OK) return PyLong_FromLong(st);
    PyObject *shapes = PyList_New(n_out);
    if (!shapes) return NULL;
    for (long k = 0; k < n_out; ++k) {
        PyObject *t = PyTuple_New(outs[k].rank);
        if (!t) { Py_DECREF(shapes); return NULL; }
        for (int32_t d = 0; d < outs[k].rank; ++d) PyTuple_SET_ITEM(t, d, PyLong_FromLongLong(outs[k].dim[d]));
        PyList_SET_ITEM(shapes, k, t);
    }
    return Py_BuildValue("y#N", (const char *)buf, (Py_ssize_t)len, shapes);
}

/* Device addresses of a sequence.  The count, or -1. */
static Py_ssize_t addresses_from(PyObject *seq, void **out, Py_ssize_t room) {
    PyObject *fast = PySequence_Fast(seq, "a sequence of addresses");
    if (!fast) return -1;
    Py_ssize_t n = PySequence_Fast_GET_SIZE(fast);
    for (Py_ssize_t i = 0; i < n && i < room; ++i)          /* (the caller looks at the count) */
        if (address_of(PySequence_Fast_GET_ITEM(fast, i), &out[i]) != 0) { n = -1; break; }
    Py_DECREF(fast);
    return n;
}

/* run(ctx, code, addresses, stream) -> status */
static PyObject *py_run(PyObject *self, PyObject *const *a, Py_ssize_t na) {
    (void)self;
    if (na != 4) return PyErr_Format(PyExc_TypeError, "run takes 4 arguments");
    void *ctx, *stream, *ptrs[DVM_MAX_TENSORS];
    char *code;
    Py_ssize_t len;
    if (address_of(a[0], &ctx) != 0 || address_of(a[3], &stream) != 0 || PyBytes_AsStringAndSize(a[1], &code, &len) != 0) return NULL;
    const Py_ssize_t n = addresses_from(a[2], ptrs, DVM_MAX_TENSORS);
    if (n < 0) return NULL;
    if (n > DVM_MAX_TENSORS) return PyLong_FromLong(DVM_E_ARGS);
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = lib.run(ctx, code, (size_t)len, ptrs, (int)n, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

/* run_batched(ctx, code, sets, table, table_bytes, stream) -> status; sets of unequal size: None */
static PyObject *py_run_batched(PyObject *self, PyObject *const *a, Py_ssize_t na) {
    (void)self;
    if (na != 6) return PyErr_Format(PyExc_TypeError, "run_batched takes 6 arguments");
    void *ctx, *table, *stream;
    char *code;
    Py_ssize_t len;
    if (address_of(a[0], &ctx) != 0 || address_of(a[3], &table) != 0 || address_of(a[5], &stream) != 0 || PyBytes_AsStringAndSize(a[1], &code, &len) != 0) return NULL;
    const size_t table_bytes = PyLong_AsSize_t(a[4]);
    if (PyErr_Occurred()) return NULL;
    PyObject *sets = PySequence_Fast(a[2], "a sequence of sets");
    if (!sets) return NULL;
    const Py_ssize_t n_sets = PySequence_Fast_GET_SIZE(sets);
    Py_ssize_t n = 0;
    void **flat = NULL;
    PyObject *result = NULL;
    for (Py_ssize_t k = 0; k < n_sets; ++k) {
        PyObject *set = PySequence_Fast(PySequence_Fast_GET_ITEM(sets, k), "a set of addresses");      /* (any iterable, taken once) */
        if (!set) goto done;
        if (k == 0) {
            n = PySequence_Fast_GET_SIZE(set);
            flat = (void **)PyMem_Malloc(sizeof(void *) * (size_t)(n > 0 ? n : 1) * (size_t)n_sets);
            if (!flat) { PyErr_NoMemory(); Py_DECREF(set); goto done; }
        }
        const Py_ssize_t got = PySequence_Fast_GET_SIZE(set) == n ? addresses_from(set, flat + k * n, n) : n + 1;
        Py_DECREF(set);
        if (got < 0) goto done;
        if (got != n) {
            result = Py_None;
            Py_INCREF(result);
            goto done;
        }
    }
    {
        int st;
        Py_BEGIN_ALLOW_THREADS
        st = lib.run_batched(ctx, code, (size_t)len, flat, (int)n, (int)n_sets, table, table_bytes, stream);
        Py_END_ALLOW_THREADS
        result = PyLong_FromLong(st);
    }
done:
    PyMem_Free(flat);
    Py_DECREF(sets);
    return result;
}

/* stack([bytes, ..], spatial) -> bytes, or a status */
static PyObject *py_stack(PyObject *self, PyObject *const *a, Py_ssize_t na) {
    (void)self;
    if (na != 2) return PyErr_Format(PyExc_TypeError, "stack takes 2 arguments");
    const int spatial = PyObject_IsTrue(a[1]);
    PyObject *fast = PySequence_Fast(a[0], "a sequence of bytecodes");
    if (!fast) return NULL;
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(fast);
    const void *codes[DVM_MAX_TENSORS];
    size_t lens[DVM_MAX_TENSORS];
    PyObject *result = NULL;
    if (n > DVM_MAX_TENSORS) {          /* (every part has a tensor) */
        result = PyLong_FromLong(DVM_E_LIMIT);
        goto done;
    }
    for (Py_ssize_t i = 0; i < n; ++i) {
        char *p;
        Py_ssize_t len;
        if (PyBytes_AsStringAndSize(PySequence_Fast_GET_ITEM(fast, i), &p, &len) != 0) goto done;
        codes[i] = p;
        lens[i] = (size_t)len;
    }
    {
        unsigned char buf[ENC_CAP];
        size_t len = 0;
        const int st = (spatial ? lib.stack_spatial : lib.stack)(codes, lens, (int)n, buf, sizeof(buf), &len);
        result = st != DVM_OK ? PyLong_FromLong(st) : PyBytes_FromStringAndSize((const char *)buf, (Py_ssize_t)len);
    }
done:
    Py_DECREF(fast);
    return result;
}

/* A method of a tensor without arguments that gives an int; -1 with an exception. */
static long long number(PyObject *o, PyObject *name) {
    PyObject *v = PyObject_CallMethodNoArgs(o, name);
    if (!v) return -1;
    const long long n = PyLong_AsLongLong(v);
    Py_DECREF(v);
    return n;
}

/* check(code, tensors): every tensor's storage covers what the bytecode touches.  None; a status; or (index, bytes needed, bytes there) */
static PyObject *py_check(PyObject *self, PyObject *const *a, Py_ssize_t na) {
    (void)self;
    if (na != 2) return PyErr_Format(PyExc_TypeError, "check takes 2 arguments");
    char *code;
    Py_ssize_t len;
    if (PyBytes_AsStringAndSize(a[0], &code, &len) != 0) return NULL;
    PyObject *fast = PySequence_Fast(a[1], "a sequence of tensors");
    if (!fast) return NULL;
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(fast);
    PyObject *result = NULL;
    int64_t need[DVM_MAX_TENSORS];
    const int st = n > DVM_MAX_TENSORS ? DVM_E_ARGS : lib.min_bytes(code, (size_t)len, need, (int)n);
    if (st != DVM_OK) {
        result = PyLong_FromLong(st);
        goto done;
    }
    for (Py_ssize_t i = 0; i < n; ++i) {
        PyObject *t = PySequence_Fast_GET_ITEM(fast, i);
        PyObject *storage = PyObject_CallMethodNoArgs(t, s_untyped_storage);       /* (may have been resized below what the tensor's shape says) */
        if (!storage) goto done;
        long long have = number(storage, s_nbytes);
        Py_DECREF(storage);
        const long long offset = PyErr_Occurred() ? -1 : number(t, s_storage_offset);
        if (PyErr_Occurred()) goto done;
        if (offset != 0) {
            const long long es = number(t, s_element_size);
            if (PyErr_Occurred()) goto done;
            have -= offset * es;
        }
        const long long numel = number(t, s_numel);
        if (PyErr_Occurred()) goto done;
        if (need[i] > have || (numel == 0 && need[i] > 0)) {
            result = Py_BuildValue("nLL", i, (long long)need[i], numel != 0 ? have : 0LL);
            goto done;
        }
    }
    result = Py_None;
    Py_INCREF(result);
done:
    Py_DECREF(fast);
    return result;
}

/* needs_workspace(code): whether the launch's last tensor is its workspace; or a status */
static PyObject *py_needs_workspace(PyObject *self, PyObject *arg) {
    (void)self;
    char *code;
    Py_ssize_t len;
    if (PyBytes_AsStringAndSize(arg, &code, &len) != 0) return NULL;
    dvm_code_info info;
    int st = lib.info(code, (size_t)len, &info), kind = 0;
    if (st == DVM_OK && info.n_tensors > 0) st = lib.tensor(code, (size_t)len, info.n_tensors - 1, NULL, &kind, NULL, NULL);
    if (st != DVM_OK) return PyLong_FromLong(st);
    return PyBool_FromLong(kind == 2);
}

static PyMethodDef methods[] = {
    {"encode", (PyCFunction)(void (*)(void))py_encode, METH_FASTCALL, NULL},
    {"run", (PyCFunction)(void (*)(void))py_run, METH_FASTCALL, NULL},
    {"run_batched", (PyCFunction)(void (*)(void))py_run_batched, METH_FASTCALL, NULL},
    {"stack", (PyCFunction)(void (*)(void))py_stack, METH_FASTCALL, NULL},
    {"bind", (PyCFunction)(void (*)(void))py_bind, METH_FASTCALL, NULL},
    {"check", (PyCFunction)(void (*)(void))py_check, METH_FASTCALL, NULL},
    {"needs_workspace", py_needs_workspace, METH_O, NULL},
    {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_dvm", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__dvm(void) {
    struct { PyObject **at; const char *text; } names[] = {
        {&s_shape, "shape"}, {&s_stride, "stride"}, {&s_data_ptr, "data_ptr"}, {&s_untyped_storage, "untyped_storage"}, {&s_nbytes, "nbytes"},
        {&s_storage_offset, "storage_offset"}, {&s_element_size, "element_size"}, {&s_numel, "numel"}, {&s_value, "value"}};
    for (size_t i = 0; i < sizeof(names) / sizeof(names[0]); ++i)
        if (!(*names[i].at = PyUnicode_InternFromString(names[i].text))) return NULL;
    return PyModule_Create(&module);
}
