/* The binding's way into the library for the calls that programs make in a loop.
 *
 * A small call is bound by its host side: of 4.9 us (bf16 64 x 64 x 64 through ctypes) the launch takes 2.9, the library 0.4 and
 * converting fifteen arguments the rest; through this it is 3.6.  make(name, address, ...) returns a callable that takes the binding's own arguments in
 * order - tensors or addresses, a workspace tensor or None, a stream or None - and calls the function at `address` without
 * the interpreter lock.  The three functions that find the current stream may be None: such an entry takes calls that name theirs.
 * Whatever is not plain (a subclass of int, a value out of range, an object without data_ptr) it
 * leaves to the caller by returning NotImplemented, so that there is one place that says what an argument may be. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

typedef struct {
    void *fn;
    PyObject *initialized, *device, *raw_stream;        /* torch's: is there a device context, which device, its current stream; or None */
} Entry;

static PyObject *data_ptr_name, *nbytes_name, *stream_name;

/* Each returns 0, or -1 where the argument is not plain (with or without an exception set). */
static int get_int(PyObject *o, int64_t lo, int64_t hi, int64_t *out)
{
    int overflow = 0;
    if (!PyLong_CheckExact(o) && !PyBool_Check(o))
        return -1;
    *out = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow || *out < lo || *out > hi ? -1 : 0;
}
static int get_i32(PyObject *o, int *out)
{
    int64_t v;
    if (get_int(o, INT32_MIN, INT32_MAX, &v))
        return -1;
    *out = (int)v;
    return 0;
}
static int get_i64(PyObject *o, int64_t *out) { return get_int(o, INT64_MIN, INT64_MAX, out); }
static int get_truth(PyObject *o, int *out) { return (*out = PyObject_IsTrue(o)) < 0 ? -1 : 0; }
static int get_float(PyObject *o, float *out)
{
    if (PyFloat_CheckExact(o)) {
        *out = (float)PyFloat_AS_DOUBLE(o);
        return 0;
    }
    int64_t v;
    if (get_int(o, -(1 << 24), 1 << 24, &v))
        return -1;
    *out = (float)v;
    return 0;
}
static int get_address(PyObject *o, void **out)
{
    int64_t v;
    if (get_int(o, 0, INT64_MAX, &v))
        return -1;
    *out = (void *)(intptr_t)v;
    return 0;
}
static int get_ptr(PyObject *o, void **out)
{
    if (o == Py_None) {
        *out = NULL;
        return 0;
    }
    if (PyLong_Check(o))
        return get_address(o, out);
    PyObject *p = PyObject_CallMethodNoArgs(o, data_ptr_name);
    if (!p)
        return -1;
    const int rc = get_address(p, out);
    Py_DECREF(p);
    return rc;
}
static int get_workspace(PyObject *o, void **ws, size_t *bytes)
{
    *ws = NULL;
    *bytes = 0;
    if (o == Py_None)
        return 0;
    if (PyLong_Check(o) || get_ptr(o, ws))
        return -1;
    PyObject *n = PyObject_GetAttr(o, nbytes_name);
    int64_t v;
    const int rc = n ? get_int(n, 0, INT64_MAX, &v) : -1;
    Py_XDECREF(n);
    if (rc == 0)
        *bytes = (size_t)v;
    return rc;
}
static int get_stream(const Entry *e, PyObject *o, void **out)
{
    if (o != Py_None) {
        if (PyLong_Check(o))
            return get_address(o, out);
        PyObject *s = PyObject_GetAttr(o, stream_name);
        const int rc = s ? get_address(s, out) : -1;
        Py_XDECREF(s);
        return rc;
    }
    if (e->initialized == Py_None)
        return -1;
    PyObject *yes = PyObject_CallNoArgs(e->initialized);
    const int is = yes ? PyObject_IsTrue(yes) : -1;
    Py_XDECREF(yes);
    if (is != 1)
        return -1;
    PyObject *dev = PyObject_CallNoArgs(e->device);
    PyObject *raw = dev ? PyObject_CallOneArg(e->raw_stream, dev) : NULL;
    const int rc = raw ? get_address(raw, out) : -1;
    Py_XDECREF(raw);
    Py_XDECREF(dev);
    return rc;
}

static PyObject *not_plain(void)
{
    PyErr_Clear();
    Py_RETURN_NOTIMPLEMENTED;
}

#define ENTRY(count)                                                          \
    const Entry *e = (const Entry *)PyCapsule_GetPointer(self, NULL);         \
    if (!e || n != (count))                                                   \
        return not_plain();
#define RETURN_CALL(...)                                                      \
    do {                                                                      \
        int rc_;                                                              \
        Py_BEGIN_ALLOW_THREADS                                                \
        rc_ = __VA_ARGS__;                                                    \
        Py_END_ALLOW_THREADS                                                  \
        return PyLong_FromLong(rc_);                                          \
    } while (0)

/* transA, transB, M, N, K, A, lda, B, ldb, beta, C, ldc, workspace, stream */
static PyObject *call_f32(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    int tA, tB;
    int64_t M, N, K, lda, ldb, ldc;
    void *A, *B, *C, *ws, *st;
    size_t nb;
    float beta;
    ENTRY(14)
    if (get_i32(a[0], &tA) || get_i32(a[1], &tB) || get_i64(a[2], &M) || get_i64(a[3], &N) || get_i64(a[4], &K) || get_ptr(a[5], &A) ||
        get_i64(a[6], &lda) || get_ptr(a[7], &B) || get_i64(a[8], &ldb) || get_float(a[9], &beta) || get_ptr(a[10], &C) ||
        get_i64(a[11], &ldc) || get_workspace(a[12], &ws, &nb) || get_stream(e, a[13], &st))
        return not_plain();
    typedef int (*fn)(int, int, int64_t, int64_t, int64_t, const void *, int64_t, const void *, int64_t, float, void *, int64_t, void *, size_t, void *);
    RETURN_CALL(((fn)e->fn)(tA, tB, M, N, K, A, lda, B, ldb, beta, C, ldc, ws, nb, st));
}

/* the same with c_is_f32 before the workspace */
static PyObject *call_half(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    int tA, tB, c32;
    int64_t M, N, K, lda, ldb, ldc;
    void *A, *B, *C, *ws, *st;
    size_t nb;
    float beta;
    ENTRY(15)
    if (get_i32(a[0], &tA) || get_i32(a[1], &tB) || get_i64(a[2], &M) || get_i64(a[3], &N) || get_i64(a[4], &K) || get_ptr(a[5], &A) ||
        get_i64(a[6], &lda) || get_ptr(a[7], &B) || get_i64(a[8], &ldb) || get_float(a[9], &beta) || get_ptr(a[10], &C) ||
        get_i64(a[11], &ldc) || get_truth(a[12], &c32) || get_workspace(a[13], &ws, &nb) || get_stream(e, a[14], &st))
        return not_plain();
    typedef int (*fn)(int, int, int64_t, int64_t, int64_t, const void *, int64_t, const void *, int64_t, float, void *, int64_t, int, void *, size_t, void *);
    RETURN_CALL(((fn)e->fn)(tA, tB, M, N, K, A, lda, B, ldb, beta, C, ldc, c32, ws, nb, st));
}

/* transA, transB, M, N, K, A, lda, B, ldb, accumulate, C, ldc, stream */
static PyObject *call_s8(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    int tA, tB, acc;
    int64_t M, N, K, lda, ldb, ldc;
    void *A, *B, *C, *st;
    ENTRY(13)
    if (get_i32(a[0], &tA) || get_i32(a[1], &tB) || get_i64(a[2], &M) || get_i64(a[3], &N) || get_i64(a[4], &K) || get_ptr(a[5], &A) ||
        get_i64(a[6], &lda) || get_ptr(a[7], &B) || get_i64(a[8], &ldb) || get_truth(a[9], &acc) || get_ptr(a[10], &C) ||
        get_i64(a[11], &ldc) || get_stream(e, a[12], &st))
        return not_plain();
    typedef int (*fn)(int, int, int64_t, int64_t, int64_t, const void *, int64_t, const void *, int64_t, int, void *, int64_t, void *);
    RETURN_CALL(((fn)e->fn)(tA, tB, M, N, K, A, lda, B, ldb, acc, C, ldc, st));
}

/* transA, transB, M, N, K, batch, A, A_off, lda, B, B_off, ldb, beta, C, ldc, workspace, stream */
static PyObject *call_brgemm(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    int tA, tB;
    int64_t M, N, K, batch, lda, ldb, ldc;
    void *A, *Ao, *B, *Bo, *C, *ws, *st;
    size_t nb;
    float beta;
    ENTRY(17)
    if (get_i32(a[0], &tA) || get_i32(a[1], &tB) || get_i64(a[2], &M) || get_i64(a[3], &N) || get_i64(a[4], &K) || get_i64(a[5], &batch) ||
        get_ptr(a[6], &A) || get_ptr(a[7], &Ao) || get_i64(a[8], &lda) || get_ptr(a[9], &B) || get_ptr(a[10], &Bo) || get_i64(a[11], &ldb) ||
        get_float(a[12], &beta) || get_ptr(a[13], &C) || get_i64(a[14], &ldc) || get_workspace(a[15], &ws, &nb) || get_stream(e, a[16], &st))
        return not_plain();
    typedef int (*fn)(int, int, int64_t, int64_t, int64_t, int64_t, const void *, const void *, int64_t, const void *, const void *, int64_t, float, void *,
                      int64_t, void *, size_t, void *);
    RETURN_CALL(((fn)e->fn)(tA, tB, M, N, K, batch, A, Ao, lda, B, Bo, ldb, beta, C, ldc, ws, nb, st));
}

/* in_dtype, transA, transB, M, N, K, batch, A, A_off, lda, B, B_off, ldb, beta, C, ldc, c_is_f32, bias, epilogue, workspace, stream */
static PyObject *call_fused(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    int dt, tA, tB, c32, epi;
    int64_t M, N, K, batch, lda, ldb, ldc;
    void *A, *Ao, *B, *Bo, *C, *bias, *ws, *st;
    size_t nb;
    float beta;
    ENTRY(21)
    if (get_i32(a[0], &dt) || get_i32(a[1], &tA) || get_i32(a[2], &tB) || get_i64(a[3], &M) || get_i64(a[4], &N) || get_i64(a[5], &K) ||
        get_i64(a[6], &batch) || get_ptr(a[7], &A) || get_ptr(a[8], &Ao) || get_i64(a[9], &lda) || get_ptr(a[10], &B) || get_ptr(a[11], &Bo) ||
        get_i64(a[12], &ldb) || get_float(a[13], &beta) || get_ptr(a[14], &C) || get_i64(a[15], &ldc) || get_truth(a[16], &c32) ||
        get_ptr(a[17], &bias) || get_i32(a[18], &epi) || get_workspace(a[19], &ws, &nb) || get_stream(e, a[20], &st))
        return not_plain();
    typedef int (*fn)(int, int, int, int64_t, int64_t, int64_t, int64_t, const void *, const void *, int64_t, const void *, const void *, int64_t, float,
                      void *, int64_t, int, const void *, int, void *, size_t, void *);
    RETURN_CALL(((fn)e->fn)(dt, tA, tB, M, N, K, batch, A, Ao, lda, B, Bo, ldb, beta, C, ldc, c32, bias, epi, ws, nb, st));
}

/* transA, M, N, K, A, lda, packedB, beta, C, ldc, c_is_f32, bias, epilogue, workspace, stream */
static PyObject *call_packed(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    int tA, c32, epi;
    int64_t M, N, K, lda, ldc;
    void *A, *B, *C, *bias, *ws, *st;
    size_t nb;
    float beta;
    ENTRY(15)
    if (get_i32(a[0], &tA) || get_i64(a[1], &M) || get_i64(a[2], &N) || get_i64(a[3], &K) || get_ptr(a[4], &A) || get_i64(a[5], &lda) ||
        get_ptr(a[6], &B) || get_float(a[7], &beta) || get_ptr(a[8], &C) || get_i64(a[9], &ldc) || get_truth(a[10], &c32) || get_ptr(a[11], &bias) ||
        get_i32(a[12], &epi) || get_workspace(a[13], &ws, &nb) || get_stream(e, a[14], &st))
        return not_plain();
    typedef int (*fn)(int, int64_t, int64_t, int64_t, const void *, int64_t, const void *, float, void *, int64_t, int, const void *, int, void *, size_t, void *);
    RETURN_CALL(((fn)e->fn)(tA, M, N, K, A, lda, B, beta, C, ldc, c32, bias, epi, ws, nb, st));
}

/* transA, transB, M, N, K, nmat, A, lda, strideA, B, ldb, strideB, beta, C, ldc, strideC, [c_is_f32,] stream */
static PyObject *batched(PyObject *self, PyObject *const *a, Py_ssize_t n, int half)
{
    int tA, tB, c32 = 0;
    int64_t M, N, K, nmat, lda, sa, ldb, sb, ldc, sc;
    void *A, *B, *C, *st;
    float beta;
    ENTRY(17 + half)
    if (get_i32(a[0], &tA) || get_i32(a[1], &tB) || get_i64(a[2], &M) || get_i64(a[3], &N) || get_i64(a[4], &K) || get_i64(a[5], &nmat) ||
        get_ptr(a[6], &A) || get_i64(a[7], &lda) || get_i64(a[8], &sa) || get_ptr(a[9], &B) || get_i64(a[10], &ldb) || get_i64(a[11], &sb) ||
        get_float(a[12], &beta) || get_ptr(a[13], &C) || get_i64(a[14], &ldc) || get_i64(a[15], &sc) || (half && get_truth(a[16], &c32)) ||
        get_stream(e, a[16 + half], &st))
        return not_plain();
    if (half) {
        typedef int (*fn)(int, int, int64_t, int64_t, int64_t, int64_t, const void *, int64_t, int64_t, const void *, int64_t, int64_t, float, void *, int64_t,
                          int64_t, int, void *);
        RETURN_CALL(((fn)e->fn)(tA, tB, M, N, K, nmat, A, lda, sa, B, ldb, sb, beta, C, ldc, sc, c32, st));
    }
    typedef int (*fn)(int, int, int64_t, int64_t, int64_t, int64_t, const void *, int64_t, int64_t, const void *, int64_t, int64_t, float, void *, int64_t,
                      int64_t, void *);
    RETURN_CALL(((fn)e->fn)(tA, tB, M, N, K, nmat, A, lda, sa, B, ldb, sb, beta, C, ldc, sc, st));
}
static PyObject *call_batched_half(PyObject *self, PyObject *const *a, Py_ssize_t n) { return batched(self, a, n, 1); }
static PyObject *call_batched_f32(PyObject *self, PyObject *const *a, Py_ssize_t n) { return batched(self, a, n, 0); }

#define DEF(name, fn) {name, (PyCFunction)(void (*)(void))fn, METH_FASTCALL, NULL}
static PyMethodDef entries[] = {
    DEF("gemm_f32", call_f32), DEF("gemm_bf16", call_half), DEF("gemm_f16", call_half), DEF("gemm_f8", call_half), DEF("gemm_bf8", call_half),
    DEF("gemm_s8", call_s8), DEF("brgemm_bf16", call_brgemm), DEF("brgemm_fused", call_fused), DEF("gemm_bf16_packed", call_packed),
    DEF("gemm_bf16_batched", call_batched_half), DEF("gemm_f32_batched", call_batched_f32)};

static PyObject *make(PyObject *self, PyObject *args)
{
    const char *name;
    unsigned long long address;
    PyObject *initialized, *device, *raw_stream;
    (void)self;
    if (!PyArg_ParseTuple(args, "sKOOO", &name, &address, &initialized, &device, &raw_stream))
        return NULL;
    for (size_t i = 0; i < sizeof entries / sizeof *entries; ++i) {
        if (strcmp(entries[i].ml_name, name))
            continue;
        Entry *e = (Entry *)PyMem_Malloc(sizeof *e);        /* as long as the process, like the library */
        if (!e)
            return PyErr_NoMemory();
        *e = (Entry){(void *)(uintptr_t)address, initialized, device, raw_stream};
        Py_INCREF(initialized);
        Py_INCREF(device);
        Py_INCREF(raw_stream);
        PyObject *capsule = PyCapsule_New(e, NULL, NULL);
        PyObject *f = capsule ? PyCFunction_New(&entries[i], capsule) : NULL;
        Py_XDECREF(capsule);
        return f;
    }
    return PyErr_Format(PyExc_KeyError, "%s", name);
}

static PyMethodDef methods[] = {{"make", make, METH_VARARGS, NULL}, {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__fastcall(void)
{
    data_ptr_name = PyUnicode_InternFromString("data_ptr");
    nbytes_name = PyUnicode_InternFromString("nbytes");
    stream_name = PyUnicode_InternFromString("cuda_stream");
    return data_ptr_name && nbytes_name && stream_name ? PyModule_Create(&module) : NULL;
}
