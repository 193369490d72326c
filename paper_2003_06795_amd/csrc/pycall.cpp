// Argument marshalling of the GEMM entry points for Python, in C: what binding.py does through ctypes, for the arguments
// that GEMM calls are made of (plain integers and floats, tensors, addresses, streams, None).  Anything else is answered
// with NotImplemented, before any side effect but the operands' data_ptr(), and binding.py makes the call through ctypes.
// ctypes converts some twenty arguments in 1.2 us, the Python around it takes as long again; a small GEMM's launch takes 2.5
// and its kernel 3: 128^3 5.5 -> 4.4 us a call among others, 37 x 1001 x 515 with a bias 6.1 -> 5.1.
// Host only.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <limits.h>
#include <stdint.h>

namespace {

PyObject *g_dataPtr = nullptr, *g_cudaStream = nullptr;      // "data_ptr", "cuda_stream"
PyObject *g_initialized = nullptr, *g_device = nullptr, *g_rawStream = nullptr;

enum Got { OK, OTHER, ERROR };

Got integer(PyObject *o, int64_t &v) {
    if (!PyLong_Check(o)) return OTHER;
    int over = 0;
    v = PyLong_AsLongLongAndOverflow(o, &over);
    return over ? OTHER : OK;
}
Got integer32(PyObject *o, int &v) {
    int64_t x = 0;
    if (integer(o, x) != OK || x < INT_MIN || x > INT_MAX) return OTHER;
    v = (int)x;
    return OK;
}
Got real(PyObject *o, float &v) {
    if (PyFloat_CheckExact(o)) {
        v = (float)PyFloat_AS_DOUBLE(o);
        return OK;
    }
    if (!PyLong_CheckExact(o)) return OTHER;
    const double x = PyLong_AsDouble(o);
    if (x == -1.0 && PyErr_Occurred()) {
        PyErr_Clear();
        return OTHER;
    }
    v = (float)x;
    return OK;
}
Got address(PyObject *o, void *&v) {
    int64_t x = 0;
    v = nullptr;
    if (o == Py_None) return OK;
    if (PyLong_CheckExact(o)) {
        if (integer(o, x) != OK || x < 0) return OTHER;
        v = (void *)(intptr_t)x;
        return OK;
    }
    PyObject *method = PyObject_GetAttr(o, g_dataPtr);
    if (!method) {
        if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return ERROR;
        PyErr_Clear();
        return OTHER;
    }
    PyObject *r = PyObject_CallNoArgs(method);
    Py_DECREF(method);
    if (!r) return ERROR;
    const Got g = integer(r, x) == OK && x >= 0 ? OK : OTHER;
    Py_DECREF(r);
    v = (void *)(intptr_t)x;
    return g;
}
// handle of a stream, or of the current stream of the current device (never kept)
Got stream_handle(PyObject *o, void *&v) {
    int64_t x = 0;
    if (o != Py_None) {
        PyObject *handle = o;
        if (PyLong_CheckExact(o)) {
            Py_INCREF(handle);
        } else if (!(handle = PyObject_GetAttr(o, g_cudaStream))) {
            if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return ERROR;
            PyErr_Clear();
            return OTHER;
        }
        const bool plain = PyLong_CheckExact(handle) && integer(handle, x) == OK && x >= 0;
        Py_DECREF(handle);
        v = (void *)(intptr_t)x;
        return plain ? OK : OTHER;
    }
    if (!g_initialized) return OTHER;
    PyObject *r = PyObject_CallNoArgs(g_initialized);
    if (!r) return ERROR;
    const bool ready = r == Py_True;
    Py_DECREF(r);
    if (!ready) return OTHER;
    PyObject *device = PyObject_CallNoArgs(g_device);
    if (!device) return ERROR;
    r = PyObject_CallOneArg(g_rawStream, device);
    Py_DECREF(device);
    if (!r) return ERROR;
    const Got g = integer(r, x) == OK && x >= 0 ? OK : OTHER;
    Py_DECREF(r);
    v = (void *)(intptr_t)x;
    return g;
}

#define KS_HEAD int, int, int64_t, int64_t, int64_t, float, const void *, int64_t, const void *, int64_t, float, void *, int64_t
#define KS_TAIL int64_t, int64_t, int64_t, int64_t
typedef int (*Plain)(KS_HEAD, KS_TAIL, void *);                                     // ks_gemm_f32 / bf16 / f16
typedef int (*Member)(int, KS_HEAD, KS_TAIL, void *);                               // ..._with_kernel
typedef int (*Typed)(int, int, KS_HEAD, KS_TAIL, void *);                           // ks_gemm_static_scratch
typedef int (*Bias)(int, int, KS_HEAD, const void *, KS_TAIL, void *);              // ks_gemm_bias, ks_gemm_out_bf16
typedef int (*Scratch)(int, int, KS_HEAD, KS_TAIL, void *, size_t, void *);         // ks_gemm_with_workspace

enum Form { PLAIN, MEMBER, TYPED, BIAS, SCRATCH };
// gemm(entry address, its form, dtype, kernel id, transA, transB, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc,
//      batch, strideA, strideB, strideC, stream, bias or workspace, bytes of the latter) -> status or NotImplemented;
// what a form does not have is 0 or None
PyObject *gemm(PyObject *, PyObject *const *a, Py_ssize_t n) {
    enum { ENTRY, FORM, DTYPE, KERNEL, TA, TB, M, N, K, ALPHA, A, LDA, B, LDB, BETA, C, LDC, BATCH, SA, SB, SC, STREAM, EXTRA, BYTES, COUNT };
    if (n != COUNT) {
        PyErr_Format(PyExc_TypeError, "gemm: %d arguments", (int)COUNT);
        return nullptr;
    }
    void *entry = nullptr, *pa = nullptr, *pb = nullptr, *pc = nullptr, *extra = nullptr, *stream = nullptr;
    int form = 0, dtype = 0, kernel = 0, tA = 0, tB = 0;
    int64_t m, nn, k, lda, ldb, ldc, batch, sA, sB, sC, bytes = 0;
    float alpha, beta;
    Got g;
#define KS_GET(call)                              \
    do {                                          \
        if ((g = (call)) == ERROR) return nullptr; \
        if (g == OTHER) Py_RETURN_NOTIMPLEMENTED; \
    } while (0)
    KS_GET(address(a[ENTRY], entry));
    KS_GET(integer32(a[FORM], form));
    KS_GET(integer32(a[DTYPE], dtype));
    KS_GET(integer32(a[KERNEL], kernel));
    KS_GET(integer32(a[TA], tA));
    KS_GET(integer32(a[TB], tB));
    KS_GET(integer(a[M], m));
    KS_GET(integer(a[N], nn));
    KS_GET(integer(a[K], k));
    KS_GET(real(a[ALPHA], alpha));
    KS_GET(integer(a[LDA], lda));
    KS_GET(integer(a[LDB], ldb));
    KS_GET(real(a[BETA], beta));
    KS_GET(integer(a[LDC], ldc));
    KS_GET(integer(a[BATCH], batch));
    KS_GET(integer(a[SA], sA));
    KS_GET(integer(a[SB], sB));
    KS_GET(integer(a[SC], sC));
    KS_GET(integer(a[BYTES], bytes));
    if (!entry || bytes < 0 || form < PLAIN || form > SCRATCH) Py_RETURN_NOTIMPLEMENTED;
    KS_GET(stream_handle(a[STREAM], stream));            // before the operands: what it does not take costs no more than that
    KS_GET(address(a[A], pa));
    KS_GET(address(a[B], pb));
    KS_GET(address(a[C], pc));
    KS_GET(address(a[EXTRA], extra));
#undef KS_GET
    int rc;
#define KS_ARGS tA, tB, m, nn, k, alpha, pa, lda, pb, ldb, beta, pc, ldc
    Py_BEGIN_ALLOW_THREADS
    switch (form) {
        case PLAIN: rc = ((Plain)entry)(KS_ARGS, batch, sA, sB, sC, stream); break;
        case MEMBER: rc = ((Member)entry)(kernel, KS_ARGS, batch, sA, sB, sC, stream); break;
        case TYPED: rc = ((Typed)entry)(dtype, kernel, KS_ARGS, batch, sA, sB, sC, stream); break;
        case BIAS: rc = ((Bias)entry)(dtype, kernel, KS_ARGS, extra, batch, sA, sB, sC, stream); break;
        default: rc = ((Scratch)entry)(dtype, kernel, KS_ARGS, batch, sA, sB, sC, extra, (size_t)bytes, stream); break;
    }
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// streams(is_initialized, current device, raw stream of a device): how torch is asked for its current stream
PyObject *streams(PyObject *, PyObject *args) {
    PyObject *i, *d, *r;
    if (!PyArg_ParseTuple(args, "OOO", &i, &d, &r)) return nullptr;
    Py_INCREF(i); Py_INCREF(d); Py_INCREF(r);
    Py_XSETREF(g_initialized, i);
    Py_XSETREF(g_device, d);
    Py_XSETREF(g_rawStream, r);
    Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {{"gemm", (PyCFunction)(void (*)(void))gemm, METH_FASTCALL, nullptr},
                          {"streams", streams, METH_VARARGS, nullptr},
                          {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_pycall", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pycall(void) {
    g_dataPtr = PyUnicode_InternFromString("data_ptr");
    g_cudaStream = PyUnicode_InternFromString("cuda_stream");
    return g_dataPtr && g_cudaStream ? PyModule_Create(&kModule) : nullptr;
}
