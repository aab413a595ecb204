// CPython entry to the product calls: the arguments of gemm_f32 and its siblings, handed to the library without ctypes.
//
// A small product takes the GPU 3 us, and its call took the host 4.2 us from Python, of which the library's own
// share is 1.5: the rest was a Python function, three attribute look-ups and thirteen ctypes conversions.  Here
// whole-number arguments are converted directly.  Whatever is not plain (keywords, a missing argument, anything but whole
// numbers in range, errors to be raised) goes to the ctypes function of the same name, which alone defines what is
// accepted and what is raised.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

typedef int (*product_fn)(int64_t, int64_t, int64_t, const void *, int, int64_t, const void *, int, int64_t, void *, int, int64_t,
                          void *);

static const int kProducts = 5;
static product_fn g_product[kProducts];   // null until the library is loaded
static PyObject *g_general[kProducts];    // the ctypes functions
static PyObject *g_check;                 // raises for a status
static PyObject *g_data_ptr;              // the string "data_ptr"

// a plain Python whole number that fits; false (no error set) otherwise
static inline bool whole(PyObject *x, int64_t *out)
{
    if (!PyLong_CheckExact(x)) return false;
    int overflow = 0;
    const long long v = PyLong_AsLongLongAndOverflow(x, &overflow);
    if (overflow) return false;
    *out = v;
    return true;
}

// a device address: None, a whole number, or what an object's data_ptr() returns; 0 no, 1 yes, -1 error set
static inline int address(PyObject *x, void **out)
{
    int64_t v;
    if (x == Py_None) {
        *out = nullptr;
        return 1;
    }
    if (PyLong_CheckExact(x)) {
        if (!whole(x, &v)) return 0;
        *out = (void *)(uintptr_t)v;
        return 1;
    }
    PyObject *p = PyObject_CallMethodNoArgs(x, g_data_ptr);
    if (p == nullptr) {
        if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return -1;
        PyErr_Clear();
        return 0;
    }
    const bool ok = whole(p, &v);
    Py_DECREF(p);
    *out = (void *)(uintptr_t)v;
    return ok ? 1 : 0;
}

static PyObject *call(int which, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    int64_t n[12];
    void *ptr[4] = {nullptr, nullptr, nullptr, nullptr};  // A, B, C, stream
    bool plain = g_product[which] != nullptr && kwnames == nullptr && nargs >= 12 && nargs <= 14;
    for (int i = 0; plain && i < 12; ++i) {
        if (i == 3 || i == 6 || i == 9) {
            const int ok = address(args[i], &ptr[i / 3 - 1]);
            if (ok < 0) return nullptr;
            plain = ok != 0;
        } else {
            plain = whole(args[i], &n[i]) && (i % 3 != 1 || i < 4 || (n[i] >= INT32_MIN && n[i] <= INT32_MAX));
        }
    }
    if (plain && nargs > 12) {
        int64_t v = 0;
        plain = args[12] == Py_None || whole(args[12], &v);
        ptr[3] = (void *)(uintptr_t)v;
    }
    const bool check = nargs < 14 || args[13] == Py_True;
    if (plain && !check) plain = args[13] == Py_False;
    if (plain) {
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = g_product[which](n[0], n[1], n[2], ptr[0], (int)n[4], n[5], ptr[1], (int)n[7], n[8], ptr[2], (int)n[10], n[11], ptr[3]);
        Py_END_ALLOW_THREADS
        PyObject *const status = PyLong_FromLong(rc);
        if (rc == 0 || !check || status == nullptr) return status;
        PyObject *const r = PyObject_CallOneArg(g_check, status);
        Py_DECREF(status);
        return r;
    }
    return PyObject_Vectorcall(g_general[which], args, (size_t)nargs, kwnames);
}

#define PRODUCT(I, NAME, DOC)                                                                                             \
    static PyObject *py_##NAME(PyObject *, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)                     \
    {                                                                                                                      \
        return call(I, args, nargs, kwnames);                                                                              \
    }                                                                                                                      \
    PyDoc_STRVAR(doc_##NAME, #NAME "(M, N, K, A, layoutA, lda, B, layoutB, ldb, C, layoutC, ldc, stream=None, check=True)\n--\n\n" DOC);
PRODUCT(0, gemm_f32, "C = A*B, binary32. A, B, C: device addresses or tensors; stream: hipStream_t as int.")
PRODUCT(1, gemm_f16f32, "C = A*B, binary16 operands, binary32 accumulation and result.")
PRODUCT(2, gemm_f16f16, "C = A*B, binary16 operands, binary32 accumulation, C rounded to binary16 (16-bit patterns).")
PRODUCT(3, gemm_bf16f32, "C = A*B, bfloat16 operands (16-bit patterns), binary32 accumulation and result.")
PRODUCT(4, gemm_f16f32_noalloc, "gemm_f16f32 that never allocates: K-slice partials go to the library's fixed per-GPU array.")

// general(index, function): the ctypes function calls fall back to
static PyObject *py_general(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    int64_t i;
    if (nargs != 2 || !whole(args[0], &i) || i < 0 || i >= kProducts) {
        PyErr_SetString(PyExc_TypeError, "general(index, function)");
        return nullptr;
    }
    Py_INCREF(args[1]);
    Py_XSETREF(g_general[i], args[1]);
    Py_RETURN_NONE;
}

// bind(check, address, ...): what raises for a status, and the loaded library's functions in the order above
static PyObject *py_bind(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    int64_t v[kProducts];
    for (int i = 0; i < kProducts; ++i) {
        if (nargs != kProducts + 1 || !whole(args[i + 1], &v[i])) {
            PyErr_SetString(PyExc_TypeError, "bind: a function and five addresses");
            return nullptr;
        }
    }
    Py_INCREF(args[0]);
    Py_XSETREF(g_check, args[0]);
    for (int i = 0; i < kProducts; ++i) g_product[i] = (product_fn)(uintptr_t)v[i];
    Py_RETURN_NONE;
}

#define ENTRY(NAME) {#NAME, (PyCFunction)(void (*)(void))py_##NAME, METH_FASTCALL | METH_KEYWORDS, doc_##NAME}
static PyMethodDef methods[] = {ENTRY(gemm_f32), ENTRY(gemm_f16f32), ENTRY(gemm_f16f16), ENTRY(gemm_bf16f32), ENTRY(gemm_f16f32_noalloc),
                                {"general", (PyCFunction)(void (*)(void))py_general, METH_FASTCALL, nullptr},
                                {"bind", (PyCFunction)(void (*)(void))py_bind, METH_FASTCALL, nullptr},
                                {nullptr, nullptr, 0, nullptr}};
static PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

PyMODINIT_FUNC PyInit__binding(void)
{
    g_data_ptr = PyUnicode_InternFromString("data_ptr");
    return g_data_ptr == nullptr ? nullptr : PyModule_Create(&module);
}
