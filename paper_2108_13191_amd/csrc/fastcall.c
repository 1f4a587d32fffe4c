/* Calls from Python into the GEMM entry points of the C ABI, without ctypes' marshalling.
 *
 * The smallest calls are bound by the host: 256^3 f32, launches in a row, 3.9 us a call of which HIP's launch takes 2.4, the
 * choice of a plan 0.25, and ctypes with the Python around it took 1.2.
 *
 * A function takes the address of the C function and its arguments: an int, or for a pointer None, an int or an object with
 * data_ptr().  Integers are converted as ctypes converts them (modulo 2^64, an int modulo 2^32).  Given anything else -- another
 * type, an object whose data_ptr() raises, another number of arguments -- it calls nothing and returns NotImplemented, and
 * the caller takes the general way, which accepts or refuses the arguments as it always has.  The GIL is released around the
 * call, as ctypes does. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

static PyObject* s_data_ptr;

/* 1: converted; 0: no argument for this way (an exception is left set only where it is none of Exception's, an interrupt) */
static int to_word(PyObject* x, uint64_t* out)
{
    if (!PyLong_Check(x)) return 0;
    *out = PyLong_AsUnsignedLongLongMask(x);
    if (*out == UINT64_MAX && PyErr_Occurred()) { PyErr_Clear(); return 0; }
    return 1;
}

static int to_pointer(PyObject* x, void** out)
{
    uint64_t w = 0;
    int ok = 1;
    if (PyLong_CheckExact(x)) ok = to_word(x, &w);
    else if (x != Py_None) {
        PyObject* const v = PyObject_CallMethodNoArgs(x, s_data_ptr);
        if (!v) { if (PyErr_ExceptionMatches(PyExc_Exception)) PyErr_Clear(); return 0; }
        ok = PyLong_CheckExact(v) && to_word(v, &w);
        Py_DECREF(v);
    }
    *out = (void*)(uintptr_t)w;
    return ok;
}

/* the arguments that all entry points begin with: address, M, N, K, A, lda, B, ldb, C, ldc */
typedef struct { void *address, *A, *B, *C; int64_t M, N, K, lda, ldb, ldc; } Operands;
static int to_operands(PyObject* const* a, Operands* o)
{
    uint64_t f, m, n, k, la, lb, lc;
    if (!(to_word(a[0], &f) && to_word(a[1], &m) && to_word(a[2], &n) && to_word(a[3], &k) && to_pointer(a[4], &o->A) && to_word(a[5], &la) &&
          to_pointer(a[6], &o->B) && to_word(a[7], &lb) && to_pointer(a[8], &o->C) && to_word(a[9], &lc))) return 0;
    o->address = (void*)(uintptr_t)f;
    o->M = (int64_t)m; o->N = (int64_t)n; o->K = (int64_t)k; o->lda = (int64_t)la; o->ldb = (int64_t)lb; o->ldc = (int64_t)lc;
    return 1;
}

static PyObject* other_way(void)
{
    if (PyErr_Occurred()) return NULL;
    Py_RETURN_NOTIMPLEMENTED;
}

typedef int (*plain_fn)(int64_t, int64_t, int64_t, const void*, int64_t, const void*, int64_t, void*, int64_t, void*);
static PyObject* plain(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    Operands o;
    void* stream;
    int rc;
    if (n != 11 || !to_operands(a, &o) || !to_pointer(a[10], &stream)) return other_way();
    Py_BEGIN_ALLOW_THREADS
    rc = ((plain_fn)o.address)(o.M, o.N, o.K, o.A, o.lda, o.B, o.ldb, o.C, o.ldc, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

typedef int (*bias_act_fn)(int64_t, int64_t, int64_t, const void*, int64_t, const void*, int64_t, void*, int64_t, const void*, int, void*);
static PyObject* bias_act(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    Operands o;
    void *bias, *stream;
    uint64_t act;
    int rc;
    if (n != 13 || !to_operands(a, &o) || !to_pointer(a[10], &bias) || !to_word(a[11], &act) || !to_pointer(a[12], &stream)) return other_way();
    Py_BEGIN_ALLOW_THREADS
    rc = ((bias_act_fn)o.address)(o.M, o.N, o.K, o.A, o.lda, o.B, o.ldb, o.C, o.ldc, bias, (int)(uint32_t)act, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

typedef int (*workspace_fn)(int64_t, int64_t, int64_t, const void*, int64_t, const void*, int64_t, void*, int64_t, void*, int64_t, void*);
static PyObject* workspace(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    Operands o;
    void *ws, *stream;
    uint64_t bytes;
    int rc;
    if (n != 13 || !to_operands(a, &o) || !to_pointer(a[10], &ws) || !to_word(a[11], &bytes) || !to_pointer(a[12], &stream)) return other_way();
    Py_BEGIN_ALLOW_THREADS
    rc = ((workspace_fn)o.address)(o.M, o.N, o.K, o.A, o.lda, o.B, o.ldb, o.C, o.ldc, ws, (int64_t)bytes, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

static PyMethodDef methods[] = {
    {"plain", (PyCFunction)(void (*)(void))plain, METH_FASTCALL, "plain(address, M, N, K, A, lda, B, ldb, C, ldc, stream)"},
    {"bias_act", (PyCFunction)(void (*)(void))bias_act, METH_FASTCALL, "bias_act(address, M, N, K, A, lda, B, ldb, C, ldc, bias, act, stream)"},
    {"workspace", (PyCFunction)(void (*)(void))workspace, METH_FASTCALL, "workspace(address, M, N, K, A, lda, B, ldb, C, ldc, workspace, workspace_bytes, stream)"},
    {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", "Calls into the C ABI of libgemm_f16.so", -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__fastcall(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    return s_data_ptr ? PyModule_Create(&module) : NULL;
}
