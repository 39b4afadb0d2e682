/* Arguments of the Python binding's calls, from Python objects to C, for the entry points of include/pasa.h that are called once per
 * layer and step.  Each function takes the address of an entry point, what makes the same call through ctypes, and the arguments in
 * order (the fields of pasa_opts spread out), and returns the entry point's status.  Through ctypes alone a call of
 * pasa_attn_fwd_ex costs 4.4 us on the host before anything is launched, which for the smallest calls is as long as their kernels
 * take; here 1.3.
 *
 * Taken here: addresses, and objects whose data_ptr() or cuda_stream is one; sizes that are Python integers; options that int() and
 * float() take.  A call with anything else (a size that is a numpy integer, say), or that raises on the way, is made again through
 * ctypes, so that ctypes alone says what is accepted and what is refused, and how. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "pasa.h"

static PyObject *s_data_ptr, *s_cuda_stream;

/* a: address, the call through ctypes, its arguments */
static PyObject* through_ctypes(PyObject* const* a, Py_ssize_t n)
{
    if (n < 2) {
        PyErr_SetString(PyExc_TypeError, "an address, the call through ctypes and its arguments");
        return NULL;
    }
    if (PyErr_Occurred()) {
        if (!PyErr_ExceptionMatches(PyExc_Exception)) return NULL;     /* an interrupt is no refusal */
        PyErr_Clear();
    }
    return PyObject_Vectorcall(a[1], a + 2, n - 2, NULL);
}

/* None, an address or an object with data_ptr() */
static int get_ptr(PyObject* x, void** out)
{
    *out = NULL;
    if (x == Py_None) return 1;
    if (PyLong_Check(x)) {
        *out = (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(x);
        return !PyErr_Occurred();
    }
    PyObject* p = PyObject_CallMethodNoArgs(x, s_data_ptr);
    if (p == NULL) return 0;
    const int ok = PyLong_Check(p) || p == Py_None;
    if (ok && p != Py_None) *out = (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(p);
    Py_DECREF(p);
    return ok && !PyErr_Occurred();
}

/* None, an address or an object with cuda_stream */
static int get_stream(PyObject* x, void** out)
{
    *out = NULL;
    if (x == Py_None) return 1;
    if (PyLong_Check(x)) return get_ptr(x, out);
    PyObject* p = PyObject_GetAttr(x, s_cuda_stream);
    if (p == NULL) return 0;
    const int ok = PyLong_Check(p) || p == Py_None;
    if (ok && p != Py_None) *out = (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(p);
    Py_DECREF(p);
    return ok && !PyErr_Occurred();
}

/* sizes: the low 32 bits, as ctypes takes them */
static int get_size(PyObject* x, int* out)
{
    if (!PyLong_Check(x)) return 0;
    *out = (int)(unsigned)PyLong_AsUnsignedLongLongMask(x);
    return !PyErr_Occurred();
}

/* options: int(x), float(x) */
static int get_int(PyObject* x, unsigned long long* out)
{
    PyObject* n = PyLong_CheckExact(x) ? (Py_INCREF(x), x) : PyNumber_Long(x);
    if (n == NULL) return 0;
    *out = PyLong_AsUnsignedLongLongMask(n);
    Py_DECREF(n);
    return !PyErr_Occurred();
}
static int get_float(PyObject* x, float* out)
{
    double f;
    if (PyFloat_CheckExact(x)) {
        f = PyFloat_AS_DOUBLE(x);
    } else {
        PyObject* n = PyNumber_Float(x);
        if (n == NULL) return 0;
        f = PyFloat_AS_DOUBLE(n);
        Py_DECREF(n);
    }
    *out = (float)f;
    return 1;
}

/* beta, variant, shift_tile, overflow_s, nonfinite_o, shift_mode, io_dtype */
#define OPTS 7
static int get_opts(PyObject* const* a, pasa_opts* o)
{
    unsigned long long variant, tile, mode, type;
    void *ovf, *bad;
    if (!get_float(a[0], &o->beta) || !get_int(a[1], &variant) || !get_int(a[2], &tile) || !get_ptr(a[3], &ovf) ||
        !get_ptr(a[4], &bad) || !get_int(a[5], &mode) || !get_int(a[6], &type))
        return 0;
    o->variant = (int)(unsigned)variant;
    o->shift_tile = (int)(unsigned)tile;
    o->overflow_s = (unsigned long long*)ovf;
    o->nonfinite_o = (unsigned long long*)bad;
    o->shift_mode = (int)(unsigned)mode;
    o->io_dtype = (int)(unsigned)type;
    return 1;
}

static int get_ptrs(PyObject* const* a, int n, void** out)
{
    for (int i = 0; i < n; ++i)
        if (!get_ptr(a[i], out + i)) return 0;
    return 1;
}
static int get_sizes(PyObject* const* a, int n, int* out)
{
    for (int i = 0; i < n; ++i)
        if (!get_size(a[i], out + i)) return 0;
    return 1;
}

#define CALL(status, expression)     \
    do {                             \
        Py_BEGIN_ALLOW_THREADS       \
        status = (expression);       \
        Py_END_ALLOW_THREADS         \
    } while (0)

/* address, ctypes, q, k, v, o, B, Hq, Hkv, N, d, causal, scale, stream */
static PyObject* plain(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    void *f, *p[4], *stream;
    int s[5], status;
    unsigned long long causal;
    float scale;
    if (n != 14 || !get_ptr(a[0], &f) || !get_ptrs(a + 2, 4, p) || !get_sizes(a + 6, 5, s) || !get_int(a[11], &causal) ||
        !get_float(a[12], &scale) || !get_stream(a[13], &stream))
        return through_ctypes(a, n);
    CALL(status, ((int (*)(const void*, const void*, const void*, void*, int, int, int, int, int, int, float, void*))f)(
                     p[0], p[1], p[2], p[3], s[0], s[1], s[2], s[3], s[4], (int)(unsigned)causal, scale, stream));
    return PyLong_FromLong(status);
}

/* address, ctypes, q, k, v, o, B, Hq, Hkv, N, d, causal, scale, workspace, bytes, stream, options, no options at all */
static PyObject* whole(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    void *f, *p[4], *ws, *stream;
    int s[5], status, none;
    unsigned long long causal, bytes;
    float scale;
    pasa_opts opts;
    if (n != 16 + OPTS + 1 || !get_ptr(a[0], &f) || !get_ptrs(a + 2, 4, p) || !get_sizes(a + 6, 5, s) || !get_int(a[11], &causal) ||
        !get_float(a[12], &scale) || !get_ptr(a[13], &ws) || !get_int(a[14], &bytes) || !get_stream(a[15], &stream) ||
        !get_opts(a + 16, &opts) || (none = PyObject_IsTrue(a[16 + OPTS])) < 0)
        return through_ctypes(a, n);
    CALL(status, ((int (*)(const void*, const void*, const void*, void*, int, int, int, int, int, int, float, const pasa_opts*, void*,
                           size_t, void*))f)(p[0], p[1], p[2], p[3], s[0], s[1], s[2], s[3], s[4], (int)(unsigned)causal, scale,
                                             none ? NULL : &opts, ws, (size_t)bytes, stream));
    return PyLong_FromLong(status);
}

/* address, ctypes, k, v, B, Hkv, N, d, scale, workspace, bytes, stream, options */
static PyObject* prepare(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    void *f, *p[2], *ws, *stream;
    int s[4], status;
    unsigned long long bytes;
    float scale;
    pasa_opts opts;
    if (n != 12 + OPTS || !get_ptr(a[0], &f) || !get_ptrs(a + 2, 2, p) || !get_sizes(a + 4, 4, s) || !get_float(a[8], &scale) ||
        !get_ptr(a[9], &ws) || !get_int(a[10], &bytes) || !get_stream(a[11], &stream) || !get_opts(a + 12, &opts))
        return through_ctypes(a, n);
    CALL(status, ((int (*)(const void*, const void*, int, int, int, int, float, const pasa_opts*, void*, size_t, void*))f)(
                     p[0], p[1], s[0], s[1], s[2], s[3], scale, &opts, ws, (size_t)bytes, stream));
    return PyLong_FromLong(status);
}

/* address, ctypes, q, o, B, Hq, Hkv, Nq, row0, N, d, causal, scale, workspace, bytes, stream, options */
static PyObject* chunk(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    void *f, *p[2], *ws, *stream;
    int s[7], status;
    unsigned long long causal, bytes;
    float scale;
    pasa_opts opts;
    if (n != 16 + OPTS || !get_ptr(a[0], &f) || !get_ptrs(a + 2, 2, p) || !get_sizes(a + 4, 7, s) || !get_int(a[11], &causal) ||
        !get_float(a[12], &scale) || !get_ptr(a[13], &ws) || !get_int(a[14], &bytes) || !get_stream(a[15], &stream) ||
        !get_opts(a + 16, &opts))
        return through_ctypes(a, n);
    CALL(status, ((int (*)(const void*, void*, int, int, int, int, int, int, int, int, float, const pasa_opts*, void*, size_t, void*))f)(
                     p[0], p[1], s[0], s[1], s[2], s[3], s[4], s[5], s[6], (int)(unsigned)causal, scale, &opts, ws, (size_t)bytes,
                     stream));
    return PyLong_FromLong(status);
}

static PyMethodDef methods[] = {
    {"plain", (PyCFunction)(void (*)(void))plain, METH_FASTCALL, NULL},
    {"whole", (PyCFunction)(void (*)(void))whole, METH_FASTCALL, NULL},
    {"prepare", (PyCFunction)(void (*)(void))prepare, METH_FASTCALL, NULL},
    {"chunk", (PyCFunction)(void (*)(void))chunk, METH_FASTCALL, NULL},
    {NULL, NULL, 0, NULL},
};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__calls(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (s_data_ptr == NULL || s_cuda_stream == NULL) return NULL;
    return PyModule_Create(&module);
}
