/* One call of sqllm_dense_sparse_matvec from Python without ctypes: takes the arguments apart, asks the tensors for their addresses and the
 * runtime for the current stream, and calls the library.  The call of a small layer is bound by the host: through ctypes 256x4096 takes
 * 5.6 us and 4096x4096 at 4 bits 5.8, this way 4.5 and 4.5 (their kernels run for 3.0 and 4.4).  Arguments that are not plain ints, None or
 * objects with data_ptr() are left to the ctypes path (None is returned), which accepts or refuses them as it always has. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>

typedef int (*matvec_fn)(int, int, int, long long, int, const void*, const void*, const int*, const int*, const void*, const void*, const void*, void*, void*);

static matvec_fn g_matvec;
static PyObject *g_device, *g_stream;      /* torch.cuda.current_device, device -> raw handle of its current stream */
static PyObject *s_data_ptr, *s_cuda_stream;

static PyObject* bind(PyObject* self, PyObject* args) {
    unsigned long long address;
    PyObject *device, *stream;
    (void)self;
    if (!PyArg_ParseTuple(args, "KOO", &address, &device, &stream)) return NULL;
    Py_INCREF(device);
    Py_INCREF(stream);
    Py_XSETREF(g_device, device);
    Py_XSETREF(g_stream, stream);
    g_matvec = (matvec_fn)(uintptr_t)address;
    Py_RETURN_NONE;
}

/* 1: *out is set, 0: not for this path, -1: an error is set */
static int address_of(PyObject* o, PyObject* method, int call, void** out) {
    PyObject* v;
    if (o == Py_None) { *out = NULL; return 1; }
    if (PyLong_Check(o)) { Py_INCREF(o); v = o; }
    else {
        v = call ? PyObject_CallMethodNoArgs(o, method) : PyObject_GetAttr(o, method);
        if (!v) return -1;
        if (!PyLong_Check(v)) { Py_DECREF(v); return 0; }
    }
    *out = (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(v);        /* as ctypes takes integers: the low bits */
    Py_DECREF(v);
    return PyErr_Occurred() ? -1 : 1;
}

/* matvec(M, N, bits, nnz, B, qidx, lut, rowptr, cols, vals, plan, x, y, stream) -> status, or None */
static PyObject* matvec(PyObject* self, PyObject* const* a, Py_ssize_t n) {
    long long v[5];
    void* p[9];
    int i, st;
    (void)self;
    if (n != 14 || !g_matvec) Py_RETURN_NONE;
    for (i = 0; i < 5; ++i) {
        if (!PyLong_Check(a[i])) Py_RETURN_NONE;
        v[i] = (long long)PyLong_AsUnsignedLongLongMask(a[i]);
        if (PyErr_Occurred()) return NULL;
    }
    for (i = 0; i < 8; ++i) {
        st = address_of(a[5 + i], s_data_ptr, 1, &p[i]);
        if (st < 0) return NULL;
        if (st == 0) Py_RETURN_NONE;
    }
    if (a[13] == Py_None) {
        PyObject *dev = PyObject_CallNoArgs(g_device), *s;
        if (!dev) return NULL;
        s = PyObject_CallOneArg(g_stream, dev);
        Py_DECREF(dev);
        if (!s) return NULL;
        st = PyLong_Check(s) ? address_of(s, NULL, 0, &p[8]) : 0;
        Py_DECREF(s);
    } else {
        st = address_of(a[13], s_cuda_stream, 0, &p[8]);
    }
    if (st < 0) return NULL;
    if (st == 0) Py_RETURN_NONE;
    Py_BEGIN_ALLOW_THREADS
    st = g_matvec((int)v[0], (int)v[1], (int)v[2], v[3], (int)v[4], p[0], p[1], (const int*)p[2], (const int*)p[3], p[4], p[5], p[6], p[7], p[8]);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

static PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, NULL},
    {"matvec", (PyCFunction)(void (*)(void))matvec, METH_FASTCALL, NULL},
    {NULL, NULL, 0, NULL},
};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pycall", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__pycall(void) {
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (!s_data_ptr || !s_cuda_stream) return NULL;
    return PyModule_Create(&module);
}
