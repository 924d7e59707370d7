/* Argument marshalling of the Python binding for the compute entry points: integers, device addresses and the coefficient
 * array's buffer go straight to the C ABI.  Through ctypes a call spent 2.2 us on this (1.1 us of it on asking numpy for the
 * array's address), which a kernel of 3 us does not hide; here it is 0.3 us.  The interpreter lock is released around the
 * call, as ctypes does. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

typedef int (*conv2d_fn)(const void*, void*, int, int, const void*, int, int, int, int, int, int, void*);
typedef int (*conv3d_fn)(const void*, void*, int, int, int, const void*, int, int, int, int, int, int, int, int, void*);
typedef int (*stencil2d_fn)(const void*, void*, int, int, const void*, int, int, int, int, void*);
typedef int (*stencil3d_fn)(const void*, void*, int, int, int, const void*, int, int, int, int, int, void*);
typedef int (*iterate_fn)(void*, void*, int, int, int, const void*, int, int, int, int, int, int, void*, void**);
typedef int (*scan_fn)(const void*, void*, long long, int, void*, size_t, void*);

static conv2d_fn p_conv2d;
static conv3d_fn p_conv3d;
static stencil2d_fn p_stencil2d;
static stencil3d_fn p_stencil3d;
static iterate_fn p_iterate;
static scan_fn p_scan;

static void* ptr(PyObject* o) { return (void*)(uintptr_t)PyLong_AsUnsignedLongLong(o); }
static int num(PyObject* o) { return (int)PyLong_AsLong(o); }

static int arity(Py_ssize_t have, Py_ssize_t want)
{
    if (have == want) return 1;
    PyErr_Format(PyExc_TypeError, "%zd arguments, %zd expected", have, want);
    return 0;
}

/* The coefficients: a C-contiguous array of `ndim` dimensions of the element size of dtype (0 = 4 bytes, 1 = 8 bytes). */
static int coefs(PyObject* o, Py_buffer* b, int ndim, int dtype)
{
    if (PyObject_GetBuffer(o, b, PyBUF_ND | PyBUF_FORMAT) != 0) return 0;
    if (b->ndim == ndim && b->itemsize == (dtype == 0 ? 4 : 8)) return 1;
    PyBuffer_Release(b);
    PyErr_SetString(PyExc_ValueError, "coefficient array of the wrong rank or element size");
    return 0;
}

static PyObject* bind(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    if (!arity(n, 6)) return NULL;
    p_conv2d = (conv2d_fn)ptr(a[0]);
    p_conv3d = (conv3d_fn)ptr(a[1]);
    p_stencil2d = (stencil2d_fn)ptr(a[2]);
    p_stencil3d = (stencil3d_fn)ptr(a[3]);
    p_iterate = (iterate_fn)ptr(a[4]);
    p_scan = (scan_fn)ptr(a[5]);
    if (PyErr_Occurred()) return NULL;
    Py_RETURN_NONE;
}

/* conv2d(d_in, d_out, W, H, filter, ax, ay, boundary, dtype, stream) */
static PyObject* conv2d(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    if (!arity(n, 10)) return NULL;
    void *in = ptr(a[0]), *out = ptr(a[1]), *stream = ptr(a[9]);
    const int W = num(a[2]), H = num(a[3]), ax = num(a[5]), ay = num(a[6]), bnd = num(a[7]), dt = num(a[8]);
    Py_buffer b;
    int rc;
    if (PyErr_Occurred() || !coefs(a[4], &b, 2, dt)) return NULL;
    Py_BEGIN_ALLOW_THREADS
    rc = p_conv2d(in, out, W, H, b.buf, (int)b.shape[1], (int)b.shape[0], ax, ay, bnd, dt, stream);
    Py_END_ALLOW_THREADS
    PyBuffer_Release(&b);
    return PyLong_FromLong(rc);
}

/* conv3d(d_in, d_out, W, H, D, filter, ax, ay, az, boundary, dtype, stream) */
static PyObject* conv3d(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    if (!arity(n, 12)) return NULL;
    void *in = ptr(a[0]), *out = ptr(a[1]), *stream = ptr(a[11]);
    const int W = num(a[2]), H = num(a[3]), D = num(a[4]), ax = num(a[6]), ay = num(a[7]), az = num(a[8]), bnd = num(a[9]),
              dt = num(a[10]);
    Py_buffer b;
    int rc;
    if (PyErr_Occurred() || !coefs(a[5], &b, 3, dt)) return NULL;
    Py_BEGIN_ALLOW_THREADS
    rc = p_conv3d(in, out, W, H, D, b.buf, (int)b.shape[2], (int)b.shape[1], (int)b.shape[0], ax, ay, az, bnd, dt, stream);
    Py_END_ALLOW_THREADS
    PyBuffer_Release(&b);
    return PyLong_FromLong(rc);
}

/* stencil2d(d_in, d_out, W, H, coef, boundary, dtype, stream) */
static PyObject* stencil2d(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    if (!arity(n, 8)) return NULL;
    void *in = ptr(a[0]), *out = ptr(a[1]), *stream = ptr(a[7]);
    const int W = num(a[2]), H = num(a[3]), bnd = num(a[5]), dt = num(a[6]);
    Py_buffer b;
    int rc;
    if (PyErr_Occurred() || !coefs(a[4], &b, 2, dt)) return NULL;
    Py_BEGIN_ALLOW_THREADS
    rc = p_stencil2d(in, out, W, H, b.buf, (int)b.shape[1] / 2, (int)b.shape[0] / 2, bnd, dt, stream);
    Py_END_ALLOW_THREADS
    PyBuffer_Release(&b);
    return PyLong_FromLong(rc);
}

/* stencil3d(d_in, d_out, W, H, D, coef, boundary, dtype, stream) */
static PyObject* stencil3d(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    if (!arity(n, 9)) return NULL;
    void *in = ptr(a[0]), *out = ptr(a[1]), *stream = ptr(a[8]);
    const int W = num(a[2]), H = num(a[3]), D = num(a[4]), bnd = num(a[6]), dt = num(a[7]);
    Py_buffer b;
    int rc;
    if (PyErr_Occurred() || !coefs(a[5], &b, 3, dt)) return NULL;
    Py_BEGIN_ALLOW_THREADS
    rc = p_stencil3d(in, out, W, H, D, b.buf, (int)b.shape[2] / 2, (int)b.shape[1] / 2, (int)b.shape[0] / 2, bnd, dt, stream);
    Py_END_ALLOW_THREADS
    PyBuffer_Release(&b);
    return PyLong_FromLong(rc);
}

/* iterate(d_a, d_b, W, H, D, coef, boundary, dtype, steps, stream) -> (status, address of the result); coef 2D: D = 1 */
static PyObject* iterate(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    if (!arity(n, 10)) return NULL;
    void *pa = ptr(a[0]), *pb = ptr(a[1]), *stream = ptr(a[9]), *result = NULL;
    const int W = num(a[2]), H = num(a[3]), D = num(a[4]), bnd = num(a[6]), dt = num(a[7]), steps = num(a[8]);
    Py_buffer b;
    int rc, rx, ry, rz, d2;
    if (PyErr_Occurred()) return NULL;
    if (PyObject_GetBuffer(a[5], &b, PyBUF_ND | PyBUF_FORMAT) != 0) return NULL;
    d2 = b.ndim == 2;
    PyBuffer_Release(&b);
    if (!coefs(a[5], &b, d2 ? 2 : 3, dt)) return NULL;
    rx = (int)b.shape[d2 ? 1 : 2] / 2;
    ry = (int)b.shape[d2 ? 0 : 1] / 2;
    rz = d2 ? 0 : (int)b.shape[0] / 2;
    Py_BEGIN_ALLOW_THREADS
    rc = p_iterate(pa, pb, W, H, D, b.buf, rx, ry, rz, bnd, dt, steps, stream, &result);
    Py_END_ALLOW_THREADS
    PyBuffer_Release(&b);
    return Py_BuildValue("iK", rc, (unsigned long long)(uintptr_t)result);
}

/* scan(d_in, d_out, n, dtype, d_work, work_bytes, stream) */
static PyObject* scan(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    if (!arity(n, 7)) return NULL;
    void *in = ptr(a[0]), *out = ptr(a[1]), *work = ptr(a[4]), *stream = ptr(a[6]);
    const long long count = PyLong_AsLongLong(a[2]);
    const int dt = num(a[3]);
    const size_t bytes = (size_t)PyLong_AsUnsignedLongLong(a[5]);
    int rc;
    if (PyErr_Occurred()) return NULL;
    Py_BEGIN_ALLOW_THREADS
    rc = p_scan(in, out, count, dt, work, bytes, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, NULL}
static PyMethodDef methods[] = {FAST(bind),      FAST(conv2d), FAST(conv3d), FAST(stencil2d),
                                FAST(stencil3d), FAST(iterate), FAST(scan),  {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", NULL, -1, methods, NULL, NULL, NULL, NULL};
PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&module); }
