/* The fused call's arguments, taken from Python objects and handed to the library without ctypes.
 *
 * Bound by host work: a decode step of a few microseconds is issued as fast as its arguments are marshalled.  One call,
 * arguments to return, without the launch: 4.0 us through ctypes and the binding's own Python lines, 1.2 here (15 arguments, four
 * tensors).  The same attributes and methods of the same objects are asked for as the binding does; nothing is kept from one call for the next.
 * Whatever is not as expected is left to the binding's general path: None is returned and nothing has happened.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

typedef int (*fused_fn)(const void *, int, int64_t, int64_t, int64_t, const float *, float, float, const void *, int64_t, float *,
                        int64_t, void *, size_t, void *);

static PyObject *s_is_cuda, *s_shape, *s_dtype, *s_data_ptr, *s_stride, *s_numel, *s_K, *s_rows, *s_buf, *zero;

static int is_true(PyObject *o, PyObject *name)
{
    PyObject *v = PyObject_GetAttr(o, name);
    const int t = v == Py_True;
    Py_XDECREF(v);
    return t;
}

/* an integer result, which is consumed; *bad is set where it is none */
static int64_t integer(PyObject *v, int *bad)
{
    int64_t r = 0;
    if (v != NULL && PyLong_Check(v)) {
        r = PyLong_AsLongLong(v);
        if (r == -1 && PyErr_Occurred()) *bad = 1;
    } else {
        *bad = 1;
    }
    Py_XDECREF(v);
    return r;
}

/* (from here on: nothing is asked for once something was bad, an exception may be pending) */
static int64_t attribute(PyObject *o, PyObject *name, int *bad)
{
    return *bad ? 0 : integer(PyObject_GetAttr(o, name), bad);
}

static void *pointer(PyObject *tensor, int *bad)
{
    if (*bad) return NULL;
    PyObject *const args[1] = {tensor};
    PyObject *v = PyObject_VectorcallMethod(s_data_ptr, args, 1, NULL);
    void *p = NULL;
    if (v != NULL && PyLong_Check(v)) p = PyLong_AsVoidPtr(v);
    if (v == NULL || !PyLong_Check(v) || PyErr_Occurred()) *bad = 1;
    Py_XDECREF(v);
    return p;
}

static int64_t row_stride(PyObject *tensor, int *bad)
{
    PyObject *const args[2] = {tensor, zero};
    return *bad ? 0 : integer(PyObject_VectorcallMethod(s_stride, args, 2, NULL), bad);
}

static int64_t elements(PyObject *tensor, int *bad)
{
    PyObject *const args[1] = {tensor};
    return *bad ? 0 : integer(PyObject_VectorcallMethod(s_numel, args, 1, NULL), bad);
}

static double number(PyObject *o, int *bad)
{
    if (*bad) return 0.0;
    if (PyFloat_CheckExact(o)) return PyFloat_AS_DOUBLE(o);
    PyObject *v = PyNumber_Float(o);
    const double d = v != NULL ? PyFloat_AS_DOUBLE(v) : 0.0;
    if (v == NULL) *bad = 1;
    Py_XDECREF(v);
    return d;
}

/* quant_gemm_fused(entry point, torch.float32, torch.bfloat16, X, fisher, threshold, scale, packed W, out, workspace, stream)
 * -> status, or None */
static PyObject *quant_gemm_fused(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    (void)self;
    if (n != 11) {
        PyErr_SetString(PyExc_TypeError, "eleven arguments expected");
        return NULL;
    }
    PyObject *const X = a[3], *const fisher = a[4], *const pW = a[7], *const out = a[8], *const workspace = a[9];
    int bad = 0;
    int64_t M = 0, K = 0;
    PyObject *v = NULL;

    if (!is_true(X, s_is_cuda) || !is_true(fisher, s_is_cuda)) goto general;
    v = PyObject_GetAttr(X, s_shape);
    if (v == NULL || !PyTuple_Check(v) || PyTuple_GET_SIZE(v) != 2) goto general;
    Py_INCREF(PyTuple_GET_ITEM(v, 0));
    Py_INCREF(PyTuple_GET_ITEM(v, 1));
    M = integer(PyTuple_GET_ITEM(v, 0), &bad);
    K = integer(PyTuple_GET_ITEM(v, 1), &bad);
    Py_CLEAR(v);
    if (bad) goto general;
    v = PyObject_GetAttr(X, s_dtype);
    const int dt = v == a[1] ? 0 : v == a[2] ? 1 : -1;
    Py_CLEAR(v);
    if (dt < 0) goto general;
    if (attribute(pW, s_K, &bad) != K) goto general;
    const int64_t N = attribute(pW, s_rows, &bad);
    if (bad) goto general;
    v = PyObject_GetAttr(pW, s_buf);
    if (v == NULL) goto general;
    const void *const w = pointer(v, &bad);
    Py_CLEAR(v);
    const void *const x = pointer(X, &bad);
    const int64_t ldx = row_stride(X, &bad);
    const float *const f = (const float *)pointer(fisher, &bad);
    float *const y = (float *)pointer(out, &bad);
    const int64_t ldy = row_stride(out, &bad);
    void *const ws = pointer(workspace, &bad);
    const int64_t ws_bytes = elements(workspace, &bad);
    const float T = (float)number(a[5], &bad), S = (float)number(a[6], &bad);
    if (bad) goto general;
    const fused_fn fn = (fused_fn)PyLong_AsVoidPtr(a[0]);
    void *const stream = fn != NULL ? PyLong_AsVoidPtr(a[10]) : NULL;
    if (fn == NULL || PyErr_Occurred()) goto general;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = fn(x, dt, M, K, ldx, f, T, S, w, N, y, ldy, ws, (size_t)ws_bytes, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
general:
    Py_XDECREF(v);
    PyErr_Clear();
    Py_RETURN_NONE;
}

static PyMethodDef methods[] = {{"quant_gemm_fused", (PyCFunction)(void (*)(void))quant_gemm_fused, METH_FASTCALL, NULL}, {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fgmp_call", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__fgmp_call(void)
{
    struct { PyObject **at; const char *name; } const names[] = {{&s_is_cuda, "is_cuda"}, {&s_shape, "shape"}, {&s_dtype, "dtype"},
        {&s_data_ptr, "data_ptr"}, {&s_stride, "stride"}, {&s_numel, "numel"}, {&s_K, "K"}, {&s_rows, "rows"}, {&s_buf, "buf"}};
    for (size_t i = 0; i < sizeof names / sizeof names[0]; ++i)
        if ((*names[i].at = PyUnicode_InternFromString(names[i].name)) == NULL) return NULL;
    if ((zero = PyLong_FromLong(0)) == NULL) return NULL;
    return PyModule_Create(&module);
}
