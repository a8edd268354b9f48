/* The host side of the binding's three calls (transform, convolution over the im2win tensor, workspace-free convolution) as one C call each:
 * the checks on tensors and sizes, the current stream and the library call.  A layer of a few microseconds is bound by its host side: a call
 * through ctypes and the checks in Python take 5.4 us, of which the library, from its checks to the enqueued launch, 3.6; see binding.py for what a call takes here.
 *
 * Only what needs no judgement is decided here: exact ints, exact torch tensors (or Parameters), fp32, on the GPU, contiguous, of the expected number of
 * elements.  For anything else, and for any error on the way, the call returns None with nothing launched, and the binding's general path
 * accepts or refuses the arguments as it always did.  No state is kept but what setup() is given. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stddef.h>

typedef int (*transform_fn)(const void *, void *, int, int, int, int, int, int, int, int, void *);
typedef int (*conv_fn)(const void *, const void *, void *, int, int, int, int, int, int, int, int, int, void *);
typedef int (*bytes_fn)(int, int, int, int, int, int, int, int, size_t *);
typedef int (*shape_fn)(int, int, int, int, int, int, int *, int *);

static PyObject *tensor_type, *parameter_type, *float32, *get_device, *get_stream;
static PyObject *s_is_cuda, *s_dtype, *s_is_contiguous, *s_numel, *s_data_ptr;
static transform_fn transform;
static conv_fn convs[2];
static bytes_fn workspace_bytes;
static shape_fn out_shape;

static PyObject *setup(PyObject *self, PyObject *args)
{
    PyObject *t, *p, *f, *d, *s;
    unsigned long long a[5];
    (void)self;
    if (!PyArg_ParseTuple(args, "OOOOOKKKKK", &t, &p, &f, &d, &s, &a[0], &a[1], &a[2], &a[3], &a[4])) return NULL;
    Py_INCREF(t); Py_INCREF(p); Py_INCREF(f); Py_INCREF(d); Py_INCREF(s);
    Py_XSETREF(tensor_type, t); Py_XSETREF(parameter_type, p); Py_XSETREF(float32, f); Py_XSETREF(get_device, d); Py_XSETREF(get_stream, s);
    transform = (transform_fn)a[0];
    convs[0] = (conv_fn)a[1];
    convs[1] = (conv_fn)a[2];
    workspace_bytes = (bytes_fn)a[3];
    out_shape = (shape_fn)a[4];
    Py_RETURN_NONE;
}

/* The tensor's address; 0 where it is not plainly an fp32 tensor on the GPU, contiguous, of `elems` elements. */
static int tensor_address(PyObject *t, unsigned long long elems, void **at)
{
    PyObject *v;
    int ok;
    unsigned long long n;
    if ((PyObject *)Py_TYPE(t) != tensor_type && (PyObject *)Py_TYPE(t) != parameter_type) return 0;
    if (!(v = PyObject_GetAttr(t, s_is_cuda))) return 0;
    ok = v == Py_True;
    Py_DECREF(v);
    if (!ok || !(v = PyObject_GetAttr(t, s_dtype))) return 0;
    ok = v == float32;
    Py_DECREF(v);
    if (!ok || !(v = PyObject_CallMethodNoArgs(t, s_is_contiguous))) return 0;
    ok = v == Py_True;
    Py_DECREF(v);
    if (!ok || !(v = PyObject_CallMethodNoArgs(t, s_numel))) return 0;
    n = PyLong_CheckExact(v) ? PyLong_AsUnsignedLongLong(v) : ~0ull;
    Py_DECREF(v);
    if (PyErr_Occurred() || n != elems || !(v = PyObject_CallMethodNoArgs(t, s_data_ptr))) return 0;
    *at = PyLong_CheckExact(v) ? PyLong_AsVoidPtr(v) : NULL;
    Py_DECREF(v);
    return !PyErr_Occurred() && *at != NULL;
}

/* The stream's handle: torch's current one on the current device for None, else the object's cuda_stream (an int). */
static int stream_handle(PyObject *stream, void **st)
{
    PyObject *d, *v;
    if (stream == Py_None) {
        if (!(d = PyObject_CallNoArgs(get_device))) return 0;
        v = PyObject_CallOneArg(get_stream, d);
        Py_DECREF(d);
    } else {
        v = PyObject_GetAttrString(stream, "cuda_stream");
    }
    if (!v) return 0;
    *st = PyLong_CheckExact(v) ? PyLong_AsVoidPtr(v) : NULL;
    d = PyLong_CheckExact(v) ? v : NULL;
    Py_DECREF(v);
    return d != NULL && !PyErr_Occurred();
}

static int plain_ints(PyObject *const *args, int n, int *out)
{
    int i, over;
    for (i = 0; i < n; ++i) {
        long v;
        if (!PyLong_CheckExact(args[i])) return 0;
        v = PyLong_AsLongAndOverflow(args[i], &over);
        if (over || v < -2147483647L - 1 || v > 2147483647L) return 0;
        out[i] = (int)v;
    }
    return 1;
}

static PyObject *general(void)
{
    PyErr_Clear();
    Py_RETURN_NONE;
}

/* call_transform(input, window, N, Ci, Hi, Wi, Hf, Wf, stride, pad, stream) */
static PyObject *call_transform(PyObject *self, PyObject *const *args, Py_ssize_t nargs)
{
    int d[8], status;
    size_t bytes;
    void *in, *win, *st;
    (void)self;
    if (nargs != 11 || !transform || !plain_ints(args + 2, 8, d)) return general();
    if (workspace_bytes(d[0], d[1], d[2], d[3], d[4], d[5], d[6], d[7], &bytes) != 0) return general();
    if (!tensor_address(args[0], (unsigned long long)d[0] * d[1] * ((unsigned long long)d[2] * d[3]), &in)) return general();
    if (!tensor_address(args[1], bytes / 4, &win) || !stream_handle(args[10], &st)) return general();
    Py_BEGIN_ALLOW_THREADS
    status = transform(in, win, d[0], d[1], d[2], d[3], d[4], d[5], d[6], d[7], st);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

/* call_conv(which, source, filter, output, N, Ci, Hi, Wi, Co, Hf, Wf, stride, pad, stream); which: 0 over the im2win tensor, 1 over the input */
static PyObject *call_conv(PyObject *self, PyObject *const *args, Py_ssize_t nargs)
{
    int d[9], which, Ho, Wo, status;
    size_t bytes;
    void *src, *flt, *out, *st;
    (void)self;
    if (nargs != 14 || !transform || !plain_ints(args, 1, &which) || !plain_ints(args + 4, 9, d)) return general();
    if ((which & ~1) || d[4] < 1 || workspace_bytes(d[0], d[1], d[2], d[3], d[5], d[6], d[7], d[8], &bytes) != 0) return general();
    if (out_shape(d[2], d[3], d[5], d[6], d[7], d[8], &Ho, &Wo) != 0) return general();
    if (!tensor_address(args[1], which ? (unsigned long long)d[0] * d[1] * ((unsigned long long)d[2] * d[3]) : bytes / 4, &src)) return general();
    if (!tensor_address(args[2], (unsigned long long)d[4] * d[1] * ((unsigned long long)d[5] * d[6]), &flt)) return general();
    if (!tensor_address(args[3], (unsigned long long)d[0] * d[4] * ((unsigned long long)Ho * Wo), &out) || !stream_handle(args[13], &st)) return general();
    Py_BEGIN_ALLOW_THREADS
    status = convs[which](src, flt, out, d[0], d[1], d[2], d[3], d[4], d[5], d[6], d[7], d[8], st);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

static PyMethodDef methods[] = {
    {"setup", setup, METH_VARARGS, NULL},
    {"call_transform", (PyCFunction)(void (*)(void))call_transform, METH_FASTCALL, NULL},
    {"call_conv", (PyCFunction)(void (*)(void))call_conv, METH_FASTCALL, NULL},
    {NULL, NULL, 0, NULL},
};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__native(void)
{
    if (!(s_is_cuda = PyUnicode_InternFromString("is_cuda")) || !(s_dtype = PyUnicode_InternFromString("dtype")) ||
        !(s_is_contiguous = PyUnicode_InternFromString("is_contiguous")) || !(s_numel = PyUnicode_InternFromString("numel")) ||
        !(s_data_ptr = PyUnicode_InternFromString("data_ptr")))
        return NULL;
    return PyModule_Create(&module);
}
