// Call path of the Python binding's small calls: tensor descriptors, output
// allocation and the library call in one C function.
//
// A doubling of a 64x64 image takes the GPU 4.6 us, while the same steps in
// Python (ctypes structures from the shape and stride tuples, byref, argument
// conversion) took 8.9 us of host time per call, 4.2 of them in the library
// and the HIP launch; here it is 5.9 (zoom2x_ 6.3 -> 4.2, the adjoint 9.3 -> 7.0).  Only the common forms are taken:
// anything else returns None, and the caller goes the general way, which also
// raises the errors.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "weno_zoom.h"

typedef int (*fn_zoom)(const weno_tensor_t*, const weno_tensor_t*, const weno_params_t*, void*);
typedef int (*fn_bwd)(const weno_tensor_t*, const weno_tensor_t*, const weno_tensor_t*, const weno_params_t*, void*);

// torch objects, set once by init()
static PyObject *g_u8, *g_f32, *g_empty, *g_raw_stream, *g_tensor;
// interned names
static PyObject *s_is_cuda, *s_dtype, *s_shape, *s_stride, *s_data_ptr, *s_device, *s_get_device, *s_kw_dtype_device;

// plain tensors only: a subclass may redefine any of the attributes read here
static int is_plain(PyObject* t) { return (PyObject*)Py_TYPE(t) == g_tensor; }

static int to_i64(PyObject* o, int64_t* v)
{
    *v = PyLong_AsLongLong(o);
    return *v == -1 && PyErr_Occurred() ? -1 : 0;
}

// 1: d describes t; 0: not a form for this path; -1: Python error.  *device
// (optional) is t's device index.
static int describe(PyObject* t, weno_tensor_t* d, int* device)
{
    if (!is_plain(t)) return 0;
    PyObject* o = PyObject_GetAttr(t, s_is_cuda);
    if (!o) return -1;
    const int cuda = o == Py_True;
    Py_DECREF(o);
    if (!cuda) return 0;
    o = PyObject_GetAttr(t, s_dtype);
    if (!o) return -1;
    d->dtype = o == g_f32 ? WENO_F32 : WENO_U8;
    const int known = o == g_f32 || o == g_u8;
    Py_DECREF(o);
    if (!known) return 0;
    PyObject* shape = PyObject_GetAttr(t, s_shape);
    if (!shape) return -1;
    PyObject* stride = PyObject_CallMethodNoArgs(t, s_stride);
    if (!stride) {
        Py_DECREF(shape);
        return -1;
    }
    int rc = 0;
    int64_t n[4] = {1, 1, 1, 1}, s[4] = {0, 0, 0, 0};
    const Py_ssize_t nd = PyTuple_Check(shape) && PyTuple_Check(stride) ? PyTuple_GET_SIZE(shape) : 0;
    if (nd >= 2 && nd <= 4 && PyTuple_GET_SIZE(stride) == nd) {
        rc = 1;
        for (Py_ssize_t i = 0; i < nd; ++i)
            if (to_i64(PyTuple_GET_ITEM(shape, i), &n[4 - nd + i]) || to_i64(PyTuple_GET_ITEM(stride, i), &s[4 - nd + i]))
                rc = -1;
        // missing leading dims: size 1, the stride of torch's unsqueeze(0)
        if (nd == 2) s[1] = n[2] * s[2];
        if (nd <= 3) s[0] = n[1] * s[1];
        for (int i = 0; i < 4; ++i)
            if (rc == 1 && (n[i] < 0 || n[i] > INT32_MAX)) rc = 0;
    }
    Py_DECREF(shape);
    Py_DECREF(stride);
    if (rc != 1) return rc;
    o = PyObject_CallMethodNoArgs(t, s_data_ptr);
    if (!o) return -1;
    d->data = PyLong_AsVoidPtr(o);
    Py_DECREF(o);
    if (!d->data && PyErr_Occurred()) return -1;
    d->n = (int32_t)n[0];
    d->c = (int32_t)n[1];
    d->h = (int32_t)n[2];
    d->w = (int32_t)n[3];
    d->sn = s[0];
    d->sc = s[1];
    d->sh = s[2];
    d->sw = s[3];
    if (device) {
        o = PyObject_CallMethodNoArgs(t, s_get_device);
        if (!o) return -1;
        *device = (int)PyLong_AsLong(o);
        Py_DECREF(o);
        if (*device == -1 && PyErr_Occurred()) return -1;
    }
    return 1;
}

// handle of torch's current stream on a device
static int current_stream(int device, void** stream)
{
    PyObject* idx = PyLong_FromLong(device);
    if (!idx) return -1;
    PyObject* o = PyObject_CallOneArg(g_raw_stream, idx);
    Py_DECREF(idx);
    if (!o) return -1;
    *stream = PyLong_AsVoidPtr(o);
    Py_DECREF(o);
    return !*stream && PyErr_Occurred() ? -1 : 0;
}

static void* address(PyObject* o) { return PyLong_AsVoidPtr(o); }

// zoom2x_(fn, params, x, out) -> status, or None
static PyObject* native_zoom2x_into(PyObject* self, PyObject* const* a, Py_ssize_t na)
{
    (void)self;
    if (na != 4) return PyErr_Format(PyExc_TypeError, "zoom2x_ takes 4 arguments");
    const fn_zoom fn = (fn_zoom)address(a[0]);
    const weno_params_t* p = (const weno_params_t*)address(a[1]);
    if (!fn || !p) return PyErr_Occurred() ? NULL : PyErr_Format(PyExc_ValueError, "null address");
    weno_tensor_t s, d;
    int dev = 0;
    int rc = describe(a[2], &s, &dev);
    if (rc == 1) rc = describe(a[3], &d, NULL);
    if (rc < 0) return NULL;
    if (rc == 0) Py_RETURN_NONE;
    void* st;
    if (current_stream(dev, &st)) return NULL;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = fn(&s, &d, p, st);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

// zoom2x(fn, params, x, dtype or None) -> the new output, a status, or None:
// planar inputs only, into a contiguous output
static PyObject* native_zoom2x(PyObject* self, PyObject* const* a, Py_ssize_t na)
{
    (void)self;
    if (na != 4) return PyErr_Format(PyExc_TypeError, "zoom2x takes 4 arguments");
    const fn_zoom fn = (fn_zoom)address(a[0]);
    const weno_params_t* p = (const weno_params_t*)address(a[1]);
    if (!fn || !p) return PyErr_Occurred() ? NULL : PyErr_Format(PyExc_ValueError, "null address");
    weno_tensor_t s, d;
    int dev = 0;
    int rc = describe(a[2], &s, &dev);
    if (rc < 0) return NULL;
    if (rc == 0) Py_RETURN_NONE;   // s is not filled
    PyObject* dtype = a[3] == Py_None ? (s.dtype == WENO_F32 ? g_f32 : g_u8) : a[3];
    // interleaved channels take an output of their own layout
    if ((s.sc == 1 && s.c > 1) || (dtype != g_f32 && dtype != g_u8) || s.h > INT32_MAX / 2 ||
        s.w > INT32_MAX / 2)
        Py_RETURN_NONE;
    PyObject* shape = PyObject_GetAttr(a[2], s_shape);
    if (!shape) return NULL;
    const Py_ssize_t nd = PyTuple_GET_SIZE(shape);
    Py_DECREF(shape);
    d.n = s.n;
    d.c = s.c;
    d.h = 2 * s.h;
    d.w = 2 * s.w;
    d.dtype = dtype == g_f32 ? WENO_F32 : WENO_U8;
    d.sw = 1;
    d.sh = d.w;
    d.sc = (int64_t)d.h * d.w;
    d.sn = d.c * d.sc;
    PyObject* size = nd == 2   ? Py_BuildValue("(ii)", d.h, d.w)
                     : nd == 3 ? Py_BuildValue("(iii)", d.c, d.h, d.w)
                               : Py_BuildValue("(iiii)", d.n, d.c, d.h, d.w);
    PyObject* device = PyObject_GetAttr(a[2], s_device);
    if (!size || !device) {
        Py_XDECREF(size);
        Py_XDECREF(device);
        return NULL;
    }
    PyObject* args[3] = {size, dtype, device};
    PyObject* out = PyObject_Vectorcall(g_empty, args, 1, s_kw_dtype_device);
    Py_DECREF(size);
    Py_DECREF(device);
    if (!out) return NULL;
    PyObject* ptr = PyObject_CallMethodNoArgs(out, s_data_ptr);
    void* st;
    if (!ptr || current_stream(dev, &st)) {
        Py_XDECREF(ptr);
        Py_DECREF(out);
        return NULL;
    }
    d.data = PyLong_AsVoidPtr(ptr);
    Py_DECREF(ptr);
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = fn(&s, &d, p, st);
    Py_END_ALLOW_THREADS
    if (status == WENO_OK) return out;
    Py_DECREF(out);
    return PyLong_FromLong(status);
}

// zoom2x_backward(fn, params, x, grad_y, grad_x) -> status, or None
static PyObject* native_backward(PyObject* self, PyObject* const* a, Py_ssize_t na)
{
    (void)self;
    if (na != 5) return PyErr_Format(PyExc_TypeError, "zoom2x_backward takes 5 arguments");
    const fn_bwd fn = (fn_bwd)address(a[0]);
    const weno_params_t* p = (const weno_params_t*)address(a[1]);
    if (!fn || !p) return PyErr_Occurred() ? NULL : PyErr_Format(PyExc_ValueError, "null address");
    weno_tensor_t x, gy, gx;
    int dev = 0;
    int rc = describe(a[2], &x, &dev);
    if (rc == 1) rc = describe(a[3], &gy, NULL);
    if (rc == 1) rc = describe(a[4], &gx, NULL);
    if (rc < 0) return NULL;
    if (rc == 0) Py_RETURN_NONE;
    void* st;
    if (current_stream(dev, &st)) return NULL;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = fn(&x, &gy, &gx, p, st);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

// init(torch.uint8, torch.float32, torch.empty, raw stream query, torch.Tensor)
static PyObject* native_init(PyObject* self, PyObject* const* a, Py_ssize_t na)
{
    (void)self;
    if (na != 5) return PyErr_Format(PyExc_TypeError, "init takes 5 arguments");
    PyObject** dst[5] = {&g_u8, &g_f32, &g_empty, &g_raw_stream, &g_tensor};
    for (int i = 0; i < 5; ++i) {
        Py_INCREF(a[i]);
        Py_XDECREF(*dst[i]);
        *dst[i] = a[i];
    }
    Py_RETURN_NONE;
}

static PyMethodDef kMethods[] = {
    {"init", (PyCFunction)(void (*)(void))native_init, METH_FASTCALL, NULL},
    {"zoom2x_", (PyCFunction)(void (*)(void))native_zoom2x_into, METH_FASTCALL, NULL},
    {"zoom2x", (PyCFunction)(void (*)(void))native_zoom2x, METH_FASTCALL, NULL},
    {"zoom2x_backward", (PyCFunction)(void (*)(void))native_backward, METH_FASTCALL, NULL},
    {NULL, NULL, 0, NULL},
};

static struct PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_native", NULL, -1, kMethods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__native(void)
{
    s_is_cuda = PyUnicode_InternFromString("is_cuda");
    s_dtype = PyUnicode_InternFromString("dtype");
    s_shape = PyUnicode_InternFromString("shape");
    s_stride = PyUnicode_InternFromString("stride");
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_device = PyUnicode_InternFromString("device");
    s_get_device = PyUnicode_InternFromString("get_device");
    s_kw_dtype_device = Py_BuildValue("(OO)", s_dtype, s_device);
    if (!s_is_cuda || !s_dtype || !s_shape || !s_stride || !s_data_ptr || !s_device || !s_get_device ||
        !s_kw_dtype_device)
        return NULL;
    return PyModule_Create(&kModule);
}
