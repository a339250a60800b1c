// CPython extension: torch tensors to bellman_tensor_t descriptors and one
// library call, without the ctypes structures in between.  A decode step of
// two library calls spent 18 of its 33 us of host time building thirteen
// ctypes descriptors and looking the current stream up.
//
// call() handles plain device tensors of the library's element types and
// returns the library's status; for anything else it returns None before the
// library is called, and the caller's general path raises the right error.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>

#include "../../include/bellman.h"

namespace {

PyObject *g_tensor, *g_parameter;             // the exact types taken
PyObject* g_dtype[5];                         // torch dtypes, and their codes
int32_t g_code[5];
PyObject *g_raw_stream, *g_device;            // current stream of a device, current device
PyObject *s_is_cuda, *s_dtype, *s_shape, *s_stride, *s_data_ptr, *s_is_contiguous;
int g_float32 = -1;                           // index of float32 in g_dtype

struct Ref {                                  // an owned reference, or an error
    PyObject* p;
    explicit Ref(PyObject* o) : p(o) {}
    ~Ref() { Py_XDECREF(p); }
    Ref(const Ref&) = delete;
    Ref& operator=(const Ref&) = delete;
};

bool is_true(PyObject* t, PyObject* name) {
    Ref r(PyObject_GetAttr(t, name));
    return r.p == Py_True;
}

bool address(PyObject* t, void** out) {
    Ref r(PyObject_CallMethodNoArgs(t, s_data_ptr));
    if (!r.p) return false;
    *out = PyLong_AsVoidPtr(r.p);
    return !PyErr_Occurred();
}

bool device_tensor(PyObject* t) {
    PyObject* type = (PyObject*)Py_TYPE(t);
    return (type == g_tensor || type == g_parameter) && is_true(t, s_is_cuda);
}

int dtype_index(PyObject* t) {
    Ref r(PyObject_GetAttr(t, s_dtype));
    for (int i = 0; i < 5; ++i)
        if (r.p == g_dtype[i]) return i;
    return -1;
}

bool ints(PyObject* seq, int64_t* out) {      // a tuple (or torch.Size) of plain ints
    if (!PyTuple_Check(seq)) return false;
    const Py_ssize_t n = PyTuple_GET_SIZE(seq);
    for (Py_ssize_t i = 0; i < n; ++i) {
        PyObject* v = PyTuple_GET_ITEM(seq, i);
        if (!PyLong_CheckExact(v)) return false;
        out[i] = PyLong_AsLongLong(v);
        if (out[i] == -1 && PyErr_Occurred()) return false;
    }
    return true;
}

// false: not a case for this path (a Python error may be set)
bool fill(PyObject* t, PyObject* scale, bellman_tensor_t* d) {
    if (!device_tensor(t)) return false;
    const int dt = dtype_index(t);
    if (dt < 0) return false;
    *d = bellman_tensor_t{};
    d->dtype = g_code[dt];
    Ref shape(PyObject_GetAttr(t, s_shape));
    if (!shape.p || !PyTuple_Check(shape.p) || PyTuple_GET_SIZE(shape.p) > BELLMAN_MAX_DIMS) return false;
    d->ndim = (int32_t)PyTuple_GET_SIZE(shape.p);
    Ref stride(PyObject_CallMethodNoArgs(t, s_stride));
    if (!stride.p || !PyTuple_Check(stride.p) || PyTuple_GET_SIZE(stride.p) != d->ndim) return false;
    if (!ints(shape.p, d->shape) || !ints(stride.p, d->stride)) return false;
    bool empty = false;
    for (int i = 0; i < d->ndim; ++i) empty = empty || d->shape[i] == 0;
    if (!empty && !address(t, &d->data)) return false;
    if (scale != Py_None) {
        if (!device_tensor(scale) || dtype_index(scale) != g_float32) return false;
        Ref c(PyObject_CallMethodNoArgs(scale, s_is_contiguous));
        void* p = nullptr;
        if (c.p != Py_True || !address(scale, &p)) return false;
        d->dequant_scale = (const float*)p;
    }
    return true;
}

// The calls' forms: tensors before and after the softmax scale, the position
// of k_pages (v_pages follows), and whether the options come before the stream.
struct Form {
    int before, after, pages;
    bool opts;
};
const Form kForms[] = {
    {6, 0, 2, false},   // 0 kv_append
    {5, 1, 1, false},   // 1 decode_attention
    {5, 1, 1, true},    // 2 decode_attention_noalloc
    {7, 1, 3, true},    // 3 decode_step
    {7, 0, 2, false},   // 4 kv_write
    {6, 1, 1, false},   // 5 prefill_attention
};

typedef bellman_tensor_t T;

int invoke(void* fn, int form, T* d, float scale, void* opts, void* stream) {
    switch (form) {
        case 0: return ((int (*)(T*, T*, T*, T*, T*, T*, void*))fn)(d, d + 1, d + 2, d + 3, d + 4, d + 5, stream);
        case 1: return ((int (*)(T*, T*, T*, T*, T*, float, T*, void*))fn)(d, d + 1, d + 2, d + 3, d + 4, scale, d + 5, stream);
        case 2: return ((int (*)(T*, T*, T*, T*, T*, float, T*, void*, void*))fn)(d, d + 1, d + 2, d + 3, d + 4, scale, d + 5, opts, stream);
        case 3: return ((int (*)(T*, T*, T*, T*, T*, T*, T*, float, T*, void*, void*))fn)(d, d + 1, d + 2, d + 3, d + 4, d + 5, d + 6, scale, d + 7, opts, stream);
        case 4: return ((int (*)(T*, T*, T*, T*, T*, T*, T*, void*))fn)(d, d + 1, d + 2, d + 3, d + 4, d + 5, d + 6, stream);
        default: return ((int (*)(T*, T*, T*, T*, T*, T*, float, T*, void*))fn)(d, d + 1, d + 2, d + 3, d + 4, d + 5, scale, d + 6, stream);
    }
}

// call(function address, form, stream or None, scale, options address,
//      k_scale, v_scale, tensor, ...)
PyObject* call(PyObject*, PyObject* const* a, Py_ssize_t n) {
    constexpr int kFixed = 7;
    if (n < kFixed || !g_tensor) {
        PyErr_SetString(PyExc_TypeError, "call: too few arguments, or setup() has not run");
        return nullptr;
    }
    void* fn = PyLong_AsVoidPtr(a[0]);
    const long form = PyLong_AsLong(a[1]);
    void* opts = PyLong_AsVoidPtr(a[4]);
    if (PyErr_Occurred()) return nullptr;
    if (form < 0 || form >= (long)(sizeof kForms / sizeof kForms[0]) ||
        n - kFixed != kForms[form].before + kForms[form].after) {
        PyErr_SetString(PyExc_TypeError, "call: unknown form, or the wrong number of tensors for it");
        return nullptr;
    }
    const Form& f = kForms[form];
    T d[8];
    for (int i = 0; i < (int)(n - kFixed); ++i) {
        PyObject* s = i == f.pages ? a[5] : i == f.pages + 1 ? a[6] : Py_None;
        if (!fill(a[kFixed + i], s, &d[i])) {
            PyErr_Clear();
            Py_RETURN_NONE;
        }
    }
    const double scale = f.after ? PyFloat_AsDouble(a[3]) : 0.0;
    if (PyErr_Occurred()) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    void* stream;
    if (a[2] == Py_None) {
        Ref dev(PyObject_CallNoArgs(g_device));
        if (!dev.p) return nullptr;
        Ref raw(PyObject_CallOneArg(g_raw_stream, dev.p));
        if (!raw.p) return nullptr;
        stream = PyLong_AsVoidPtr(raw.p);
    } else {
        stream = PyLong_AsVoidPtr(a[2]);
    }
    if (PyErr_Occurred()) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = invoke(fn, (int)form, d, (float)scale, opts, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// setup(Tensor, Parameter, ((dtype, code), ...5), float32, raw_stream, device)
PyObject* setup(PyObject*, PyObject* args) {
    PyObject *tensor, *parameter, *dtypes, *f32, *raw, *dev;
    if (!PyArg_ParseTuple(args, "OOO!OOO", &tensor, &parameter, &PyTuple_Type, &dtypes, &f32, &raw, &dev)) return nullptr;
    if (PyTuple_GET_SIZE(dtypes) != 5) {
        PyErr_SetString(PyExc_ValueError, "setup: five element types");
        return nullptr;
    }
    for (int i = 0; i < 5; ++i) {
        PyObject* dt;
        int code;
        if (!PyArg_ParseTuple(PyTuple_GET_ITEM(dtypes, i), "Oi", &dt, &code)) return nullptr;
        Py_INCREF(dt);
        Py_XDECREF(g_dtype[i]);
        g_dtype[i] = dt;
        g_code[i] = code;
        if (dt == f32) g_float32 = i;
    }
    PyObject** const slots[] = {&g_tensor, &g_parameter, &g_raw_stream, &g_device};
    PyObject* const vals[] = {tensor, parameter, raw, dev};
    for (int i = 0; i < 4; ++i) {
        Py_INCREF(vals[i]);
        Py_XDECREF(*slots[i]);
        *slots[i] = vals[i];
    }
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"call", (PyCFunction)(void (*)(void))call, METH_FASTCALL, "one library call on device tensors; None if it is not a case for this path"},
    {"setup", setup, METH_VARARGS, "the torch objects call() compares with"},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) {
    s_is_cuda = PyUnicode_InternFromString("is_cuda");
    s_dtype = PyUnicode_InternFromString("dtype");
    s_shape = PyUnicode_InternFromString("shape");
    s_stride = PyUnicode_InternFromString("stride");
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
    if (!s_is_cuda || !s_dtype || !s_shape || !s_stride || !s_data_ptr || !s_is_contiguous) return nullptr;
    return PyModule_Create(&module);
}
