// CPython module `_native`: the launching entry points of libtetri as fast calls.
//
// What bounds a small decode iteration, a chunk-level transfer or a short prompt's chunk is the host: the launch
// itself takes about 2.5 us of host time, the same call through ctypes with its arguments wrapped one by one and the
// stream looked up through torch.cuda.current_stream() took 8-10 us.  Here the arguments of a call go straight from the
// Python objects (tensors, numbers, None) to the C function: about 1 us on top of the launch.
// The functions of the library are found by name in the library that the package has loaded, so that another build
// of it can be chosen in one place.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <dlfcn.h>
#include <stdint.h>
#include <tuple>
#include <utility>

#include "tetri.h"

namespace {

PyObject *s_data_ptr, *s_cuda_stream, *s_value, *s_ctypes, *s_data;     // interned names
PyObject *g_ndarray;                                                    // numpy.ndarray
PyObject *g_get_device, *g_get_stream;                                  // torch's current device / raw current stream of a device

struct ConvError {};

uint64_t number(PyObject *x)
{
    const uint64_t v = PyLong_AsUnsignedLongLongMask(x);
    if (v == (uint64_t)-1 && PyErr_Occurred()) throw ConvError();
    return v;
}

// An address from what a caller may pass as one: None, a number, a tensor (data_ptr()), a ctypes pointer (value), a
// NumPy array (ctypes.data), whatever converts to a number.
void *address(PyObject *x)
{
    if (x == Py_None) return nullptr;
    if (PyLong_Check(x)) return (void *)(uintptr_t)number(x);
    if ((PyObject *)Py_TYPE(x) == g_ndarray) {       // (0.1 us; through its `ctypes` attribute 2 us)
        Py_buffer view;
        if (PyObject_GetBuffer(x, &view, PyBUF_SIMPLE) == 0) {
            void *p = view.buf;
            PyBuffer_Release(&view);                 // the caller's argument keeps the array alive during the call
            return p;
        }
        PyErr_Clear();                               // (not contiguous)
    }
    PyObject *r = PyObject_CallMethodNoArgs(x, s_data_ptr);
    if (!r) {
        PyErr_Clear();
        r = PyObject_GetAttr(x, s_value);
        if (!r) {
            PyErr_Clear();
            if (PyObject *c = PyObject_GetAttr(x, s_ctypes)) {
                r = PyObject_GetAttr(c, s_data);
                Py_DECREF(c);
            } else {
                PyErr_Clear();
                r = PyNumber_Long(x);
            }
            if (!r) throw ConvError();
        }
    }
    void *p = r == Py_None ? nullptr : (void *)(uintptr_t)PyLong_AsUnsignedLongLongMask(r);
    Py_DECREF(r);
    if (PyErr_Occurred()) throw ConvError();
    return p;
}

// The stream of a call: None is torch's current stream on the current device.
void *stream_of(PyObject *x)
{
    if (x == Py_None) {
        PyObject *dev = PyObject_CallNoArgs(g_get_device);
        if (!dev) throw ConvError();
        PyObject *st = PyObject_CallOneArg(g_get_stream, dev);
        Py_DECREF(dev);
        if (!st) throw ConvError();
        void *p = (void *)(uintptr_t)PyLong_AsUnsignedLongLongMask(st);
        Py_DECREF(st);
        if (PyErr_Occurred()) throw ConvError();
        return p;
    }
    if (!PyLong_Check(x)) {
        if (PyObject *r = PyObject_GetAttr(x, s_cuda_stream)) {
            void *p = (void *)(uintptr_t)PyLong_AsUnsignedLongLongMask(r);
            Py_DECREF(r);
            if (PyErr_Occurred()) throw ConvError();
            return p;
        }
        PyErr_Clear();
    }
    return address(x);
}

template <typename T> struct Conv;
template <typename T> struct Conv<T *> {
    static T *from(PyObject *x) { return static_cast<T *>(address(x)); }
};
template <> struct Conv<int32_t> {
    static int32_t from(PyObject *x)
    {
        if (PyLong_Check(x)) return (int32_t)number(x);
        PyObject *n = PyNumber_Long(x);
        if (!n) throw ConvError();
        const int32_t v = (int32_t)PyLong_AsUnsignedLongLongMask(n);
        Py_DECREF(n);
        return v;
    }
};
template <> struct Conv<int64_t> {
    static int64_t from(PyObject *x)
    {
        if (PyLong_Check(x)) return (int64_t)number(x);
        PyObject *n = PyNumber_Long(x);
        if (!n) throw ConvError();
        const int64_t v = (int64_t)PyLong_AsUnsignedLongLongMask(n);
        Py_DECREF(n);
        return v;
    }
};
template <> struct Conv<float> {
    static float from(PyObject *x)
    {
        const double v = PyFloat_AsDouble(x);
        if (v == -1.0 && PyErr_Occurred()) throw ConvError();
        return (float)v;
    }
};

// One entry point: converts the arguments in order (the last one is the stream), calls with the interpreter lock
// released (as ctypes does: a launch may wait for room in the queue), returns the status.
template <typename... A, size_t... I>
PyObject *invoke(tetri_status (*fn)(A...), PyObject *const *args, std::index_sequence<I...>)
{
    constexpr size_t N = sizeof...(A);
    try {
        std::tuple<A...> a{[&]() -> A {
            if constexpr (I + 1 == N) return static_cast<A>(stream_of(args[I]));
            else return Conv<A>::from(args[I]);
        }()...};
        tetri_status st;
        Py_BEGIN_ALLOW_THREADS
        st = std::apply(fn, a);
        Py_END_ALLOW_THREADS
        return PyLong_FromLong((long)st);
    } catch (const ConvError &) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "an argument is neither a tensor, an array, a number nor None");
        return nullptr;
    }
}

template <typename F> struct Entry;
template <typename... A> struct Entry<tetri_status(A...)> {
    typedef tetri_status (*fn_t)(A...);
    static PyObject *call(fn_t fn, const char *name, PyObject *const *args, Py_ssize_t n)
    {
        if (!fn) return PyErr_Format(PyExc_RuntimeError, "%s: the library is not bound", name);
        if (n != (Py_ssize_t)sizeof...(A)) return PyErr_Format(PyExc_TypeError, "%s takes %zd arguments (%zd given)", name, (Py_ssize_t)sizeof...(A), n);
        return invoke(fn, args, std::make_index_sequence<sizeof...(A)>());
    }
};

#define TETRI_ENTRIES(X) \
    X(tetri_kv_append) X(tetri_chunk_prefill_attn) X(tetri_chunk_prefill_attn_append) X(tetri_chunk_prefill_attn_fp8) \
    X(tetri_decode_attn) X(tetri_decode_attn_static) X(tetri_decode_attn_append) X(tetri_decode_attn_fp8) \
    X(tetri_kv_export) X(tetri_kv_import) X(tetri_kv_export_fp8) X(tetri_kv_import_fp8) \
    X(tetri_chunk_prefill_planned) X(tetri_batch_upload) X(tetri_batch_launch) X(tetri_batch_step)

#define X(f) \
    decltype(&f) g_##f = nullptr; \
    PyObject *py_##f(PyObject *, PyObject *const *args, Py_ssize_t n) { return Entry<decltype(f)>::call(g_##f, #f, args, n); }
TETRI_ENTRIES(X)
#undef X

// bind(path of libtetri, torch's current-device function, torch's raw-current-stream function)
PyObject *py_bind(PyObject *, PyObject *args)
{
    const char *path;
    PyObject *dev, *st;
    if (!PyArg_ParseTuple(args, "sOO", &path, &dev, &st)) return nullptr;
    void *so = dlopen(path, RTLD_NOW | RTLD_LOCAL);
    if (!so) return PyErr_Format(PyExc_ImportError, "%s", dlerror());
#define X(f) \
    if (!(g_##f = reinterpret_cast<decltype(&f)>(dlsym(so, #f)))) return PyErr_Format(PyExc_ImportError, "%s does not export %s", path, #f);
    TETRI_ENTRIES(X)
#undef X
    Py_INCREF(dev), Py_INCREF(st);
    Py_XSETREF(g_get_device, dev);
    Py_XSETREF(g_get_stream, st);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", py_bind, METH_VARARGS, "Find the entry points in a build of libtetri."},
#define X(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(py_##f)), METH_FASTCALL, nullptr},
    TETRI_ENTRIES(X)
#undef X
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "Fast calls of libtetri's launching entry points.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    s_value = PyUnicode_InternFromString("value");
    s_ctypes = PyUnicode_InternFromString("ctypes");
    s_data = PyUnicode_InternFromString("data");
    PyObject *numpy = PyImport_ImportModule("numpy");
    if (!numpy) return nullptr;
    g_ndarray = PyObject_GetAttrString(numpy, "ndarray");
    Py_DECREF(numpy);
    if (!g_ndarray) return nullptr;
    return PyModule_Create(&module);
}
