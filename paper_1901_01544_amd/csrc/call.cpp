// The Python binding's way into the library: arguments of the hot calls -> the C functions of include/iwp.h.  Argument
// marshalling only; the library itself is opened by iwp.py, which hands over its functions' addresses (bind).
//
// Bound by the host: a call is a few launches of 3 us each, and through ctypes the arguments of one took 4 to 8 us (0.4 us per
// tensor for its three checks, 0.9 us per table of workers, 1.1 us for the call).  A small exchange (two calls, one launch
// each, two workers) 17.4 -> 9.9 us; the first pass on a new state 10 to 40 us less, whatever its size.
//
// The converters follow from the functions' types: a pointer takes a tensor (on the device and contiguous), an address or
// None; a pointer to pointers a sequence of those; numbers what ctypes took.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>
#include <tuple>
#include <utility>

#include "../../include/iwp.h"

namespace {

PyObject *s_is_cuda, *s_is_contiguous, *s_data_ptr;      // interned

bool address(PyObject* o, uintptr_t* out) {
    if (o == Py_None) {
        *out = 0;
        return true;
    }
    if (PyLong_Check(o)) {
        *out = (uintptr_t)PyLong_AsUnsignedLongLongMask(o);
        return !PyErr_Occurred();
    }
    PyObject* x = PyObject_GetAttr(o, s_is_cuda);
    if (!x) return false;
    int ok = PyObject_IsTrue(x);
    Py_DECREF(x);
    if (ok == 1) {
        x = PyObject_CallMethodNoArgs(o, s_is_contiguous);
        if (!x) return false;
        ok = PyObject_IsTrue(x);
        Py_DECREF(x);
    }
    if (ok != 1) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_AssertionError, "contiguous device tensor required");
        return false;
    }
    x = PyObject_CallMethodNoArgs(o, s_data_ptr);
    if (!x) return false;
    *out = (uintptr_t)PyLong_AsUnsignedLongLong(x);
    Py_DECREF(x);
    return !PyErr_Occurred();
}

template <class T> struct Arg;
template <class T> struct Arg<T*> {
    uintptr_t at = 0;
    bool from(PyObject* o) { return address(o, &at); }
    T* get() { return reinterpret_cast<T*>(at); }
};
template <class T> struct Arg<T* const*> {               // one entry per worker
    static constexpr Py_ssize_t FEW = IWP_MAX_WORKERS;
    uintptr_t few[FEW];
    uintptr_t* at = few;
    bool from(PyObject* o) {
        PyObject* seq = PySequence_Fast(o, "a sequence of tensors, one per worker");
        if (!seq) return false;
        const Py_ssize_t n = PySequence_Fast_GET_SIZE(seq);
        bool ok = true;
        if (n > FEW) {                                   // the library turns such a call away, by the number of workers
            at = static_cast<uintptr_t*>(PyMem_Malloc(n * sizeof(uintptr_t)));
            if (!at) {
                PyErr_NoMemory();
                ok = false;
            }
        }
        for (Py_ssize_t p = 0; ok && p < n; ++p) ok = address(PySequence_Fast_GET_ITEM(seq, p), at + p);
        Py_DECREF(seq);
        return ok;
    }
    ~Arg() { if (at != few) PyMem_Free(at); }
    T* const* get() { return reinterpret_cast<T* const*>(at); }
};
template <class T> bool unsigned_from(PyObject* o, T* out) {
    PyObject* x = PyNumber_Index(o);
    if (!x) return false;
    *out = (T)PyLong_AsUnsignedLongLongMask(x);
    Py_DECREF(x);
    return !PyErr_Occurred();
}
template <> struct Arg<uint32_t> {
    uint32_t x = 0;
    bool from(PyObject* o) { return unsigned_from(o, &x); }
    uint32_t get() { return x; }
};
template <> struct Arg<uint64_t> {
    uint64_t x = 0;
    bool from(PyObject* o) { return unsigned_from(o, &x); }
    uint64_t get() { return x; }
};
template <> struct Arg<float> {
    double x = 0;
    bool from(PyObject* o) { x = PyFloat_AsDouble(o); return x != -1.0 || !PyErr_Occurred(); }
    float get() { return (float)x; }
};
template <> struct Arg<double> {
    double x = 0;
    bool from(PyObject* o) { x = PyFloat_AsDouble(o); return x != -1.0 || !PyErr_Occurred(); }
    double get() { return x; }
};

template <class... A, size_t... I>
PyObject* call_with(int (*f)(A...), PyObject* const* args, std::index_sequence<I...>) {
    std::tuple<Arg<A>...> a;
    if (!(std::get<I>(a).from(args[I]) && ...)) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f(std::get<I>(a).get()...);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

template <class... A>
PyObject* call(const char* name, int (*f)(A...), PyObject* const* args, Py_ssize_t n) {
    if (!f) return PyErr_Format(PyExc_RuntimeError, "%s: the library is not loaded", name);
    if (n != (Py_ssize_t)sizeof...(A))
        return PyErr_Format(PyExc_TypeError, "%s takes %zd arguments, not %zd", name, (Py_ssize_t)sizeof...(A), n);
    return call_with(f, args, std::index_sequence_for<A...>());
}

#define EACH_HOT_CALL(DO)                                                                                         \
    DO(compress_layer) DO(select_threshold) DO(compact_pairs) DO(gather_sum_at_indices) DO(apply_sparse_update)   \
    DO(compress_segmented) DO(compress_segmented_static) DO(iwp_step_segmented) DO(select_threshold_segmented)    \
    DO(compact_pairs_segmented) DO(iwp_step_threshold_segmented) DO(iwp_step_threshold_random_segmented)          \
    DO(iwp_step_layerwise_segmented)

#define DO(name)                                                                    \
    decltype(&::name) f_##name = nullptr;                                           \
    PyObject* py_##name(PyObject*, PyObject* const* args, Py_ssize_t n) {           \
        return call(#name, f_##name, args, n);                                      \
    }
EACH_HOT_CALL(DO)
#undef DO

// bind({name: address}): where the loaded library's functions are.
PyObject* bind(PyObject*, PyObject* addresses) {
    if (!PyDict_Check(addresses)) return PyErr_Format(PyExc_TypeError, "a dict of addresses");
#define DO(name)                                                                                              \
    {                                                                                                         \
        PyObject* o = PyDict_GetItemString(addresses, #name);                                                 \
        if (!o) return PyErr_Format(PyExc_KeyError, #name);                                                   \
        const uintptr_t at = (uintptr_t)PyLong_AsUnsignedLongLong(o);                                         \
        if (PyErr_Occurred()) return nullptr;                                                                 \
        f_##name = reinterpret_cast<decltype(&::name)>(at);                                                   \
    }
    EACH_HOT_CALL(DO)
#undef DO
    Py_RETURN_NONE;
}

PyObject* names(PyObject*, PyObject*) {
    PyObject* out = PyList_New(0);
#define DO(name)                                                   \
    if (out) {                                                     \
        PyObject* s = PyUnicode_FromString(#name);                 \
        if (!s || PyList_Append(out, s)) { Py_CLEAR(out); }        \
        Py_XDECREF(s);                                             \
    }
    EACH_HOT_CALL(DO)
#undef DO
    return out;
}

PyMethodDef methods[] = {
#define DO(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_##name)), METH_FASTCALL, nullptr},
    EACH_HOT_CALL(DO)
#undef DO
    {"bind", bind, METH_O, nullptr},
    {"names", names, METH_NOARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__call(void) {
    s_is_cuda = PyUnicode_InternFromString("is_cuda");
    s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    if (!s_is_cuda || !s_is_contiguous || !s_data_ptr) return nullptr;
    return PyModule_Create(&module);
}
