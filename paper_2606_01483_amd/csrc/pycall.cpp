// Python entry to the per-step calls of libmurmur (include/murmur.h): converts
// the arguments of one call in C and makes it.  murmur.py's ctypes calls did
// the same in about 4.4 us for a decode step of 22 arguments, more than the
// launch itself; this takes about 1.2 us.  Each function takes the C function's
// address (from the library that murmur.py has loaded) and its arguments, and
// returns the status, or NotImplemented for an argument of a type it does not
// take, which murmur.py then hands to ctypes.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <tuple>
#include <utility>

#include "murmur.h"

namespace {

PyObject *g_data_ptr;  // "data_ptr"
// murmur.py's classes of the two structures (structures(), called once when it is imported)
PyTypeObject *g_kv_type, *g_ring_type;

// One argument: get() is false when the object is not taken (with or without
// an exception set).
template <typename T>
struct Arg;

template <typename T>
struct Arg<T *> {  // device or host address: None, an int, or an object with data_ptr()
    T *v = nullptr;
    bool get(PyObject *o) {
        if (o == Py_None) return true;
        PyObject *n = o;
        if (PyLong_Check(o)) {
            Py_INCREF(n);
        } else {
            n = PyObject_CallMethodNoArgs(o, g_data_ptr);
            if (!n) return false;
        }
        const unsigned long long a = PyLong_AsUnsignedLongLongMask(n);
        Py_DECREF(n);
        if (a == (unsigned long long)-1 && PyErr_Occurred()) return false;
        v = reinterpret_cast<T *>(a);
        return true;
    }
};

template <typename T, PyTypeObject *&type>
struct StructArg {  // None, or the ctypes structure itself, by its buffer
    Py_buffer b{};
    const T *v = nullptr;
    bool get(PyObject *o) {
        if (o == Py_None) return true;
        if (!type || !PyObject_TypeCheck(o, type)) return false;
        if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) {
            PyErr_Clear();
            return false;
        }
        if (b.len < (Py_ssize_t)sizeof(T)) return false;
        v = static_cast<const T *>(b.buf);
        return true;
    }
    ~StructArg() {
        if (b.obj) PyBuffer_Release(&b);
    }
};
template <>
struct Arg<const murmur_kv *> : StructArg<murmur_kv, g_kv_type> {};
template <>
struct Arg<const murmur_ring *> : StructArg<murmur_ring, g_ring_type> {};

template <>
struct Arg<int32_t> {
    int32_t v = 0;
    bool get(PyObject *o) {
        if (!PyLong_Check(o)) return false;
        int over = 0;
        const long x = PyLong_AsLongAndOverflow(o, &over);
        v = (int32_t)x;
        return over == 0 && (long)v == x;
    }
};
template <>
struct Arg<size_t> {
    size_t v = 0;
    bool get(PyObject *o) {
        if (!PyLong_Check(o)) return false;
        int over = 0;
        const long x = PyLong_AsLongAndOverflow(o, &over);
        v = (size_t)x;
        return over == 0 && x >= 0;
    }
};
template <>
struct Arg<float> {
    float v = 0.f;
    bool get(PyObject *o) {
        if (!PyFloat_Check(o)) return false;
        v = (float)PyFloat_AS_DOUBLE(o);
        return true;
    }
};

template <typename... A, size_t... I>
PyObject *call(int (*)(A...), PyObject *const *args, std::index_sequence<I...>) {
    const unsigned long long address = PyLong_AsUnsignedLongLong(args[0]);
    if (PyErr_Occurred()) return nullptr;
    std::tuple<Arg<A>...> v;
    if (!(std::get<I>(v).get(args[1 + I]) && ...)) {
        if (PyErr_Occurred()) return nullptr;
        Py_RETURN_NOTIMPLEMENTED;
    }
    const auto fn = reinterpret_cast<int (*)(A...)>(address);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = fn(std::get<I>(v).v...);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

template <typename... A>
std::integral_constant<size_t, sizeof...(A)> arity_of(int (*)(A...));

#define ENTRY(name)                                                                                       \
    PyObject *name(PyObject *, PyObject *const *args, Py_ssize_t n) {                                     \
        constexpr size_t count = decltype(arity_of(&murmur_##name))::value;                               \
        if (n != (Py_ssize_t)count + 1) {                                                                 \
            PyErr_SetString(PyExc_TypeError, #name ": wrong number of arguments");                        \
            return nullptr;                                                                               \
        }                                                                                                 \
        return call(static_cast<decltype(&murmur_##name)>(nullptr), args, std::make_index_sequence<count>{}); \
    }

ENTRY(evict_compact)
ENTRY(evict_compact_paged)
ENTRY(decode_attn)
ENTRY(decode_step)
ENTRY(decode_step_static)
ENTRY(decode_step_ring)
ENTRY(paged_step)

PyObject *structures(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != 2 || !PyType_Check(args[0]) || !PyType_Check(args[1])) {
        PyErr_SetString(PyExc_TypeError, "structures: the classes of murmur_kv and murmur_ring");
        return nullptr;
    }
    Py_INCREF(args[0]);
    Py_INCREF(args[1]);
    Py_XDECREF(g_kv_type);
    Py_XDECREF(g_ring_type);
    g_kv_type = reinterpret_cast<PyTypeObject *>(args[0]);
    g_ring_type = reinterpret_cast<PyTypeObject *>(args[1]);
    Py_RETURN_NONE;
}

#define METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {METHOD(evict_compact),      METHOD(evict_compact_paged), METHOD(decode_attn),
                           METHOD(decode_step),        METHOD(decode_step_static),  METHOD(decode_step_ring),
                           METHOD(paged_step),         METHOD(structures),          {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_pycall", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pycall(void) {
    g_data_ptr = PyUnicode_InternFromString("data_ptr");
    return g_data_ptr ? PyModule_Create(&g_module) : nullptr;
}
