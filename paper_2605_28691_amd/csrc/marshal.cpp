// The calls of the Python binding, marshalled natively: every entry point of include/skiparse.h that launches kernels as a function of a CPython
// module, with the argument list of the C function, tensors in the places of device pointers.
//
// A small call is bound by what it costs to issue it: a kernel of 3 us behind 5.2 us of host work.  Of these the native call takes 3.9, nearly all of it the
// launch (a fill of a tensor by torch, one launch as well, takes 4.0), the result's tensor 1.1 and the checks and look-ups in Python 0.5.  By way of ctypes, with
// an address asked for tensor by tensor in Python, the call took 2 us more.  Here an argument costs nanoseconds.
//
// Only plain arguments are taken: torch.Tensor itself, on the GPU and contiguous, int and float themselves.  With anything else, and to turn a
// code into an exception, the module calls the functions that the binding has given it, so that what those accept, refuse and raise does not
// depend on this module.
//
// The module is not linked to the library: the binding hands it the addresses in the copy that it has opened itself, so that a process that
// rebuilds the library calls one copy only.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>
#include <tuple>
#include <utility>

#include "../../include/skiparse.h"

namespace {

#ifndef BUILT_FOR
#error "the torch that the headers belong to"
#endif

PyObject* g_general = nullptr;  // (name, *arguments): the same call by way of ctypes
PyObject* g_failed = nullptr;   // (code, name): raises

template <typename T>
struct Arg;
template <>
struct Arg<int> {
    static bool get(PyObject* o, int& v) {
        if (!PyLong_CheckExact(o)) return false;
        v = (int)PyLong_AsUnsignedLongMask(o);  // as ctypes does, without a range check
        return true;
    }
};
template <>
struct Arg<unsigned> {
    static bool get(PyObject* o, unsigned& v) {
        if (!PyLong_CheckExact(o)) return false;
        v = (unsigned)PyLong_AsUnsignedLongMask(o);
        return true;
    }
};
template <>
struct Arg<size_t> {
    static bool get(PyObject* o, size_t& v) {
        if (!PyLong_CheckExact(o)) return false;
        v = (size_t)PyLong_AsUnsignedLongLongMask(o);
        return true;
    }
};
template <>
struct Arg<float> {
    static bool get(PyObject* o, float& v) {
        if (!PyFloat_CheckExact(o)) return false;
        v = (float)PyFloat_AS_DOUBLE(o);
        return true;
    }
};
template <typename P>
struct Arg<P*> {
    static bool get(PyObject* o, P*& v) {
        if (!THPVariable_CheckExact(o)) return false;
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.is_cuda() || !t.is_contiguous()) return false;
        v = (P*)t.data_ptr();
        return true;
    }
};

// Argument I of N: the last one is the stream's handle; argument NONE may be None.
template <size_t I, size_t N, size_t NONE, typename T>
bool get_arg(PyObject* o, T& v) {
    if constexpr (I + 1 == N) {
        if (!PyLong_CheckExact(o)) return false;
        v = (T)(uintptr_t)PyLong_AsUnsignedLongLongMask(o);
        return true;
    } else {
        if constexpr (I == NONE) {
            if (o == Py_None) {
                v = nullptr;
                return true;
            }
        }
        return Arg<T>::get(o, v);
    }
}

// The arguments as they came, with one more in front.
PyObject* pass_on(PyObject* callable, PyObject* first, PyObject* const* args, Py_ssize_t n) {
    PyObject* all = PyTuple_New(n + 1);
    if (all == nullptr) return nullptr;
    Py_INCREF(first);
    PyTuple_SET_ITEM(all, 0, first);
    for (Py_ssize_t i = 0; i < n; i++) {
        Py_INCREF(args[i]);
        PyTuple_SET_ITEM(all, i + 1, args[i]);
    }
    PyObject* r = PyObject_CallObject(callable, all);
    Py_DECREF(all);
    return r;
}

PyObject* general(const char* name, PyObject* const* args, Py_ssize_t n) {
    if (g_general == nullptr) {
        PyErr_SetString(PyExc_RuntimeError, "the binding has not been set up");
        return nullptr;
    }
    PyObject* first = PyUnicode_FromString(name);
    if (first == nullptr) return nullptr;
    PyObject* r = pass_on(g_general, first, args, n);
    Py_DECREF(first);
    return r;
}

template <size_t NONE, typename... A, size_t... I>
PyObject* call_with(int (*fn)(A...), const char* name, PyObject* const* args, Py_ssize_t n, std::index_sequence<I...>) {
    std::tuple<A...> v;
    bool plain = n == (Py_ssize_t)sizeof...(A) && g_general != nullptr && g_failed != nullptr;
    try {
        plain = plain && (get_arg<I, sizeof...(A), NONE>(args[I], std::get<I>(v)) && ...);
    } catch (...) {  // a tensor without storage: the general way says so
        plain = false;
    }
    if (!plain) return general(name, args, n);
    int code;
    Py_BEGIN_ALLOW_THREADS
    code = fn(std::get<I>(v)...);
    Py_END_ALLOW_THREADS
    if (code == SKIPARSE_OK) Py_RETURN_NONE;
    return PyObject_CallFunction(g_failed, "is", code, name);
}

template <size_t NONE, typename... A>
PyObject* call(int (*fn)(A...), const char* name, PyObject* const* args, Py_ssize_t n) {
    return call_with<NONE>(fn, name, args, n, std::index_sequence_for<A...>{});
}

constexpr size_t NEVER = ~(size_t)0;
// address of the C function: none until the binding has opened the library, and the general way is taken (which opens it)
#define SLOT(name, none) decltype(&::name) g_##name = nullptr;
// argument that may be None: the workspace of the forward layer, which the fused form does not need
#define ENTRY(name, none)                                                 \
    PyObject* py_##name(PyObject*, PyObject* const* args, Py_ssize_t n) { \
        return g_##name ? call<none>(g_##name, #name, args, n) : general(#name, args, n); \
    }
#define BIND(name, none) \
    if (strcmp(what, #name) == 0) g_##name = (decltype(g_##name))address;
#define LISTED(name, none) {#name, (PyCFunction)(void (*)(void))py_##name, METH_FASTCALL, nullptr},
#define ENTRIES(X) \
    X(skiparse_attn_fwd, 15) \
    X(skiparse_permute, NEVER) \
    X(skiparse_unpermute, NEVER) \
    X(skiparse_switch_pattern, NEVER) \
    X(skiparse_ssp_pack, NEVER) \
    X(skiparse_ssp_unpack, NEVER) \
    X(dense_attn_fwd, NEVER) \
    X(skiparse_attn_fwd_sparse, NEVER) \
    X(skiparse_attn_fwd_lse, NEVER) \
    X(skiparse_attn_bwd, NEVER) \
    X(skiparse_attn_bwd_static, NEVER) \
    X(skiparse_quantize_fp8_ex, NEVER) \
    X(skiparse_attn_fwd_fp8_ex, NEVER)
ENTRIES(SLOT)
ENTRIES(ENTRY)

PyObject* set_up(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != 2 || !PyCallable_Check(args[0]) || !PyCallable_Check(args[1])) {
        PyErr_SetString(PyExc_TypeError, "set_up(general, failed)");
        return nullptr;
    }
    Py_INCREF(args[0]);
    Py_INCREF(args[1]);
    Py_XDECREF(g_general);
    Py_XDECREF(g_failed);
    g_general = args[0];
    g_failed = args[1];
    Py_RETURN_NONE;
}

PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n) {
    const char* what = n == 2 ? PyUnicode_AsUTF8(args[0]) : nullptr;
    void* address = what != nullptr ? PyLong_AsVoidPtr(args[1]) : nullptr;
    if (PyErr_Occurred()) return nullptr;
    if (address == nullptr) {
        PyErr_SetString(PyExc_TypeError, "bind(name, address)");
        return nullptr;
    }
    ENTRIES(BIND)
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {ENTRIES(LISTED){"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, nullptr},
                         {"set_up", (PyCFunction)(void (*)(void))set_up, METH_FASTCALL, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", "Native marshalling of the binding's calls.", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject* PyInit__marshal() {
    PyObject* m = PyModule_Create(&module);
    if (m != nullptr && PyModule_AddStringConstant(m, "BUILT_FOR", BUILT_FOR) != 0) Py_CLEAR(m);
    return m;
}
