// Python calls of the library's execute entry points, without ctypes: argument conversion in C.
//
// A pass over a small tensor is bound by the host (a kernel of 3 us; the launch itself takes 3.3), and
// ctypes spends 0.5 us of it on four pointer objects and the foreign call, 0.9 on the two argument
// arrays of the one-call interface.  These functions take the same Python objects with the same
// conversions (int() of extents and permutation entries; None or an int for a pointer) and release the
// interpreter lock around the call, as ctypes does.  They return the status; binding.py raises.
//
// The library is not linked: bind() receives the entry points' addresses from the one copy that
// binding.py has loaded.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include "../../include/tperm.h"

namespace {

decltype(&tperm_execute) g_execute, g_accumulate;
decltype(&tperm_execute_verified) g_verified;
decltype(&tperm_transpose) g_transpose, g_transpose_accumulate;
decltype(&tperm_product_accumulate) g_product;

// None or an int; anything else is a TypeError.
bool to_pointer(PyObject* o, void** p) {
    if (o == Py_None) {
        *p = nullptr;
        return true;
    }
    if (!PyLong_Check(o)) {
        PyErr_Format(PyExc_TypeError, "cannot be converted to pointer: %.100s", Py_TYPE(o)->tp_name);
        return false;
    }
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);
    if (v == (unsigned long long)-1 && PyErr_Occurred()) return false;
    *p = (void*)(uintptr_t)v;
    return true;
}

// int(o), reduced to 64 bits.
bool to_int64(PyObject* o, int64_t* v) {
    PyObject* n = PyNumber_Long(o);
    if (n == nullptr) return false;
    const unsigned long long u = PyLong_AsUnsignedLongLongMask(n);
    Py_DECREF(n);
    if (u == (unsigned long long)-1 && PyErr_Occurred()) return false;
    *v = (int64_t)u;
    return true;
}

bool count_is(const char* name, Py_ssize_t n, Py_ssize_t want) {
    if (n == want) return true;
    PyErr_Format(PyExc_TypeError, "%s takes %zd arguments (%zd given)", name, want, n);
    return false;
}

bool pointers(PyObject* const* args, int n, void** p) {
    for (int i = 0; i < n; ++i)
        if (!to_pointer(args[i], &p[i])) return false;
    return true;
}

PyObject* plain(const char* name, decltype(&tperm_execute) f, PyObject* const* args, Py_ssize_t n) {
    void* p[4];
    if (!count_is(name, n, 4) || !pointers(args, 4, p)) return nullptr;
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = f((tperm_plan_t)p[0], p[1], p[2], p[3]);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

PyObject* execute(PyObject*, PyObject* const* args, Py_ssize_t n) { return plain("execute", g_execute, args, n); }
PyObject* accumulate(PyObject*, PyObject* const* args, Py_ssize_t n) { return plain("accumulate", g_accumulate, args, n); }

// plan, in, out, stream, verdict, workspace, bytes
PyObject* verified(PyObject*, PyObject* const* args, Py_ssize_t n) {
    void* p[6];
    int64_t bytes;
    if (!count_is("verified", n, 7) || !pointers(args, 6, p) || !to_int64(args[6], &bytes)) return nullptr;
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = g_verified((tperm_plan_t)p[0], p[1], p[2], p[3], (uint64_t*)p[4], p[5], (size_t)bytes);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

// product, left, right, out, workspace, stream, bytes
PyObject* product(PyObject*, PyObject* const* args, Py_ssize_t n) {
    void* p[6];
    int64_t bytes;
    if (!count_is("product", n, 7) || !pointers(args, 6, p) || !to_int64(args[6], &bytes)) return nullptr;
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = g_product((tperm_product_t)p[0], p[1], p[2], p[3], p[4], (size_t)bytes, p[5]);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

// The entries of an iterable as integers; up to TPERM_MAX_RANK of them (the library refuses longer ones
// by their number alone).  Returns their number, -1 with an exception set.  A conversion may run Python
// code, and so may change the iterable: a tuple stays as it is, anything else goes through its
// iterator, which holds a reference to each entry and ends where the entries do.
template <typename Int>
Py_ssize_t entries(PyObject* o, Int* out) {
    Py_ssize_t n = 0;
    int64_t v;
    if (PyTuple_CheckExact(o)) {
        const Py_ssize_t size = PyTuple_GET_SIZE(o);
        for (; n < size; ++n) {
            if (!to_int64(PyTuple_GET_ITEM(o, n), &v)) return -1;
            if (n < TPERM_MAX_RANK) out[n] = (Int)v;
        }
        return n;
    }
    PyObject* it = PyObject_GetIter(o);
    if (it == nullptr) return -1;
    while (PyObject* item = PyIter_Next(it)) {
        const bool ok = to_int64(item, &v);
        Py_DECREF(item);
        if (!ok) break;
        if (n < TPERM_MAX_RANK) out[n] = (Int)v;
        ++n;
    }
    Py_DECREF(it);
    return PyErr_Occurred() ? -1 : n;
}

// dims, perm, element size, in, out, stream, accumulate
PyObject* transpose(PyObject*, PyObject* const* args, Py_ssize_t n) {
    int64_t dims[TPERM_MAX_RANK] = {}, elem;
    int perm[TPERM_MAX_RANK] = {};
    void* p[3];
    if (!count_is("transpose", n, 7)) return nullptr;
    if (PyObject_Size(args[0]) < 0) return nullptr;  // extents come as a sequence: an iterator is a TypeError
    const Py_ssize_t rank = entries(args[0], dims);
    if (rank < 0) return nullptr;
    const Py_ssize_t given = entries(args[1], perm);
    if (given < 0) return nullptr;
    if (given > (rank > 1 ? rank : 1)) {
        PyErr_SetString(PyExc_IndexError, "more permutation entries than extents");
        return nullptr;
    }
    if (!to_int64(args[2], &elem) || !pointers(args + 3, 3, p)) return nullptr;
    const int acc = PyObject_IsTrue(args[6]);
    if (acc < 0) return nullptr;
    const decltype(&tperm_transpose) f = acc ? g_transpose_accumulate : g_transpose;
    const int r = rank > 1000 ? 1000 : (int)rank;
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = f(r, dims, perm, (size_t)elem, p[0], p[1], p[2]);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n) {
    void* p[6];
    if (!count_is("bind", n, 6) || !pointers(args, 6, p)) return nullptr;
    g_execute = (decltype(g_execute))p[0];
    g_accumulate = (decltype(g_accumulate))p[1];
    g_verified = (decltype(g_verified))p[2];
    g_transpose = (decltype(g_transpose))p[3];
    g_transpose_accumulate = (decltype(g_transpose_accumulate))p[4];
    g_product = (decltype(g_product))p[5];
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, nullptr},
    {"execute", (PyCFunction)(void (*)(void))execute, METH_FASTCALL, nullptr},
    {"accumulate", (PyCFunction)(void (*)(void))accumulate, METH_FASTCALL, nullptr},
    {"verified", (PyCFunction)(void (*)(void))verified, METH_FASTCALL, nullptr},
    {"product", (PyCFunction)(void (*)(void))product, METH_FASTCALL, nullptr},
    {"transpose", (PyCFunction)(void (*)(void))transpose, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall(void) { return PyModule_Create(&module); }
