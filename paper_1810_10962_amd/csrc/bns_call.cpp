// The calls that a program makes for every layer and step, as a CPython extension: what bns.py would hand to ctypes, marshalled in C.
// ctypes converts each argument through a type object of its own: of the 5.1 us that bns_forward took on the host, 2.7 are the library
// and the launch.  What is added to those is 0.8 us with this (8x16x8x8 f32, whose two kernels take 6.7 us on the device, with a launch that
// takes 3.7 us: a pass 10.1 -> 8.8 us; 2x512x14x14 N x H x W x C 10.6 -> 9.5).
//
// The extension knows nothing of torch: a tensor is an object with data_ptr(), None is a null pointer.  It is bound to the functions of
// the library that bns.py has loaded.  It takes the arguments that a program has in earnest: the two structures, integers, whatever has a
// floating-point value, tensors.  For anything else (ctypes scalars, objects with _as_parameter_, wrong types, a data_ptr() that fails) a
// function returns None without having called the library, and bns.py makes the call through ctypes: what that accepts is accepted, and what
// it refuses raises its exceptions.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <string.h>

#include "../../include/bns.h"

namespace {

decltype(&bns_forward) g_forward;
decltype(&bns_backward) g_backward;
decltype(&bns_forward_mixed) g_forward_mixed;
decltype(&bns_backward_mixed) g_backward_mixed;
decltype(&bns_inference) g_inference;
PyObject *g_shape_type, *g_spec_type, *g_data_ptr;

// Reads positional arguments one after the other; after one that is left to ctypes nothing more is read.  No exception stays set.
struct Reader {
    PyObject* const* at;
    bool ok;

    Reader(PyObject* const* args, Py_ssize_t given, Py_ssize_t wanted) : at(args), ok(g_shape_type && given == wanted) {}

    void leave() {
        PyErr_Clear();
        ok = false;
    }
    template <typename S>
    S structure(PyObject* type) {
        S s;
        memset(&s, 0, sizeof s);
        if (!ok) return s;
        PyObject* o = *at++;
        Py_buffer b;
        if (!PyObject_TypeCheck(o, reinterpret_cast<PyTypeObject*>(type)) || PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) {
            leave();
            return s;
        }
        if (b.len >= Py_ssize_t(sizeof s)) memcpy(&s, b.buf, sizeof s);
        else ok = false;
        PyBuffer_Release(&b);
        return s;
    }
    bns_shape shape() { return structure<bns_shape>(g_shape_type); }
    bns_spec spec() { return structure<bns_spec>(g_spec_type); }

    // an integer, reduced modulo 2^64 as ctypes does
    unsigned long long integer() {
        if (!ok) return 0;
        PyObject* o = *at++;
        ok = PyLong_Check(o);
        return ok ? PyLong_AsUnsignedLongLongMask(o) : 0;
    }
    float real() {
        if (!ok) return 0.f;
        const double v = PyFloat_AsDouble(*at++);
        if (v == -1.0 && PyErr_Occurred()) leave();
        return float(v);
    }
    void* pointer() {
        if (!ok) return nullptr;
        PyObject* o = *at++;
        if (o == Py_None) return nullptr;
        PyObject* address = PyObject_CallMethodNoArgs(o, g_data_ptr);
        void* p = nullptr;
        if (!address || !PyLong_Check(address)) leave();
        else if (!(p = PyLong_AsVoidPtr(address)) && PyErr_Occurred()) leave();
        Py_XDECREF(address);
        return p;
    }
    float* vector() { return static_cast<float*>(pointer()); }
    void* stream() { return reinterpret_cast<void*>(integer()); }
};

// (the lock is released as ctypes releases it: other threads may enqueue work meanwhile)
template <typename Call>
PyObject* finish(const Reader& r, Call&& call) {
    if (!r.ok) Py_RETURN_NONE;
    bns_status s;
    Py_BEGIN_ALLOW_THREADS
    s = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(long(s));
}

PyObject* forward(PyObject*, PyObject* const* args, Py_ssize_t n) {
    Reader r(args, n, 16);
    const bns_shape shape = r.shape();
    const bns_spec spec = r.spec();
    const uint64_t seed = r.integer();
    const void* x = r.pointer();
    const float *gamma = r.vector(), *beta = r.vector();
    const float eps = r.real(), momentum = r.real();
    void* y = r.pointer();
    float *mean = r.vector(), *invstd = r.vector(), *running_mean = r.vector(), *running_var = r.vector();
    void* workspace = r.pointer();
    const size_t bytes = r.integer();
    void* stream = r.stream();
    return finish(r, [&] {
        return g_forward(&shape, &spec, seed, x, gamma, beta, eps, momentum, y, mean, invstd, running_mean, running_var, workspace, bytes,
                         stream);
    });
}

PyObject* backward(PyObject*, PyObject* const* args, Py_ssize_t n) {
    Reader r(args, n, 14);
    const bns_shape shape = r.shape();
    const bns_spec spec = r.spec();
    const uint64_t seed = r.integer();
    const void *x = r.pointer(), *dy = r.pointer();
    const float *gamma = r.vector(), *mean = r.vector(), *invstd = r.vector();
    void* dx = r.pointer();
    float *dgamma = r.vector(), *dbeta = r.vector();
    void* workspace = r.pointer();
    const size_t bytes = r.integer();
    void* stream = r.stream();
    return finish(r, [&] {
        return g_backward(&shape, &spec, seed, x, dy, gamma, mean, invstd, dx, dgamma, dbeta, workspace, bytes, stream);
    });
}

PyObject* forward_mixed(PyObject*, PyObject* const* args, Py_ssize_t n) {
    Reader r(args, n, 19);
    const bns_shape shape = r.shape();
    const bns_spec spec = r.spec();
    const uint64_t seed = r.integer();
    const int32_t n_v = int32_t(r.integer());
    const float mix_beta = r.real();
    const void* x = r.pointer();
    const float *gamma = r.vector(), *beta = r.vector();
    const float eps = r.real(), momentum = r.real();
    void* y = r.pointer();
    float *mean = r.vector(), *invstd = r.vector(), *parts = r.vector(), *running_mean = r.vector(), *running_var = r.vector();
    void* workspace = r.pointer();
    const size_t bytes = r.integer();
    void* stream = r.stream();
    return finish(r, [&] {
        return g_forward_mixed(&shape, &spec, seed, n_v, mix_beta, x, gamma, beta, eps, momentum, y, mean, invstd, parts, running_mean,
                               running_var, workspace, bytes, stream);
    });
}

PyObject* backward_mixed(PyObject*, PyObject* const* args, Py_ssize_t n) {
    Reader r(args, n, 17);
    const bns_shape shape = r.shape();
    const bns_spec spec = r.spec();
    const uint64_t seed = r.integer();
    const int32_t n_v = int32_t(r.integer());
    const float mix_beta = r.real();
    const void *x = r.pointer(), *dy = r.pointer();
    const float *gamma = r.vector(), *mean = r.vector(), *invstd = r.vector(), *parts = r.vector();
    void* dx = r.pointer();
    float *dgamma = r.vector(), *dbeta = r.vector();
    void* workspace = r.pointer();
    const size_t bytes = r.integer();
    void* stream = r.stream();
    return finish(r, [&] {
        return g_backward_mixed(&shape, &spec, seed, n_v, mix_beta, x, dy, gamma, mean, invstd, parts, dx, dgamma, dbeta, workspace, bytes,
                                stream);
    });
}

PyObject* inference(PyObject*, PyObject* const* args, Py_ssize_t n) {
    Reader r(args, n, 9);
    const bns_shape shape = r.shape();
    const void* x = r.pointer();
    const float *gamma = r.vector(), *beta = r.vector(), *mean = r.vector(), *var = r.vector();
    const float eps = r.real();
    void* y = r.pointer();
    void* stream = r.stream();
    return finish(r, [&] { return g_inference(&shape, x, gamma, beta, mean, var, eps, y, stream); });
}

// bind(type of bns_shape, type of bns_spec, addresses of the five functions)
PyObject* bind(PyObject*, PyObject* args) {
    PyObject *shape, *spec;
    unsigned long long f, b, fm, bm, i;
    if (!PyArg_ParseTuple(args, "O!O!KKKKK", &PyType_Type, &shape, &PyType_Type, &spec, &f, &b, &fm, &bm, &i)) return nullptr;
    g_forward = reinterpret_cast<decltype(g_forward)>(f);
    g_backward = reinterpret_cast<decltype(g_backward)>(b);
    g_forward_mixed = reinterpret_cast<decltype(g_forward_mixed)>(fm);
    g_backward_mixed = reinterpret_cast<decltype(g_backward_mixed)>(bm);
    g_inference = reinterpret_cast<decltype(g_inference)>(i);
    Py_INCREF(shape);
    Py_INCREF(spec);
    Py_XSETREF(g_shape_type, shape);
    Py_XSETREF(g_spec_type, spec);
    Py_RETURN_NONE;
}

#define BNS_FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&name)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {{"bind", &bind, METH_VARARGS, nullptr}, BNS_FAST(forward), BNS_FAST(backward), BNS_FAST(forward_mixed),
                           BNS_FAST(backward_mixed),               BNS_FAST(inference), {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_bnscall", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__bnscall() {
    if (!g_data_ptr && !(g_data_ptr = PyUnicode_InternFromString("data_ptr"))) return nullptr;
    return PyModule_Create(&g_module);
}
