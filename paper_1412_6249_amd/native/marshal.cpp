// Native argument marshalling of the operator calls (binding.py): torch tensors to purine_tensor descriptors, the current
// stream, the call. Built as the Python module _marshal.
//
// Bound: host time per call. A descriptor made with ctypes costs 1.6 us, a call with five tensors and its stream about
// 10, more than its launches: most small layers were bound by it. Here an argument costs tens of nanoseconds.
//
// Every function takes its entry point's arguments in the C order (scratch and its size as one argument) and returns the
// status, or None for any argument that is not the plain case (a tensor's descriptor made by hand, another kind of object, a
// tensor that the operators refuse): the caller then takes the general path, which says what is wrong. Convolution and
// pooling descriptors are instances of the two ctypes structures that descriptor_types() is given, as ctypes itself asks.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>
#include <tuple>
#include <type_traits>

#include "purine.h"

namespace {

constexpr int MAX_TENSORS = 5;

struct Call {
    PyObject* const* args;
    Py_ssize_t n, next = 0;
    unsigned optional;                       // tensor arguments that may be None
    purine_tensor t[MAX_TENSORS];
    int tensors = 0;
    void* ws = nullptr;
    size_t ws_bytes = 0;
    bool ws_taken = false;
    Py_buffer desc{};
    bool ok = true;                          // the plain case so far
    ~Call() { if (desc.obj) PyBuffer_Release(&desc); }
    PyObject* arg() {
        if (next >= n) { ok = false; return nullptr; }
        return args[next++];
    }
};

PyTypeObject* descriptor_type[2] = {nullptr, nullptr};     // purine_conv_desc, purine_pool_desc

bool is_descriptor(PyObject* o, int which) { return descriptor_type[which] && PyObject_TypeCheck(o, descriptor_type[which]); }

bool fill(purine_tensor& d, PyObject* o) {
    if (!THPVariable_Check(o)) return false;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided) return false;
    const auto dims = t.dim();
    if (dims < 1 || dims > 4) return false;
    switch (t.scalar_type()) {
        case at::kFloat: d.dtype = PURINE_F32; break;
        case at::kBFloat16: d.dtype = PURINE_BF16; break;
        case at::kInt: d.dtype = PURINE_I32; break;
        default: return false;
    }
    d.nstride = 0;
    for (int i = 0; i < 4; ++i) d.dim[i] = i < dims ? t.size(i) : 0;
    if (!t.is_contiguous()) {                // a channel slice of a contiguous NCHW tensor
        if (dims != 4 || t.stride(3) != 1 || t.stride(2) != d.dim[3] || t.stride(1) != d.dim[2] * d.dim[3] ||
            t.stride(0) < d.dim[1] * d.dim[2] * d.dim[3]) return false;
        d.nstride = t.stride(0);
    }
    d.data = t.data_ptr();
    d.ndim = (int32_t)dims;
    return true;
}

template <typename A, int POINTERS>
A take(Call& c) {
    if constexpr (std::is_same_v<A, const purine_tensor*> || std::is_same_v<A, purine_tensor*>) {
        PyObject* o = c.arg();
        const int i = c.tensors++;
        if (!c.ok || i >= MAX_TENSORS) { c.ok = false; return nullptr; }
        if (o == Py_None && (c.optional >> i & 1)) return nullptr;
        if (!fill(c.t[i], o)) c.ok = false;
        return &c.t[i];
    } else if constexpr (std::is_same_v<A, const purine_conv_desc*> || std::is_same_v<A, const purine_pool_desc*>) {
        PyObject* o = c.arg();
        constexpr int which = std::is_same_v<A, const purine_pool_desc*> ? 1 : 0;
        if (!c.ok || !is_descriptor(o, which) || PyObject_GetBuffer(o, &c.desc, PyBUF_SIMPLE) != 0) { PyErr_Clear(); c.ok = false; return nullptr; }
        if (c.desc.len < (Py_ssize_t)sizeof(std::remove_pointer_t<A>)) c.ok = false;
        return (A)c.desc.buf;
    } else if constexpr (std::is_same_v<A, float>) {
        PyObject* o = c.arg();
        const double v = c.ok ? PyFloat_AsDouble(o) : 0.0;
        if (PyErr_Occurred()) { PyErr_Clear(); c.ok = false; }
        return (float)v;
    } else if constexpr (std::is_same_v<A, int>) {
        PyObject* o = c.arg();
        if (!c.ok || !PyLong_Check(o)) { c.ok = false; return 0; }      // (True and False are ints)
        int overflow = 0;
        const long v = PyLong_AsLongAndOverflow(o, &overflow);
        if (overflow || v != (int)v) c.ok = false;
        return (int)v;
    } else if constexpr (std::is_same_v<A, size_t>) {
        return c.ws_bytes;
    } else {
        static_assert(std::is_same_v<A, void*>);
        PyObject* o = c.arg();
        if (!c.ok) return nullptr;
        if (POINTERS == 2 && !c.ws_taken) {                             // scratch
            c.ws_taken = true;
            if (o == Py_None) return nullptr;
            if (!THPVariable_Check(o)) { c.ok = false; return nullptr; }
            const at::Tensor& t = THPVariable_Unpack(o);
            if (!t.defined() || t.layout() != at::kStrided) { c.ok = false; return nullptr; }
            c.ws_bytes = (size_t)t.numel() * t.element_size();
            return c.ws = t.data_ptr();
        }
        if (o == Py_None) return (void*)c10::hip::getCurrentHIPStream().stream();
        if (!PyLong_Check(o)) { c.ok = false; return nullptr; }
        void* s = PyLong_AsVoidPtr(o);
        if (PyErr_Occurred()) { PyErr_Clear(); c.ok = false; }
        return s;
    }
}

template <typename... A>
PyObject* invoke(int (*fn)(A...), PyObject* const* args, Py_ssize_t n, unsigned optional) {
    constexpr int POINTERS = (0 + ... + (std::is_same_v<A, void*> ? 1 : 0));
    try {
        Call c{args, n};
        c.optional = optional;
        std::tuple<A...> a{take<A, POINTERS>(c)...};                    // (braces: in order)
        if (!c.ok || c.next != n) Py_RETURN_NONE;
        // (noexcept: an exception out of a C entry ends the program, as from ctypes; it must not be taken for "not the plain case")
        auto call = [&]() noexcept { return std::apply(fn, a); };
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = call();
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    } catch (const std::exception&) {
        PyErr_Clear();
        Py_RETURN_NONE;                                                 // a tensor without storage, no device: as above
    }
}

#define ENTRY(NAME, OPTIONAL)                                                                    \
    PyObject* call_##NAME(PyObject*, PyObject* const* args, Py_ssize_t n) { return invoke(&NAME, args, n, OPTIONAL); }
#define ENTRIES(X)                                                                               \
    X(purine_conv_fwd, 0) X(purine_conv_fwd_bias_relu, 4) X(purine_conv_bwd_data, 0) X(purine_conv_bwd_data_relu, 0)        \
    X(purine_conv_bwd_weight, 0) X(purine_conv_bwd_weight_bias, 0) X(purine_conv_bwd_weight_static, 0)                     \
    X(purine_grouped_conv_fwd, 4) X(purine_grouped_conv_bwd_data, 0) X(purine_grouped_conv_bwd_weight, 8)                  \
    X(purine_fc_fwd, 4) X(purine_fc_bwd_data, 0) X(purine_fc_bwd_weight, 8) X(purine_sgd_update, 0)                        \
    X(purine_bias_fwd, 0) X(purine_bias_bwd, 0) X(purine_relu_fwd, 0) X(purine_relu_bwd, 0)                                \
    X(purine_maxpool_fwd, 0) X(purine_maxpool_bwd, 0) X(purine_maxpool_bwd_relu, 0)
ENTRIES(ENTRY)

PyObject* descriptor_types(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != 2 || !PyType_Check(args[0]) || !PyType_Check(args[1])) {
        PyErr_SetString(PyExc_TypeError, "descriptor_types(purine_conv_desc, purine_pool_desc)");
        return nullptr;
    }
    for (int i = 0; i < 2; ++i) {
        Py_INCREF(args[i]);
        Py_XDECREF((PyObject*)descriptor_type[i]);
        descriptor_type[i] = (PyTypeObject*)args[i];
    }
    Py_RETURN_NONE;
}

// whether a convolution (0) or pooling (1) call would take the object as its descriptor
PyObject* takes_descriptor(PyObject*, PyObject* const* args, Py_ssize_t n) {
    const long which = n == 2 ? PyLong_AsLong(args[1]) : -1;
    if (which != 0 && which != 1) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "takes_descriptor(object, 0 or 1)");
        return nullptr;
    }
    return PyBool_FromLong(is_descriptor(args[0], (int)which));
}

#define METHOD(NAME, OPTIONAL) {#NAME, (PyCFunction)(void (*)(void))&call_##NAME, METH_FASTCALL, nullptr},
PyMethodDef methods[] = {ENTRIES(METHOD)
    {"descriptor_types", (PyCFunction)(void (*)(void))&descriptor_types, METH_FASTCALL, nullptr},
    {"takes_descriptor", (PyCFunction)(void (*)(void))&takes_descriptor, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&module); }
