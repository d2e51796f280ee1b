// Python entry to the calls that only enqueue work.  A call of the library costs the host about 4 us including the kernel
// launch; marshalling its arguments with ctypes cost as much again (two 4-us aggregations of a small graph: 14 us a pair,
// 11.9 with this module).  One wrapper template reads the parameter types off the C declaration and converts
// positional arguments: a pointer from None, an int, a torch tensor (data_ptr()), a numpy array or a ctypes pointer; a
// stream (the last parameter, or the last two) from None, an int or a torch stream (cuda_stream).  The interpreter lock is given up
// during the call.  Every function returns the status code.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <tuple>
#include <type_traits>
#include <utility>

#include "ntp.h"

namespace {

PyObject *s_data_ptr, *s_cuda_stream, *s_ctypes, *s_data, *s_value;

// the address an int object holds, consuming the reference
bool take_int(PyObject* v, void** out) {
    if (!v) return false;
    bool ok = true;
    if (v == Py_None) *out = nullptr;
    else {
        *out = PyLong_AsVoidPtr(v);
        ok = !(*out == nullptr && PyErr_Occurred());
    }
    Py_DECREF(v);
    return ok;
}

bool to_address(PyObject* o, PyObject* attribute, bool method, void** out) {
    if (o == Py_None) { *out = nullptr; return true; }
    if (PyLong_Check(o)) {
        *out = PyLong_AsVoidPtr(o);
        return !(*out == nullptr && PyErr_Occurred());
    }
    PyObject* v = method ? PyObject_CallMethodNoArgs(o, attribute) : PyObject_GetAttr(o, attribute);
    if (v) return take_int(v, out);
    if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return false;
    PyErr_Clear();
    if (PyObject* c = PyObject_GetAttr(o, s_ctypes)) {          // numpy array
        v = PyObject_GetAttr(c, s_data);
        Py_DECREF(c);
        return take_int(v, out);
    }
    PyErr_Clear();
    return take_int(PyObject_GetAttr(o, s_value), out);         // ctypes pointer
}

template <class P> bool convert(PyObject* o, bool stream, P* out) {
    if constexpr (std::is_pointer_v<P>) {
        void* a;
        if (!to_address(o, stream ? s_cuda_stream : s_data_ptr, !stream, &a)) return false;
        *out = static_cast<P>(a);
        return true;
    } else if constexpr (std::is_floating_point_v<P>) {
        *out = (P)PyFloat_AsDouble(o);
        return !(*out == (P)-1 && PyErr_Occurred());
    } else {
        long long v;
        if (PyLong_Check(o)) {
            v = PyLong_AsLongLong(o);
        } else {
            PyObject* i = PyNumber_Long(o);
            if (!i) return false;
            v = PyLong_AsLongLong(i);
            Py_DECREF(i);
        }
        *out = (P)v;
        return !(v == -1 && PyErr_Occurred());
    }
}

// Streams: how many of the last parameters are streams
template <auto Fn, int Streams> struct Wrap;
template <class... P, int (*Fn)(P...), int Streams>
struct Wrap<Fn, Streams> {
    template <std::size_t... I>
    static PyObject* go(PyObject* const* args, std::index_sequence<I...>) {
        std::tuple<P...> v;
        if (!(convert(args[I], I + Streams >= sizeof...(P), &std::get<I>(v)) && ...)) return nullptr;
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = Fn(std::get<I>(v)...);
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    }
    static PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t n) {
        if (n != (Py_ssize_t)sizeof...(P)) return PyErr_Format(PyExc_TypeError, "%d arguments expected, %zd given", (int)sizeof...(P), n);
        return go(args, std::index_sequence_for<P...>());
    }
};

#define ONE(name) {#name, (PyCFunction)(void (*)(void))Wrap<&name, 1>::call, METH_FASTCALL, nullptr}
#define TWO(name) {#name, (PyCFunction)(void (*)(void))Wrap<&name, 2>::call, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    ONE(ntp_aggregate_fwd), ONE(ntp_aggregate_fwd_noalloc), ONE(ntp_aggregate_bwd), ONE(ntp_aggregate_weighted),
    TWO(ntp_chunked_aggregate), TWO(ntp_aggregate_act),
    ONE(ntp_edge_softmax), ONE(ntp_edge_softmax_bwd), ONE(ntp_attention_scores_fwd), ONE(ntp_attention_scores_bwd),
    ONE(ntp_nn_fwd), ONE(ntp_nn_bwd), ONE(ntp_softmax_xent), ONE(ntp_relu_fwd), ONE(ntp_relu_bwd),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) {
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    s_ctypes = PyUnicode_InternFromString("ctypes");
    s_data = PyUnicode_InternFromString("data");
    s_value = PyUnicode_InternFromString("value");
    return PyModule_Create(&module);
}
