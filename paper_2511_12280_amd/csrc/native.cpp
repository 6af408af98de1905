// The Python side of the device entry points: turns tensors into device pointers and calls libd3tom.so.  Marshalling only, no
// arithmetic.  A merge-layer step of a short sequence is half a dozen launches of a few microseconds each, and looking up the
// attributes of some thirty tensors in Python and converting sixty arguments took a good part of the time of its kernels: the
// five calls on one crop of 729 tokens took 38.3 us on the host, 33.3 us here (most of what is left are the launches); a first
// pass over new inputs 105 us with its kernels, 79 us here.
#define PY_SSIZE_T_CLEAN
#include <torch/csrc/autograd/python_variable.h>
#include <exception>
#include <tuple>
#include <type_traits>
#include <utility>
#include "../../include/d3tom.h"

namespace {

struct PythonError {};         // a Python exception is set

PyObject* refuse() {
    PyErr_SetString(PyExc_ValueError, "device entry points take contiguous tensors on the GPU");
    throw PythonError();
}

// None or a tensor
void* pointer(PyObject* o) {
    if (o == Py_None) return nullptr;
    if (THPVariable_CheckExact(o)) {
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.is_cuda() || !t.is_contiguous()) refuse();
        return t.data_ptr();
    }
    // subclasses of Tensor: by their own attributes, whatever those do
    auto take = [](PyObject* r) { if (!r) throw PythonError(); return r; };
    auto truth = [&](PyObject* r) { take(r); const int v = PyObject_IsTrue(r); Py_DECREF(r); if (v < 0) throw PythonError(); return v != 0; };
    if (!truth(PyObject_GetAttrString(o, "is_cuda")) || !truth(PyObject_CallMethod(o, "is_contiguous", nullptr))) refuse();
    PyObject* a = take(PyObject_CallMethod(o, "data_ptr", nullptr));
    void* p = PyLong_AsVoidPtr(a);
    Py_DECREF(a);
    if (!p && PyErr_Occurred()) throw PythonError();
    return p;
}

// a stream's handle: None or an integer; the last argument of every entry point, and the only address taken as it is
void* stream(PyObject* o) {
    if (o == Py_None) return nullptr;
    void* p = PyLong_AsVoidPtr(o);
    if (!p && PyErr_Occurred()) throw PythonError();
    return p;
}

template <typename T> struct Arg;
template <typename T> struct Arg<T*> { static T* get(PyObject* o) { return static_cast<T*>(pointer(o)); } };
template <> struct Arg<int> {
    static int get(PyObject* o) {
        const unsigned long v = PyLong_AsUnsignedLongMask(o);  // the low 32 bits, as ctypes takes a C int
        if (v == (unsigned long)-1 && PyErr_Occurred()) throw PythonError();
        return (int)(unsigned)v;
    }
};
template <> struct Arg<size_t> {
    static size_t get(PyObject* o) {
        const size_t v = PyLong_AsSize_t(o);
        if (v == (size_t)-1 && PyErr_Occurred()) throw PythonError();
        return v;
    }
};
template <> struct Arg<float> {
    static float get(PyObject* o) {
        const double v = PyFloat_AsDouble(o);
        if (v == -1.0 && PyErr_Occurred()) throw PythonError();
        return (float)v;
    }
};

template <typename T> struct Type { using type = T; };

template <typename... A, size_t... I>
int call(int (*fn)(A...), PyObject* const* args, std::index_sequence<I...>) {
    constexpr size_t last = sizeof...(A) - 1;
    auto take = [&](auto type, size_t i) {
        using T = typename decltype(type)::type;
        if constexpr (std::is_same_v<T, void*>) { if (i == last) return stream(args[i]); }
        return Arg<T>::get(args[i]);
    };
    const std::tuple<A...> a{take(Type<A>{}, I)...};           // in order
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = fn(std::get<I>(a)...);
    Py_END_ALLOW_THREADS
    return status;
}

// the entry point's status as a Python int
template <typename... A>
PyObject* enter(int (*fn)(A...), PyObject* const* args, Py_ssize_t n) {
    if (n != (Py_ssize_t)sizeof...(A)) return PyErr_Format(PyExc_TypeError, "%zd arguments, the entry point takes %zd", n, (Py_ssize_t)sizeof...(A));
    try {
        return PyLong_FromLong(call(fn, args, std::index_sequence_for<A...>()));
    } catch (const PythonError&) {
        return nullptr;
    } catch (const std::exception& e) {                        // a tensor without storage
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

#define D3TOM_ENTRY(NAME) \
    PyObject* py_##NAME(PyObject*, PyObject* const* args, Py_ssize_t n) { return enter(&NAME, args, n); }
D3TOM_ENTRY(d3tom_importance)
D3TOM_ENTRY(d3tom_importance_static)
D3TOM_ENTRY(d3tom_select_topk)
D3TOM_ENTRY(d3tom_merge)
D3TOM_ENTRY(d3tom_merge_kv)
D3TOM_ENTRY(d3tom_merge_layer)
D3TOM_ENTRY(d3tom_attend)
D3TOM_ENTRY(d3tom_attend_weighted)
D3TOM_ENTRY(d3tom_update_deciders)
D3TOM_ENTRY(d3tom_rmsnorm)
D3TOM_ENTRY(d3tom_rope)
D3TOM_ENTRY(d3tom_linear)
D3TOM_ENTRY(d3tom_linear_tile)
#undef D3TOM_ENTRY

#define D3TOM_METHOD(NAME) {#NAME, (PyCFunction)(void (*)(void))py_##NAME, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    D3TOM_METHOD(d3tom_importance), D3TOM_METHOD(d3tom_importance_static), D3TOM_METHOD(d3tom_select_topk), D3TOM_METHOD(d3tom_merge),
    D3TOM_METHOD(d3tom_merge_kv), D3TOM_METHOD(d3tom_merge_layer), D3TOM_METHOD(d3tom_attend), D3TOM_METHOD(d3tom_attend_weighted),
    D3TOM_METHOD(d3tom_update_deciders), D3TOM_METHOD(d3tom_rmsnorm), D3TOM_METHOD(d3tom_rope), D3TOM_METHOD(d3tom_linear),
    D3TOM_METHOD(d3tom_linear_tile), {nullptr, nullptr, 0, nullptr}};
#undef D3TOM_METHOD
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&module); }
