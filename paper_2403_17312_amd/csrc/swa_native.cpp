// Native half of the Python binding: turns the arguments of one call (tensors, integers, None) into the C ABI's pointers and
// makes the call.  Marshalling only, as in binding.py, which keeps the general path in Python: whatever is not a plain
// tensor, an integer or None makes a function here answer None, and the caller goes that way, with its errors.
//
// What it saves is the host's time per call, which bounds small steps: 32 calls of about sixteen tensors each, on four short
// pairs, 254 -> 198 us; 32 calls on 512 pairs 305 -> 292, where the GPU is the bound again.
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <tuple>
#include <type_traits>
#include <utility>

#include "swa.h"

namespace {

enum class Arg { ok, other, failed };

PyObject* params_type = nullptr;                         // binding.py's SwaParams

// A pointer argument: None, or a plain contiguous tensor.
Arg pointer(PyObject* o, void*& out)
{
    if (o == Py_None) {
        out = nullptr;
        return Arg::ok;
    }
    if (!THPVariable_CheckExact(o)) return Arg::other;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_contiguous()) return Arg::other;           // (refused on the general path)
    out = t.data_ptr();
    return Arg::ok;
}

Arg integer(PyObject* o, int64_t& out)
{
    if (!PyLong_CheckExact(o)) return Arg::other;
    out = PyLong_AsLongLong(o);
    if (out == -1 && PyErr_Occurred()) {
        PyErr_Clear();
        return Arg::other;
    }
    return Arg::ok;
}

// One argument of the C function, by its type there.
template <typename A>
Arg convert(PyObject* o, A& out)
{
    if constexpr (std::is_pointer_v<A>) {
        void* p = nullptr;
        const Arg r = pointer(o, p);
        out = static_cast<A>(p);
        return r;
    } else {
        int64_t v = 0;
        const Arg r = integer(o, v);
        if (r != Arg::ok || v < INT32_MIN || v > INT32_MAX) return Arg::other;
        out = static_cast<A>(v);
        return Arg::ok;
    }
}

// fn(params, arguments..., stream) for one entry point; ADDR holds its address in the library that binding.py loaded.
template <typename F>
struct Entry;

template <typename... A>
struct Entry<int (*)(const swa_params*, A...)> {
    static constexpr size_t N = sizeof...(A);            // the stream is the last one

    // The arguments, or false where the general path has to look at them.
    template <size_t... I>
    static bool convert_all(PyObject* const* args, swa_params& p, std::tuple<A...>& a, std::index_sequence<I...>)
    {
        Arg r = Arg::ok;
        ((I + 1 < N && r == Arg::ok ? (void)(r = convert(args[1 + I], std::get<I>(a))) : (void)0), ...);
        if (r != Arg::ok) return false;
        if (args[N] == Py_None) {
            std::get<N - 1>(a) = reinterpret_cast<void*>(c10::hip::getCurrentHIPStream().stream());
        } else {
            if (!PyLong_CheckExact(args[N])) return false;
            std::get<N - 1>(a) = PyLong_AsVoidPtr(args[N]);
            if (PyErr_Occurred()) return false;
        }
        if (reinterpret_cast<PyObject*>(Py_TYPE(args[0])) != params_type) return false;
        Py_buffer params;
        if (PyObject_GetBuffer(args[0], &params, PyBUF_SIMPLE) != 0) return false;
        const bool fits = params.len == (Py_ssize_t)sizeof(swa_params);
        if (fits) p = *static_cast<const swa_params*>(params.buf);
        PyBuffer_Release(&params);
        return fits;
    }

    // Without the interpreter's lock.  An exception that leaves the library ends the process here, as it does by way of ctypes: caught
    // further out it would find the lock released and the call made a second time.
    static int make(void* fn, const swa_params& p, const std::tuple<A...>& a) noexcept
    {
        PyThreadState* const held = PyEval_SaveThread();
        const int rc = std::apply([&](A... v) { return reinterpret_cast<int (*)(const swa_params*, A...)>(fn)(&p, v...); }, a);
        PyEval_RestoreThread(held);
        return rc;
    }

    static PyObject* run(void* fn, PyObject* const* args, Py_ssize_t n)
    {
        if (!fn || n != (Py_ssize_t)N + 1) Py_RETURN_NONE;
        std::tuple<A...> a;
        swa_params p;
        bool ready = false;
        try {
            ready = convert_all(args, p, a, std::make_index_sequence<N>());
        } catch (...) {                                  // a tensor without storage, no device: the general path reports it
        }
        if (!ready) {
            PyErr_Clear();
            Py_RETURN_NONE;
        }
        return PyLong_FromLong(make(fn, p, a));
    }
};

#define SWA_ENTRIES(X) \
    X(swa_decode_step) \
    X(swa_decode_step_q8) \
    X(swa_decode_step_window) \
    X(swa_decode_step_window_q8) \
    X(swa_decode_step_static) \
    X(swa_compact_kv) \
    X(swa_prefill_scores) \
    X(swa_prefill_rows) \
    X(swa_prefill_attention) \
    X(swa_quantize_kv)

#define SWA_DEFINE(name) \
    void* addr_##name = nullptr; \
    PyObject* py_##name(PyObject*, PyObject* const* args, Py_ssize_t n) \
    { \
        return Entry<decltype(&name)>::run(addr_##name, args, n); \
    }
SWA_ENTRIES(SWA_DEFINE)

// bind({name: address}, SwaParams): the entry points of the library that is in use.
PyObject* bind(PyObject*, PyObject* args)
{
    PyObject *dict = nullptr, *type = nullptr;
    if (!PyArg_ParseTuple(args, "O!O", &PyDict_Type, &dict, &type)) return nullptr;
    Py_INCREF(type);
    Py_XSETREF(params_type, type);
#define SWA_BIND(name) \
    { \
        PyObject* v = PyDict_GetItemString(dict, #name); \
        void* p = v ? PyLong_AsVoidPtr(v) : nullptr; \
        if (PyErr_Occurred()) return nullptr; \
        addr_##name = p; \
    }
    SWA_ENTRIES(SWA_BIND)
    Py_RETURN_NONE;
}

#define SWA_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(&py_##name)), METH_FASTCALL, nullptr},
PyMethodDef methods[] = {{"bind", bind, METH_VARARGS, nullptr}, SWA_ENTRIES(SWA_METHOD){nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_swa_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__swa_native()
{
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", SWA_TORCH_VERSION) != 0) Py_CLEAR(m);
    return m;
}
