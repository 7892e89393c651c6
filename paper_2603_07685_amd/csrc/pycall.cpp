// Native half of binding.py: one Python-callable function per C entry point that takes device tensors, compiled from
// the declarations in moe_hip.h.  A call converts its arguments (tensor -> checked data pointer, int, float), takes the current
// stream of the current device, releases the interpreter lock and calls the library; the status comes back as an int.
//
// Why not ctypes: marshalling a call there cost 8-9 us of host time (15 conversions 2 us, four Python-level operations per
// tensor 0.54 us each, a stream object 1.5 us); a step of eleven calls whose kernels take 50 us (T 256, h 128, f 256, 8 experts)
// took 92 us, bound by that, and takes 55 now; T 1024, h 512, f 256 with a shared expert, blockwise fp8, 252 -> 232 us.
//
// The library stays the one binding.py has loaded: its symbols' addresses are handed to init(), nothing is linked against.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <tuple>
#include <type_traits>
#include <utility>

#include "moe_hip.h"

namespace {

PyObject* other_ptr = nullptr;   // binding._ptr: everything that is no plain tensor (subclasses may override the queries)

// tensor / None -> device pointer
void* pointer(PyObject* o, bool& ok) {
    if (o == Py_None) return nullptr;
    if (!THPVariable_CheckExact(o)) {
        PyObject* r = PyObject_CallOneArg(other_ptr, o);
        void* p = r && r != Py_None ? PyLong_AsVoidPtr(r) : nullptr;
        Py_XDECREF(r);
        if (PyErr_Occurred()) ok = false;
        return p;
    }
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous()) {
        PyErr_SetString(PyExc_AssertionError, "device tensors must be contiguous CUDA tensors");
        ok = false;
        return nullptr;
    }
    return t.data_ptr();
}

// a ctypes call's conversions: integers by value modulo their width (no floats), floats from anything with __float__
template <typename T>
T convert(PyObject* o, bool& ok) {
    if (!ok) return T{};
    if constexpr (std::is_pointer_v<T>) {
        return (T)pointer(o, ok);
    } else if constexpr (std::is_floating_point_v<T>) {
        const double v = PyFloat_AsDouble(o);
        if (v == -1.0 && PyErr_Occurred()) ok = false;
        return (T)v;
    } else {
        if (PyFloat_Check(o)) {
            PyErr_SetString(PyExc_TypeError, "int expected instead of float instance");
            ok = false;
            return T{};
        }
        const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);
        if (v == (unsigned long long)-1 && PyErr_Occurred()) ok = false;
        return (T)(long long)v;
    }
}

// arguments after the context and the stream
template <typename... A, size_t... I>
moe_status invoke(moe_status (*f)(moe_ctx*, void*, A...), moe_ctx* ctx, PyObject* const* args, std::index_sequence<I...>, bool& ok) {
    std::tuple<A...> v{convert<A>(args[I], ok)...};   // (braces: in order)
    if (!ok) return MOE_OK;
    void* const stream = (void*)c10::hip::getCurrentHIPStream().stream();
    moe_status st;
    Py_BEGIN_ALLOW_THREADS
    st = f(ctx, stream, std::get<I>(v)...);
    Py_END_ALLOW_THREADS
    return st;
}
template <typename... A>
constexpr size_t count(moe_status (*)(moe_ctx*, void*, A...)) { return sizeof...(A); }
template <typename... A>
PyObject* run(moe_status (*f)(moe_ctx*, void*, A...), PyObject* const* args, Py_ssize_t n, const char* name) {
    HANDLE_TH_ERRORS
    if (n != (Py_ssize_t)sizeof...(A) + 1) return PyErr_Format(PyExc_TypeError, "%s: %d arguments expected, %zd given", name, (int)sizeof...(A) + 1, n);
    if (!f) return PyErr_Format(PyExc_RuntimeError, "%s: not initialised", name);
    void* const ctx = args[0] == Py_None ? nullptr : PyLong_AsVoidPtr(args[0]);   // the context's address
    bool ok = !PyErr_Occurred();
    const moe_status st = invoke(f, (moe_ctx*)ctx, args + 1, std::index_sequence_for<A...>{}, ok);
    return ok ? PyLong_FromLong(st) : nullptr;
    END_HANDLE_TH_ERRORS
}

#define ENTRIES(X)                                                                                                         \
    X(moe_route_topk) X(moe_route_topk_grouped) X(moe_route_topk_bwd) X(moe_aux_loss) X(moe_gate_gemm) X(moe_permute)      \
    X(moe_grouped_gemm_fwd) X(moe_grouped_gemm_fwd_weighted) X(moe_grouped_gemm_fwd_quant) X(moe_grouped_gemm_fwd_quant_mx) \
    X(moe_grouped_gemm_fwd_gather) X(moe_grouped_gemm_dgrad) X(moe_grouped_gemm_dgrad_weighted)                            \
    X(moe_grouped_gemm_dgrad_quant) X(moe_grouped_gemm_dgrad_quant_mx) X(moe_grouped_gemm_dgrad_gather)                    \
    X(moe_grouped_gemm_wgrad) X(moe_grouped_gemm_wgrad_gather) X(moe_unpermute_combine) X(moe_unpermute_combine_bwd)       \
    X(moe_gather_row_prob) X(moe_scatter_row_dprob) X(moe_fp8_quantize) X(moe_fp8_quantize_rowcol)                         \
    X(moe_fp8_quantize_rowcol_gather) X(moe_mx_quantize) X(moe_mx_quantize_rowcol) X(moe_mx_quantize_rowcol_gather) X(moe_batch_end)

#define DEFINE(name)                                                              \
    decltype(&::name) fn_##name = nullptr;                                        \
    PyObject* py_##name(PyObject*, PyObject* const* args, Py_ssize_t n) { return run(fn_##name, args, n, #name); }
ENTRIES(DEFINE)

// init(addresses: name -> int, ptr: the general conversion of an object to a pointer)
PyObject* py_init(PyObject*, PyObject* args) {
    PyObject *table, *ptr;
    if (!PyArg_ParseTuple(args, "O!O", &PyDict_Type, &table, &ptr)) return nullptr;
#define TAKE(name)                                                                                   \
    {                                                                                                \
        PyObject* a = PyDict_GetItemString(table, #name);                                            \
        if (!a) return PyErr_Format(PyExc_KeyError, "no address of %s", #name);                      \
        fn_##name = (decltype(&::name))PyLong_AsVoidPtr(a);                                          \
        if (PyErr_Occurred()) return nullptr;                                                        \
    }
    ENTRIES(TAKE)
    Py_INCREF(ptr);
    Py_XDECREF(other_ptr);
    other_ptr = ptr;
    Py_RETURN_NONE;
}

#define METHOD(name) {#name, (PyCFunction)(void (*)(void))py_##name, METH_FASTCALL, nullptr},
PyMethodDef methods[] = {{"init", py_init, METH_VARARGS, nullptr}, ENTRIES(METHOD){nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pycall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pycall() { return PyModule_Create(&module); }
