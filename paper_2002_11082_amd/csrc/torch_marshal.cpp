// Argument marshalling between torch tensors and libogq's C ABI, as a CPython extension module: what binding.py's
// ogq_quantize and ogq_dequantize_average do for every call, without the interpreter.  It checks the tensors (the kernels
// trust their sizes), allocates the outputs the caller left out, and calls the library through the addresses that
// binding.py hands to bind(); nothing of the path runs here and nothing links against libogq.
//
// Why native: a call is one kernel launch (2.3 us on the host), and for gradients below about a million elements the
// kernels take less than what the same checks cost in Python with ctypes (n = 1728, host time per call: quantize
// 8.5 us, 10.5 with allocated outputs, decode of one stream 9.4, of eight 17.4).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdio>
#include <cstring>
#include <exception>

#include "ogq.h"

namespace {

using QuantizeFn = decltype(&ogq_quantize);
using AverageFn = decltype(&ogq_dequantize_average);
using CountFn = decltype(&ogq_levels_count);

// What bind() was given.
struct Bound {
    QuantizeFn quantize = nullptr;
    AverageFn average = nullptr;
    CountFn levels_count = nullptr, codes_bytes = nullptr;
    PyObject* raw_stream = nullptr;  // callable: device index -> address of torch's current stream
    PyObject* check = nullptr;       // callable: raises OgqError for a status other than 0
    PyTypeObject* params = nullptr;  // the class of the caller's parameters
} bound;

// Thrown where the Python error is already set.
struct PythonError {};

[[noreturn]] void refuse(const char* text)
{
    PyErr_SetString(PyExc_ValueError, text);
    throw PythonError{};
}

void require(bool ok, const char* text)
{
    if (!ok) refuse(text);
}

const at::Tensor& tensor(PyObject* o, const char* what)
{
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "%s: expected a tensor", what);
        throw PythonError{};
    }
    return THPVariable_Unpack(o);
}

// A contiguous CUDA tensor of `dtype` with at least `elements` elements.  what, worker: the tensor's name in the error
// text (worker < 0: none).
void holds(const at::Tensor& t, at::ScalarType dtype, size_t elements, const char* what, Py_ssize_t worker = -1)
{
    const bool kind = t.is_cuda() && t.scalar_type() == dtype && t.is_contiguous();
    if (kind && static_cast<size_t>(t.numel()) >= elements) return;
    char name[64];
    if (worker < 0) snprintf(name, sizeof name, "%s", what);
    else snprintf(name, sizeof name, "%s of worker %zd", what, worker);
    if (!kind)
        PyErr_Format(PyExc_ValueError, "%s: expected a contiguous CUDA tensor of %s", name,
                     dtype == at::kFloat ? "torch.float32" : "torch.int64");
    else
        PyErr_Format(PyExc_ValueError, "%s: %lld elements, at least %zu needed", name, static_cast<long long>(t.numel()), elements);
    throw PythonError{};
}

// The caller's Params (a ctypes structure) through the buffer protocol.  Nothing else is taken, whatever its size: its bytes
// would be read as parameters.
ogq_params_t params_of(PyObject* o)
{
    if (!PyObject_TypeCheck(o, bound.params)) {
        PyErr_Format(PyExc_TypeError, "params: expected Params, got %s", Py_TYPE(o)->tp_name);
        throw PythonError{};
    }
    Py_buffer view;
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) throw PythonError{};
    ogq_params_t p;
    const bool fits = view.len == static_cast<Py_ssize_t>(sizeof p);
    if (fits) std::memcpy(&p, view.buf, sizeof p);
    PyBuffer_Release(&view);
    require(fits, "params: not an ogq Params structure");
    return p;
}

void* stream_of(const at::Tensor& t)
{
    PyObject* index = PyLong_FromLong(t.get_device());
    if (!index) throw PythonError{};
    PyObject* stream = PyObject_CallOneArg(bound.raw_stream, index);
    Py_DECREF(index);
    if (!stream) throw PythonError{};
    void* address = PyLong_AsVoidPtr(stream);
    Py_DECREF(stream);
    if (!address && PyErr_Occurred()) throw PythonError{};
    return address;
}

void check(int status)
{
    if (status == OGQ_OK) return;
    PyObject* r = PyObject_CallFunction(bound.check, "i", status);
    Py_XDECREF(r);
    if (r) PyErr_SetString(PyExc_RuntimeError, "a status other than 0 was not turned into an error");
    throw PythonError{};
}

at::Tensor empty_like_device(size_t elements, at::ScalarType dtype, const at::Tensor& like)
{
    return at::empty({static_cast<int64_t>(elements)}, at::TensorOptions().dtype(dtype).device(like.device()));
}

// A new reference to the caller's tensor, or to the one allocated in its place.
PyObject* give_back(PyObject* given, const at::Tensor& made)
{
    if (!made.defined()) {
        Py_INCREF(given);
        return given;
    }
    return THPVariable_Wrap(made);
}

// Runs f() and turns what it throws into a Python error: torch's own exceptions (an allocation may raise them) into the types
// that torch gives them, so that a caller sees torch.OutOfMemoryError, or the error of a Python mode that was asked.
template <class F>
PyObject* guarded(F f)
{
    try {
        require(bound.check != nullptr, "bind() comes first");
        return f();
    } catch (const PythonError&) {
    } catch (const std::exception&) {
        torch::translate_exception_to_python(std::current_exception());
    }
    return nullptr;
}

bool argument_count(Py_ssize_t nargs, Py_ssize_t wanted)
{
    if (nargs == wanted) return true;
    PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", wanted, nargs);
    return false;
}

// quantize(grad, params, levels or None, codes or None) -> (levels, codes)
PyObject* quantize(PyObject*, PyObject* const* args, Py_ssize_t nargs)
{
    if (!argument_count(nargs, 4)) return nullptr;
    return guarded([&]() -> PyObject* {
        const at::Tensor& grad = tensor(args[0], "grad");
        require(grad.dim() == 1, "grad: expected a 1-D tensor");
        holds(grad, at::kFloat, 0, "grad");
        const ogq_params_t p = params_of(args[1]);
        const size_t n = static_cast<size_t>(grad.numel());
        const size_t n_levels = bound.levels_count(n, &p), n_words = bound.codes_bytes(n, &p) / 8;
        at::Tensor made_levels, made_codes;
        if (args[2] == Py_None) made_levels = empty_like_device(n_levels < 4 ? 4 : n_levels, at::kFloat, grad);
        if (args[3] == Py_None) made_codes = empty_like_device(n_words < 2 ? 2 : n_words, at::kLong, grad);
        const at::Tensor& levels = made_levels.defined() ? made_levels : tensor(args[2], "levels");
        const at::Tensor& codes = made_codes.defined() ? made_codes : tensor(args[3], "codes");
        holds(levels, at::kFloat, n_levels, "levels");
        holds(codes, at::kLong, n_words, "codes");
        require(levels.device() == grad.device() && codes.device() == grad.device(), "levels / codes: not on grad's device");
        const float* from = static_cast<const float*>(grad.const_data_ptr());
        float* to_levels = static_cast<float*>(levels.data_ptr());
        void *to_codes = codes.data_ptr(), *stream = stream_of(grad);
        int status;
        Py_BEGIN_ALLOW_THREADS
        status = bound.quantize(from, n, &p, to_levels, to_codes, stream);
        Py_END_ALLOW_THREADS
        check(status);
        PyObject* both = PyTuple_New(2);
        if (!both) throw PythonError{};
        PyTuple_SET_ITEM(both, 0, give_back(args[2], made_levels));
        PyTuple_SET_ITEM(both, 1, give_back(args[3], made_codes));
        return both;
    });
}

// The items of a Python sequence for the time of a call.
struct Items {
    PyObject* fast;
    explicit Items(PyObject* sequence) : fast(PySequence_Fast(sequence, "expected a sequence of tensors"))
    {
        if (!fast) throw PythonError{};
    }
    Items(const Items&) = delete;
    ~Items() { Py_DECREF(fast); }
    Py_ssize_t size() const { return PySequence_Fast_GET_SIZE(fast); }
    PyObject* operator[](Py_ssize_t i) const { return PySequence_Fast_GET_ITEM(fast, i); }
};

// dequantize_average(codes_list, levels_list, n, params, out or None) -> out
PyObject* dequantize_average(PyObject*, PyObject* const* args, Py_ssize_t nargs)
{
    if (!argument_count(nargs, 5)) return nullptr;
    return guarded([&]() -> PyObject* {
        const Items codes_list(args[0]), levels_list(args[1]);
        const Py_ssize_t workers = codes_list.size();
        require(workers == levels_list.size() && workers > 0, "one codes and one levels tensor per worker");
        PyObject* count = PyNumber_Index(args[2]);
        if (!count) throw PythonError{};
        const size_t n = PyLong_AsSize_t(count);
        Py_DECREF(count);
        if (n == static_cast<size_t>(-1) && PyErr_Occurred()) throw PythonError{};
        const ogq_params_t p = params_of(args[3]);
        const size_t n_levels = bound.levels_count(n, &p), n_words = bound.codes_bytes(n, &p) / 8;
        const at::Tensor& first = tensor(codes_list[0], "codes");
        const at::Device device = first.device();
        // (more workers than the library takes are its own error)
        constexpr Py_ssize_t kMost = OGQ_MAX_WORKERS;
        const void* codes[kMost];
        const float* levels[kMost];
        for (Py_ssize_t w = 0; w < workers; ++w) {
            const at::Tensor& c = tensor(codes_list[w], "codes");
            const at::Tensor& l = tensor(levels_list[w], "levels");
            holds(c, at::kLong, n_words, "codes", w);
            holds(l, at::kFloat, n_levels, "levels", w);
            if (c.device() != device || l.device() != device) {
                PyErr_Format(PyExc_ValueError, "worker %zd: tensors on different devices", w);
                throw PythonError{};
            }
            if (w < kMost) {
                codes[w] = c.const_data_ptr();
                levels[w] = static_cast<const float*>(l.const_data_ptr());
            }
        }
        at::Tensor made;
        if (args[4] == Py_None) {
            made = empty_like_device(n < 4 ? 4 : n, at::kFloat, first);
            if (n < 4) made = made.narrow(0, 0, static_cast<int64_t>(n));
        }
        const at::Tensor& out = made.defined() ? made : tensor(args[4], "out");
        holds(out, at::kFloat, n, "out");
        require(out.device() == device, "out: not on the workers' device");
        float* to = static_cast<float*>(out.data_ptr());
        void* stream = stream_of(out);
        int status;
        Py_BEGIN_ALLOW_THREADS
        status = bound.average(codes, levels, static_cast<uint32_t>(workers), n, &p, to, stream);
        Py_END_ALLOW_THREADS
        check(status);
        return give_back(args[4], made);
    });
}

// bind(address of ogq_quantize, of ogq_dequantize_average, of ogq_levels_count, of ogq_codes_bytes, raw_stream, check, Params)
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t nargs)
{
    if (!argument_count(nargs, 7)) return nullptr;
    if (!PyType_Check(args[6])) {
        PyErr_SetString(PyExc_TypeError, "Params: expected a class");
        return nullptr;
    }
    void* address[4];
    for (int i = 0; i < 4; ++i) {
        address[i] = PyLong_AsVoidPtr(args[i]);
        if (!address[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "address 0");
            return nullptr;
        }
    }
    bound.quantize = reinterpret_cast<QuantizeFn>(address[0]);
    bound.average = reinterpret_cast<AverageFn>(address[1]);
    bound.levels_count = reinterpret_cast<CountFn>(address[2]);
    bound.codes_bytes = reinterpret_cast<CountFn>(address[3]);
    Py_INCREF(args[4]);
    Py_INCREF(args[5]);
    Py_INCREF(args[6]);
    Py_XDECREF(bound.raw_stream);
    Py_XDECREF(bound.check);
    Py_XDECREF(reinterpret_cast<PyObject*>(bound.params));
    bound.raw_stream = args[4];
    bound.check = args[5];
    bound.params = reinterpret_cast<PyTypeObject*>(args[6]);
    Py_RETURN_NONE;
}

template <class F>
PyCFunction as_method(F f)
{
    return reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(f));
}

PyMethodDef methods[] = {
    {"bind", as_method(bind), METH_FASTCALL, "the library's entry points and the two callables"},
    {"quantize", as_method(quantize), METH_FASTCALL, "ogq_quantize on tensors; after bind()"},
    {"dequantize_average", as_method(dequantize_average), METH_FASTCALL, "ogq_dequantize_average on tensors; after bind()"},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&module); }
