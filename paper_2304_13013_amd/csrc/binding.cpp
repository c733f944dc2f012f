// Python side of the C ABI: the calls themselves and the two checks that every call makes of its tensors, as built-in
// functions.  A small layer's pass is bound by the host: each of its launches takes 3 us, and what Python and ctypes add
// to a call is of the same size.  The general forms of the checks stay in Python: whatever is not a plain tensor that
// passes (subclasses, function modes, wrong types and shapes) goes to those, which raise or answer as they always did.
#include <Python.h>

#include <ATen/Functions.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <torch/csrc/Device.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <tuple>
#include <type_traits>
#include <utility>

#include "../../include/switchback.h"

namespace {

PyObject *general_dev, *general_out;  // the Python functions, set once by general_forms()

struct WithoutGil {  // other Python threads run meanwhile
    PyThreadState *state = PyEval_SaveThread();
    ~WithoutGil() { PyEval_RestoreThread(state); }
};

bool plain(PyObject *o) { return THPVariable_CheckExact(o) && !at::impl::torch_function_mode_enabled(); }

PyObject *call_general(PyObject *f, PyObject *const *args, Py_ssize_t nargs) {
    if (f == nullptr) {
        PyErr_SetString(PyExc_RuntimeError, "general_forms() has not been called");
        return nullptr;
    }
    return PyObject_Vectorcall(f, args, (size_t)nargs, nullptr);
}

// dev(t, dtype, ndim=None): device address of a contiguous GPU tensor of this type (and rank).
PyObject *dev(PyObject *, PyObject *const *args, Py_ssize_t nargs) {
    if ((nargs == 2 || nargs == 3) && plain(args[0]) && THPDtype_Check(args[1])) try {
            const at::Tensor &t = THPVariable_Unpack(args[0]);
            const bool any_rank = nargs == 2 || args[2] == Py_None;
            if (t.is_cuda() && t.has_storage() && !t.is_conj() && !t.is_neg() && !t._is_zerotensor() &&
                t.layout() == at::kStrided && t.scalar_type() == reinterpret_cast<THPDtype *>(args[1])->scalar_type &&
                t.is_contiguous() && (any_rank || (PyLong_CheckExact(args[2]) && t.dim() == PyLong_AsLong(args[2]))))
                return PyLong_FromVoidPtr(t.data_ptr());
        } catch (...) {
            PyErr_Clear();
        }
    return call_general(general_dev, args, nargs);
}

// out(t, shape, dtype, device, name): a fresh output tensor, or the caller's if it has exactly this shape and type.
PyObject *out(PyObject *, PyObject *const *args, Py_ssize_t nargs) {
    constexpr Py_ssize_t MAX_RANK = 2;
    if (nargs == 5 && PyTuple_CheckExact(args[1]) && PyTuple_GET_SIZE(args[1]) <= MAX_RANK && THPDtype_Check(args[2]) &&
        THPDevice_Check(args[3])) {
        int64_t shape[MAX_RANK];
        const Py_ssize_t rank = PyTuple_GET_SIZE(args[1]);
        bool known = true;
        for (Py_ssize_t i = 0; i < rank; ++i) {
            PyObject *e = PyTuple_GET_ITEM(args[1], i);
            int overflow = 0;
            shape[i] = PyLong_CheckExact(e) ? PyLong_AsLongLongAndOverflow(e, &overflow) : -1;
            known = known && shape[i] >= 0 && !overflow;
        }
        const at::ScalarType type = reinterpret_cast<THPDtype *>(args[2])->scalar_type;
        const at::IntArrayRef sizes(shape, (size_t)rank);
        if (known && args[0] == Py_None && !at::impl::torch_function_mode_enabled()) try {
                const at::Device device = reinterpret_cast<THPDevice *>(args[3])->device;
                if (device.is_cuda()) {
                    at::Tensor t;
                    {
                        WithoutGil released;
                        t = at::empty(sizes, at::TensorOptions().dtype(type).device(device));
                    }
                    return THPVariable_Wrap(t);
                }
            } catch (...) {
                PyErr_Clear();
            }
        if (known && plain(args[0])) try {
                const at::Tensor &t = THPVariable_Unpack(args[0]);
                if (t.scalar_type() == type && t.sizes() == sizes) {
                    Py_INCREF(args[0]);
                    return args[0];
                }
            } catch (...) {
                PyErr_Clear();
            }
    }
    return call_general(general_out, args, nargs);
}

PyObject *general_forms(PyObject *, PyObject *const *args, Py_ssize_t nargs) {
    if (nargs != 2) {
        PyErr_SetString(PyExc_TypeError, "general_forms(dev, out)");
        return nullptr;
    }
    Py_INCREF(args[0]);
    Py_INCREF(args[1]);
    Py_XSETREF(general_dev, args[0]);
    Py_XSETREF(general_out, args[1]);
    Py_RETURN_NONE;
}

// What ctypes takes for these C types: integers (an address is one) modulo the type's range, None for a null pointer.
template <class T>
bool convert(PyObject *o, T &v) {
    if constexpr (std::is_pointer<T>::value) {
        if (o != Py_None && !PyLong_Check(o)) return false;
        v = o == Py_None ? nullptr : reinterpret_cast<T>((uintptr_t)PyLong_AsUnsignedLongLongMask(o));
    } else if constexpr (std::is_floating_point<T>::value) {
        v = (T)PyFloat_AsDouble(o);
    } else {
        if (!PyLong_Check(o)) return false;
        v = (T)PyLong_AsUnsignedLongLongMask(o);
    }
    return !PyErr_Occurred();
}

PyObject *refused(Py_ssize_t i) {
    PyErr_Clear();
    PyObject *m = PyImport_ImportModule("ctypes"), *e = m != nullptr ? PyObject_GetAttrString(m, "ArgumentError") : nullptr;
    if (e != nullptr) PyErr_Format(e, "argument %zd: wrong type", i + 1);
    Py_XDECREF(e);
    Py_XDECREF(m);
    return nullptr;
}

// One entry of the C ABI, its argument types taken from its declaration.
template <auto F, class... A, size_t... I>
PyObject *call_entry(int (*)(A...), PyObject *const *args, Py_ssize_t nargs, std::index_sequence<I...>) {
    if (nargs != (Py_ssize_t)sizeof...(A)) {
        PyErr_Format(PyExc_TypeError, "this function takes %zu arguments (%zd given)", sizeof...(A), nargs);
        return nullptr;
    }
    std::tuple<A...> v{};
    Py_ssize_t bad = -1;
    if (!((convert(args[I], std::get<I>(v)) || (bad = (Py_ssize_t)I, false)) && ...)) return refused(bad);
    int status;
    {
        WithoutGil released;
        status = F(std::get<I>(v)...);
    }
    return PyLong_FromLong(status);
}
template <class... A>
constexpr std::index_sequence_for<A...> indices_of(int (*)(A...)) {
    return {};
}
template <auto F>
PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t nargs) {
    return call_entry<F>(F, args, nargs, decltype(indices_of(F)){});
}

#define SB_METHOD(name, f) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
#define SB_ENTRY(name) SB_METHOD("switchback_" #name, &entry<&switchback_##name>)
PyMethodDef methods[] = {SB_METHOD("dev", &dev),
                         SB_METHOD("out", &out),
                         SB_METHOD("general_forms", &general_forms),
                         SB_ENTRY(quantize_rowwise),
                         SB_ENTRY(dequantize_rowwise),
                         SB_ENTRY(quantize_tensorwise),
                         SB_ENTRY(matmul_int8_dequant),
                         SB_ENTRY(matmul_int8_dequant_bias_layerscale),
                         SB_ENTRY(forward),
                         SB_ENTRY(forward_bias_layerscale),
                         SB_ENTRY(forward_static),
                         SB_ENTRY(backward_input),
                         SB_ENTRY(backward_weight),
                         SB_ENTRY(backward_weight_m),
                         SB_ENTRY(quantize_colwise_transpose),
                         SB_ENTRY(matmul_int8_dequant_rc),
                         SB_ENTRY(forward_q),
                         SB_ENTRY(backward_input_q),
                         SB_ENTRY(quantize_rowwise_f8),
                         SB_ENTRY(quantize_tensorwise_f8),
                         SB_ENTRY(matmul_f8_dequant),
                         SB_ENTRY(forward_f8),
                         SB_ENTRY(backward_input_f8),
                         SB_ENTRY(stable_adamw_step_multi),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
