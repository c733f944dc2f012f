// Python side of the C ABI: the calls themselves and the two checks that every call makes of its tensors, as built-in
// functions.  A small layer's pass is bound by the host: each of its launches takes 3 us, and what Python and ctypes add
// to a call is of the same size.  The general forms stay in Python (the checks) and ctypes (the calls): whatever is not a
// plain tensor that passes (subclasses, function modes, wrong types and shapes) or not a plain argument (ctypes objects,
// wrong types and numbers of them) goes to those, which raise or answer as they always did.
//
// The tensor checks read tensors through the headers of the torch that this file is compiled against, so the module says
// which one that is (built_for), and the caller uses it with no other.  It links no library of kernels: bind() gets the
// addresses of one that is loaded, and returns functions that carry them, so two libraries may be bound side by side.
#include <Python.h>

#include <ATen/Functions.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <torch/csrc/Device.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <new>
#include <tuple>
#include <type_traits>
#include <utility>

#include "../../include/switchback.h"

namespace {

struct WithoutGil {  // other Python threads run meanwhile
    PyThreadState *state = PyEval_SaveThread();
    ~WithoutGil() { PyEval_RestoreThread(state); }
};

bool plain(PyObject *o) { return THPVariable_CheckExact(o) && !at::impl::torch_function_mode_enabled(); }

struct Entry {
    void *address;
    PyObject *general;  // the ctypes function
};
// What bind() was given: the self of every function that it returns.
struct Bound {
    PyObject *dev = nullptr, *out = nullptr;  // the checks in Python
    PyObject *saved_type = nullptr;           // ctypes structure of sb_saved
    Entry entries[32] = {};
    ~Bound() {
        Py_XDECREF(dev);
        Py_XDECREF(out);
        Py_XDECREF(saved_type);
        for (Entry &e : entries) Py_XDECREF(e.general);
    }
};
Bound *bound(PyObject *self) { return static_cast<Bound *>(PyCapsule_GetPointer(self, nullptr)); }

PyObject *call_general(PyObject *f, PyObject *const *args, Py_ssize_t nargs) {
    return PyObject_Vectorcall(f, args, (size_t)nargs, nullptr);
}

// dev(t, dtype, ndim=None): device address of a contiguous GPU tensor of this type (and rank).
PyObject *dev(PyObject *self, PyObject *const *args, Py_ssize_t nargs) {
    if ((nargs == 2 || nargs == 3) && plain(args[0]) && THPDtype_Check(args[1])) try {
            const at::Tensor &t = THPVariable_Unpack(args[0]);
            int overflow = 0;
            const bool any_rank = nargs == 2 || args[2] == Py_None;
            if (t.is_cuda() && t.has_storage() && !t.is_conj() && !t.is_neg() && !t._is_zerotensor() &&
                t.layout() == at::kStrided && t.scalar_type() == reinterpret_cast<THPDtype *>(args[1])->scalar_type &&
                t.is_contiguous() && (any_rank || (PyLong_CheckExact(args[2]) && t.dim() == PyLong_AsLongAndOverflow(args[2], &overflow))))
                return PyLong_FromVoidPtr(t.data_ptr());
        } catch (...) {
            PyErr_Clear();
        }
    return call_general(bound(self)->dev, args, nargs);
}

// out(t, shape, dtype, device, name): a fresh output tensor, or the caller's if it has exactly this shape and type.
PyObject *out(PyObject *self, PyObject *const *args, Py_ssize_t nargs) {
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
    return call_general(bound(self)->out, args, nargs);
}

// What ctypes takes for these C types: integers (an address is one) modulo the type's range, None for a null pointer, the
// structure itself for a pointer to it.
template <class T>
bool convert(PyObject *o, T &v, PyObject *saved_type) {
    if constexpr (std::is_same<T, const sb_saved *>::value) {
        Py_buffer view;
        if (o == Py_None) {
            v = nullptr;
        } else if (reinterpret_cast<PyObject *>(Py_TYPE(o)) != saved_type || PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) {
            return false;
        } else {  // the caller's reference keeps it
            v = static_cast<T>(view.buf);
            PyBuffer_Release(&view);
        }
    } else if constexpr (std::is_pointer<T>::value) {
        if (o != Py_None && !PyLong_Check(o)) return false;
        v = o == Py_None ? nullptr : reinterpret_cast<T>((uintptr_t)PyLong_AsUnsignedLongLongMask(o));
    } else if constexpr (std::is_floating_point<T>::value) {
        if (!PyFloat_Check(o) && !PyLong_Check(o)) return false;
        v = (T)PyFloat_AsDouble(o);
    } else {
        if (!PyLong_Check(o)) return false;
        v = (T)PyLong_AsUnsignedLongLongMask(o);
    }
    return !PyErr_Occurred();
}

// One entry of the C ABI, its argument types taken from its declaration.
template <class... A, size_t... I>
PyObject *call_entry(int (*)(A...), const Entry &e, PyObject *saved_type, PyObject *const *args, Py_ssize_t nargs,
                     std::index_sequence<I...>) {
    std::tuple<A...> v{};
    if (nargs != (Py_ssize_t)sizeof...(A) || !(convert(args[I], std::get<I>(v), saved_type) && ...)) {
        PyErr_Clear();
        return call_general(e.general, args, nargs);
    }
    int status;
    {
        WithoutGil released;
        status = reinterpret_cast<int (*)(A...)>(e.address)(std::get<I>(v)...);
    }
    return PyLong_FromLong(status);
}
template <class... A>
constexpr std::index_sequence_for<A...> indices_of(int (*)(A...)) {
    return {};
}
template <size_t INDEX, class F>
PyObject *entry(PyObject *self, PyObject *const *args, Py_ssize_t nargs) {
    Bound *b = bound(self);
    return call_entry((F) nullptr, b->entries[INDEX], b->saved_type, args, nargs, decltype(indices_of((F) nullptr)){});
}

#define SB_METHOD(name, f) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
#define SB_ENTRY(name) SB_METHOD("switchback_" #name, (&entry<__COUNTER__ - FIRST, decltype(&switchback_##name)>))
constexpr size_t CHECKS = 2, FIRST = __COUNTER__ + 1;
PyMethodDef bound_methods[] = {SB_METHOD("dev", &dev),
                               SB_METHOD("out", &out),
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
                               SB_ENTRY(stable_adamw_step_multi)};
constexpr size_t ENTRIES = sizeof(bound_methods) / sizeof(bound_methods[0]) - CHECKS;

// bind(dev, out, saved_type, entry) -> {name: built-in function}: the general forms of the checks, the ctypes structure of
// sb_saved, and a function that gives an entry's address and ctypes function by name.
PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t nargs) {
    if (nargs != 4) {
        PyErr_SetString(PyExc_TypeError, "bind(dev, out, saved_type, entry)");
        return nullptr;
    }
    static_assert(ENTRIES <= sizeof(Bound::entries) / sizeof(Entry), "entries");
    Bound *b = new (std::nothrow) Bound;
    PyObject *self = b == nullptr ? PyErr_NoMemory() : PyCapsule_New(b, nullptr, [](PyObject *c) { delete bound(c); });
    if (self == nullptr) {
        delete b;
        return nullptr;
    }
    for (Py_ssize_t i = 0; i < 3; ++i) Py_INCREF(args[i]);
    b->dev = args[0], b->out = args[1], b->saved_type = args[2];
    PyObject *functions = PyDict_New();
    bool ok = functions != nullptr;
    for (size_t i = 0; ok && i < CHECKS + ENTRIES; ++i) {
        if (i >= CHECKS) {
            PyObject *pair = PyObject_CallFunction(args[3], "s", bound_methods[i].ml_name);
            unsigned long long address = 0;
            Entry e{nullptr, nullptr};
            ok = pair != nullptr && PyArg_ParseTuple(pair, "KO", &address, &e.general);
            if (ok) {
                e.address = reinterpret_cast<void *>((uintptr_t)address);
                Py_INCREF(e.general);
                b->entries[i - CHECKS] = e;
            }
            Py_XDECREF(pair);
        }
        PyObject *f = ok ? PyCFunction_New(&bound_methods[i], self) : nullptr;
        ok = f != nullptr && PyDict_SetItemString(functions, bound_methods[i].ml_name, f) == 0;
        Py_XDECREF(f);
    }
    Py_DECREF(self);
    if (!ok) Py_CLEAR(functions);
    return functions;
}

PyMethodDef methods[] = {SB_METHOD("bind", &bind), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() {
    PyObject *m = PyModule_Create(&module);
    if (m != nullptr && PyModule_AddStringConstant(m, "built_for", SB_BUILT_FOR) != 0) Py_CLEAR(m);
    return m;
}
