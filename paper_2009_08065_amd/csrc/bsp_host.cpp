// The C entry points as Python functions of tensors, and the allocation of results.
//
// What bounds it: a small call (one layer of 24 tokens, an update of a million weights) is 3 to 6 us on the GPU, and a
// program that issues them one after the other was bound by what the host did per call: through ctypes 6.6 us for a planned
// layer (2.5 of it the launch), 1.8 of them torch.empty from Python, 0.2 per tensor for its checks and 1 for the
// conversion of the arguments.  Here the conversions are made by the signature of the C function at compile time.
// Host time of a call: bsp_linear_planned 6.6 -> 4.9 us, an encoder layer's four 26.8 -> 20.0 (the GPU's part is 21.6),
// factors and update of 1024 x 1024 weights 12.6 -> 9.7, the layer in single precision 8.2 -> 5.3.
//
// The checks are the binding's own: a tensor is contiguous and on the GPU, and of its pointer's type where that function
// asks for it.  Only plain tensors are read directly; anything else is asked through its Python attributes, as before.
// The interpreter lock is released during the call, as ctypes does, and while results are allocated, as torch does.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>
#include <tuple>
#include <type_traits>
#include <utility>

#include "bsp.h"

namespace {

enum Check : unsigned { kNone = 0, kFloat = 1, kByte = 2, kInt = 4, kAll = 7 };

bool wrong_place() {
    PyErr_SetString(PyExc_ValueError, "tensor must be a contiguous GPU tensor");
    return false;
}

bool wrong_type(PyObject *o, const char *want) {
    PyObject *dtype = PyObject_GetAttrString(o, "dtype");
    if (!dtype) return false;
    PyErr_Format(PyExc_ValueError, "expected dtype torch.%s, got %S", want, dtype);
    Py_DECREF(dtype);
    return false;
}

// An object that is no plain tensor: by its attributes.
bool read_other(PyObject *o, const char *want, void *&out) {
    PyObject *flag = PyObject_GetAttrString(o, "is_cuda");
    if (!flag) return false;
    const int cuda = PyObject_IsTrue(flag);
    Py_DECREF(flag);
    if (cuda < 0) return false;
    if (!cuda) return wrong_place();
    PyObject *dense = PyObject_CallMethod(o, "is_contiguous", nullptr);
    if (!dense) return false;
    const int contiguous = PyObject_IsTrue(dense);
    Py_DECREF(dense);
    if (contiguous < 0) return false;
    if (!contiguous) return wrong_place();
    if (want) {
        PyObject *dtype = PyObject_GetAttrString(o, "dtype");
        if (!dtype) return false;
        PyObject *name = PyObject_Str(dtype);
        Py_DECREF(dtype);
        if (!name) return false;
        const char *text = PyUnicode_AsUTF8(name);
        const bool same = text && strncmp(text, "torch.", 6) == 0 && strcmp(text + 6, want) == 0;
        Py_DECREF(name);
        if (!same) return PyErr_Occurred() ? false : wrong_type(o, want);
    }
    PyObject *at = PyObject_CallMethod(o, "data_ptr", nullptr);
    if (!at) return false;
    out = PyLong_AsVoidPtr(at);
    Py_DECREF(at);
    return !PyErr_Occurred();
}

bool read_tensor(PyObject *o, const char *want, at::ScalarType type, void *&out) {
    if (o == Py_None) {
        out = nullptr;
        return true;
    }
    if (!THPVariable_CheckExact(o)) return read_other(o, want, out);
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous()) return wrong_place();
    if (want && t.scalar_type() != type) return wrong_type(o, want);
    out = t.data_ptr();
    return true;
}

// What else stands for a number, as for ctypes: its own scalar of the argument's type, and an object that names another as its
// _as_parameter_.  A new reference, or null with the error that was set.
PyObject *other_number(PyObject *o, const char *scalar) {
    if (!PyErr_ExceptionMatches(PyExc_TypeError)) return nullptr;
    PyObject *type, *value, *trace;
    PyErr_Fetch(&type, &value, &trace);
    PyObject *n = strcmp(Py_TYPE(o)->tp_name, scalar) == 0 ? PyObject_GetAttrString(o, "value") : nullptr;
    if (!n) {
        PyErr_Clear();
        n = PyObject_GetAttrString(o, "_as_parameter_");
    }
    if (n) {
        Py_XDECREF(type);
        Py_XDECREF(value);
        Py_XDECREF(trace);
    } else {
        PyErr_Clear();
        PyErr_Restore(type, value, trace);
    }
    return n;
}

// The number that stands in another's place, which may name one in turn (without end, if it names itself).  Takes the reference.
template <typename T>
bool read_instead(PyObject *n, bool (*read_number)(PyObject *, T &), T &out) {
    bool ok = Py_EnterRecursiveCall(" while processing _as_parameter_") == 0;
    if (ok) {
        ok = read_number(n, out);
        Py_LeaveRecursiveCall();
    }
    Py_DECREF(n);
    return ok;
}

// Whole numbers: everything with __index__ (numpy's, a tensor of one).  Of one larger than the type the low bits.
template <typename T>
bool read_whole(PyObject *o, T &out) {
    PyObject *n = PyNumber_Index(o);
    if (!n) {
        n = other_number(o, std::is_unsigned_v<T> ? "c_ulong" : (sizeof(T) == 8 ? "c_long" : "c_int"));
        return n && read_instead(n, read_whole<T>, out);
    }
    out = static_cast<T>(PyLong_AsUnsignedLongLongMask(n));
    Py_DECREF(n);
    return true;
}

bool read_real(PyObject *o, float &out) {
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) {
        PyObject *n = other_number(o, "c_float");
        return n && read_instead(n, read_real, out);
    }
    out = static_cast<float>(v);
    return true;
}

// STREAM: the argument is the stream, an address.
template <unsigned C, bool STREAM, typename T>
bool read(PyObject *o, T &out) {
    if constexpr (STREAM) {
        out = PyLong_AsVoidPtr(o);
        return !PyErr_Occurred();
    } else if constexpr (std::is_pointer_v<T>) {
        using V = std::remove_cv_t<std::remove_pointer_t<T>>;
        void *p = nullptr;
        bool ok;
        if constexpr (std::is_same_v<V, float> && (C & kFloat)) ok = read_tensor(o, "float32", at::kFloat, p);
        else if constexpr (std::is_same_v<V, uint8_t> && (C & kByte)) ok = read_tensor(o, "uint8", at::kByte, p);
        else if constexpr (std::is_same_v<V, int32_t> && (C & kInt)) ok = read_tensor(o, "int32", at::kInt, p);
        else ok = read_tensor(o, nullptr, at::kByte, p);
        out = static_cast<T>(p);
        return ok;
    } else if constexpr (std::is_floating_point_v<T>) {
        return read_real(o, out);
    } else {
        return read_whole(o, out);
    }
}

struct Unlocked {  // the interpreter lock, given up for its lifetime
    PyThreadState *state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};

template <auto Fn, unsigned C>
struct Entry;
template <typename Ret, typename... A, Ret (*Fn)(A...), unsigned C>
struct Entry<Fn, C> {
    template <size_t... I>
    static PyObject *call(PyObject *const *args, std::index_sequence<I...>) {
        std::tuple<A...> a{};
        constexpr auto is_stream = [](size_t i) { return i == sizeof...(A) - 1; };
        if (!(read<C, is_stream(I) && std::is_pointer_v<A>>(args[I], std::get<I>(a)) && ...)) return nullptr;
        Ret r;
        {
            const Unlocked unlocked;
            r = Fn(std::get<I>(a)...);
        }
        if constexpr (std::is_signed_v<Ret>) return PyLong_FromLongLong(r);
        else return PyLong_FromUnsignedLongLong(r);
    }
    static PyObject *run(PyObject *, PyObject *const *args, Py_ssize_t n) {
        HANDLE_TH_ERRORS
        if (n != (Py_ssize_t)sizeof...(A)) {
            PyErr_Format(PyExc_TypeError, "this function takes %d arguments (%zd given)", (int)sizeof...(A), n);
            return nullptr;
        }
        return call(args, std::make_index_sequence<sizeof...(A)>{});
        END_HANDLE_TH_ERRORS
    }
};

// empty() beside an object that is no plain tensor: torch.empty with the object's own device.
PyObject *empty_beside_other(PyObject *like, const char *type, const int64_t *size, int dims) {
    PyObject *torch = PyImport_ImportModule("torch");
    if (!torch) return nullptr;
    PyObject *make = PyObject_GetAttrString(torch, "empty"), *dtype = PyObject_GetAttrString(torch, type);
    PyObject *device = PyObject_GetAttrString(like, "device"), *result = nullptr;
    PyObject *args = dims == 1 ? Py_BuildValue("((L))", (long long)size[0]) : Py_BuildValue("((LL))", (long long)size[0], (long long)size[1]);
    if (make && dtype && device && args) {
        PyObject *named = Py_BuildValue("{s:O,s:O}", "dtype", dtype, "device", device);
        if (named) result = PyObject_Call(make, args, named);
        Py_XDECREF(named);
    }
    Py_DECREF(torch);
    Py_XDECREF(make);
    Py_XDECREF(dtype);
    Py_XDECREF(device);
    Py_XDECREF(args);
    return result;
}

// empty(like, type, n) or empty(like, type, n, m): a tensor on the device of `like`; type: a bsp_dtype, 3 uint8, 4 int32.
PyObject *empty(PyObject *, PyObject *const *args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 3 && n != 4) {
        PyErr_SetString(PyExc_TypeError, "empty(tensor, type, n[, m])");
        return nullptr;
    }
    constexpr at::ScalarType types[] = {at::kFloat, at::kBFloat16, at::kHalf, at::kByte, at::kInt};
    constexpr const char *names[] = {"float32", "bfloat16", "float16", "uint8", "int32"};
    const long long type = PyLong_AsLongLong(args[1]);
    int64_t size[2] = {0, 0};
    for (Py_ssize_t i = 2; i < n; ++i) size[i - 2] = PyLong_AsLongLong(args[i]);
    if (PyErr_Occurred()) return nullptr;
    if (type < 0 || type > 4) {
        PyErr_SetString(PyExc_ValueError, "unknown type");
        return nullptr;
    }
    if (!THPVariable_CheckExact(args[0])) return empty_beside_other(args[0], names[type], size, (int)n - 2);
    const auto options = at::TensorOptions().dtype(types[type]).device(THPVariable_Unpack(args[0]).device());
    at::Tensor t;
    {
        const Unlocked unlocked;  // (an allocation may wait for the device)
        t = at::empty(at::IntArrayRef(size, (size_t)(n - 2)), options);
    }
    return THPVariable_Wrap(std::move(t));
    END_HANDLE_TH_ERRORS
}

// last(tensor): the last element of a vector of whole numbers, read back; of an object that is no plain tensor int(o[-1].item()).
PyObject *last(PyObject *, PyObject *o) {
    HANDLE_TH_ERRORS
    if (!THPVariable_CheckExact(o)) {
        PyObject *at = PyLong_FromLong(-1), *element = at ? PyObject_GetItem(o, at) : nullptr;
        PyObject *value = element ? PyObject_CallMethod(element, "item", nullptr) : nullptr;
        PyObject *whole = value ? PyNumber_Long(value) : nullptr;
        Py_XDECREF(at);
        Py_XDECREF(element);
        Py_XDECREF(value);
        return whole;
    }
    const at::Tensor &t = THPVariable_Unpack(o);
    int64_t v;
    {
        const Unlocked unlocked;
        v = t.select(0, -1).item().toLong();
    }
    return PyLong_FromLongLong(v);
    END_HANDLE_TH_ERRORS
}

#define BSP_ENTRY(name, check) \
    {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&Entry<&name, check>::run)), METH_FASTCALL, nullptr}

PyMethodDef methods[] = {
    BSP_ENTRY(bsp_group_norms, kFloat),
    BSP_ENTRY(bsp_group_norms_grad, kFloat),
    BSP_ENTRY(bsp_prune_mask, kFloat | kByte),
    BSP_ENTRY(bsp_prune_mask_workspace_bytes, kNone),
    BSP_ENTRY(bsp_prune_mask_count, kAll),
    BSP_ENTRY(bsp_pack_count, kAll),
    BSP_ENTRY(bsp_pack, kAll),
    BSP_ENTRY(bsp_mask_weights, kByte),
    BSP_ENTRY(bsp_adam_step, kFloat | kByte),
    BSP_ENTRY(bsp_linear_workspace_bytes, kNone),
    BSP_ENTRY(bsp_linear_sized, kNone),
    BSP_ENTRY(bsp_linear_transposed_workspace_bytes, kNone),
    BSP_ENTRY(bsp_linear_transposed_ws, kNone),
    BSP_ENTRY(bsp_linear_dvals_workspace_bytes, kNone),
    BSP_ENTRY(bsp_linear_dvals, kNone),
    BSP_ENTRY(bsp_linear_plan_bytes, kNone),
    BSP_ENTRY(bsp_linear_plan, kNone),
    BSP_ENTRY(bsp_linear_planned, kNone),
    BSP_ENTRY(bsp_linear_planned_fused, kNone),
    {"empty", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&empty)), METH_FASTCALL, nullptr},
    {"last", last, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_bsp_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__bsp_host() { return PyModule_Create(&module_def); }
