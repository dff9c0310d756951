// Argument marshalling of the Python binding's calls in native code: the module _dab_call.
//
// A call through ctypes with its checks in Python cost 2.8 us more than one from here (six
// tensors: four attribute reads each, then one conversion per argument), which is what bounded a
// chain of small layers (nine calls of one sketch: 54 us, now 40).  Here a function is made
// from the signature of the entry point that it calls:
//   float* / int32_t* / uint8_t*    an fp32 / int32 / uint8 tensor on the GPU, contiguous, or None
//   void*                           any tensor or None (a workspace); the last one is the stream
//   const dab_conv_desc*            the binding's structure of that name
//   int32_t, size_t, float          numbers
// What is not plainly right is left to the binding's own Python: a tensor of another type, a subclass of
// Tensor or an active torch-function mode to its check, which either returns the address or raises, and
// what is no Python int or float (a scalar of numpy, a tensor of one element) to ctypes' conversion.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <array>
#include <tuple>
#include <type_traits>
#include <utility>

#include "dab.h"

namespace {

PyObject* g_pointer;         // (object, kind, name) -> address or None, or raises
PyObject* g_failed;          // (name, status): raises
PyObject* g_number;          // (object, kind) -> int or float as ctypes converts it, or raises
PyObject* g_desc_type;       // the binding's dab_conv_desc
PyObject* g_argument_error;  // ctypes.ArgumentError

template <typename T>
constexpr char kind_of() {
    using V = std::remove_const_t<T>;
    if constexpr (std::is_same_v<V, float>) return 'f';
    if constexpr (std::is_same_v<V, int32_t> || std::is_same_v<V, uint32_t>) return 'i';
    if constexpr (std::is_same_v<V, uint8_t>) return 'b';
    return 'v';
}

// A tensor's address.  name: what the binding calls the argument, or NULL where it checks nothing.
bool pointer(PyObject* o, char kind, const char* name, void** out) {
    if (o == Py_None) {
        *out = nullptr;
        return true;
    }
    if (name == nullptr) kind = 'v';
    if (THPVariable_CheckExact(o) && !at::impl::torch_function_mode_enabled()) {
        try {
            const at::Tensor& t = THPVariable_Unpack(o);
            const auto type = t.scalar_type();
            const bool same = kind == 'f' ? type == at::kFloat : kind == 'i' ? type == at::kInt : type == at::kByte;
            if (kind == 'v' || (same && t.is_cuda() && t.is_contiguous())) {
                *out = t.data_ptr();
                return true;
            }
        } catch (...) {
            // the Python check meets the same error and reports it
        }
    }
    PyObject* r = PyObject_CallFunction(g_pointer, "OCs", o, kind, name);
    if (r == nullptr) return false;
    *out = r == Py_None ? nullptr : PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    return !PyErr_Occurred();
}

bool wrong_type() {
    PyErr_SetString(g_argument_error, "wrong type");
    return false;
}

// A Python int or float.
template <typename T>
bool number(PyObject* o, T* out) {
    if constexpr (std::is_floating_point_v<T>) *out = static_cast<T>(PyFloat_AsDouble(o));
    else *out = static_cast<T>(PyLong_AsUnsignedLongLongMask(o));
    return !PyErr_Occurred();
}

template <typename T>
bool convert(PyObject* o, const char* name, T* out) {
    if constexpr (std::is_same_v<T, const dab_conv_desc*>) {
        Py_buffer view;
        if (!PyObject_TypeCheck(o, reinterpret_cast<PyTypeObject*>(g_desc_type))) return wrong_type();
        if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) return false;
        *out = static_cast<const dab_conv_desc*>(view.buf);      // alive as long as the caller's argument
        PyBuffer_Release(&view);
        return true;
    } else if constexpr (std::is_pointer_v<T>) {
        void* p = nullptr;
        if (!pointer(o, kind_of<std::remove_pointer_t<T>>(), name, &p)) return false;
        *out = static_cast<T>(p);
        return true;
    } else {
        constexpr bool kFloat = std::is_floating_point_v<T>;
        if (!PyLong_Check(o) && !(kFloat && PyFloat_Check(o))) {
            PyObject* r = PyObject_CallFunction(g_number, "OC", o, kFloat ? 'f' : sizeof(T) == 8 ? 'z' : 'i');
            if (r == nullptr) return false;
            const bool ok = number(r, out);
            Py_DECREF(r);
            return ok;
        }
        return number(o, out);
    }
}

// One entry point: its name and the names of its arguments (NULL: an unchecked tensor or a number).
template <auto Fn>
struct Entry;

template <typename R, typename... P, R (*Fn)(P...)>
struct Entry<Fn> {
    static inline const char* name;
    static inline const char* args[sizeof...(P) + 1];
    // a status is checked, and the stream supplied; sizes are returned
    static constexpr bool kStatus = std::is_same_v<R, int>;
    static constexpr size_t kArgs = sizeof...(P) - (kStatus ? 1 : 0);

    template <size_t... I>
    static bool convert_all(std::tuple<P...>& v, PyObject* const* a, std::index_sequence<I...>) {
        return (convert(a[I], args[I], &std::get<I>(v)) && ...);
    }

    static PyObject* call(PyObject*, PyObject* const* a, Py_ssize_t n) {
        if (n != static_cast<Py_ssize_t>(kArgs)) {
            PyErr_Format(PyExc_TypeError, "%s takes %zu arguments, got %zd", name, kArgs, n);
            return nullptr;
        }
        std::tuple<P...> v{};
        if (!convert_all(v, a, std::make_index_sequence<kArgs>{})) return nullptr;
        if constexpr (kStatus) {
            try {
                std::get<sizeof...(P) - 1>(v) = c10::hip::getCurrentHIPStream().stream();
            } catch (const std::exception& e) {
                PyErr_SetString(PyExc_RuntimeError, e.what());
                return nullptr;
            }
        }
        R r;
        Py_BEGIN_ALLOW_THREADS
        r = std::apply(Fn, v);
        Py_END_ALLOW_THREADS
        if constexpr (!kStatus) return PyLong_FromSize_t(r);
        if (r == 0) Py_RETURN_NONE;
        return PyObject_CallFunction(g_failed, "si", name, static_cast<int>(r));
    }

    template <typename... N>
    static PyMethodDef def(const char* entry, N... arg_names) {
        static_assert(sizeof...(N) == kArgs, "one name per argument");
        name = entry;
        size_t i = 0;
        ((args[i++] = arg_names), ...);
        return PyMethodDef{entry, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&call)), METH_FASTCALL, nullptr};
    }
};

PyObject* setup(PyObject*, PyObject* args) {
    PyObject *pointer_fn, *failed_fn, *number_fn, *desc, *error;
    if (!PyArg_ParseTuple(args, "OOOOO", &pointer_fn, &failed_fn, &number_fn, &desc, &error)) return nullptr;
    Py_INCREF(pointer_fn), Py_INCREF(failed_fn), Py_INCREF(number_fn), Py_INCREF(desc), Py_INCREF(error);
    g_pointer = pointer_fn, g_failed = failed_fn, g_number = number_fn, g_desc_type = desc, g_argument_error = error;
    Py_RETURN_NONE;
}

constexpr std::nullptr_t _ = nullptr;
#define ENTRY(fn, ...) Entry<&fn>::def(#fn, __VA_ARGS__)

PyMethodDef* methods() {
    static PyMethodDef m[] = {
        ENTRY(dab_estimate_alpha_beta, "W", _, _, _, _, _, _, _, _, _, _),
        ENTRY(dab_estimate_alpha_beta_bounded, "W", _, _, "K_prev", "alpha_is_upper_prev", _, "alpha", "beta", "K", "thr_val",
              "thr_idx", "alpha_is_upper", _, _),
        ENTRY(dab_estimate_sign_split, "W", _, _, _, _, _, _, _, _),
        ENTRY(dab_estimate_workspace_bytes, _, _),
        ENTRY(dab_pack_weights, "W", _, _, _, _, "thr_val", "thr_idx", "alpha_is_upper", "E_packed", "ecnt"),
        ENTRY(dab_pack_activations, "X", _, _, _, _, _, "tau", "A_packed"),
        ENTRY(dab_binconv2d, _, "A_packed", "E_packed", "alpha", "beta", "Y", _, _, _),
        ENTRY(dab_binconv2d_workspace_bytes, _),
        ENTRY(dab_binfc, _, _, _, "A_packed", "E_packed", "alpha", "beta", "Y", _, _, _),
        ENTRY(dab_binfc_workspace_bytes, _, _, _),
        ENTRY(dab_binconv2d_bits, _, "A_packed", "E_packed", "alpha", "beta", "tau_out", "A_next", _, _),
        ENTRY(dab_binfc_bits, _, _, _, "A_packed", "E_packed", "alpha", "beta", "tau_out", "A_next", _, _),
        ENTRY(dab_pool_bits, "A_packed", _, _, _, _, _, _, _, _, "A_pooled"),
        ENTRY(dab_wbin_conv2d, _, "X", "E_packed", "alpha", "beta", "Y", _, _),
        ENTRY(dab_wbin_conv2d_workspace_bytes, _),
        ENTRY(dab_wbin_fc, _, _, _, "X", "E_packed", "alpha", "beta", "Y", _, _),
        ENTRY(dab_wbin_fc_workspace_bytes, _, _, _),
        ENTRY(dab_mean_center_clamp, "W", _, _, _, _, _, _, "W_out"),
        ENTRY(dab_binarized_weights, "W", _, _, "alpha", "beta", "thr_val", "thr_idx", "alpha_is_upper", "W_tilde"),
        ENTRY(dab_weight_gradient, "W", _, _, "thr_val", "thr_idx", "alpha_is_upper", "upstream", "G_out"),
        {"setup", setup, METH_VARARGS, nullptr},
        {nullptr, nullptr, 0, nullptr},
    };
    return m;
}

}  // namespace

PyMODINIT_FUNC PyInit__dab_call() {
    static PyModuleDef def = {PyModuleDef_HEAD_INIT, "_dab_call", nullptr, -1, methods()};
    return PyModule_Create(&def);
}
