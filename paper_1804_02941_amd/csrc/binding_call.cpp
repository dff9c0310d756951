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
#include <ATen/ops/empty.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
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

// ---------------------------------------------------------------- whole calls
// A layer's call with nothing unusual about it, sizes, output and workspace included: the tensors plain fp32 / int32
// ones on the GPU, contiguous and not empty, numbers Python ints, no mode active.  Whatever is not so is left to the binding's
// Python, which does the same by the entry points above or raises: the functions then return None, before anything is
// launched.  Sizes read, the output allocated and the checks done in Python were 1 us of a call of 5: 16 x 4096 -> 4096,
// packing and product with new outputs, 12.6 -> 10.3 us; one sketch through six layers, nine calls into kept buffers, 38.6 -> 37.3.
struct Unusual {};

const at::Tensor& plain(PyObject* o, at::ScalarType type) {
    if (!THPVariable_CheckExact(o)) throw Unusual{};
    const at::Tensor& t = THPVariable_Unpack(o);
    if (t.scalar_type() != type || !t.is_cuda() || !t.is_contiguous() || t.numel() == 0) throw Unusual{};
    return t;
}
template <typename T>
T* address(PyObject* o) {
    return static_cast<T*>(plain(o, std::is_same_v<std::remove_const_t<T>, float> ? at::kFloat : at::kInt).data_ptr());
}
template <typename T>
T* address_or_none(PyObject* o) {
    return o == Py_None ? nullptr : address<T>(o);
}
int32_t whole(int64_t v) {
    if (v < 1 || v > INT32_MAX) throw Unusual{};
    return static_cast<int32_t>(v);
}
int32_t small_int(PyObject* o) {
    int overflow = 0;
    if (!PyLong_CheckExact(o)) throw Unusual{};
    const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow || v < 0 || v > INT32_MAX) throw Unusual{};
    return static_cast<int32_t>(v);
}
dab_conv_desc layer(PyObject* o) {
    const dab_conv_desc* d = nullptr;
    if (!PyObject_TypeCheck(o, reinterpret_cast<PyTypeObject*>(g_desc_type)) || !convert(o, nullptr, &d)) {
        PyErr_Clear();
        throw Unusual{};
    }
    if (d->stride_h < 1 || d->stride_w < 1) throw Unusual{};
    return *d;
}
int64_t extent(int32_t in, int32_t pad, int32_t k, int32_t stride) {
    const int64_t room = int64_t{in} + 2 * int64_t{pad} - k;
    if (room < 0) throw Unusual{};
    return room / stride + 1;
}
int64_t words(int64_t n) { return (n + 31) / 32; }

// The buffers of a call: the output and the workspace (if one is needed) are the caller's, or new ones.  (A missing workspace left
// to Python cost an exception and the output allocated twice: 8192 x 2400 -> 1284 without one 7.9 us of host time, 10.2 with a new
// output, by Python alone 6.4 and 7.9, now 5.8 and 6.3.)
struct Buffers {
    PyObject* given;
    at::ScalarType type;
    c10::SmallVector<int64_t, 4> shape;
    c10::Device device;
    size_t ws_bytes = 0;
    at::Tensor made, scratch;
    void *out = nullptr, *ws = nullptr;

    Buffers(PyObject* o, at::ScalarType t, std::initializer_list<int64_t> s, const at::Tensor& beside)
        : given(o), type(t), shape(s), device(beside.device()) {
        if (o != Py_None) out = plain(o, t).data_ptr();
    }
    Buffers& workspace(size_t nbytes, PyObject* o) {
        ws_bytes = nbytes;
        if (nbytes == 0 || o == Py_None) return *this;
        if (!THPVariable_CheckExact(o)) throw Unusual{};
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.is_cuda()) throw Unusual{};
        if (t.nbytes() >= nbytes) ws = t.data_ptr();
        return *this;
    }
    void allocate() {
        if (out == nullptr) {
            made = at::empty(shape, at::TensorOptions().dtype(type).device(device));
            out = made.data_ptr();
        }
        if (ws_bytes != 0 && ws == nullptr) {
            scratch = at::empty({static_cast<int64_t>(ws_bytes)}, at::TensorOptions().dtype(at::kByte).device(device));
            ws = scratch.data_ptr();
        }
    }
    PyObject* result() {
        if (given == Py_None) return THPVariable_Wrap(std::move(made));
        Py_INCREF(given);
        return given;
    }
};
struct WithoutGil {
    PyThreadState* state = PyEval_SaveThread();
    ~WithoutGil() { PyEval_RestoreThread(state); }
};

// Sizes and pointers by `prepare` (which may find the call unusual), then the new buffers and the launch, without the
// interpreter's lock: an allocation may wait for the device, and other threads run on meanwhile, as during torch.empty.
template <size_t N, typename Prepare>
PyObject* whole_call(const char* name, Py_ssize_t n, Prepare&& prepare) {
    if (n != static_cast<Py_ssize_t>(N)) return PyErr_Format(PyExc_TypeError, "%s takes %zu arguments, got %zd", name, N, n);
    try {
        if (at::impl::torch_function_mode_enabled() || c10::impl::dispatch_mode_enabled()) Py_RETURN_NONE;
        auto [buffers, enqueue] = prepare();
        int rc;
        {
            WithoutGil released;
            buffers.allocate();
            rc = enqueue(buffers, c10::hip::getCurrentHIPStream().stream());
        }
        if (rc != 0) return PyObject_CallFunction(g_failed, "si", name, rc);
        return buffers.result();
    } catch (...) {
        // not a plain call, or torch has refused something: Python meets the same and reports it
        Py_RETURN_NONE;
    }
}

// (X, layout, tau, out)
PyObject* pack_activations(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return whole_call<4>("dab_pack_activations", n, [&] {
        const at::Tensor& X = plain(a[0], at::kFloat);
        const int32_t layout = small_int(a[1]);
        if ((X.dim() != 2 && X.dim() != 4) || layout > DAB_LAYOUT_NCHW) throw Unusual{};
        const bool flat = X.dim() == 2, nhwc = layout == DAB_LAYOUT_NHWC;
        const int32_t B = whole(X.size(0)), C = whole(flat ? X.size(1) : X.size(nhwc ? 3 : 1));
        const int32_t H = flat ? 1 : whole(X.size(nhwc ? 1 : 2)), W = flat ? 1 : whole(X.size(nhwc ? 2 : 3));
        const float *x = address<const float>(a[0]), *tau = address_or_none<const float>(a[2]);
        return std::pair(Buffers(a[3], at::kInt, {B, H, W, words(C)}, X), [=](const Buffers& b, void* st) {
            return ::dab_pack_activations(x, layout, B, C, H, W, tau, static_cast<uint32_t*>(b.out), st);
        });
    });
}
// (desc, A_packed, E_packed, alpha, beta, out, ws)
PyObject* binconv2d(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return whole_call<7>("dab_binconv2d", n, [&] {
        const dab_conv_desc d = layer(a[0]);
        const at::Tensor& A = plain(a[1], at::kInt);
        const auto *bits = reinterpret_cast<const uint32_t*>(A.data_ptr()), *E = reinterpret_cast<const uint32_t*>(address<int32_t>(a[2]));
        const float *alpha = address<const float>(a[3]), *beta = address<const float>(a[4]);
        Buffers Y(a[5], at::kFloat, {whole(d.B), extent(d.H, d.pad_h, d.kh, d.stride_h), extent(d.W, d.pad_w, d.kw, d.stride_w), whole(d.F)}, A);
        Y.workspace(::dab_binconv2d_workspace_bytes(&d), a[6]);
        return std::pair(std::move(Y), [=](const Buffers& b, void* st) {
            return ::dab_binconv2d(&d, bits, E, alpha, beta, static_cast<float*>(b.out), nullptr, b.ws, b.ws_bytes, st);
        });
    });
}
// (desc, A_packed, E_packed, alpha, beta, tau_out, out, ws)
PyObject* binconv2d_bits(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return whole_call<8>("dab_binconv2d_bits", n, [&] {
        const dab_conv_desc d = layer(a[0]);
        const at::Tensor& A = plain(a[1], at::kInt);
        const auto *bits = reinterpret_cast<const uint32_t*>(A.data_ptr()), *E = reinterpret_cast<const uint32_t*>(address<int32_t>(a[2]));
        const float *alpha = address<const float>(a[3]), *beta = address<const float>(a[4]), *tau = address_or_none<const float>(a[5]);
        Buffers next(a[6], at::kInt,
                     {whole(d.B), extent(d.H, d.pad_h, d.kh, d.stride_h), extent(d.W, d.pad_w, d.kw, d.stride_w), words(whole(d.F))}, A);
        next.workspace(::dab_binconv2d_workspace_bytes(&d), a[7]);
        return std::pair(std::move(next), [=](const Buffers& b, void* st) {
            return ::dab_binconv2d_bits(&d, bits, E, alpha, beta, tau, static_cast<uint32_t*>(b.out), b.ws, b.ws_bytes, st);
        });
    });
}
// (A_packed, E_packed, alpha, beta, Kin, out, ws)
PyObject* binfc(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return whole_call<7>("dab_binfc", n, [&] {
        const at::Tensor &A = plain(a[0], at::kInt), &al = plain(a[2], at::kFloat);
        if (A.dim() < 1 || al.dim() < 1) throw Unusual{};
        const int32_t B = whole(A.size(0)), F = whole(al.size(0)), Kin = small_int(a[4]);
        const auto *bits = reinterpret_cast<const uint32_t*>(A.data_ptr()), *E = reinterpret_cast<const uint32_t*>(address<int32_t>(a[1]));
        const float *alpha = address<const float>(a[2]), *beta = address<const float>(a[3]);
        Buffers Y(a[5], at::kFloat, {B, F}, A);
        Y.workspace(::dab_binfc_workspace_bytes(B, Kin, F), a[6]);
        return std::pair(std::move(Y), [=](const Buffers& b, void* st) {
            return ::dab_binfc(B, Kin, F, bits, E, alpha, beta, static_cast<float*>(b.out), nullptr, b.ws, b.ws_bytes, st);
        });
    });
}
// (A_packed, C, kh, kw, stride_h, stride_w, out)
PyObject* pool_bits(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return whole_call<7>("dab_pool_bits", n, [&] {
        const at::Tensor& A = plain(a[0], at::kInt);
        if (A.dim() != 4) throw Unusual{};
        const int32_t B = whole(A.size(0)), H = whole(A.size(1)), W = whole(A.size(2));
        const int32_t C = small_int(a[1]), kh = small_int(a[2]), kw = small_int(a[3]), sh = whole(small_int(a[4])), sw = whole(small_int(a[5]));
        const auto* bits = reinterpret_cast<const uint32_t*>(A.data_ptr());
        return std::pair(Buffers(a[6], at::kInt, {B, extent(H, 0, kh, sh), extent(W, 0, kw, sw), A.size(3)}, A), [=](const Buffers& b, void* st) {
            return ::dab_pool_bits(bits, B, C, H, W, kh, kw, sh, sw, static_cast<uint32_t*>(b.out), st);
        });
    });
}
// (desc, X, E_packed, alpha, beta, out, ws)
PyObject* wbin_conv2d(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return whole_call<7>("dab_wbin_conv2d", n, [&] {
        const dab_conv_desc d = layer(a[0]);
        const at::Tensor& X = plain(a[1], at::kFloat);
        const float* x = address<const float>(a[1]);
        const auto* E = reinterpret_cast<const uint32_t*>(address<int32_t>(a[2]));
        const float *alpha = address<const float>(a[3]), *beta = address<const float>(a[4]);
        Buffers Y(a[5], at::kFloat, {whole(d.B), extent(d.H, d.pad_h, d.kh, d.stride_h), extent(d.W, d.pad_w, d.kw, d.stride_w), whole(d.F)}, X);
        Y.workspace(::dab_wbin_conv2d_workspace_bytes(&d), a[6]);
        return std::pair(std::move(Y), [=](const Buffers& b, void* st) {
            return ::dab_wbin_conv2d(&d, x, E, alpha, beta, static_cast<float*>(b.out), b.ws, b.ws_bytes, st);
        });
    });
}
// (X, E_packed, alpha, beta, out, ws)
PyObject* wbin_fc(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return whole_call<6>("dab_wbin_fc", n, [&] {
        const at::Tensor &X = plain(a[0], at::kFloat), &al = plain(a[2], at::kFloat);
        if (X.dim() != 2 || al.dim() < 1) throw Unusual{};
        const int32_t B = whole(X.size(0)), Kin = whole(X.size(1)), F = whole(al.size(0));
        const float* x = address<const float>(a[0]);
        const auto* E = reinterpret_cast<const uint32_t*>(address<int32_t>(a[1]));
        const float *alpha = address<const float>(a[2]), *beta = address<const float>(a[3]);
        Buffers Y(a[4], at::kFloat, {B, F}, X);
        Y.workspace(::dab_wbin_fc_workspace_bytes(B, Kin, F), a[5]);
        return std::pair(std::move(Y), [=](const Buffers& b, void* st) {
            return ::dab_wbin_fc(B, Kin, F, x, E, alpha, beta, static_cast<float*>(b.out), b.ws, b.ws_bytes, st);
        });
    });
}
PyMethodDef whole_def(const char* name, PyObject* (*fn)(PyObject*, PyObject* const*, Py_ssize_t)) {
    return PyMethodDef{name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(fn)), METH_FASTCALL, nullptr};
}

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
        whole_def("pack_activations", pack_activations), whole_def("binconv2d", binconv2d), whole_def("binconv2d_bits", binconv2d_bits),
        whole_def("binfc", binfc), whole_def("pool_bits", pool_bits), whole_def("wbin_conv2d", wbin_conv2d), whole_def("wbin_fc", wbin_fc),
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
