// The native half of binding.py: turns a Python call's tensors and numbers into a call of the C entry point, and makes
// output tensors.  Host code only; every argument conversion follows from the entry point's own prototype in lsq.h.
//
// What a small call costs is host time: a layer of 12 small calls (512 tokens x 512, 16 kernels) took 155 us through ctypes and
// torch.empty, 101 this way.  Singly: an output 0.8 instead of 1.4 us (torch.empty's argument parser), eight checks 0.2 instead of 1.5,
// a call with six pointers 0.5 instead of 2.2 (0.19 per pointer and 1.1 for ctypes), all without the launch.  Whatever is not a plain
// tensor (a subclass, an active function mode) takes the Python way.
#include <ATen/ATen.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <tuple>
#include <utility>

#include "../../include/lsq.h"

namespace {

// from binding.py (setup): the error class, ctypes.ArgumentError, the stream query and the general forms of what follows
PyObject *g_error, *g_bad_argument, *g_stream, *g_ptr, *g_need, *g_empty, *g_empty_like;

struct Raised {};                                                 // a Python error is set

bool plain(PyObject* o) { return THPVariable_CheckExact(o) && !at::impl::torch_function_mode_enabled(); }

// ---- arguments.  Numbers convert as ctypes converts them: any object with __index__, truncated to the parameter's width; no floats for ints.
unsigned long long as_int(PyObject* o)
{
    if (PyFloat_Check(o)) {
        PyErr_SetString(g_bad_argument, "int expected instead of float instance");
        throw Raised{};
    }
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);
    if (v == static_cast<unsigned long long>(-1) && PyErr_Occurred()) {
        PyErr_SetString(g_bad_argument, "int expected");
        throw Raised{};
    }
    return v;
}

void* as_pointer(PyObject* o)
{
    if (o == Py_None) return nullptr;
    if (plain(o)) {
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.is_cuda()) { PyErr_SetString(g_error, "tensors must live on the GPU (there is no CPU path)"); throw Raised{}; }
        if (!t.is_contiguous()) { PyErr_SetString(g_error, "tensors must be contiguous"); throw Raised{}; }
        return t.data_ptr();
    }
    if (PyLong_Check(o)) return reinterpret_cast<void*>(static_cast<uintptr_t>(as_int(o)));
    PyObject* a = PyObject_CallOneArg(g_ptr, o);
    if (!a) throw Raised{};
    void* p = reinterpret_cast<void*>(static_cast<uintptr_t>(PyLong_AsUnsignedLongLongMask(a)));
    Py_DECREF(a);
    return p;
}

template <typename A> struct Arg {
    static A from(PyObject* o) { return static_cast<A>(as_int(o)); }
};
template <typename A> struct Arg<A*> {
    static A* from(PyObject* o) { return static_cast<A*>(as_pointer(o)); }
};
template <> struct Arg<float> {
    static float from(PyObject* o)
    {
        const double v = PyFloat_AsDouble(o);
        if (v == -1.0 && PyErr_Occurred()) { PyErr_SetString(g_bad_argument, "float expected"); throw Raised{}; }
        return static_cast<float>(v);
    }
};
template <> struct Arg<lsq_dtype> {                               // a torch dtype, or the number itself
    static lsq_dtype from(PyObject* o)
    {
        if (!THPDtype_Check(o)) return static_cast<lsq_dtype>(as_int(o));
        switch (reinterpret_cast<THPDtype*>(o)->scalar_type) {
            case at::kHalf: return LSQ_F16;
            case at::kBFloat16: return LSQ_BF16;
            case at::kFloat: return LSQ_F32;
            default: PyErr_Format(g_error, "unsupported dtype %S", o); throw Raised{};
        }
    }
};

void* current_stream()
{
    PyObject* a = PyObject_CallNoArgs(g_stream);
    if (!a) throw Raised{};
    void* p = reinterpret_cast<void*>(static_cast<uintptr_t>(PyLong_AsUnsignedLongLongMask(a)));
    Py_DECREF(a);
    return p;
}

// the call of an entry point from all arguments but the last, which is the current stream
template <typename... A, size_t... I>
PyObject* invoke(lsq_status (*fn)(A...), const char* name, PyObject* const* args, Py_ssize_t n, std::index_sequence<I...>)
{
    if (n != static_cast<Py_ssize_t>(sizeof...(I))) {
        PyErr_Format(PyExc_TypeError, "%s takes %zd arguments (%zd given)", name, static_cast<Py_ssize_t>(sizeof...(I)), n);
        return nullptr;
    }
    using All = std::tuple<A...>;
    const std::tuple<std::tuple_element_t<I, All>...> v{Arg<std::tuple_element_t<I, All>>::from(args[I])...};     // left to right
    void* s = current_stream();
    lsq_status st;
    Py_BEGIN_ALLOW_THREADS
    st = fn(std::get<I>(v)..., s);
    Py_END_ALLOW_THREADS
    if (st != LSQ_OK) {
        PyErr_Format(g_error, "%s failed: %s", name, lsq_status_string(st));
        return nullptr;
    }
    Py_RETURN_NONE;
}
template <typename... A>
PyObject* invoke(lsq_status (*fn)(A...), const char* name, PyObject* const* args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    try {
        return invoke(fn, name, args, n, std::make_index_sequence<sizeof...(A) - 1>{});
    } catch (const Raised&) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}
#define LSQ_CALL(NAME) \
    PyObject* call_##NAME(PyObject*, PyObject* const* args, Py_ssize_t n) { return invoke(&NAME, #NAME, args, n); }
#define LSQ_CALLS(X)                                                                                                            \
    X(lsq_layernorm_fwd) X(lsq_layernorm_bwd) X(lsq_layernorm_bwd_noalloc) X(lsq_bias_dropout_residual_fwd)                     \
    X(lsq_bias_dropout_residual_bwd) X(lsq_softmax_fwd) X(lsq_softmax_bwd) X(lsq_ls_xent_fwd) X(lsq_ls_xent_bwd)                \
    X(lsq_ls_xent_fwd_bwd) X(lsq_adam_step) X(lsq_bias_act_dropout_fwd) X(lsq_bias_act_dropout_bwd) X(lsq_adam_step_lp)         \
    X(lsq_sgd_step) X(lsq_split_heads_fwd) X(lsq_split_heads_bwd) X(lsq_merge_heads_fwd) X(lsq_merge_heads_bwd)                 \
    X(lsq_embedding_fwd) X(lsq_embedding_bwd) X(lsq_bdr_layernorm_fwd) X(lsq_bdr_layernorm_bwd) X(lsq_adam_state_pack)          \
    X(lsq_adam_state_unpack) X(lsq_adam_step_blocked) X(lsq_trainer_state_pack) X(lsq_trainer_state_unpack)                     \
    X(lsq_sgd_step_blocked) X(lsq_adam_step_lp_blocked) X(lsq_pad_offsets) X(lsq_pad_remove) X(lsq_pad_restore)                 \
    X(lsq_softmax_varlen_fwd) X(lsq_softmax_varlen_bwd) X(lsq_calib_stream)
LSQ_CALLS(LSQ_CALL)

// ---- need(name, tensor, elements, dtype or None, ...): every tensor (None: none) holds at least `elements` of the dtype
PyObject* need(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    for (Py_ssize_t i = 0; i + 3 < n; i += 4) {
        PyObject *t = args[i + 1], *dt = args[i + 3];
        if (t == Py_None) continue;
        if (plain(t) && PyLong_Check(args[i + 2]) && (dt == Py_None || THPDtype_Check(dt))) {
            const at::Tensor& v = THPVariable_Unpack(t);
            int over = 0;
            const long long least = PyLong_AsLongLongAndOverflow(args[i + 2], &over);
            if (over <= 0 && v.numel() >= least && (dt == Py_None || v.scalar_type() == reinterpret_cast<THPDtype*>(dt)->scalar_type)) continue;
        }
        PyObject* r = PyObject_CallFunctionObjArgs(g_need, args[i], t, args[i + 2], dt, nullptr);     // says what is wrong
        if (!r) return nullptr;
        Py_DECREF(r);
    }
    Py_RETURN_NONE;
    END_HANDLE_TH_ERRORS
}

// ---- outputs, through torch's dispatcher (modes, deterministic fills and the caching allocator as in torch.empty)
PyObject* make(const at::Tensor& like, at::IntArrayRef sizes, at::ScalarType dt)
{
    at::Tensor o;
    {
        pybind11::gil_scoped_release no_gil;
        o = at::empty(sizes, at::TensorOptions().dtype(dt).device(like.device()));
    }
    return THPVariable_Wrap(std::move(o));
}

// strides as a new contiguous tensor has them: then empty() makes the same tensor as empty_like(), 0.8 instead of 1.1 us
bool ordinary(const at::Tensor& t)
{
    if (t.layout() != at::kStrided) return false;
    int64_t stride = 1;
    for (int64_t d = t.dim(); d-- > 0;) {
        if (t.stride(d) != stride) return false;
        stride *= t.size(d) > 1 ? t.size(d) : 1;
    }
    return true;
}

PyObject* empty_like(PyObject*, PyObject* t)
{
    HANDLE_TH_ERRORS
    if (!plain(t)) return PyObject_CallOneArg(g_empty_like, t);
    const at::Tensor& like = THPVariable_Unpack(t);
    if (ordinary(like)) return make(like, like.sizes(), like.scalar_type());
    at::Tensor o;
    {
        pybind11::gil_scoped_release no_gil;
        o = at::empty_like(like, like.options().requires_grad(false));
    }
    return THPVariable_Wrap(std::move(o));
    END_HANDLE_TH_ERRORS
}

// empty(like, dtype or None for like's, size, size, ...): a tensor on `like`'s device
PyObject* empty(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    bool easy = n >= 2 && n <= 7 && plain(args[0]) && (args[1] == Py_None || THPDtype_Check(args[1]));
    int64_t sizes[5];
    for (Py_ssize_t i = 2; easy && i < n; ++i) {
        int over = 0;
        easy = PyLong_Check(args[i]) != 0;
        if (easy) sizes[i - 2] = PyLong_AsLongLongAndOverflow(args[i], &over);
        easy = easy && over == 0 && sizes[i - 2] >= 0;
    }
    if (!easy) return PyObject_Vectorcall(g_empty, args, static_cast<size_t>(n), nullptr);
    const at::Tensor& like = THPVariable_Unpack(args[0]);
    return make(like, at::IntArrayRef(sizes, static_cast<size_t>(n - 2)),
                args[1] == Py_None ? like.scalar_type() : reinterpret_cast<THPDtype*>(args[1])->scalar_type);
    END_HANDLE_TH_ERRORS
}

// workspace_bytes(op, rows, cols)
PyObject* workspace_bytes(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 3) { PyErr_SetString(PyExc_TypeError, "op, rows, cols"); return nullptr; }
    try {
        return PyLong_FromSize_t(lsq_workspace_bytes(Arg<int32_t>::from(args[0]), Arg<int64_t>::from(args[1]), Arg<int32_t>::from(args[2])));
    } catch (const Raised&) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

PyObject* setup(PyObject*, PyObject* args)
{
    PyObject** const to[] = {&g_error, &g_bad_argument, &g_stream, &g_ptr, &g_need, &g_empty, &g_empty_like};
    if (PyTuple_GET_SIZE(args) != 7) { PyErr_SetString(PyExc_TypeError, "seven objects"); return nullptr; }
    for (int i = 0; i < 7; ++i) {
        PyObject* o = PyTuple_GET_ITEM(args, i);
        Py_INCREF(o);
        Py_XSETREF(*to[i], o);
    }
    Py_RETURN_NONE;
}

#define LSQ_METHOD(NAME) {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&call_##NAME)), METH_FASTCALL, nullptr},
PyMethodDef methods[] = {
    LSQ_CALLS(LSQ_METHOD)
    {"need", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&need)), METH_FASTCALL, nullptr},
    {"empty", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&empty)), METH_FASTCALL, nullptr},
    {"empty_like", &empty_like, METH_O, nullptr},
    {"workspace_bytes", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&workspace_bytes)), METH_FASTCALL, nullptr},
    {"setup", &setup, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// It is compiled against torch's own headers (THPDtype, the tensor's layout), which promise nothing from one version to the next:
// binding.py compares `torch_version` before it uses anything else here.
PyMODINIT_FUNC PyInit__calls()
{
    PyObject* m = PyModule_Create(&module_def);
    if (m && PyModule_AddStringConstant(m, "torch_version", LSQ_TORCH_VERSION) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
