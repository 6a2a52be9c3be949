// Argument marshalling of the tensor calls in native code (Python extension module _torch_marshal).
//
// What bounds a decoding call is the host: in Python the checks, the output allocation and the ctypes
// call took 8.0 us (forward), 10.1 us (forward + residual + statistic) and 16.4 us (backward), for
// kernels of 2 to 3 us.  Here the same calls take 4.3, 5.3 and 10.4 us, of which a launch is 2.9 us
// and an allocation 0.8 us.  These functions do the same for the calls that a program makes all the
// time -- plain tensors on the current device and stream, all arguments valid -- and return None for
// every other call, which binding.py then takes through its own code: the checks and their messages
// stand there, once.
//
//   None            not a call for this path (wrong type, shape, dtype, device, layout; no tokens; a
//                   subclass or a wrapped tensor; an active torch function or dispatch mode)
//   int             the library's non-zero status
//   tensor, tuple   the outputs, as binding.py returns them
//
// layer() is the differentiable call (autograd.py) as a node of torch's C++ autograd: as a Python Function the
// forward and backward of a training step of few tokens took 90 us of host time, here 67 (a product by a constant
// and its backward: 43), a call without gradients 10.6 and 7.4.  What it saves, views and returns is what the Python Function does; it declines where a
// transform, a trace, forward-mode differentiation or a mode is active, and the Python Function, which knows how
// to answer there, takes the call.
//
// Nothing is kept between calls but the addresses of the library's entry points, the function
// that names the current stream and the one that takes the backward calls declined here.
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty_cuda_dispatch.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/core/impl/VirtualGuardImpl.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/forward_grad.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/wht_affine.h"

namespace {

decltype(&wht_affine_forward) lib_forward;
decltype(&wht_affine_forward_residual) lib_forward_residual;
decltype(&wht_affine_forward_residual_stats) lib_forward_residual_stats;
decltype(&wht_affine_backward_workspace_bytes) lib_workspace_bytes;
decltype(&wht_affine_backward) lib_backward;
decltype(&wht_affine_backward_static) lib_backward_static;
PyObject* raw_stream_of;                // torch._C._cuda_getCurrentRawStream
PyObject* general_backward;             // binding.wht_affine_backward

// A tensor with memory of its own and nothing wrapped around it.
bool is_plain(const at::Tensor& t) {
    static const c10::DispatchKeySet ordinary({c10::DispatchKey::CUDA, c10::DispatchKey::ADInplaceOrView,
                                               c10::DispatchKey::AutogradCUDA, c10::DispatchKey::AutocastCUDA});
    return t.defined() && (t.key_set() | ordinary) == ordinary && t.is_cuda() && t.is_contiguous();
}
const at::Tensor* plain(PyObject* obj) {
    if (!THPVariable_CheckExact(obj)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(obj);
    return is_plain(t) ? &t : nullptr;
}
// As torch::empty makes it on the GPU, without the dispatcher in front (no mode is active here), which was 0.1 us of an
// allocation's 0.9.
at::Tensor new_empty(c10::IntArrayRef sizes, const at::TensorOptions& options) { return at::cuda::empty(sizes, options); }

bool modes_active() {
    return at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set();
}
bool on_current_device(const at::Tensor& t) {
    const c10::impl::VirtualGuardImpl guard(c10::DeviceType::CUDA);
    return guard.getDevice() == t.device();
}
// The library's code for a tensor's dtype, or -1.
int32_t dtype_code(const at::Tensor& t) {
    return t.scalar_type() == at::kFloat ? WHT_DTYPE_F32 : t.scalar_type() == at::kBFloat16 ? WHT_DTYPE_BF16 : -1;
}
bool is_vec(const at::Tensor& t, int64_t n, const at::Tensor& x) {
    return is_plain(t) && t.dim() == 1 && t.size(0) == n && t.scalar_type() == at::kFloat && t.device() == x.device();
}
// The current stream of a device (with the GIL).
bool current_stream(c10::Device device, void** stream) {
    PyObject* index = PyLong_FromLong(device.index());
    if (!index) return false;
    PyObject* handle = PyObject_CallOneArg(raw_stream_of, index);
    Py_DECREF(index);
    if (!handle) return false;
    *stream = PyLong_AsVoidPtr(handle);
    Py_DECREF(handle);
    return !PyErr_Occurred();
}

// The tensors of one call: x (or dy) sets shape, dtype and device, the others are checked against it.
struct Call {
    const at::Tensor* x = nullptr;
    int64_t N = 0, d = 0;
    int32_t dtype = 0;
    void* stream = nullptr;
    bool ok = false;

    explicit Call(PyObject* obj) {
        if (modes_active()) return;
        x = plain(obj);
        if (!x || x->dim() != 2) return;
        N = x->size(0);
        d = x->size(1);
        if (N == 0 || d > WHT_MAX_D) return;
        dtype = dtype_code(*x);
        ok = dtype >= 0 && on_current_device(*x);
    }
    bool is_none(PyObject* obj) const { return obj == Py_None; }
    // [N,d] like x
    void* io(PyObject* obj) {
        const at::Tensor* t = plain(obj);
        if (!t || t->dim() != 2 || t->size(0) != N || t->size(1) != d || t->scalar_type() != x->scalar_type() ||
            t->device() != x->device()) { ok = false; return nullptr; }
        return t->data_ptr();
    }
    // float32 [n]
    void* vec(PyObject* obj, int64_t n) {
        const at::Tensor* t = plain(obj);
        if (!t || !is_vec(*t, n, *x)) { ok = false; return nullptr; }
        return t->data_ptr();
    }
    bool find_stream() { return current_stream(x->device(), &stream); }
};

// An output: the caller's tensor, or a new one.
struct Out {
    PyObject* obj = nullptr;            // owned
    void* ptr = nullptr;
    ~Out() { Py_XDECREF(obj); }
    void take(PyObject* given, void* p) { Py_INCREF(given); obj = given; ptr = p; }
    bool make(c10::IntArrayRef sizes, const at::TensorOptions& options) {
        at::Tensor t = new_empty(sizes, options);
        ptr = t.data_ptr();
        obj = THPVariable_Wrap(std::move(t));
        return obj != nullptr;
    }
    PyObject* release() { PyObject* o = obj ? obj : Py_NewRef(Py_None); obj = nullptr; return o; }
};

PyObject* none() { Py_RETURN_NONE; }
PyObject* pack(Out& a, Out& b) {
    PyObject* t = PyTuple_New(2);
    if (!t) return nullptr;
    PyTuple_SET_ITEM(t, 0, a.release());
    PyTuple_SET_ITEM(t, 1, b.release());
    return t;
}
PyObject* pack(Out& a, Out& b, Out& c) {
    PyObject* t = PyTuple_New(3);
    if (!t) return nullptr;
    PyTuple_SET_ITEM(t, 0, a.release());
    PyTuple_SET_ITEM(t, 1, b.release());
    PyTuple_SET_ITEM(t, 2, c.release());
    return t;
}
bool expect(Py_ssize_t got, Py_ssize_t want) {
    if (got == want) return true;
    PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, got);
    return false;
}

// forward(x, alpha, beta, resid | None, y | None, sumsq | None, with_resid, with_stats)
PyObject* forward(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    if (!expect(nargs, 8)) return nullptr;
    const bool with_resid = args[6] == Py_True, with_stats = args[7] == Py_True;
    Call c(args[0]);
    if (!c.ok) return none();
    const void* x = c.x->data_ptr();
    const float* alpha = static_cast<float*>(c.vec(args[1], c.d));
    const float* beta = static_cast<float*>(c.vec(args[2], c.d));
    const void* resid = with_resid ? c.io(args[3]) : nullptr;
    void* given_y = c.is_none(args[4]) ? nullptr : c.io(args[4]);
    void* given_s = !with_stats || c.is_none(args[5]) ? nullptr : c.vec(args[5], c.N);
    if (!c.ok) return none();
    Out y, s;
    if (given_y) y.take(args[4], given_y);
    else if (!y.make(c.x->sizes(), c.x->options())) return nullptr;
    if (given_s) s.take(args[5], given_s);
    else if (with_stats && !s.make({c.N}, c.x->options().dtype(at::kFloat))) return nullptr;
    if (!c.find_stream()) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    if (with_stats)
        rc = lib_forward_residual_stats(x, alpha, beta, resid, y.ptr, static_cast<float*>(s.ptr), c.N, (int32_t)c.d,
                                        c.dtype, c.stream);
    else if (with_resid)
        rc = lib_forward_residual(x, alpha, beta, resid, y.ptr, c.N, (int32_t)c.d, c.dtype, c.stream);
    else
        rc = lib_forward(x, alpha, beta, y.ptr, c.N, (int32_t)c.d, c.dtype, c.stream);
    Py_END_ALLOW_THREADS
    if (rc != WHT_OK) return PyLong_FromLong(rc);
    return with_stats ? pack(y, s) : y.release();
    END_HANDLE_TH_ERRORS
}

// backward(dy, x | None, alpha, dx | None, dalpha | None, dbeta | None, workspace | None, want_dx,
//          want_param_grads, own_scratch)
PyObject* backward(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    if (!expect(nargs, 10)) return nullptr;
    const bool want_dx = args[7] == Py_True, want_pg = args[8] == Py_True, own_scratch = args[9] == Py_True;
    if (!want_dx && !want_pg) return none();
    Call c(args[0]);
    if (!c.ok || (want_pg && c.is_none(args[1]))) return none();
    const void* dy = c.x->data_ptr();
    const void* x = c.is_none(args[1]) ? nullptr : c.io(args[1]);
    const float* alpha = static_cast<float*>(c.vec(args[2], c.d));
    void* given[3] = {nullptr, nullptr, nullptr};
    if (want_dx && !c.is_none(args[3])) given[0] = c.io(args[3]);
    for (int i = 1; i < 3; ++i)
        if (want_pg && !c.is_none(args[3 + i])) given[i] = c.vec(args[3 + i], c.d);
    if (!c.ok) return none();
    Out dx, dalpha, dbeta;
    const auto f32 = c.x->options().dtype(at::kFloat);
    if (given[0]) dx.take(args[3], given[0]);
    else if (want_dx && !dx.make(c.x->sizes(), c.x->options())) return nullptr;
    if (given[1]) dalpha.take(args[4], given[1]);
    else if (want_pg && !dalpha.make({c.d}, f32)) return nullptr;
    if (given[2]) dbeta.take(args[5], given[2]);
    else if (want_pg && !dbeta.make({c.d}, f32)) return nullptr;
    at::Tensor scratch;
    size_t ws_bytes = 0;
    void* ws = nullptr;
    if (want_pg && !own_scratch) {
        if (c.is_none(args[6])) {
            const int64_t need = (int64_t)lib_workspace_bytes(c.N, (int32_t)c.d, c.dtype);
            scratch = new_empty({need > 16 ? need : 16}, c.x->options().dtype(at::kByte));
            ws = scratch.data_ptr();
            ws_bytes = scratch.nbytes();
        } else {
            const at::Tensor* t = plain(args[6]);
            if (!t || t->device() != c.x->device()) return none();
            ws = t->data_ptr();
            ws_bytes = t->nbytes();
        }
    }
    if (!c.find_stream()) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    if (own_scratch)
        rc = lib_backward_static(dy, x, alpha, dx.ptr, static_cast<float*>(dalpha.ptr), static_cast<float*>(dbeta.ptr), c.N,
                                 (int32_t)c.d, c.dtype, c.stream);
    else
        rc = lib_backward(dy, want_pg ? x : nullptr, alpha, dx.ptr, static_cast<float*>(dalpha.ptr),
                          static_cast<float*>(dbeta.ptr), c.N, (int32_t)c.d, c.dtype, ws, ws_bytes, c.stream);
    Py_END_ALLOW_THREADS
    if (rc != WHT_OK) return PyLong_FromLong(rc);
    return pack(dx, dalpha, dbeta);
    END_HANDLE_TH_ERRORS
}

// The Python error that is set, as an exception (with the GIL).
[[noreturn]] void raise() {
    python_error error;
    error.persist();
    throw error;
}

struct Declined {};                     // the library refused the call: binding.py's code says why

}  // namespace

// (named: the graph's nodes and torch's error messages show the type)
struct WhtAffineFunction : torch::autograd::Function<WhtAffineFunction> {
    static at::Tensor forward(torch::autograd::AutogradContext* ctx, const at::Tensor& x, const at::Tensor& alpha,
                              const at::Tensor& beta, const std::optional<at::Tensor>& resid) {
        const int64_t d = x.size(-1), N = x.numel() / d;
        const at::Tensor x2 = x.reshape({N, d}), y = new_empty({N, d}, x.options());
        void* stream = nullptr;
        if (!current_stream(x.device(), &stream)) raise();
        const auto a = static_cast<const float*>(alpha.data_ptr()), b = static_cast<const float*>(beta.data_ptr());
        int rc;
        Py_BEGIN_ALLOW_THREADS
        if (resid)
            rc = lib_forward_residual(x.data_ptr(), a, b, resid->data_ptr(), y.data_ptr(), N, (int32_t)d, dtype_code(x), stream);
        else
            rc = lib_forward(x.data_ptr(), a, b, y.data_ptr(), N, (int32_t)d, dtype_code(x), stream);
        Py_END_ALLOW_THREADS
        if (rc != WHT_OK) throw Declined{};
        ctx->save_for_backward({x2, alpha});
        ctx->saved_data["resid"] = resid.has_value();
        return y.view(x.sizes());
    }

    static torch::autograd::variable_list backward(torch::autograd::AutogradContext* ctx, const torch::autograd::variable_list& grads) {
        const auto saved = ctx->get_saved_variables();
        const at::Tensor &x2 = saved[0], &alpha = saved[1], &dy = grads[0];
        const bool want_dx = ctx->needs_input_grad(0), want_pg = ctx->needs_input_grad(1) || ctx->needs_input_grad(2);
        torch::autograd::variable_list out(4);
        if (want_dx || want_pg) {
            at::Tensor dy2 = dy.reshape({-1, x2.size(1)});
            if (!dy2.is_contiguous()) dy2 = dy2.contiguous();
            if (!native(dy2, x2, alpha, want_dx, want_pg, out)) general(dy2, x2, alpha, want_dx, want_pg, out);
            if (out[0].defined()) out[0] = out[0].view(dy.sizes());
        }
        if (ctx->saved_data["resid"].toBool() && ctx->needs_input_grad(3)) out[3] = dy;     // the residual stream's gradient is dy itself
        return out;
    }

    static bool native(const at::Tensor& dy, const at::Tensor& x, const at::Tensor& alpha, bool want_dx, bool want_pg,
                       torch::autograd::variable_list& out) {
        if (modes_active() || !is_plain(dy) || !is_plain(x) || dy.sizes() != x.sizes() || dy.scalar_type() != x.scalar_type() ||
            dy.device() != x.device() || dtype_code(dy) < 0 || !is_vec(alpha, x.size(1), x) || !on_current_device(dy))
            return false;
        const int64_t N = dy.size(0), d = dy.size(1);
        const auto f32 = dy.options().dtype(at::kFloat);
        at::Tensor dx, dalpha, dbeta, scratch;
        if (want_dx) dx = new_empty({N, d}, dy.options());
        if (want_pg) {
            dalpha = new_empty({d}, f32);
            dbeta = new_empty({d}, f32);
            const int64_t need = (int64_t)lib_workspace_bytes(N, (int32_t)d, dtype_code(dy));
            scratch = new_empty({need > 16 ? need : 16}, dy.options().dtype(at::kByte));
        }
        void* stream = nullptr;
        {
            const PyGILState_STATE gil = PyGILState_Ensure();
            const bool found = current_stream(dy.device(), &stream);
            if (!found) PyErr_Clear();
            PyGILState_Release(gil);
            if (!found) return false;
        }
        auto at = [](const at::Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; };
        const int rc = lib_backward(dy.data_ptr(), want_pg ? x.data_ptr() : nullptr, static_cast<const float*>(alpha.data_ptr()), at(dx),
                                    static_cast<float*>(at(dalpha)), static_cast<float*>(at(dbeta)), N, (int32_t)d,
                                    dtype_code(dy), at(scratch), want_pg ? scratch.nbytes() : 0, stream);
        if (rc != WHT_OK) return false;
        out[0] = dx;
        out[1] = dalpha;
        out[2] = dbeta;
        return true;
    }

    // general_backward(dy, x, alpha, dx, dalpha, dbeta, workspace, stream, want_dx, want_param_grads)
    static void general(const at::Tensor& dy, const at::Tensor& x, const at::Tensor& alpha, bool want_dx, bool want_pg,
                        torch::autograd::variable_list& out) {
        const PyGILState_STATE gil = PyGILState_Ensure();
        PyObject *args[10] = {}, *result = nullptr;
        for (int i = 3; i < 8; ++i) args[i] = Py_NewRef(Py_None);
        args[0] = THPVariable_Wrap(dy);
        args[1] = THPVariable_Wrap(x);
        args[2] = THPVariable_Wrap(alpha);
        args[8] = PyBool_FromLong(want_dx);
        args[9] = PyBool_FromLong(want_pg);
        if (args[0] && args[1] && args[2]) result = PyObject_Vectorcall(general_backward, args, 10, nullptr);
        for (PyObject* a : args) Py_XDECREF(a);
        bool ok = result && PyTuple_Check(result) && PyTuple_GET_SIZE(result) == 3;
        for (int i = 0; ok && i < 3; ++i) {
            PyObject* t = PyTuple_GET_ITEM(result, i);
            if (THPVariable_Check(t)) out[i] = THPVariable_Unpack(t);
        }
        if (result && !ok) PyErr_SetString(PyExc_TypeError, "wht_affine_backward returns three tensors");
        Py_XDECREF(result);
        python_error error;
        if (!ok) error.persist();
        PyGILState_Release(gil);
        if (!ok) throw error;
    }
};

namespace {

// layer(x, alpha, beta, resid | None)
PyObject* layer(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    if (!expect(nargs, 4)) return nullptr;
    // transforms, traces and modes are keys that the thread includes beyond the ordinary ones
    if (modes_active() || c10::impl::tls_local_dispatch_key_set().included_ != c10::default_included_set ||
        torch::autograd::ForwardADLevel::try_get_by_idx(0)) return none();
    const at::Tensor *x = plain(args[0]), *alpha = plain(args[1]), *beta = plain(args[2]);
    const at::Tensor* resid = args[3] == Py_None ? nullptr : plain(args[3]);
    if (!x || !alpha || !beta || (args[3] != Py_None && !resid) || x->dim() < 1 || x->numel() == 0) return none();
    const int64_t d = x->size(-1);
    if (d > WHT_MAX_D || dtype_code(*x) < 0 || !is_vec(*alpha, d, *x) || !is_vec(*beta, d, *x) || !on_current_device(*x) ||
        (resid && (resid->sizes() != x->sizes() || resid->scalar_type() != x->scalar_type() || resid->device() != x->device())))
        return none();
    try {
        return THPVariable_Wrap(WhtAffineFunction::apply(*x, *alpha, *beta, resid ? std::optional<at::Tensor>(*resid) : std::nullopt));
    } catch (const Declined&) {
        return none();
    }
    END_HANDLE_TH_ERRORS
}

// bind(addresses of the six entry points in the order below, torch._C._cuda_getCurrentRawStream, binding.wht_affine_backward)
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    if (!expect(nargs, 8)) return nullptr;
    void* p[6];
    for (int i = 0; i < 6; ++i) {
        p[i] = PyLong_AsVoidPtr(args[i]);
        if (PyErr_Occurred()) return nullptr;
    }
    lib_forward = reinterpret_cast<decltype(lib_forward)>(p[0]);
    lib_forward_residual = reinterpret_cast<decltype(lib_forward_residual)>(p[1]);
    lib_forward_residual_stats = reinterpret_cast<decltype(lib_forward_residual_stats)>(p[2]);
    lib_workspace_bytes = reinterpret_cast<decltype(lib_workspace_bytes)>(p[3]);
    lib_backward = reinterpret_cast<decltype(lib_backward)>(p[4]);
    lib_backward_static = reinterpret_cast<decltype(lib_backward_static)>(p[5]);
    Py_INCREF(args[6]);
    Py_XSETREF(raw_stream_of, args[6]);
    Py_INCREF(args[7]);
    Py_XSETREF(general_backward, args[7]);
    Py_RETURN_NONE;
}

#define FAST(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(f))
PyMethodDef methods[] = {{"bind", FAST(bind), METH_FASTCALL, nullptr},
                         {"forward", FAST(forward), METH_FASTCALL, nullptr},
                         {"backward", FAST(backward), METH_FASTCALL, nullptr},
                         {"layer", FAST(layer), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_torch_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// torch_version: the torch this was compiled for (named by build.py); binding.py uses the module with no other.
PyMODINIT_FUNC PyInit__torch_marshal(void) {
    PyObject* m = PyModule_Create(&module_def);
    if (m && PyModule_AddStringConstant(m, "torch_version", WHT_TORCH_VERSION) < 0) Py_CLEAR(m);
    return m;
}
