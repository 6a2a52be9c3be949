// Argument marshalling of the tensor calls in native code (Python extension module _torch_marshal).
//
// What bounds a decoding call is the host: in Python the checks, the output allocation and the ctypes
// call took 8.0 us (forward), 10.1 us (forward + residual + statistic) and 16.4 us (backward), for
// kernels of 2 to 3 us.  Here the same calls take 4.4, 5.5 and 10.3 us, of which a launch is 3.3 us
// and an allocation 0.6 us.  These functions do the same for the calls that a program makes all the
// time -- plain tensors on the current device and stream, all arguments valid -- and return None for
// every other call, which binding.py then takes through its own code: the checks and their messages
// stand there, once.
//
//   None            not a call for this path (wrong type, shape, dtype, device, layout; no tokens; a
//                   subclass or a wrapped tensor; an active torch function or dispatch mode)
//   int             the library's non-zero status
//   tensor, tuple   the outputs, as binding.py returns them
//
// Nothing is kept between calls but the addresses of the library's entry points and the function
// that names the current stream.
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/core/impl/VirtualGuardImpl.h>
#include <torch/csrc/Exceptions.h>
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

// A tensor with memory of its own and nothing wrapped around it.
const at::Tensor* plain(PyObject* obj) {
    if (!THPVariable_CheckExact(obj)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(obj);
    static const c10::DispatchKeySet ordinary({c10::DispatchKey::CUDA, c10::DispatchKey::ADInplaceOrView,
                                               c10::DispatchKey::AutogradCUDA, c10::DispatchKey::AutocastCUDA});
    if (!t.defined() || (t.key_set() | ordinary) != ordinary || !t.is_cuda() || !t.is_contiguous()) return nullptr;
    return &t;
}

// The tensors of one call: x (or dy) sets shape, dtype and device, the others are checked against it.
struct Call {
    const at::Tensor* x = nullptr;
    int64_t N = 0, d = 0;
    int32_t dtype = 0;
    void* stream = nullptr;
    bool ok = false;

    explicit Call(PyObject* obj) {
        if (at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set()) return;
        x = plain(obj);
        if (!x || x->dim() != 2) return;
        N = x->size(0);
        d = x->size(1);
        if (N == 0 || d > WHT_MAX_D) return;
        if (x->scalar_type() == at::kFloat) dtype = WHT_DTYPE_F32;
        else if (x->scalar_type() == at::kBFloat16) dtype = WHT_DTYPE_BF16;
        else return;
        const c10::impl::VirtualGuardImpl guard(c10::DeviceType::CUDA);
        ok = guard.getDevice() == x->device();
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
        if (!t || t->dim() != 1 || t->size(0) != n || t->scalar_type() != at::kFloat || t->device() != x->device()) {
            ok = false;
            return nullptr;
        }
        return t->data_ptr();
    }
    bool find_stream() {
        PyObject* index = PyLong_FromLong(x->device().index());
        if (!index) return false;
        PyObject* handle = PyObject_CallOneArg(raw_stream_of, index);
        Py_DECREF(index);
        if (!handle) return false;
        stream = PyLong_AsVoidPtr(handle);
        Py_DECREF(handle);
        return !PyErr_Occurred();
    }
};

// An output: the caller's tensor, or a new one.
struct Out {
    PyObject* obj = nullptr;            // owned
    void* ptr = nullptr;
    ~Out() { Py_XDECREF(obj); }
    void take(PyObject* given, void* p) { Py_INCREF(given); obj = given; ptr = p; }
    bool make(c10::IntArrayRef sizes, const at::TensorOptions& options) {
        at::Tensor t = at::empty(sizes, options);
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
            scratch = at::empty({need > 16 ? need : 16}, c.x->options().dtype(at::kByte));
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

// bind(addresses of the six entry points in the order below, torch._C._cuda_getCurrentRawStream)
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    if (!expect(nargs, 7)) return nullptr;
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
    Py_RETURN_NONE;
}

#define FAST(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(f))
PyMethodDef methods[] = {{"bind", FAST(bind), METH_FASTCALL, nullptr},
                         {"forward", FAST(forward), METH_FASTCALL, nullptr},
                         {"backward", FAST(backward), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_torch_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// torch_version: the torch this was compiled for (named by build.py); binding.py uses the module with no other.
PyMODINIT_FUNC PyInit__torch_marshal(void) {
    PyObject* m = PyModule_Create(&module_def);
    if (m && PyModule_AddStringConstant(m, "torch_version", WHT_TORCH_VERSION) < 0) Py_CLEAR(m);
    return m;
}
