// The binding's plain calls without an interpreter between the checks, the outputs and the library: a Python extension
// with one function per entry point that a training loop calls over and over.
//
// A call is plain when its tensors are exactly torch.Tensor, its numbers exactly int, float and bool, its workspace given
// and nothing traces or transforms it; every function here returns None for any other call, also for one whose checks
// fail, and binding.py then goes the general way, which says what is wrong.  The smallest calls are bound by the host: a
// prompt step of 16 prompts is three calls with five outputs, of 1.3 us each out of the interpreter, and three launches of 4
// (25 us in all through ctypes, 16 here).
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/TensorBody.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "spo.h"

namespace {

PyObject *g_error = nullptr;  // binding.SpoError

PyObject *refused(int status, const char *where) {
    if (PyObject *e = PyObject_CallFunction(g_error, "is", status, where)) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    }
    return nullptr;
}

// Under a transform (grad, jvp, functionalize, vmap of torch.func), functionalization or a trace, outputs made here are not
// plain tensors, whatever the inputs are.
bool plain_context() {
    using c10::DispatchKey;
    constexpr c10::DispatchKeySet transforms({DispatchKey::FuncTorchDynamicLayerFrontMode, DispatchKey::FuncTorchDynamicLayerBackMode,
                                              DispatchKey::FuncTorchVmapMode, DispatchKey::VmapMode, DispatchKey::Functionalize,
                                              DispatchKey::Tracer, DispatchKey::PreDispatch, DispatchKey::PythonDispatcher,
                                              DispatchKey::Python, DispatchKey::PythonTLSSnapshot});
    return !at::impl::torch_function_mode_enabled() && !c10::impl::TorchDispatchModeTLS::any_modes_set() &&
           !c10::impl::tls_local_dispatch_key_set().included_.has_any(transforms);
}

// NULL: not a plain tensor
const at::Tensor *tensor(PyObject *o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    const auto *impl = t.unsafeGetTensorImpl();
    using c10::DispatchKey;
    const auto keys = impl->key_set();
    if (!t.is_cuda() || !impl->has_storage() || impl->is_python_dispatch() || keys.has(DispatchKey::FuncTorchBatched) ||
        keys.has(DispatchKey::FuncTorchGradWrapper) || keys.has(DispatchKey::Functionalize) || keys.has(DispatchKey::Batched))
        return nullptr;
    return &t;
}
// ... of this type, dense, and with n elements (n < 0: any number)
const at::Tensor *dense(PyObject *o, at::ScalarType type, int64_t n) {
    const at::Tensor *t = tensor(o);
    return t && t->scalar_type() == type && t->is_contiguous() && (n < 0 || t->numel() == n) ? t : nullptr;
}
const at::Tensor *workspace(PyObject *o, size_t bytes) {
    const at::Tensor *t = tensor(o);
    return t && t->scalar_type() == at::kByte && static_cast<size_t>(t->numel()) >= bytes &&
                   reinterpret_cast<uintptr_t>(t->data_ptr()) % 256 == 0 ? t : nullptr;
}
bool number(PyObject *o, double &v) {
    if (PyFloat_CheckExact(o)) v = PyFloat_AS_DOUBLE(o);
    else if (PyLong_CheckExact(o)) v = PyLong_AsDouble(o);
    else return false;
    if (!PyErr_Occurred()) return true;
    PyErr_Clear();  // an int past the largest double: the general way says so
    return false;
}
bool whole(PyObject *o, int64_t lo, int64_t hi, int64_t &v) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return !overflow && v >= lo && v <= hi;
}
bool flag(PyObject *o, int &v) {
    v = o == Py_True;
    return PyBool_Check(o);
}
at::Tensor fresh(at::IntArrayRef shape, at::ScalarType type, const at::Tensor &like) {
    return at::empty(shape, at::TensorOptions().dtype(type).device(like.device()));
}
spo_stream_t stream() { return reinterpret_cast<spo_stream_t>(c10::hip::getCurrentHIPStream().stream()); }
template <typename T> T *ptr(const at::Tensor *t) { return t ? static_cast<T *>(t->data_ptr()) : nullptr; }
template <typename T> T *ptr(const at::Tensor &t) { return static_cast<T *>(t.data_ptr()); }

// Other threads run meanwhile, as through ctypes.  The lock is taken again on every way out: an exception (a tensor that has
// no memory) is turned into Python's by the caller, which needs it.
template <typename F> int unlocked(F call) {
    struct Unlocked {
        PyThreadState *state = PyEval_SaveThread();
        ~Unlocked() { PyEval_RestoreThread(state); }
    } lock;
    return call();
}
template <typename... T> PyObject *tuple_of(T &&...t) { return PyTuple_Pack(sizeof...(t), t...); }
// a tuple of new references
template <typename... T> PyObject *pack(T... o) {
    PyObject *r = (o && ...) ? tuple_of(o...) : nullptr;
    (Py_XDECREF(o), ...);
    return r;
}
PyObject *wrap(const at::Tensor &t) { return THPVariable_Wrap(t); }
PyObject *none() { Py_RETURN_NONE; }

// (alpha, beta, B, eps_explore, seed, iteration, replace, max_attempts, workspace) -> (idx, info)
PyObject *sample_prompts(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 9 || !plain_context()) return none();
    const at::Tensor *alpha = dense(a[0], at::kFloat, -1), *beta = alpha ? dense(a[1], at::kFloat, alpha->numel()) : nullptr;
    int64_t B, most;
    double eps;
    int replace;
    if (!beta || !whole(a[2], 1, INT32_MAX, B) || !number(a[3], eps) || !PyLong_CheckExact(a[4]) || !PyLong_CheckExact(a[5]) ||
        !flag(a[6], replace) || !whole(a[7], 0, UINT32_MAX, most))
        return none();
    const int64_t N = alpha->numel();
    const at::Tensor *ws = workspace(a[8], spo_sample_prompts_workspace_bytes(N, static_cast<int32_t>(B)));
    if (!ws) return none();
    const uint64_t seed = PyLong_AsUnsignedLongLongMask(a[4]), iteration = PyLong_AsUnsignedLongLongMask(a[5]);
    const at::Tensor idx = fresh({B}, at::kInt, *alpha), info = fresh({2}, at::kInt, *alpha);
    const spo_stream_t s = stream();
    const int rc = unlocked([&] {
        return spo_sample_prompts(ptr<float>(alpha), ptr<float>(beta), N, static_cast<int32_t>(B), eps, seed, iteration, replace,
                                  static_cast<uint32_t>(most), ptr<int32_t>(idx), ptr<int32_t>(info), ws->data_ptr(), ws->numel(), s);
    });
    return rc ? refused(rc, "spo_sample_prompts") : pack(wrap(idx), wrap(info));
    END_HANDLE_TH_ERRORS
}

// (alpha, beta, idx, reward, ddof, eps_norm, workspace or None) -> (raw, normalised, stats); with the baseline, no info
PyObject *advantages(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 7 || !plain_context()) return none();
    const at::Tensor *reward = dense(a[3], at::kFloat, -1), *alpha = dense(a[0], at::kFloat, -1);
    if (!reward || !alpha) return none();
    const int64_t B = reward->numel(), N = alpha->numel();
    const at::Tensor *beta = dense(a[1], at::kFloat, N), *idx = dense(a[2], at::kInt, B);
    const at::Tensor *ws = a[6] == Py_None ? nullptr : tensor(a[6]);
    int64_t ddof;
    double eps;
    if (!beta || !idx || B < 1 || B > INT32_MAX || (!ws && a[6] != Py_None) || !whole(a[4], INT32_MIN, INT32_MAX, ddof) || !number(a[5], eps))
        return none();
    const at::Tensor raw = fresh({B}, at::kFloat, *reward), nrm = fresh({B}, at::kFloat, *reward), st = fresh({2}, at::kFloat, *reward);
    const spo_stream_t s = stream();
    const int rc = unlocked([&] {
        return spo_advantages(ptr<float>(alpha), ptr<float>(beta), N, ptr<int32_t>(idx), ptr<float>(reward), static_cast<int32_t>(B),
                              static_cast<int>(ddof), static_cast<float>(eps), 1, ptr<float>(raw), ptr<float>(nrm), ptr<float>(st), nullptr,
                              ptr<void>(ws), ws ? ws->numel() : 0, s);
    });
    return rc ? refused(rc, "spo_advantages") : pack(wrap(raw), wrap(nrm), wrap(st));
    END_HANDLE_TH_ERRORS
}

// (raw, reward, tau_tight, tau_loose) -> diag
PyObject *advantage_diagnostics(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 4 || !plain_context()) return none();
    const at::Tensor *raw = dense(a[0], at::kFloat, -1), *reward = raw ? dense(a[1], at::kFloat, raw->numel()) : nullptr;
    double tight, loose;
    if (!reward || raw->numel() < 1 || raw->numel() > INT32_MAX || !number(a[2], tight) || !number(a[3], loose)) return none();
    const at::Tensor diag = fresh({4}, at::kFloat, *raw);
    const spo_stream_t s = stream();
    const int rc = unlocked([&] {
        return spo_advantage_diagnostics(ptr<float>(raw), ptr<float>(reward), static_cast<int32_t>(raw->numel()), static_cast<float>(tight),
                                         static_cast<float>(loose), ptr<float>(diag), s);
    });
    return rc ? refused(rc, "spo_advantage_diagnostics") : wrap(diag);
    END_HANDLE_TH_ERRORS
}

// (alpha, beta, idx, reward, kl, d_half, rho_min, rho_max, ids_unique, workspace or None) -> True; no counters, baselines or info
PyObject *tracker_update(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 10 || !plain_context()) return none();
    const at::Tensor *alpha = dense(a[0], at::kFloat, -1), *idx = dense(a[2], at::kInt, -1);
    if (!alpha || !idx) return none();
    const int64_t N = alpha->numel(), B = idx->numel();
    const at::Tensor *beta = dense(a[1], at::kFloat, N), *reward = dense(a[3], at::kFloat, B), *kl = dense(a[4], at::kFloat, B);
    const at::Tensor *ws = a[9] == Py_None ? nullptr : tensor(a[9]);
    double d_half, lo, hi;
    int unique;
    if (!beta || !reward || !kl || B < 1 || B > INT32_MAX || !number(a[5], d_half) || !number(a[6], lo) || !number(a[7], hi) ||
        !flag(a[8], unique) || (!ws && (a[9] != Py_None || !unique)))
        return none();
    const spo_stream_t s = stream();
    const int rc = unlocked([&] {
        return spo_tracker_update(ptr<float>(alpha), ptr<float>(beta), N, ptr<int32_t>(idx), ptr<float>(reward), ptr<float>(kl),
                                  static_cast<int32_t>(B), static_cast<float>(d_half), static_cast<float>(lo), static_cast<float>(hi), unique,
                                  nullptr, nullptr, nullptr, ptr<void>(ws), ws ? ws->numel() : 0, s);
    });
    if (rc) return refused(rc, "spo_tracker_update");
    Py_RETURN_TRUE;
    END_HANDLE_TH_ERRORS
}

// The descriptor of a call: its address, and its target tensor (the device).  False: not plain.
bool descriptor(PyObject *address, PyObject *target, const spo_pg_desc *&d, const at::Tensor *&like) {
    if (!PyLong_CheckExact(address)) return false;
    d = static_cast<const spo_pg_desc *>(PyLong_AsVoidPtr(address));
    like = tensor(target);
    return d && like && d->T > 0;
}
at::ScalarType type_of(int dtype) { return dtype == SPO_FP32 ? at::kFloat : at::kBFloat16; }
// the caller's d_W: the first V * H of its elements are written, in order
const at::Tensor *head_gradient(PyObject *o, const spo_pg_desc *d) {
    const at::Tensor *t = tensor(o);
    return t && (t->scalar_type() == at::kFloat || t->scalar_type() == at::kBFloat16) && t->is_contiguous() && t->numel() >= d->V * d->H ? t : nullptr;
}
int code_of(const at::Tensor &t) { return t.scalar_type() == at::kFloat ? SPO_FP32 : SPO_BF16; }

// (descriptor, target, workspace) -> (loss, logp, lse, stats)
PyObject *pg_loss_fwd(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    const spo_pg_desc *d;
    const at::Tensor *like;
    if (n != 3 || !plain_context() || !descriptor(a[0], a[1], d, like)) return none();
    const at::Tensor *ws = workspace(a[2], spo_pg_loss_fwd_workspace_bytes(d));
    if (!ws) return none();
    const at::Tensor loss = fresh({1}, at::kFloat, *like), logp = fresh({d->T}, at::kFloat, *like), lse = fresh({d->T}, at::kFloat, *like),
                     st = fresh({4}, at::kFloat, *like);
    const spo_stream_t s = stream();
    const int rc = unlocked([&] {
        return spo_pg_loss_fwd(d, ptr<float>(loss), ptr<float>(logp), ptr<float>(lse), ptr<float>(st), ws->data_ptr(), ws->numel(), s);
    });
    return rc ? refused(rc, "spo_pg_loss_fwd") : pack(wrap(loss), wrap(logp), wrap(lse), wrap(st));
    END_HANDLE_TH_ERRORS
}

// (descriptor, target, logp, lse, grad_loss, d_W (None for the logits-in form), accumulate_dW, chunk_tokens, workspace)
// -> d_logits, or (d_hidden in the type of the hidden states, d_W)
PyObject *pg_loss_bwd(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    const spo_pg_desc *d;
    const at::Tensor *like;
    if (n != 9 || !plain_context() || !descriptor(a[0], a[1], d, like)) return none();
    const at::Tensor *logp = dense(a[2], at::kFloat, d->T), *lse = dense(a[3], at::kFloat, d->T);
    double grad;
    int accumulate;
    int64_t chunk;
    if (!logp || !lse || !number(a[4], grad) || !flag(a[6], accumulate) || !whole(a[7], INT64_MIN, INT64_MAX, chunk)) return none();
    const at::Tensor *ws = workspace(a[8], spo_pg_loss_bwd_workspace_bytes(d, chunk));
    if (!ws) return none();
    if (d->logits) {
        const at::Tensor dl = fresh({d->T, d->V}, type_of(d->dtype), *like);
        const spo_stream_t s = stream();
        const int rc = unlocked([&] {
            return spo_pg_loss_bwd(d, ptr<float>(logp), ptr<float>(lse), static_cast<float>(grad), nullptr, 0, nullptr, 0, 0, dl.data_ptr(),
                                   chunk, ws->data_ptr(), ws->numel(), s);
        });
        return rc ? refused(rc, "spo_pg_loss_bwd") : wrap(dl);
    }
    const at::Tensor *dw = head_gradient(a[5], d);
    if (!dw) return none();
    const at::Tensor dx = fresh({d->T, d->H}, type_of(d->dtype), *like);
    const spo_stream_t s = stream();
    const int rc = unlocked([&] {
        return spo_pg_loss_bwd(d, ptr<float>(logp), ptr<float>(lse), static_cast<float>(grad), dx.data_ptr(), d->dtype, dw->data_ptr(),
                               code_of(*dw), accumulate, nullptr, chunk, ws->data_ptr(), ws->numel(), s);
    });
    if (rc) return refused(rc, "spo_pg_loss_bwd");
    Py_INCREF(a[5]);
    return pack(wrap(dx), a[5]);
    END_HANDLE_TH_ERRORS
}

// (descriptor, target, grad_loss, d_W, accumulate_dW, chunk_tokens, workspace) -> (loss, logp, lse, stats, d_hidden, d_W)
PyObject *pg_loss_fwd_bwd(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    const spo_pg_desc *d;
    const at::Tensor *like;
    if (n != 7 || !plain_context() || !descriptor(a[0], a[1], d, like) || d->logits) return none();
    const at::Tensor *dw = head_gradient(a[3], d);
    double grad;
    int accumulate;
    int64_t chunk;
    if (!dw || !number(a[2], grad) || !flag(a[4], accumulate) || !whole(a[5], INT64_MIN, INT64_MAX, chunk)) return none();
    const at::Tensor *ws = workspace(a[6], spo_pg_loss_fwd_bwd_workspace_bytes(d, chunk));
    if (!ws) return none();
    const at::Tensor loss = fresh({1}, at::kFloat, *like), logp = fresh({d->T}, at::kFloat, *like), lse = fresh({d->T}, at::kFloat, *like),
                     st = fresh({4}, at::kFloat, *like), dx = fresh({d->T, d->H}, type_of(d->dtype), *like);
    const spo_stream_t s = stream();
    const int rc = unlocked([&] {
        return spo_pg_loss_fwd_bwd(d, static_cast<float>(grad), ptr<float>(loss), ptr<float>(logp), ptr<float>(lse), ptr<float>(st),
                                   dx.data_ptr(), d->dtype, dw->data_ptr(), code_of(*dw), accumulate, chunk, ws->data_ptr(), ws->numel(), s);
    });
    if (rc) return refused(rc, "spo_pg_loss_fwd_bwd");
    Py_INCREF(a[3]);
    return pack(wrap(loss), wrap(logp), wrap(lse), wrap(st), wrap(dx), a[3]);
    END_HANDLE_TH_ERRORS
}

PyObject *set_error(PyObject *, PyObject *type) {
    Py_INCREF(type);
    Py_XSETREF(g_error, type);
    Py_RETURN_NONE;
}

#define FAST(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(sample_prompts), FAST(advantages), FAST(advantage_diagnostics), FAST(tracker_update), FAST(pg_loss_fwd),
                         FAST(pg_loss_bwd), FAST(pg_loss_fwd_bwd), {"set_error", set_error, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_spo_calls", "plain calls of the binding", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__spo_calls() { return PyModule_Create(&module); }
