// The differentiable operators of functional.py as native autograd nodes: argument checks, allocation and the calls of the C ABI
// (na2d.h, na1d.h) without the interpreter in between.  Every gradient comes from the library's kernels, as there.
//
// Each function of the module returns the operator's output, or None where something is not as the plain case has it (a tensor that is
// not dense on one GPU or a subclass, shapes or types that do not fit, a functorch transform, forward-mode differentiation, tracing, a dispatch or
// torch-function mode, a call that the library refuses): the caller then takes the interpreted functions, which serve those or raise.  A pass of a small operator
// is bound by this path, not by its kernels (us a pass of 1 x 8 x 14 x 14 fp16, k = 7, inference, and of 5 x 3 x 61 x 45 bf16, k = 5, without a
// bias, forward and backward; through ctypes and Python's autograd functions / here: 20 / 6.4, 159 / 71; of the latter 34 are what a pass of any operator takes in autograd).
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/PyInterpreter.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/forward_grad.h>
#include <torch/csrc/autograd/function.h>
#include <torch/csrc/autograd/functions/utils.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/autograd/saved_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>

#include <cmath>
#include <limits>
#include <optional>

#include "na_typed.h"

namespace {

using at::Tensor;
using torch::autograd::AutogradContext;
using torch::autograd::SavedVariable;
using torch::autograd::variable_list;

// ---- checks ------------------------------------------------------------------------------------------------------------

// a strided tensor on a GPU with nothing wrapped around it
bool plain(const Tensor &t) {
    static const c10::DispatchKeySet allowed{c10::DispatchKey::CUDA, c10::DispatchKey::AutogradCUDA, c10::DispatchKey::ADInplaceOrView, c10::DispatchKey::AutocastCUDA};
    return t.defined() && t.is_cuda() && (t.key_set() | allowed) == allowed;
}
bool plain_context() {
    static const c10::DispatchKeySet modes{c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot, c10::DispatchKey::PythonDispatcher,
                                           c10::DispatchKey::FuncTorchDynamicLayerFrontMode, c10::DispatchKey::FuncTorchDynamicLayerBackMode,
                                           c10::DispatchKey::Functionalize, c10::DispatchKey::Tracer, c10::DispatchKey::PreDispatch};
    // (a functorch transform shows in the modes; its thread-local state outlives it)
    return !c10::impl::tls_local_dispatch_key_set().included_.has_any(modes) && !torch::jit::tracer::isTracing() &&
           !torch::autograd::ForwardADLevel::try_get_by_idx(0);
}

std::optional<int> dtype_code(at::ScalarType t) {
    switch (t) {
        case at::kFloat: return NA2D_F32;
        case at::kHalf: return NA2D_F16;
        case at::kBFloat16: return NA2D_BF16;
        default: return std::nullopt;
    }
}
bool fits(int64_t n) { return n >= 0 && n <= std::numeric_limits<int32_t>::max(); }

std::optional<na2d_problem> problem_2d(at::IntArrayRef s, at::ScalarType type, int64_t k) {
    const auto code = dtype_code(type);
    if (s.size() != 5 || !code || !fits(k)) return std::nullopt;
    for (int64_t n : s)
        if (!fits(n)) return std::nullopt;
    const na2d_problem p{(int32_t)s[0], (int32_t)s[1], (int32_t)s[2], (int32_t)s[3], (int32_t)s[4], (int32_t)k, *code};
    return na2d_validate_problem(&p) == NA2D_OK ? std::optional(p) : std::nullopt;
}
std::optional<na1d_problem> problem_1d(at::IntArrayRef s, at::ScalarType type, int64_t k) {
    const auto code = dtype_code(type);
    if (s.size() != 4 || !code || !fits(k)) return std::nullopt;
    for (int64_t n : s)
        if (!fits(n)) return std::nullopt;
    const na1d_problem p{(int32_t)s[0], (int32_t)s[1], (int32_t)s[2], (int32_t)s[3], (int32_t)k, *code};
    return na1d_validate_problem(&p) == NA2D_OK ? std::optional(p) : std::nullopt;
}
// `t` (a tensor the operator takes beside `of`) is plain, on the same device, of the same type and of these sizes
bool matches(const Tensor &t, const Tensor &of, at::IntArrayRef sizes) {
    return plain(t) && t.scalar_type() == of.scalar_type() && t.device() == of.device() && t.sizes() == sizes;
}

// ---- calls -------------------------------------------------------------------------------------------------------------

void *stream() {   // of the current device, as the interpreted binding takes it
    return c10::hip::getCurrentHIPStreamMasqueradingAsCUDA().stream();
}
void *ptr(const Tensor &t) { return t.defined() ? t.data_ptr() : nullptr; }
Tensor workspace(size_t bytes, const Tensor &like) { return at::empty({(int64_t)(bytes < 16 ? 16 : bytes)}, like.options().dtype(at::kByte)); }
Tensor fp32(at::IntArrayRef sizes, const Tensor &like) { return at::empty(sizes, like.options().dtype(at::kFloat)); }

// a call that the library refused inside a backward pass: the error the interpreted binding raises
void check(int status) {
    if (status == NA2D_OK) return;
    const PyGILState_STATE gil = PyGILState_Ensure();
    if (PyObject *m = PyImport_ImportModule("paper_2204_07143_amd.binding")) {
        Py_XDECREF(PyObject_CallMethod(m, "_check", "i", status));
        Py_DECREF(m);
    }
    python_error err;
    if (PyErr_Occurred()) err.persist();
    PyGILState_Release(gil);
    throw std::move(err);
}
// What a backward pass reads comes from autograd: a saved-tensor hook may hand back a tensor of another form, an upstream gradient may be
// wrapped.  The kernels read memory, so what is not dense, of the expected type and sizes and on `of`'s device is refused, with the errors of the
// interpreted binding.
const Tensor &readable(const Tensor &t, const Tensor &of, at::ScalarType type, at::IntArrayRef sizes) {
    TORCH_CHECK_VALUE(plain(t) && t.device() == of.device(), "na2d takes GPU tensors only");
    TORCH_CHECK_VALUE(t.is_contiguous(), "na2d takes contiguous tensors only");
    TORCH_CHECK_VALUE(t.scalar_type() == type, "expected dtype ", type, ", got ", t.scalar_type());
    TORCH_CHECK_VALUE(t.sizes() == sizes, "expected shape ", sizes, ", got ", t.sizes());
    return t;
}
const Tensor &readable(const Tensor &t, const Tensor &of, at::IntArrayRef sizes) { return readable(t, of, of.scalar_type(), sizes); }
// the upstream gradient, dense (autograd has checked its type, sizes and device against the output)
Tensor upstream(const Tensor &grad) {
    const Tensor g = (grad.is_neg() ? grad.resolve_neg() : grad).contiguous();
    return readable(g, g, g.sizes());
}
template <typename Problem> const Problem &valid(const std::optional<Problem> &p) {
    TORCH_CHECK_VALUE(p, "not a problem of the forward pass");
    return *p;
}
struct Refused {};   // a forward call that the library refused
void forward_check(int status) {
    if (status != NA2D_OK) throw Refused{};
}

bool wants_grad(std::initializer_list<const Tensor *> in) {
    if (!at::GradMode::is_enabled()) return false;
    for (const Tensor *t : in)
        if (t->defined() && t->requires_grad()) return true;
    return false;
}

// ---- the whole operator in 2D --------------------------------------------------------------------------------------------

struct NA2D : torch::autograd::Function<NA2D> {
    // lse: where the log-sum-exp is kept for the backward pass
    static Tensor run(const Tensor &q, const Tensor &k, const Tensor &v, const Tensor &rpb, const na2d_problem &p, double scale, Tensor *lse) {
        Tensor out = at::empty(q.sizes(), q.options());
        if (lse) *lse = fp32(q.sizes().slice(0, 4), q);
        forward_check(na2d_fused_fwd(&p, ptr(q), ptr(k), ptr(v), ptr(rpb), (float)scale, ptr(out), lse ? (float *)ptr(*lse) : nullptr, stream()));
        return out;
    }
    static Tensor forward(AutogradContext *ctx, const Tensor &q_, const Tensor &k_, const Tensor &v_, const std::optional<Tensor> &rpb_, int64_t ks, double scale) {
        const Tensor q = q_.contiguous(), k = k_.contiguous(), v = v_.contiguous(), rpb = rpb_ ? rpb_->contiguous() : Tensor();
        Tensor lse;
        Tensor out = run(q, k, v, rpb, *problem_2d(q.sizes(), q.scalar_type(), ks), scale, &lse);
        ctx->save_for_backward({q, k, v, lse, rpb});
        ctx->saved_data["k"] = ks;
        ctx->saved_data["scale"] = scale;
        ctx->saved_data["want"] = rpb_ && rpb_->requires_grad();
        return out;
    }
    static variable_list backward(AutogradContext *ctx, variable_list grads) {
        const auto saved = ctx->get_saved_variables();
        const float scale = (float)ctx->saved_data["scale"].toDouble();
        const bool want = ctx->saved_data["want"].toBool();
        const int64_t ks = ctx->saved_data["k"].toInt();
        const Tensor dout = upstream(grads[0]);
        const auto s = dout.sizes();
        const na2d_problem p = valid(problem_2d(s, dout.scalar_type(), ks));
        const Tensor &q = readable(saved[0], dout, s), &k = readable(saved[1], dout, s), &v = readable(saved[2], dout, s);
        const Tensor &lse = readable(saved[3], dout, at::kFloat, s.slice(0, 4));
        const Tensor &rpb = saved[4].defined() ? readable(saved[4], dout, {s[1], 2 * ks - 1, 2 * ks - 1}) : saved[4];
        Tensor dq = at::empty(q.sizes(), q.options()), dk = at::empty(q.sizes(), q.options()), dv = at::empty(q.sizes(), q.options());
        Tensor d_rpb = want ? at::empty(rpb.sizes(), rpb.options()) : Tensor();   // (rpb is of q's type)
        const size_t direct = na2d_direct_bwd_workspace_bytes(&p);   // 0: not for this problem
        const Tensor ws = workspace(direct ? direct : na2d_workspace_bytes(&p, NA2D_WS_FUSED_BWD), q);
        check((direct ? na2d_direct_bwd_typed : na2d_fused_bwd_typed)(&p, ptr(q), ptr(k), ptr(v), ptr(rpb), scale, (const float *)ptr(lse), ptr(dout), ptr(dq), ptr(dk), ptr(dv),
                                                                      ptr(d_rpb), ptr(ws), (size_t)ws.numel(), stream()));
        variable_list r{dq, dk, dv, d_rpb};
        r.resize(6);
        return r;
    }
};

// ---- the whole operator in 1D --------------------------------------------------------------------------------------------

struct NA1D : torch::autograd::Function<NA1D> {
    static Tensor run(const Tensor &q, const Tensor &k, const Tensor &v, const Tensor &rpb, const na1d_problem &p, double scale, Tensor *lse) {
        Tensor out = at::empty(q.sizes(), q.options());
        if (lse) *lse = fp32(q.sizes().slice(0, 3), q);
        forward_check(na1d_fused_fwd(&p, ptr(q), ptr(k), ptr(v), ptr(rpb), (float)scale, ptr(out), lse ? (float *)ptr(*lse) : nullptr, stream()));
        return out;
    }
    static Tensor forward(AutogradContext *ctx, const Tensor &q_, const Tensor &k_, const Tensor &v_, const std::optional<Tensor> &rpb_, int64_t ks, double scale) {
        const Tensor q = q_.contiguous(), k = k_.contiguous(), v = v_.contiguous(), rpb = rpb_ ? rpb_->contiguous() : Tensor();
        Tensor lse;
        Tensor out = run(q, k, v, rpb, *problem_1d(q.sizes(), q.scalar_type(), ks), scale, &lse);
        ctx->save_for_backward({q, k, v, lse, rpb});
        ctx->saved_data["k"] = ks;
        ctx->saved_data["scale"] = scale;
        ctx->saved_data["want"] = rpb_ && rpb_->requires_grad();
        return out;
    }
    static variable_list backward(AutogradContext *ctx, variable_list grads) {
        const auto saved = ctx->get_saved_variables();
        const bool want = ctx->saved_data["want"].toBool();
        const int64_t ks = ctx->saved_data["k"].toInt();
        const Tensor dout = upstream(grads[0]);
        const auto s = dout.sizes();
        const na1d_problem p = valid(problem_1d(s, dout.scalar_type(), ks));
        const Tensor &q = readable(saved[0], dout, s), &k = readable(saved[1], dout, s), &v = readable(saved[2], dout, s);
        const Tensor &lse = readable(saved[3], dout, at::kFloat, s.slice(0, 3));
        const Tensor &rpb = saved[4].defined() ? readable(saved[4], dout, {s[1], 2 * ks - 1}) : saved[4];
        Tensor dq = at::empty(q.sizes(), q.options()), dk = at::empty(q.sizes(), q.options()), dv = at::empty(q.sizes(), q.options());
        Tensor d_rpb = want ? at::empty(rpb.sizes(), rpb.options()) : Tensor();
        const Tensor ws = workspace(na1d_fused_bwd_workspace_bytes(&p), q);
        check(na1d_fused_bwd_typed(&p, ptr(q), ptr(k), ptr(v), ptr(rpb), (float)ctx->saved_data["scale"].toDouble(), (const float *)ptr(lse), ptr(dout), ptr(dq), ptr(dk), ptr(dv),
                                   ptr(d_rpb), ptr(ws), (size_t)ws.numel(), stream()));
        variable_list r{dq, dk, dv, d_rpb};
        r.resize(6);
        return r;
    }
};

// ---- the steps of the unfused operator ---------------------------------------------------------------------------------

Tensor attention_like(const Tensor &q, int64_t ks) {
    const auto s = q.sizes();
    return at::empty({s[0], s[1], s[2], s[3], ks * ks}, q.options());
}

// Where the softmax and its backward work in place, and where grad-v stands: by what still lies in the 256 MB last-level cache.  us of the forward and of the whole pass,
// always with another tensor and grad-v behind grad-a / by the rule: 39 MB of weights (64 x 2 x 56 x 56 fp16, k = 7) 57 and 174 / the same; from 48 MB on the backward in place:
// 59 MB (96 items) - and 256 / 253, 62 MB (16 x 4 x 56 x 56 fp32, 16 channels, k = 9) - and 408 / 398, 65 MB (k = 9) - and 287 / 277, 79 MB (fp32, k = 7) - and 827 / 816, 512 x 8 x 14 x 14
// fp16 - and 340 / 343; from 90 MB on the forward in place, grad-v first: 97 MB (k = 11) 102 / 100 and 397 / 390, 136 MB (k = 13) 139 / 126 and 490 / 481, 118 MB (768 x 8 x 14 x 14, k = 7)
// 161 / 166 and 508 / 514, 157 MB (256 items) 217 / 209 and 636 / 636, 272 MB (128 items, k = 13) 270 / 265 and 955 / 954.
bool large(const Tensor &t) { return t.nbytes() >= (size_t)90 << 20; }
bool in_place(const Tensor &dp) { return dp.nbytes() >= (size_t)48 << 20 && !large(dp); }

// attn: where the weights are kept for the backward pass
Tensor unfused(const Tensor &q, const Tensor &k, const Tensor &v, const Tensor &rpb, const na2d_problem &p, double scale, Tensor &attn) {
    const Tensor logits = attention_like(q, p.k);
    forward_check(na2d_qk_rpb(&p, ptr(q), ptr(k), ptr(rpb), (float)scale, ptr(logits), stream()));
    attn = large(logits) ? logits : attention_like(q, p.k);
    forward_check(na2d_softmax(&p, ptr(logits), ptr(attn), stream()));
    Tensor out = at::empty(v.sizes(), v.options());
    forward_check(na2d_av(&p, ptr(attn), ptr(v), ptr(out), stream()));
    return out;
}

// One node for the three steps: the kernels and the results are those of the separate functions, and a pass goes through autograd once
// (us a pass of 1 x 1 x 8 x 8 fp16, k = 7, forward and backward: three nodes 119, one 100).
// It keeps, and unpacks in a pass, what the separate nodes would: q and k only for gradients that need them, so that a program that does not ask for those may
// have changed q and k in between.
struct Unfused : torch::autograd::Node {
    SavedVariable q, k, v, attn;
    int64_t ks;
    float scale;
    std::string name() const override { return "NA2DUnfusedBackward"; }
    void release_variables() override {
        const std::lock_guard<std::mutex> lock(mutex_);
        for (SavedVariable *s : {&q, &k, &v, &attn}) s->reset_data();
    }
    variable_list apply(variable_list &&grads) override {
        const std::lock_guard<std::mutex> lock(mutex_);
        // (of this pass: what nothing asks for is not computed)
        const bool want_q = task_should_compute_output(0), want_k = task_should_compute_output(1), want_v = task_should_compute_output(2), want_rpb = task_should_compute_output(3);
        const bool want_ds = want_q || want_k || want_rpb;
        const Tensor v_ = v.unpack(), attn_ = attn.unpack(), q_ = want_ds ? q.unpack() : Tensor(), k_ = want_ds ? k.unpack() : Tensor();
        const Tensor dout = upstream(grads[0].defined() ? grads[0] : at::zeros_like(v_));
        const auto s = dout.sizes();
        const na2d_problem p = valid(problem_2d(s, dout.scalar_type(), ks));
        readable(v_, dout, s), readable(attn_, dout, {s[0], s[1], s[2], s[3], ks * ks});
        if (want_ds) readable(q_, dout, s), readable(k_, dout, s);
        Tensor dq, dk, dv, d_rpb, dp;
        const auto grad_v = [&] {
            dv = at::empty(s, dout.options());
            check(na2d_av_bwd_v(&p, ptr(attn_), ptr(dout), ptr(dv), ::stream()));
        };
        if (want_v && large(attn_)) grad_v();
        if (want_ds) {
            dp = attention_like(dout, ks);
            check(na2d_av_bwd_p(&p, ptr(dout), ptr(v_), ptr(dp), ::stream()));
        }
        if (want_v && !large(attn_)) grad_v();   // (the weights are read once more right behind)
        if (want_ds) {
            const Tensor ds = in_place(dp) ? dp : attention_like(dout, ks);
            check(na2d_softmax_bwd(&p, ptr(attn_), ptr(dp), ptr(ds), ::stream()));
            if (want_q) {
                dq = at::empty(s, dout.options());
                check(na2d_qk_bwd_q(&p, ptr(ds), ptr(k_), scale, ptr(dq), ::stream()));
            }
            if (want_k) {
                dk = at::empty(s, dout.options());
                check(na2d_qk_bwd_k(&p, ptr(ds), ptr(q_), scale, ptr(dk), ::stream()));
            }
            if (want_rpb) {
                d_rpb = at::empty({s[1], 2 * ks - 1, 2 * ks - 1}, dout.options());
                const Tensor ws = workspace(na2d_workspace_bytes(&p, NA2D_WS_QK_BWD_RPB), dout);
                check(na2d_qk_bwd_rpb_typed(&p, ptr(ds), ptr(d_rpb), ptr(ws), (size_t)ws.numel(), ::stream()));
            }
        }
        return {dq, dk, dv, d_rpb};
    }
    static Tensor of(const Tensor &q_, const Tensor &k_, const Tensor &v_, const Tensor &rpb_, const na2d_problem &p, double scale, bool record) {
        Tensor out, attn;
        std::shared_ptr<Unfused> node;
        {
            const at::AutoGradMode off(false);
            const Tensor q = q_.contiguous(), k = k_.contiguous(), v = v_.contiguous();
            out = unfused(q, k, v, rpb_.defined() ? rpb_.contiguous() : rpb_, p, scale, attn);
            if (!record) return out;
            node = std::shared_ptr<Unfused>(new Unfused, torch::autograd::deleteNode);
            const bool want_ds = q_.requires_grad() || k_.requires_grad() || (rpb_.defined() && rpb_.requires_grad());
            if (want_ds) node->q = SavedVariable(q, false), node->k = SavedVariable(k, false);
            node->v = SavedVariable(v, false);
            node->attn = SavedVariable(attn, false);
            node->ks = p.k;
            node->scale = (float)scale;
        }
        node->set_next_edges(torch::autograd::collect_next_edges(q_, k_, v_, rpb_));
        torch::autograd::set_history(out, node);
        return out;
    }
};

// ---- module ------------------------------------------------------------------------------------------------------------

struct NoGil {
    PyThreadState *state = PyEval_SaveThread();
    ~NoGil() { PyEval_RestoreThread(state); }
};

// args[i] as a tensor (or a parameter; a subclass may have a __torch_function__ to be asked); undefined for None where that is allowed.
// false: it is neither.
bool tensor_arg(PyObject *o, Tensor &t, bool optional = false) {
    if (optional && o == Py_None) return true;
    if (!THPVariable_CheckExact(o)) return false;
    t = THPVariable_Unpack(o);
    return true;
}
// No torch-function mode is to be asked.  (The mode of torch.set_default_device, on for as long as a program likes, only looks at calls that
// create tensors without naming a device.)
bool plain_modes() {
    if (!at::impl::torch_function_mode_enabled()) return true;
    static PyObject *default_device = nullptr;   // (under the interpreter lock)
    if (!default_device) {
        PyObject *module = PyImport_ImportModule("torch.utils._device");
        if (module) default_device = PyObject_GetAttrString(module, "DeviceContext");
        Py_XDECREF(module);
        PyErr_Clear();
    }
    for (int64_t i = 0; i < at::impl::PythonTorchFunctionTLS::stack_len(); ++i) {
        PyObject *mode = at::impl::PythonTorchFunctionTLS::get_stack_at(i)->ptr(getPyInterpreter());
        if ((PyObject *)Py_TYPE(mode) != default_device) return false;
    }
    return true;
}
std::optional<Tensor> maybe(const Tensor &t) { return t.defined() ? std::optional(t) : std::nullopt; }

// BODY computes `out`; anything that the plain case does not have leaves it undefined
template <typename Body> PyObject *guarded(Body body) {
    HANDLE_TH_ERRORS
    Tensor out;
    {
        NoGil no_gil;
        try {
            if (plain_context()) out = body();
        } catch (const Refused &) {
        }
    }
    if (!out.defined()) Py_RETURN_NONE;
    return THPVariable_Wrap(std::move(out));
    END_HANDLE_TH_ERRORS
}

// (q, k, v, rpb or None, kernel size, scale or None)
struct Args {
    Tensor q, k, v, rpb;
    int64_t ks = 0;
    double scale = 0;
    bool ok = false;
    Args(PyObject *const *a, Py_ssize_t n) {
        if (n != 6 || !plain_modes() || !tensor_arg(a[0], q) || !tensor_arg(a[1], k) || !tensor_arg(a[2], v) || !tensor_arg(a[3], rpb, true)) return;
        ks = PyLong_AsLongLong(a[4]);
        scale = a[5] == Py_None ? (q.dim() > 0 ? std::pow((double)q.size(-1), -0.5) : 0.) : PyFloat_AsDouble(a[5]);
        ok = !PyErr_Occurred();
        if (!ok) PyErr_Clear();
    }
    bool check(at::IntArrayRef table) const {
        return plain(q) && matches(k, q, q.sizes()) && matches(v, q, q.sizes()) && (!rpb.defined() || matches(rpb, q, table));
    }
};

PyObject *py_na2d(PyObject *, PyObject *const *a, Py_ssize_t n) {
    const Args x(a, n);
    if (!x.ok) Py_RETURN_NONE;
    return guarded([&]() -> Tensor {
        const auto p = problem_2d(x.q.sizes(), x.q.scalar_type(), x.ks);
        if (!p || !x.check({x.q.size(1), 2 * x.ks - 1, 2 * x.ks - 1})) return Tensor();
        if (wants_grad({&x.q, &x.k, &x.v, &x.rpb})) return NA2D::apply(x.q, x.k, x.v, maybe(x.rpb), x.ks, x.scale);
        return NA2D::run(x.q.contiguous(), x.k.contiguous(), x.v.contiguous(), x.rpb.defined() ? x.rpb.contiguous() : x.rpb, *p, x.scale, nullptr);
    });
}

PyObject *py_na1d(PyObject *, PyObject *const *a, Py_ssize_t n) {
    const Args x(a, n);
    if (!x.ok) Py_RETURN_NONE;
    return guarded([&]() -> Tensor {
        const auto p = problem_1d(x.q.sizes(), x.q.scalar_type(), x.ks);
        if (!p || !x.check({x.q.size(1), 2 * x.ks - 1})) return Tensor();
        if (wants_grad({&x.q, &x.k, &x.v, &x.rpb})) return NA1D::apply(x.q, x.k, x.v, maybe(x.rpb), x.ks, x.scale);
        return NA1D::run(x.q.contiguous(), x.k.contiguous(), x.v.contiguous(), x.rpb.defined() ? x.rpb.contiguous() : x.rpb, *p, x.scale, nullptr);
    });
}

// QK + bias, softmax and AV by their own kernels
PyObject *py_na2d_unfused(PyObject *, PyObject *const *a, Py_ssize_t n) {
    const Args x(a, n);
    if (!x.ok) Py_RETURN_NONE;
    return guarded([&]() -> Tensor {
        const auto p = problem_2d(x.q.sizes(), x.q.scalar_type(), x.ks);
        if (!p || !x.check({x.q.size(1), 2 * x.ks - 1, 2 * x.ks - 1})) return Tensor();
        return Unfused::of(x.q, x.k, x.v, x.rpb, *p, x.scale, wants_grad({&x.q, &x.k, &x.v, &x.rpb}));
    });
}

PyMethodDef methods[] = {{"na2d", (PyCFunction)(void (*)(void))py_na2d, METH_FASTCALL, nullptr},
                         {"na1d", (PyCFunction)(void (*)(void))py_na1d, METH_FASTCALL, nullptr},
                         {"na2d_unfused", (PyCFunction)(void (*)(void))py_na2d_unfused, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "na2d_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_na2d_torch() { return PyModule_Create(&module); }
