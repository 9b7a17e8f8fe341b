// lnmod_torch.cpp -- the host path of the autograd functions and of the plain forward in C++: checks,
// output and workspace allocation, the call through the C ABI and the autograd node.
//
// Why: a step (forward, autograd, backward) took 80 to 200 us of host time per call in Python -- the
// autograd engine handing the interpreter lock to its own thread, torch.empty nine times, ctypes with
// up to twenty arguments, per-tensor checks -- where its kernels take 18 us on 512 x 1536 fp32 rows and
// 100 us on 32 760 x 1536 bf16 rows, so everything up to about 200 MB per step waited for the host.
//
// Nothing is decided here that the Python binding does not decide: whatever is not the plain case (any
// check that fails, a tensor subclass, functorch, a dispatch mode, a tracer, another current device, a
// status other than LNMOD_OK) goes back to the Python path, which raises its own errors.  The kernels,
// their arguments and the saved tensors with their order are the same either way.
#include <torch/extension.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_cpp_function.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>
#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <torch/version.h>

#include "lnmod.h"

namespace {

using at::Tensor;
using torch::autograd::AutogradContext;
using torch::autograd::variable_list;

struct NotPlain {};      // thrown to leave a call to the Python path; nothing has been launched

// ---- what counts as the plain case ---------------------------------------------------------------
const c10::DispatchKeySet kSpecial({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched,
                                    c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize,
                                    c10::DispatchKey::ZeroTensor, c10::DispatchKey::Negative,
                                    c10::DispatchKey::Conjugate});

bool plain_state() {
    if (c10::impl::TorchDispatchModeTLS::any_modes_set()) return false;
    if (torch::jit::tracer::isTracing()) return false;
    return !c10::impl::tls_local_dispatch_key_set().included_.has(c10::DispatchKey::FuncTorchDynamicLayerFrontMode);
}

// A tensor of exactly torch's own type (or a Parameter), without a forward-mode tangent.
bool plain_object(const py::object& o) {
    return THPVariable_CheckExact(o.ptr()) && !THPVariable_Unpack(o.ptr())._fw_grad(0).defined();
}

bool plain(const Tensor& t, at::IntArrayRef shape, at::ScalarType type, const at::Device& dev) {
    return t.defined() && t.layout() == at::kStrided && t.device() == dev && t.scalar_type() == type &&
           !(t.key_set() & kSpecial).has_any(kSpecial) && t.sizes() == shape && t.is_contiguous();
}

// x itself: on the current device, an element type the kernels know
bool plain_first(const Tensor& x) {
    return x.defined() && x.is_cuda() && (x.scalar_type() == at::kBFloat16 || x.scalar_type() == at::kFloat) &&
           x.device().index() == c10::hip::current_device() && plain(x, x.sizes(), x.scalar_type(), x.device());
}

int code_of(const Tensor& x) { return x.scalar_type() == at::kBFloat16 ? LNMOD_BF16 : LNMOD_F32; }

void* stream_of(const Tensor& x) {
    return c10::hip::getCurrentHIPStreamMasqueradingAsCUDA(x.device().index()).stream();
}

const void* ptr(const Tensor& t) { return t.defined() ? t.const_data_ptr() : nullptr; }
void* out(const Tensor& t) { return t.mutable_data_ptr(); }
const int32_t* cu_ptr(const Tensor& cu) { return cu.defined() ? cu.const_data_ptr<int32_t>() : nullptr; }
const float* f32(const Tensor& t) { return t.defined() ? t.const_data_ptr<float>() : nullptr; }
float* f32_out(const Tensor& t) { return t.mutable_data_ptr<float>(); }

// The batch of a call: [B, S, D], or [T, D] with cu_seqlens.
struct Batch {
    int64_t n, s_or_t, T, D;
    bool ok;
};

Batch batch_of(const Tensor& x, const Tensor& cu) {
    if (!cu.defined()) {
        if (x.dim() != 3) return {0, 0, 0, 0, false};
        return {x.size(0), x.size(1), x.size(0) * x.size(1), x.size(2), true};
    }
    if (x.dim() != 2 || cu.dim() != 1 || cu.numel() < 1 || !plain(cu, cu.sizes(), at::kInt, x.device()))
        return {0, 0, 0, 0, false};
    return {cu.numel() - 1, x.size(0), x.size(0), x.size(1), true};
}

at::TensorOptions f32_like(const Tensor& x) { return x.options().dtype(at::kFloat); }

Tensor scratch(size_t bytes, const Tensor& x) {
    return at::empty({static_cast<int64_t>(bytes < 16 ? 16 : bytes)}, x.options().dtype(at::kByte));
}

// ---- the Python path, for a backward that is not the plain case ------------------------------------
py::object to_python(const Tensor& t) { return t.defined() ? py::cast(t) : py::none(); }
py::object to_python(double v) { return py::float_(v); }

// name(args...) of functional.py, with None for an undefined tensor.  Runs on a thread of the autograd engine,
// without the interpreter lock: no Python object is made before it is taken here.  The function's exception (a ValueError of a check, an LnmodError) is kept
// alive across the engine's threads
template <typename... A>
variable_list python_backward(const char* name, size_t outputs, const A&... args) {
    py::gil_scoped_acquire gil;
    try {
        py::tuple r = py::module_::import("paper_2605_17923_amd.functional").attr(name)(to_python(args)...);
        variable_list got;
        for (size_t i = 0; i < outputs; ++i) got.push_back(r[i].cast<Tensor>());
        return got;
    } catch (py::error_already_set& e) {
        e.restore();
        python_error err;
        err.persist();
        throw err;
    }
}

// ---- LayerNorm-Modulate ------------------------------------------------------------------------------
bool ln_shapes(const Tensor& x, const Tensor& scale, const Tensor& cu, Batch* b, bool* token) {
    if (!plain_first(x)) return false;
    *b = batch_of(x, cu);
    if (!b->ok || !scale.defined()) return false;
    *token = !cu.defined() && scale.dim() == 3;
    const int64_t rows[] = {b->n, b->D};
    return plain(scale, *token ? x.sizes() : at::IntArrayRef(rows, 2), x.scalar_type(), x.device());
}

// y and the statistics; throws NotPlain
std::tuple<Tensor, Tensor, Tensor> ln_forward(const Tensor& x, const Tensor& shift, const Tensor& scale,
                                              const Tensor& cu, double eps) {
    Batch b;
    bool token;
    if (!ln_shapes(x, scale, cu, &b, &token) || !plain(shift, scale.sizes(), x.scalar_type(), x.device()))
        throw NotPlain();
    Tensor y = at::empty_like(x);
    Tensor mean = cu.defined() ? at::empty({b.T}, f32_like(x)) : at::empty({b.n, b.s_or_t}, f32_like(x));
    Tensor rstd = at::empty_like(mean);
    const float e = static_cast<float>(eps);
    const int st = cu.defined() ? lnmod_forward_varlen(ptr(x), ptr(shift), ptr(scale), cu_ptr(cu), b.n, b.T, b.D, e,
                                                       stream_of(x), out(y), f32_out(mean), f32_out(rstd), code_of(x))
                                : lnmod_forward(ptr(x), ptr(shift), ptr(scale), b.n, b.s_or_t, b.D, e, stream_of(x),
                                                out(y), f32_out(mean), f32_out(rstd), code_of(x),
                                                token ? LNMOD_PER_TOKEN : LNMOD_PER_SAMPLE);
    if (st != LNMOD_OK) throw NotPlain();
    return {y, mean, rstd};
}

struct LnModulate : public torch::autograd::Function<LnModulate> {
    static Tensor forward(AutogradContext* ctx, const Tensor& x, const Tensor& shift, const Tensor& scale,
                          const std::optional<Tensor>& cu_seqlens, double eps, bool save_stats) {
        const Tensor cu = cu_seqlens.value_or(Tensor());
        auto [y, mean, rstd] = ln_forward(x, shift, scale, cu, eps);
        ctx->saved_data["eps"] = eps;
        if (!save_stats) mean = rstd = Tensor();          // the backward forms them again from x
        ctx->save_for_backward({x, scale, cu, mean, rstd});
        return y;
    }

    static variable_list backward(AutogradContext* ctx, variable_list grads) {
        const variable_list s = ctx->get_saved_variables();
        const Tensor &x = s[0], &scale = s[1], &cu = s[2], &mean = s[3], &rstd = s[4];
        const double eps = ctx->saved_data["eps"].toDouble();
        const Tensor dy = grads[0].contiguous();
        Batch b;
        bool token = false;
        if (plain_state() && ln_shapes(x, scale, cu, &b, &token) && plain(dy, x.sizes(), x.scalar_type(), x.device()) &&
            mean.defined() == rstd.defined() &&
            (!mean.defined() || (plain(mean, mean.sizes(), at::kFloat, x.device()) && mean.numel() == b.T &&
                                 plain(rstd, mean.sizes(), at::kFloat, x.device())))) {
            // With a modulation row per token dshift equals dy, but it is a tensor of its own: a leaf's .grad, a hook or
            // torch.autograd.grad's caller may write to it, and whether dy's memory has another user cannot be told here
            // (a view in front of the operator gives dy a fresh tensor over memory that is still the caller's).
            Tensor dx = at::empty_like(x), dshift = at::empty_like(scale), dscale = at::empty_like(scale);
            int st;
            if (token) {
                st = lnmod_backward(ptr(dy), ptr(x), nullptr, ptr(scale), b.n, b.s_or_t, b.D, static_cast<float>(eps),
                                    stream_of(x), f32(mean), f32(rstd), out(dx), out(dshift), out(dscale), nullptr, 0,
                                    code_of(x), LNMOD_PER_TOKEN);
            } else {
                const Tensor ws = scratch(lnmod_backward_workspace_bytes(b.n, b.T, b.D, LNMOD_PER_SAMPLE), x);
                st = lnmod_backward_io(ptr(dy), ptr(x), ptr(scale), cu_ptr(cu), b.n, b.s_or_t, b.D,
                                       static_cast<float>(eps), stream_of(x), f32(mean), f32(rstd), out(dx),
                                       out(dshift), out(dscale), out(ws), static_cast<size_t>(ws.numel()), code_of(x));
            }
            if (st == LNMOD_OK) return {dx, dshift, dscale, Tensor(), Tensor(), Tensor()};
        }
        variable_list r = python_backward("_ln_backward", 3, dy, x, scale, cu, mean, rstd, eps);
        return {r[0], r[1], r[2], Tensor(), Tensor(), Tensor()};
    }
};

// ---- gated residual + LayerNorm-Modulate ---------------------------------------------------------------
bool gated_shapes(const Tensor& x, const Tensor& u, const Tensor& gate, const Tensor& scale, const Tensor& cu, Batch* b) {
    if (!plain_first(x)) return false;
    *b = batch_of(x, cu);
    const int64_t rows[] = {b->n, b->D};
    const auto mod = at::IntArrayRef(rows, 2);
    return b->ok && plain(u, x.sizes(), x.scalar_type(), x.device()) && plain(gate, mod, x.scalar_type(), x.device()) &&
           plain(scale, mod, x.scalar_type(), x.device());
}

struct GatedLnModulate : public torch::autograd::Function<GatedLnModulate> {
    static variable_list forward(AutogradContext* ctx, const Tensor& x, const Tensor& u, const Tensor& gate,
                                 const Tensor& shift, const Tensor& scale, const std::optional<Tensor>& cu_seqlens,
                                 double eps) {
        const Tensor cu = cu_seqlens.value_or(Tensor());
        Batch b;
        if (!gated_shapes(x, u, gate, scale, cu, &b) || !plain(shift, scale.sizes(), x.scalar_type(), x.device()))
            throw NotPlain();
        Tensor h = at::empty_like(x), y = at::empty_like(x);
        Tensor mean = at::empty({b.T}, f32_like(x)), rstd = at::empty({b.T}, f32_like(x));
        const int st = lnmod_gated_forward(ptr(x), ptr(u), ptr(gate), ptr(shift), ptr(scale), cu_ptr(cu), b.n, b.s_or_t,
                                           b.D, static_cast<float>(eps), stream_of(x), out(h), out(y), f32_out(mean),
                                           f32_out(rstd), code_of(x));
        if (st != LNMOD_OK) throw NotPlain();
        ctx->saved_data["eps"] = eps;
        ctx->save_for_backward({h, u, gate, scale, cu, mean, rstd});
        return {h, y};
    }

    static variable_list backward(AutogradContext* ctx, variable_list grads) {
        const variable_list s = ctx->get_saved_variables();
        const Tensor &h = s[0], &u = s[1], &gate = s[2], &scale = s[3], &cu = s[4], &mean = s[5], &rstd = s[6];
        const double eps = ctx->saved_data["eps"].toDouble();
        const Tensor dh = grads[0].contiguous(), dy = grads[1].contiguous();
        Batch b;
        if (plain_state() && gated_shapes(h, u, gate, scale, cu, &b) &&
            plain(dh, h.sizes(), h.scalar_type(), h.device()) && plain(dy, h.sizes(), h.scalar_type(), h.device()) &&
            plain(mean, at::IntArrayRef(&b.T, 1), at::kFloat, h.device()) &&
            plain(rstd, at::IntArrayRef(&b.T, 1), at::kFloat, h.device())) {
            Tensor dx = at::empty_like(h), du = at::empty_like(h);
            Tensor dgate = at::empty_like(gate), dshift = at::empty_like(gate), dscale = at::empty_like(gate);
            const Tensor ws = scratch(lnmod_gated_backward_workspace_bytes(b.n, b.T, b.D), h);
            const int st = lnmod_gated_backward_io(
                ptr(dy), ptr(dh), ptr(h), ptr(u), ptr(gate), ptr(scale), cu_ptr(cu), b.n, b.s_or_t, b.D,
                static_cast<float>(eps), stream_of(h), f32(mean), f32(rstd), out(dx), out(du), out(dgate), out(dshift),
                out(dscale), out(ws), static_cast<size_t>(ws.numel()), code_of(h));
            if (st == LNMOD_OK) return {dx, du, dgate, dshift, dscale, Tensor(), Tensor()};
        }
        variable_list r = python_backward("_gated_backward", 5, dy, dh, h, u, gate, scale, mean, rstd, cu, eps);
        r.resize(7);
        return r;
    }
};

// ---- Q-Norm + K-Norm -------------------------------------------------------------------------------------
bool qk_shapes(const Tensor& q, const Tensor& k, const Tensor& wq, const Tensor& wk, int64_t* N, int64_t* D) {
    if (!plain_first(q) || q.dim() < 1) return false;
    *D = q.size(-1);
    *N = q.numel() / (*D > 0 ? *D : 1);
    const auto w = at::IntArrayRef(D, 1);
    return plain(k, q.sizes(), q.scalar_type(), q.device()) && plain(wq, w, q.scalar_type(), q.device()) &&
           plain(wk, w, q.scalar_type(), q.device());
}

struct QkNorm : public torch::autograd::Function<QkNorm> {
    static variable_list forward(AutogradContext* ctx, const Tensor& q, const Tensor& k, const Tensor& wq,
                                 const Tensor& wk, double eps) {
        int64_t N, D;
        if (!qk_shapes(q, k, wq, wk, &N, &D)) throw NotPlain();
        Tensor qn = at::empty_like(q), kn = at::empty_like(k);
        Tensor rq = at::empty({N}, f32_like(q)), rk = at::empty({N}, f32_like(q));
        const int st = lnmod_qknorm_forward(ptr(q), ptr(k), ptr(wq), ptr(wk), N, D, static_cast<float>(eps),
                                            stream_of(q), out(qn), out(kn), f32_out(rq), f32_out(rk), code_of(q));
        if (st != LNMOD_OK) throw NotPlain();
        ctx->saved_data["eps"] = eps;
        ctx->save_for_backward({q, k, wq, wk, rq, rk});
        return {qn, kn};
    }

    static variable_list backward(AutogradContext* ctx, variable_list grads) {
        const variable_list s = ctx->get_saved_variables();
        const Tensor &q = s[0], &k = s[1], &wq = s[2], &wk = s[3], &rq = s[4], &rk = s[5];
        const double eps = ctx->saved_data["eps"].toDouble();
        const Tensor dqn = grads[0].contiguous(), dkn = grads[1].contiguous();
        int64_t N, D;
        if (plain_state() && qk_shapes(q, k, wq, wk, &N, &D) && plain(dqn, q.sizes(), q.scalar_type(), q.device()) &&
            plain(dkn, q.sizes(), q.scalar_type(), q.device()) &&
            plain(rq, at::IntArrayRef(&N, 1), at::kFloat, q.device()) &&
            plain(rk, at::IntArrayRef(&N, 1), at::kFloat, q.device())) {
            Tensor dq = at::empty_like(q), dk = at::empty_like(k), dwq = at::empty_like(wq), dwk = at::empty_like(wk);
            const Tensor ws = scratch(lnmod_qknorm_backward_workspace_bytes(N, D), q);
            const int st = lnmod_qknorm_backward_io(ptr(dqn), ptr(dkn), ptr(q), ptr(k), ptr(wq), ptr(wk), N, D,
                                                    static_cast<float>(eps), stream_of(q), f32(rq), f32(rk), out(dq),
                                                    out(dk), out(dwq), out(dwk), out(ws),
                                                    static_cast<size_t>(ws.numel()), code_of(q));
            if (st == LNMOD_OK) return {dq, dk, dwq, dwk, Tensor()};
        }
        variable_list r = python_backward("_qk_backward", 4, dqn, dkn, q, k, wq, wk, rq, rk, eps);
        r.resize(5);
        return r;
    }
};

// ---- Python entry points: None where the call is left to the Python path ------------------------------------
template <typename F>
py::object attempt(const std::vector<py::object>& tensors, const py::object& cu, F&& call) {
    if (!plain_state()) return py::none();
    for (const auto& o : tensors)
        if (!plain_object(o)) return py::none();
    if (!cu.is_none() && !plain_object(cu)) return py::none();
    variable_list r;
    try {
        // the launch may wait for room in the queue, and saved-tensor hooks take the lock themselves
        py::gil_scoped_release nogil;
        r = call();
    } catch (const NotPlain&) {
        return py::none();
    }
    if (r.size() == 1) return py::cast(r[0]);
    py::tuple t(r.size());
    for (size_t i = 0; i < r.size(); ++i) t[i] = py::cast(r[i]);
    return t;
}

const Tensor& unpack(const py::object& o) { return THPVariable_Unpack(o.ptr()); }
std::optional<Tensor> unpack_or(const py::object& o) {
    return o.is_none() ? std::nullopt : std::optional<Tensor>(unpack(o));
}

py::object forward(const py::object& x, const py::object& shift, const py::object& scale, const py::object& cu, double eps) {
    return attempt({x, shift, scale}, cu, [&] {
        auto [y, mean, rstd] = ln_forward(unpack(x), unpack(shift), unpack(scale), unpack_or(cu).value_or(Tensor()), eps);
        return variable_list{y, mean, rstd};
    });
}

py::object ln_modulate(const py::object& x, const py::object& shift, const py::object& scale, const py::object& cu,
                       double eps, bool save_stats) {
    return attempt({x, shift, scale}, cu, [&] {
        return variable_list{LnModulate::apply(unpack(x), unpack(shift), unpack(scale), unpack_or(cu), eps, save_stats)};
    });
}

py::object gated_ln_modulate(const py::object& x, const py::object& u, const py::object& gate, const py::object& shift,
                             const py::object& scale, const py::object& cu, double eps) {
    return attempt({x, u, gate, shift, scale}, cu, [&] {
        return GatedLnModulate::apply(unpack(x), unpack(u), unpack(gate), unpack(shift), unpack(scale), unpack_or(cu), eps);
    });
}

py::object qk_norm(const py::object& q, const py::object& k, const py::object& wq, const py::object& wk, double eps) {
    return attempt({q, k, wq, wk}, py::none(), [&] {
        return QkNorm::apply(unpack(q), unpack(k), unpack(wq), unpack(wk), eps);
    });
}

// ---- what y.grad_fn shows --------------------------------------------------------------------------------------
// The node's Python type, with the saved tensors that the Python classes' nodes show (the same ones in the same order,
// None where nothing was saved; an error once the backward has freed them).
template <typename Op>
PyObject* saved_tensors(PyObject* self, void*) {
    HANDLE_TH_ERRORS
    auto& node = static_cast<torch::autograd::CppNode<Op>&>(*reinterpret_cast<torch::autograd::THPCppFunction*>(self)->cdata);
    const variable_list saved = node.ctx_.get_saved_variables();
    py::tuple t(saved.size());
    for (size_t i = 0; i < saved.size(); ++i) t[i] = to_python(saved[i]);
    return t.release().ptr();
    END_HANDLE_TH_ERRORS
}

template <typename Op>
void register_node(const char* name) {
    using namespace torch::autograd;                   // the property macro names functions of it
    static PyTypeObject type;
    static PyGetSetDef properties[] = {THP_FUNCTION_DEFAULT_PROPERTIES,
                                       {"saved_tensors", saved_tensors<Op>, nullptr, nullptr, nullptr},
                                       {nullptr, nullptr, nullptr, nullptr, nullptr}};
    if (!_initFunctionPyTypeObject(type, name, properties, nullptr)) throw py::error_already_set();
    registerCppFunction(typeid(CppNode<Op>), &type);
}

}  // namespace

PYBIND11_MODULE(TORCH_EXTENSION_NAME, m) {
    m.doc() = "Host path of the lnmod operators; every function returns None for a call it leaves to the Python path.";
    m.attr("built_for") = TORCH_VERSION;
    register_node<LnModulate>("LnModulateBackward");
    register_node<GatedLnModulate>("GatedLnModulateBackward");
    register_node<QkNorm>("QkNormBackward");
    m.def("forward", &forward);
    m.def("ln_modulate", &ln_modulate);
    m.def("gated_ln_modulate", &gated_ln_modulate);
    m.def("qk_norm", &qk_norm);
}
