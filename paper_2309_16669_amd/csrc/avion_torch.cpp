// The autograd front end's calls as native functions: what paper_2309_16669_amd/autograd.py does in
// Python for every call -- checks, allocations, one entry point of the C ABI, the autograd node -- without
// the interpreter.  A forward and backward pass of layer_norm spent 140 us there (the kernels take 86), a
// caption's forward 18 us (kernel 6); the node's backward also no longer takes the interpreter lock on
// autograd's thread.  Nothing is computed here.
//
// Each function takes plain calls only (see `plain`): exact torch tensors on the GPU in the expected
// formats and shapes, with no transform, mode, tracer or tangent in force.  For anything else it returns
// None, and the caller goes through the Python classes, which raise or behave as they always did.  Errors
// of the library are raised as the binding's AvionError.
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>
#include <torch/csrc/utils/pybind.h>
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>

#include "avion_attn.h"

namespace {

using at::Tensor;
using torch::autograd::AutogradContext;
using torch::autograd::variable_list;

void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

// AvionError of the binding, also from autograd's own threads
void check(int rc)
{
    if (rc == AVION_OK) return;
    pybind11::gil_scoped_acquire gil;
    try {
        pybind11::module_::import("paper_2309_16669_amd").attr("_check")(rc);
    } catch (pybind11::error_already_set& e) {
        e.restore();
    }
    python_error err;
    err.persist();
    throw err;
}

unsigned format_flag(const Tensor& t) { return t.scalar_type() == at::kHalf ? AVION_FLAG_F16 : 0u; }
bool element_format(const Tensor& t) { return t.scalar_type() == at::kHalf || t.scalar_type() == at::kBFloat16; }

// nothing that would have to see or replace the tensors' operations is in force on this thread
bool plain_thread()
{
    return !c10::impl::TorchDispatchModeTLS::any_modes_set() && !at::impl::torch_function_mode_enabled() &&
           !torch::jit::tracer::isTracing() &&
           !c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::FuncTorchDynamicLayerFrontMode);
}

// an exact torch.Tensor or Parameter with data on the GPU, without a tangent
bool plain(PyObject* obj, const Tensor** out)
{
    if (!THPVariable_CheckExact(obj)) return false;
    const Tensor& t = THPVariable_Unpack(obj);
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || t.is_conj() || t.is_neg() || t.numel() == 0 ||
        t._fw_grad(0).defined())
        return false;
    *out = &t;
    return true;
}
bool parameter(PyObject* obj, int64_t width, const Tensor& like, const Tensor** out)
{
    return plain(obj, out) && (*out)->scalar_type() == at::kFloat && (*out)->dim() == 1 && (*out)->size(0) == width &&
           (*out)->device() == like.device();
}

// The binding's checks (`_require`) before an address is taken.  A saved tensor is whatever the unpack hook of
// torch.autograd.graph.saved_tensors_hooks returned: other strides, another format, on the host, shorter.  The
// incoming gradient has the shape, format and device of the forward's output (autograd checks that).
void require(const Tensor& t, const char* name, at::IntArrayRef shape, at::ScalarType dtype, const Tensor& grad)
{
    TORCH_CHECK_VALUE(t.defined() && t.layout() == at::kStrided && t.is_cuda() && t.device() == grad.device(), name,
                      " must live on the GPU of the gradient");
    TORCH_CHECK_VALUE(t.scalar_type() == dtype, name, " must be ", dtype, ", got ", t.scalar_type());
    TORCH_CHECK_VALUE(t.is_contiguous(), name, " must be contiguous");
    TORCH_CHECK_VALUE(t.sizes() == shape, name, " must have shape ", shape, ", got ", t.sizes());
}

// Runs a call without the interpreter lock, as torch's own functions and ctypes do: an allocation that goes to the
// driver or a launch that waits for room in the queue stops this thread only.  The caller's frame holds the arguments.
template <typename F>
pybind11::object without_lock(F call)
{
    Tensor out;
    {
        pybind11::gil_scoped_release release;
        out = call();
    }
    return pybind11::cast(out);
}

// whether a node has to be recorded; without one a call is its allocations and its launch (a caption's forward
// 7.5 -> 6.7 us, of which the kernel runs 5.5)
bool records(std::initializer_list<const Tensor*> inputs)
{
    if (!at::GradMode::is_enabled()) return false;
    for (const Tensor* t : inputs)
        if (t->requires_grad()) return true;
    return false;
}

Tensor workspace(size_t bytes, const Tensor& like) { return at::empty({(int64_t)bytes}, like.options().dtype(at::kByte)); }

// ------------------------------------------------------------------------------------- attention
struct Shape {
    int B, H, N, d;
};
Shape shape_of(const Tensor& q, bool packed)
{
    return {(int)q.size(0), (int)q.size(packed ? 3 : 2), (int)q.size(1), (int)q.size(packed ? 4 : 3)};
}
bool fits_int(const Tensor& t)
{
    for (int64_t s : t.sizes())
        if (s > INT32_MAX) return false;
    return true;
}

// o and lse of one forward; k and v are undefined for a packed q
void attention_fwd(const Tensor& q, const Tensor& k, const Tensor& v, Tensor& o, Tensor& lse, double scale, bool causal)
{
    const bool packed = !k.defined();
    const Shape s = shape_of(q, packed);
    o = at::empty({s.B, s.N, s.H, s.d}, q.options());
    lse = at::empty({s.B, s.H, s.N}, q.options().dtype(at::kFloat));
    const unsigned flags = format_flag(q) | (causal ? AVION_FLAG_CAUSAL : 0u) | (packed ? AVION_FLAG_QKVPACKED : 0u);
    check(avion_attn_fwd_ex(q.data_ptr(), packed ? nullptr : k.data_ptr(), packed ? nullptr : v.data_ptr(), o.data_ptr(),
                            lse.data_ptr<float>(), s.B, s.H, s.N, s.d, (float)scale, flags, stream()));
}
// gradients of q, k, v (of q alone when it is packed)
variable_list attention_bwd(const Tensor& q, const Tensor& k, const Tensor& v, const Tensor& o, const Tensor& lse,
                            const Tensor& grad, double scale, bool causal)
{
    const bool packed = !k.defined();
    const Tensor dO = grad.contiguous();
    const Shape s = shape_of(dO, false);
    const at::ScalarType dt = dO.scalar_type();
    if (packed) {
        require(q, "qkv", {s.B, s.N, 3, s.H, s.d}, dt, dO);
    } else {
        require(q, "q", dO.sizes(), dt, dO);
        require(k, "k", dO.sizes(), dt, dO);
        require(v, "v", dO.sizes(), dt, dO);
    }
    require(o, "o", dO.sizes(), dt, dO);
    require(lse, "lse", {s.B, s.H, s.N}, at::kFloat, dO);
    variable_list g{at::empty_like(q)};
    if (!packed) {
        g.push_back(at::empty_like(k));
        g.push_back(at::empty_like(v));
    }
    const size_t need = avion_attn_bwd_workspace_bytes(s.B, s.H, s.N, s.d);
    const Tensor ws = workspace(need, q);
    const unsigned flags = format_flag(q) | (causal ? AVION_FLAG_CAUSAL : 0u) | (packed ? AVION_FLAG_QKVPACKED : 0u);
    check(avion_attn_bwd_ex(q.data_ptr(), packed ? nullptr : k.data_ptr(), packed ? nullptr : v.data_ptr(), o.data_ptr(),
                            lse.data_ptr<float>(), dO.data_ptr(), g[0].data_ptr(), packed ? nullptr : g[1].data_ptr(),
                            packed ? nullptr : g[2].data_ptr(), s.B, s.H, s.N, s.d, (float)scale, flags, ws.data_ptr(), need,
                            stream()));
    return g;
}

struct Attention : torch::autograd::Function<Attention> {
    static Tensor forward(AutogradContext* ctx, const Tensor& q_, const Tensor& k_, const Tensor& v_, double scale, bool causal)
    {
        const Tensor q = q_.contiguous(), k = k_.contiguous(), v = v_.contiguous();
        Tensor o, lse;
        attention_fwd(q, k, v, o, lse, scale, causal);
        ctx->save_for_backward({q, k, v, o, lse});
        ctx->saved_data["scale"] = scale;
        ctx->saved_data["causal"] = causal;
        return o;
    }
    static variable_list backward(AutogradContext* ctx, variable_list grad)
    {
        const variable_list s = ctx->get_saved_variables();
        variable_list g = attention_bwd(s[0], s[1], s[2], s[3], s[4], grad[0], ctx->saved_data["scale"].toDouble(),
                                        ctx->saved_data["causal"].toBool());
        g.resize(5);
        return g;
    }
};
struct AttentionPacked : torch::autograd::Function<AttentionPacked> {
    static Tensor forward(AutogradContext* ctx, const Tensor& qkv_, double scale, bool causal)
    {
        const Tensor qkv = qkv_.contiguous();
        Tensor o, lse;
        attention_fwd(qkv, Tensor(), Tensor(), o, lse, scale, causal);
        ctx->save_for_backward({qkv, o, lse});
        ctx->saved_data["scale"] = scale;
        ctx->saved_data["causal"] = causal;
        return o;
    }
    static variable_list backward(AutogradContext* ctx, variable_list grad)
    {
        const variable_list s = ctx->get_saved_variables();
        variable_list g = attention_bwd(s[0], Tensor(), Tensor(), s[1], s[2], grad[0], ctx->saved_data["scale"].toDouble(),
                                        ctx->saved_data["causal"].toBool());
        g.resize(3);
        return g;
    }
};

pybind11::object attention(pybind11::handle q_, pybind11::handle k_, pybind11::handle v_, double scale, bool causal)
{
    HANDLE_TH_ERRORS
    const Tensor *q, *k, *v;
    if (!plain(q_.ptr(), &q) || !plain(k_.ptr(), &k) || !plain(v_.ptr(), &v) || !plain_thread()) return pybind11::none();
    if (q->dim() != 4 || !element_format(*q) || !fits_int(*q)) return pybind11::none();
    for (const Tensor* t : {k, v})
        if (t->scalar_type() != q->scalar_type() || t->sizes() != q->sizes() || t->device() != q->device()) return pybind11::none();
    return without_lock([&] {
        if (records({q, k, v})) return Attention::apply(*q, *k, *v, scale, causal);
        Tensor o, lse;
        attention_fwd(q->contiguous(), k->contiguous(), v->contiguous(), o, lse, scale, causal);
        return o;
    });
    END_HANDLE_TH_ERRORS_PYBIND
}
pybind11::object attention_qkvpacked(pybind11::handle qkv_, double scale, bool causal)
{
    HANDLE_TH_ERRORS
    const Tensor* qkv;
    if (!plain(qkv_.ptr(), &qkv) || !plain_thread()) return pybind11::none();
    if (qkv->dim() != 5 || qkv->size(2) != 3 || !element_format(*qkv) || !fits_int(*qkv)) return pybind11::none();
    return without_lock([&] {
        if (records({qkv})) return AttentionPacked::apply(*qkv, scale, causal);
        Tensor o, lse;
        attention_fwd(qkv->contiguous(), Tensor(), Tensor(), o, lse, scale, causal);
        return o;
    });
    END_HANDLE_TH_ERRORS_PYBIND
}

// -------------------------------------------------------------------------- layer normalisation
struct LayerNorm : torch::autograd::Function<LayerNorm> {
    static Tensor forward(AutogradContext* ctx, const Tensor& x_, const Tensor& gamma, const Tensor& beta, double eps)
    {
        const int64_t D = x_.size(-1);
        const Tensor x = x_.contiguous().view({-1, D});
        const int64_t M = x.size(0);
        const Tensor y = at::empty(x_.sizes(), x.options());
        const Tensor mean = at::empty({M}, gamma.options()), rstd = at::empty({M}, gamma.options());
        check(avion_layernorm_fwd(x.data_ptr(), gamma.contiguous().data_ptr<float>(), beta.contiguous().data_ptr<float>(),
                                  y.data_ptr(), mean.data_ptr<float>(), rstd.data_ptr<float>(), M, (int)D, (float)eps,
                                  format_flag(x), stream()));
        ctx->save_for_backward({x, gamma, mean, rstd});  // the input and two floats per token; not y
        ctx->saved_data["shape"] = x_.sizes().vec();
        return y;
    }
    static variable_list backward(AutogradContext* ctx, variable_list grad)
    {
        const variable_list s = ctx->get_saved_variables();
        const Tensor &x = s[0], gamma = s[1].contiguous(), dy = grad[0].contiguous();
        const int64_t D = dy.size(-1), M = dy.numel() / D;
        require(x, "x", {M, D}, dy.scalar_type(), dy);
        require(gamma, "gamma", {D}, at::kFloat, dy);
        require(s[2], "mean", {M}, at::kFloat, dy);
        require(s[3], "rstd", {M}, at::kFloat, dy);
        const Tensor dx = at::empty_like(x), dgamma = at::empty_like(gamma), dbeta = at::empty_like(gamma);
        const size_t need = avion_layernorm_bwd_workspace_bytes(M, (int)D);
        const Tensor ws = workspace(need, x);
        check(avion_layernorm_bwd(x.data_ptr(), gamma.data_ptr<float>(), s[2].data_ptr<float>(), s[3].data_ptr<float>(),
                                  dy.data_ptr(), dx.data_ptr(), dgamma.data_ptr<float>(), dbeta.data_ptr<float>(), M, (int)D,
                                  format_flag(x), ws.data_ptr(), need, stream()));
        return {dx.view(ctx->saved_data["shape"].toIntVector()), dgamma, dbeta, Tensor()};
    }
};
pybind11::object layer_norm(pybind11::handle x_, pybind11::handle gamma_, pybind11::handle beta_, double eps)
{
    HANDLE_TH_ERRORS
    const Tensor *x, *gamma, *beta;
    if (!plain(x_.ptr(), &x) || !plain_thread()) return pybind11::none();
    if (x->dim() < 1 || !element_format(*x) || x->size(-1) > INT32_MAX) return pybind11::none();
    if (!parameter(gamma_.ptr(), x->size(-1), *x, &gamma) || !parameter(beta_.ptr(), x->size(-1), *x, &beta))
        return pybind11::none();
    return without_lock([&] { return LayerNorm::apply(*x, *gamma, *beta, eps); });
    END_HANDLE_TH_ERRORS_PYBIND
}

// ---------------------------------------------------------------------------------- bias + GELU
Tensor gelu_fwd(const Tensor& x, const Tensor& bias, at::IntArrayRef shape)
{
    const Tensor y = at::empty(shape, x.options());
    check(avion_bias_gelu_fwd(x.data_ptr(), bias.contiguous().data_ptr<float>(), y.data_ptr(), x.size(0), (int)x.size(1),
                              format_flag(x), stream()));
    return y;
}
void gelu_bwd(const Tensor& x, const Tensor& bias_, const Tensor& dy, Tensor& dx, Tensor& dbias)
{
    const Tensor bias = bias_.contiguous();
    dx = at::empty_like(x);
    dbias = at::empty_like(bias);
    const size_t need = avion_bias_gelu_bwd_workspace_bytes(x.size(0), (int)x.size(1));
    const Tensor ws = workspace(need, x);
    check(avion_bias_gelu_bwd(x.data_ptr(), bias.data_ptr<float>(), dy.data_ptr(), dx.data_ptr(), dbias.data_ptr<float>(),
                              x.size(0), (int)x.size(1), format_flag(x), ws.data_ptr(), need, stream()));
}

// d.sum(0); torch's where the rows are no multiple of 16 bytes, and where the sum is to be differentiated itself
// (create_graph, a tangent): it is linear in d
Tensor column_sum(const Tensor& d)
{
    const int64_t M = d.size(0), F = d.size(1);
    const size_t need = F <= INT32_MAX ? avion_column_sum_workspace_bytes(M, (int)F) : 0;
    if (need == 0 || !element_format(d) || reinterpret_cast<uintptr_t>(d.data_ptr()) % 16 != 0 || records({&d}) ||
        d._fw_grad(0).defined())
        return d.sum(0);
    const Tensor sum = at::empty({F}, d.options());
    check(avion_column_sum(d.data_ptr(), sum.data_ptr(), M, (int)F, format_flag(d), workspace(need, d).data_ptr(), need, stream()));
    return sum;
}

struct BiasGelu : torch::autograd::Function<BiasGelu> {
    static Tensor forward(AutogradContext* ctx, const Tensor& x_, const Tensor& bias)
    {
        const Tensor x = x_.contiguous().view({-1, x_.size(-1)});
        const Tensor y = gelu_fwd(x, bias, x_.sizes());
        ctx->save_for_backward({x, bias});  // the pre-activation only; the derivative is rebuilt from it
        ctx->saved_data["shape"] = x_.sizes().vec();
        return y;
    }
    static variable_list backward(AutogradContext* ctx, variable_list grad)
    {
        const variable_list s = ctx->get_saved_variables();
        const Tensor dy = grad[0].contiguous();
        const int64_t F = dy.size(-1);
        require(s[0], "x", {dy.numel() / F, F}, dy.scalar_type(), dy);
        require(s[1].contiguous(), "bias", {F}, at::kFloat, dy);
        Tensor dx, dbias;
        gelu_bwd(s[0], s[1], dy, dx, dbias);
        return {dx.view(ctx->saved_data["shape"].toIntVector()), dbias};
    }
};
// linear(GELU(x + bias), weight, out_bias) that keeps x only: the activation's output is rebuilt by the
// backward pass, beside dx, for the weight gradient.  The matrix products are torch's.
struct BiasGeluLinear : torch::autograd::Function<BiasGeluLinear> {
    static Tensor forward(AutogradContext* ctx, const Tensor& x_, const Tensor& bias, const Tensor& weight,
                          const std::optional<Tensor>& out_bias)
    {
        const Tensor x = x_.contiguous().view({-1, x_.size(-1)});
        const Tensor y = gelu_fwd(x, bias, x.sizes());
        const Tensor out = out_bias ? at::addmm(*out_bias, y, weight.t()) : at::matmul(y, weight.t());
        ctx->save_for_backward({x, bias, weight});
        ctx->saved_data["shape"] = x_.sizes().vec();
        ctx->saved_data["format"] = x.scalar_type();
        ctx->saved_data["has_out_bias"] = out_bias.has_value();
        std::vector<int64_t> shape = x_.sizes().vec();
        shape.back() = weight.size(0);
        return out.view(shape);
    }
    static variable_list backward(AutogradContext* ctx, variable_list grad)
    {
        const variable_list s = ctx->get_saved_variables();
        const Tensor &x = s[0], &bias = s[1], &weight = s[2];
        const std::vector<int64_t> shape = ctx->saved_data["shape"].toIntVector();
        const int64_t F = shape.back(), M = grad[0].numel() / grad[0].size(-1);
        require(x, "x", {M, F}, ctx->saved_data["format"].toScalarType(), grad[0]);
        require(bias.contiguous(), "bias", {F}, at::kFloat, grad[0]);
        const Tensor d2 = grad[0].contiguous().view({M, weight.size(0)});
        // variable_data: the product's storage without its node (create_graph) or tangent, which are not those of the
        // gradient of x that the kernel writes into it
        const Tensor dy = at::matmul(d2, weight).variable_data();
        require(dy, "dy", {M, F}, x.scalar_type(), grad[0]);  // under autocast a product comes in autocast's format
        // the gradient of x takes dy's place; y is rebuilt beside it, not kept
        const Tensor b = bias.contiguous(), y = at::empty_like(x), dbias = at::empty_like(b);
        const size_t need = avion_bias_gelu_bwd_workspace_bytes(M, (int)F);
        check(avion_bias_gelu_bwd_y(x.data_ptr(), b.data_ptr<float>(), dy.data_ptr(), dy.data_ptr(), y.data_ptr(),
                                    dbias.data_ptr<float>(), M, (int)F, format_flag(x), workspace(need, x).data_ptr(), need, stream()));
        return {dy.view(shape), dbias, at::matmul(d2.t(), y),
                ctx->saved_data["has_out_bias"].toBool() ? column_sum(d2) : Tensor()};
    }
};
bool gelu_args(pybind11::handle x_, pybind11::handle bias_, const Tensor** x, const Tensor** bias)
{
    return plain(x_.ptr(), x) && plain_thread() && (*x)->dim() >= 1 && element_format(**x) && (*x)->size(-1) <= INT32_MAX &&
           parameter(bias_.ptr(), (*x)->size(-1), **x, bias);
}
pybind11::object bias_gelu(pybind11::handle x_, pybind11::handle bias_)
{
    HANDLE_TH_ERRORS
    const Tensor *x, *bias;
    if (!gelu_args(x_, bias_, &x, &bias)) return pybind11::none();
    return without_lock([&] { return BiasGelu::apply(*x, *bias); });
    END_HANDLE_TH_ERRORS_PYBIND
}
pybind11::object bias_gelu_linear(pybind11::handle x_, pybind11::handle bias_, pybind11::handle weight_, pybind11::handle out_)
{
    HANDLE_TH_ERRORS
    const Tensor *x, *bias, *weight, *out = nullptr;
    if (!gelu_args(x_, bias_, &x, &bias) || !plain(weight_.ptr(), &weight)) return pybind11::none();
    if (weight->dim() != 2 || weight->size(1) != x->size(-1) || weight->scalar_type() != x->scalar_type() ||
        weight->device() != x->device())
        return pybind11::none();
    if (!out_.is_none()) {
        if (!plain(out_.ptr(), &out) || out->dim() != 1 || out->size(0) != weight->size(0) ||
            out->scalar_type() != x->scalar_type() || out->device() != x->device())
            return pybind11::none();
    }
    return without_lock([&] { return BiasGeluLinear::apply(*x, *bias, *weight, out ? std::optional<Tensor>(*out) : std::nullopt); });
    END_HANDLE_TH_ERRORS_PYBIND
}

}  // namespace

PYBIND11_MODULE(_avion_torch, m)
{
    m.doc() = "native calls of the autograd front end (csrc/avion_torch.cpp); each returns None for a call it does not take";
    m.def("attention", &attention);
    m.def("attention_qkvpacked", &attention_qkvpacked);
    m.def("layer_norm", &layer_norm);
    m.def("bias_gelu", &bias_gelu);
    m.def("bias_gelu_linear", &bias_gelu_linear);
}
