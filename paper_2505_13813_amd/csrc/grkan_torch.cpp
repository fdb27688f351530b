// Native autograd route of the PyTorch front end: the group-wise rational function and the layer's product
// as C++ autograd functions over the C ABI (include/grkan.h).  What runs on the device is the same as through
// the Python functions; what goes is the host time around it (argument marshalling, and small kernels that
// expand, convert and sum the coefficients of a model).
//
// Every entry returns "not taken" (an empty optional) for anything but plain dense tensors (no subclass) on the
// current GPU outside of tracing, function transforms, forward-mode differentiation, dispatch modes and function
// modes; the caller then takes the Python route, which handles or refuses the call as it always did.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>
#include <torch/csrc/utils/pybind.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>

#include <algorithm>
#include <exception>
#include <initializer_list>
#include <optional>
#include <tuple>
#include <vector>

#include "../../include/grkan.h"

namespace {

using at::Tensor;
using torch::autograd::AutogradContext;
using torch::autograd::variable_list;

constexpr c10::DispatchKeySet kNotPlain({
    c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot, c10::DispatchKey::FuncTorchBatched,
    c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::FuncTorchVmapMode, c10::DispatchKey::Batched,
    c10::DispatchKey::Functionalize, c10::DispatchKey::Negative, c10::DispatchKey::Conjugate,
    c10::DispatchKey::ZeroTensor});

bool plain(const Tensor &t, const c10::Device &dev)
{
    return t.defined() && t.device() == dev && t.layout() == at::kStrided && !t.key_set().has_any(kNotPlain) &&
           !t._fw_grad(0).defined();
}

bool plain_context()
{
    return !torch::jit::tracer::isTracing() && !c10::impl::TorchDispatchModeTLS::any_modes_set() &&
           !c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::FuncTorchDynamicLayerFrontMode);
}

bool on_current_gpu(const Tensor &t) { return t.is_cuda() && t.get_device() == c10::hip::current_device(); }

void *stream_of(const Tensor &t) { return c10::hip::getCurrentHIPStream(t.get_device()).stream(); }

std::optional<grkan_dtype_t> io_of(const Tensor &t)
{
    switch (t.scalar_type()) {
    case at::kFloat: return GRKAN_F32;
    case at::kBFloat16: return GRKAN_BF16;
    case at::kHalf: return GRKAN_F16;
    default: return std::nullopt;
    }
}

// A status of the library as the exception the Python functions raise for it.
void check(grkan_status_t st, const char *where)
{
    if (st == GRKAN_OK)
        return;
    pybind11::gil_scoped_acquire gil;
    const pybind11::object type = pybind11::module_::import("paper_2505_13813_amd.binding").attr("GrkanError");
    PyErr_SetObject(type.ptr(), type((int)st, where).ptr());
    python_error error;
    error.persist(); // (in the backward pass it crosses threads)
    throw error;
}

// A workspace from torch's allocator (its streams and lifetimes), handed out during one call of the C ABI.
struct Scratch {
    at::TensorOptions options;
    Tensor memory;
    std::exception_ptr error;

    static void *alloc(size_t bytes, void *self) noexcept
    {
        auto *s = static_cast<Scratch *>(self);
        try {
            s->memory = at::empty({(int64_t)bytes}, s->options);
            return s->memory.data_ptr();
        } catch (...) {
            s->error = std::current_exception();
            return nullptr;
        }
    }
    void rethrow() const
    {
        if (error)
            std::rethrow_exception(error);
    }
};

// Several of them.
struct Scratches {
    at::TensorOptions options;
    std::vector<Tensor> memory;
    std::exception_ptr error;

    static void *alloc(size_t bytes, void *self) noexcept
    {
        auto *s = static_cast<Scratches *>(self);
        try {
            s->memory.push_back(at::empty({(int64_t)bytes}, s->options));
            return s->memory.back().data_ptr();
        } catch (...) {
            s->error = std::current_exception();
            return nullptr;
        }
    }
};

struct Sizes {
    int64_t rows;
    int32_t D, G, m, n;
    bool shared;
};

Sizes sizes_of(const Tensor &x, const Tensor &A, const Tensor &B)
{
    const int64_t D = x.size(-1);
    return Sizes{x.numel() / D, (int32_t)D, (int32_t)B.size(0), (int32_t)A.size(-1) - 1, (int32_t)B.size(1), A.dim() == 1};
}

// The operands of a backward pass as they come back from saved-tensor hooks, which may return anything: what the
// Python function checks in front of the kernels.
void check_saved(const Tensor &x, const Tensor &dy, const Tensor &A, const Tensor &B)
{
    TORCH_CHECK_VALUE(x.is_cuda() && A.device() == x.device() && B.device() == x.device(),
                      "grkan runs on the GPU only: tensors must be on one HIP device");
    TORCH_CHECK_VALUE(x.is_contiguous() && A.is_contiguous() && B.is_contiguous(), "tensors must be contiguous");
    TORCH_CHECK_TYPE(A.scalar_type() == B.scalar_type() &&
                         (A.scalar_type() == at::kFloat || (A.scalar_type() == at::kBFloat16 && x.scalar_type() == at::kBFloat16)),
                     "A and B must be float32");
    TORCH_CHECK_VALUE(B.dim() == 2 && (A.dim() == 1 || (A.dim() == 2 && A.size(0) == B.size(0))), "A must be [G, m+1] and B [G, n]");
    TORCH_CHECK_VALUE(dy.sizes() == x.sizes() && dy.scalar_type() == x.scalar_type() && dy.device() == x.device(),
                      "dy must match x");
}

// Gradients of a backward pass that was asked for a graph of itself and has none: differentiating them with respect to
// what they depend on is an error instead of leaving it out.
struct Undifferentiable : public torch::autograd::Function<Undifferentiable> {
    static variable_list forward(AutogradContext *, const Tensor &dx, const Tensor &dA, const Tensor &dB, const Tensor &,
                                 const Tensor &, const Tensor &, const Tensor &)
    {
        return {dx.view_as(dx), dA.view_as(dA), dB.view_as(dB)};
    }
    static variable_list backward(AutogradContext *, const variable_list &)
    {
        TORCH_CHECK(false, "the group-wise rational function is not differentiable twice");
    }
};

// y = F(x); A [G, m+1] or, shared by the groups, [m+1]; all contiguous.  (A copy made in here would have no history: a second
// derivative with respect to what it was made of would not reach Undifferentiable.)  `known`: y, where it is there already and
// only its history is wanted.
struct Rational : public torch::autograd::Function<Rational> {
    static Tensor forward(AutogradContext *ctx, const Tensor &x, const Tensor &A, const Tensor &B, const std::optional<Tensor> &known)
    {
        ctx->save_for_backward({x, A, B});
        if (known)
            return known->view_as(*known);
        const Sizes s = sizes_of(x, A, B);
        Tensor y = at::empty_like(x, at::MemoryFormat::Contiguous);
        check(grkan_fwd_model(x.data_ptr(), A.data_ptr(), B.data_ptr(), y.data_ptr(), s.rows, s.D, s.G, s.m, s.n, *io_of(x),
                              *io_of(A), s.shared, stream_of(x)),
              "grkan_fwd");
        return y;
    }

    static variable_list backward(AutogradContext *ctx, const variable_list &grads)
    {
        const auto saved = ctx->get_saved_variables();
        const Tensor &x = saved[0], &A = saved[1], &B = saved[2];
        if (!grads[0].defined())
            return variable_list(4);
        variable_list out = in_backward(x, grads[0].contiguous(), A, B);
        out.resize(4); // (none for `known`)
        return out;
    }

    // {dx, dA, dB} inside a backward pass; where a graph of it is wanted, behind Undifferentiable.
    static variable_list in_backward(const Tensor &x, const Tensor &dy, const Tensor &A, const Tensor &B)
    {
        const bool graph_wanted = at::GradMode::is_enabled();
        Tensor dx, dA, dB;
        {
            at::AutoGradMode no_grad(false);
            std::tie(dx, dA, dB) = gradients(x, dy, A, B);
        }
        return graph_wanted ? Undifferentiable::apply(dx, dA, dB, x, A, B, dy) : variable_list{dx, dA, dB};
    }

    static std::tuple<Tensor, Tensor, Tensor> gradients(const Tensor &x, const Tensor &dy, const Tensor &A, const Tensor &B)
    {
        check_saved(x, dy, A, B);
        const Sizes s = sizes_of(x, A, B);
        Tensor dx = at::empty_like(x), dA = at::empty_like(A), dB = at::empty_like(B);
        Scratch scratch{x.options().dtype(at::kByte), Tensor(), nullptr};
        const grkan_status_t st =
            grkan_bwd_model(x.data_ptr(), dy.data_ptr(), A.data_ptr(), B.data_ptr(), dx.data_ptr(), dA.data_ptr(), dB.data_ptr(),
                            &Scratch::alloc, &scratch, s.rows, s.D, s.G, s.m, s.n, *io_of(x), *io_of(A), s.shared, stream_of(x));
        scratch.rethrow();
        check(st, "grkan_bwd");
        return {dx, dA, dB};
    }
};

// dW [D_out, D_in] and, where wanted, dbias [D_out] of out = y W^T + bias from the bfloat16 kernel, if it takes them.
bool weight_gradients(Tensor dout2, Tensor y2, bool want_b, Tensor &dW, Tensor &db)
{
    dout2 = dout2.contiguous();
    y2 = y2.contiguous();
    const int64_t D_in = y2.size(1), D_out = dout2.size(1);
    const size_t need = grkan_linear_wgrad_workspace_bytes(dout2.size(0), (int32_t)D_in, (int32_t)D_out);
    if (need == 0 || reinterpret_cast<uintptr_t>(dout2.data_ptr()) % 16 != 0 || reinterpret_cast<uintptr_t>(y2.data_ptr()) % 16 != 0)
        return false;
    const Tensor ws = at::empty({(int64_t)need}, dout2.options().dtype(at::kByte));
    dW = at::empty({D_out, D_in}, dout2.options());
    if (want_b)
        db = at::empty({D_out}, dout2.options());
    check(grkan_linear_wgrad(dout2.data_ptr(), y2.data_ptr(), dW.data_ptr(), want_b ? db.data_ptr() : nullptr, ws.data_ptr(), need,
                             dout2.size(0), (int32_t)D_in, (int32_t)D_out, GRKAN_BF16, stream_of(dout2)),
          "grkan_linear_wgrad");
    return true;
}

// The same of two products over the same rows (contiguous, 16-byte aligned) in one launch.
bool both_weight_gradients(const Tensor &dout1, const Tensor &y1, bool want_b1, Tensor &dW1, Tensor &db1, const Tensor &dout2, const Tensor &y2,
                           bool want_b2, Tensor &dW2, Tensor &db2)
{
    const int64_t rows = y1.size(0), in1 = y1.size(1), out1 = dout1.size(1), in2 = y2.size(1), out2 = dout2.size(1);
    const size_t need = grkan_linear_wgrad_pair_workspace_bytes(rows, (int32_t)in1, (int32_t)out1, (int32_t)in2, (int32_t)out2);
    if (need == 0)
        return false;
    const Tensor ws = at::empty({(int64_t)need}, y1.options().dtype(at::kByte));
    dW1 = at::empty({out1, in1}, y1.options());
    dW2 = at::empty({out2, in2}, y1.options());
    if (want_b1)
        db1 = at::empty({out1}, y1.options());
    if (want_b2)
        db2 = at::empty({out2}, y1.options());
    check(grkan_linear_wgrad_pair(dout1.data_ptr(), y1.data_ptr(), dW1.data_ptr(), want_b1 ? db1.data_ptr() : nullptr, (int32_t)in1,
                                  (int32_t)out1, dout2.data_ptr(), y2.data_ptr(), dW2.data_ptr(), want_b2 ? db2.data_ptr() : nullptr,
                                  (int32_t)in2, (int32_t)out2, ws.data_ptr(), need, rows, stream_of(y1)),
          "grkan_linear_wgrad_pair");
    return true;
}

// torch's linear.  The result is no view of another tensor: torch refuses to write (y += x) to an output of an autograd
// function that is one.
Tensor linear_of_rows(const Tensor &y, const Tensor &W, const std::optional<Tensor> &bias)
{
    if (y.dim() <= 2 || y.numel() == 0)
        return at::linear(y, W, bias);
    auto shape = y.sizes().vec();
    shape.back() = W.size(0);
    return at::_unsafe_view(at::linear(y.reshape({-1, y.size(-1)}), W, bias), shape);
}

// out = y W^T + bias with dW and dbias from grkan_linear_wgrad; saves what torch's linear saves: each operand where
// the gradient of the other is wanted.  `known`: out, as for Rational.  (The products are torch's: grkan_product was measured in
// whole blocks and in inference, not in a layer's training.)
struct Product : public torch::autograd::Function<Product> {
    static Tensor forward(AutogradContext *ctx, const Tensor &y, const Tensor &W, const std::optional<Tensor> &bias,
                          const std::optional<Tensor> &known)
    {
        ctx->save_for_backward({W.requires_grad() ? y : Tensor(), y.requires_grad() ? W : Tensor()});
        ctx->saved_data["has_bias"] = bias.has_value();
        if (known)
            return known->view_as(*known);
        return linear_of_rows(y, W, bias);
    }

    static variable_list backward(AutogradContext *ctx, const variable_list &grads)
    {
        const auto saved = ctx->get_saved_variables();
        const Tensor &y = saved[0], &W = saved[1];
        const Tensor &dout = grads[0];
        if (!dout.defined())
            return variable_list(4);
        const bool want_y = ctx->needs_input_grad(0), want_w = ctx->needs_input_grad(1);
        const bool want_b = ctx->saved_data["has_bias"].toBool() && ctx->needs_input_grad(2);
        const int64_t D_out = dout.size(-1);
        Tensor dout2 = dout.reshape({-1, D_out}), y2, dy, dW, db;
        if (want_y) {
            auto shape = dout.sizes().vec();
            shape.back() = W.size(1);
            dy = dout2.mm(W).view(shape);
        }
        if (want_w)
            y2 = y.reshape({-1, y.size(-1)});
        // With a graph of the backward pass wanted, operations that torch can differentiate; and what a saved-tensor
        // hook made of y is left to torch if it is not what was saved.
        if (want_w && !at::GradMode::is_enabled() && dout2.is_cuda() && plain(dout2, dout2.device()) &&
            plain(y2, dout2.device()) && dout2.scalar_type() == at::kBFloat16 && y2.scalar_type() == at::kBFloat16 &&
            y2.size(0) == dout2.size(0))
            weight_gradients(dout2, y2, want_b, dW, db);
        if (want_w && !dW.defined())
            dW = dout2.t().mm(y2);
        if (want_b && !db.defined())
            db = dout2.sum(0);
        return {dy, dW, db, Tensor()};
    }
};

bool aligned(const Tensor &t, uintptr_t to) { return reinterpret_cast<uintptr_t>(t.data_ptr()) % to == 0; }

// x W^T + bias or, transposed, x W of bfloat16 rows (contiguous, as W) from the kernel where it takes them, from torch elsewhere.
Tensor product_of_rows(const Tensor &x, const Tensor &W, const std::optional<Tensor> &bias, bool transposed)
{
    const int64_t rows = x.size(0), K = x.size(1), N = W.size(transposed ? 1 : 0);
    if (K > INT32_MAX || N > INT32_MAX || !grkan_product_supported(rows, (int32_t)K, (int32_t)N) || !aligned(x, 16) || !aligned(W, 16) ||
        (bias && !aligned(*bias, 8)))
        return transposed ? x.mm(W) : at::linear(x, W, bias);
    Tensor out = at::empty({rows, N}, x.options());
    check(grkan_product(x.data_ptr(), W.data_ptr(), bias ? bias->data_ptr() : nullptr, out.data_ptr(), rows, (int32_t)K, (int32_t)N, transposed,
                        nullptr, nullptr, 1, 0, stream_of(x)),
          "grkan_product");
    return out;
}

// The two GR-KAN layers of an MLP block: f1 = F1(x), h = f1 W1^T + b1 and f2 = F2(h), out = f2 W2^T + b2.  Where it is the
// faster route (grkan_hidden_pays, by direction) h and f2 come from one kernel, and in the backward pass the product with W2 and
// F2's gradients, so that dF2 is never written; elsewhere from grkan_product and the rational function.  The backward pass is one
// call (grkan_block_bwd).  Saves what the layers by themselves save.  `wgrad`: whether the weight gradients take this package's
// kernel (one answer for both: the second layer's sizes are the first one's in the other order).
struct Block : public torch::autograd::Function<Block> {
    static Tensor forward(AutogradContext *ctx, const Tensor &x, const Tensor &A1, const Tensor &B1, const Tensor &W1,
                          const Tensor &A2, const Tensor &B2, const Tensor &W2, const std::optional<Tensor> &b1,
                          const std::optional<Tensor> &b2, bool wgrad)
    {
        const Sizes s1 = sizes_of(x, A1, B1);
        const int64_t hidden = W1.size(0);
        Tensor f1 = at::empty_like(x, at::MemoryFormat::Contiguous);
        check(grkan_fwd_model(x.data_ptr(), A1.data_ptr(), B1.data_ptr(), f1.data_ptr(), s1.rows, s1.D, s1.G, s1.m, s1.n, GRKAN_BF16,
                              GRKAN_BF16, s1.shared, stream_of(x)),
              "grkan_fwd");
        const int32_t G2 = (int32_t)B2.size(0);
        Tensor h, f2 = at::empty({s1.rows, hidden}, x.options());
        if (grkan_hidden_pays(s1.rows, s1.D, (int32_t)hidden, G2, 0)) {
            h = at::empty_like(f2);
            check(grkan_hidden_fwd(f1.data_ptr(), W1.data_ptr(), b1 ? b1->data_ptr() : nullptr, A2.data_ptr(), B2.data_ptr(), h.data_ptr(),
                                   f2.data_ptr(), s1.rows, s1.D, (int32_t)hidden, G2, A2.dim() == 1, stream_of(x)),
                  "grkan_hidden_fwd");
        } else {
            h = product_of_rows(f1.view({s1.rows, s1.D}), W1, b1, false);
            check(grkan_fwd_model(h.data_ptr(), A2.data_ptr(), B2.data_ptr(), f2.data_ptr(), s1.rows, (int32_t)hidden, G2, 5, 4,
                                  GRKAN_BF16, GRKAN_BF16, A2.dim() == 1, stream_of(x)),
                  "grkan_fwd");
        }
        // (the biases' values are not read again: they may be written to before the backward pass)
        ctx->save_for_backward({x, A1, B1, W1, A2, B2, W2, f1, h, f2});
        if (b1)
            ctx->saved_data["b1"] = *b1;
        ctx->saved_data["biases"] = (int64_t)(b1 ? 1 : 0) + (b2 ? 2 : 0);
        ctx->saved_data["wgrad"] = wgrad;
        return at::_unsafe_view(product_of_rows(f2, W2, b2, false), x.sizes());
    }

    // A saved tensor as its hooks returned it, in the form the kernels read.
    static Tensor as_saved(const Tensor &t, const Tensor &like, at::IntArrayRef sizes)
    {
        TORCH_CHECK_VALUE(plain(t, like.device()) && t.is_cuda(), "grkan runs on the GPU only: tensors must be on one HIP device");
        TORCH_CHECK_TYPE(t.scalar_type() == at::kBFloat16, "saved tensors must be bfloat16");
        TORCH_CHECK_VALUE(t.sizes() == sizes && t.numel() > 0, "a saved tensor has another shape");
        const Tensor c = t.contiguous();
        return reinterpret_cast<uintptr_t>(c.data_ptr()) % 16 == 0 ? c : c.clone();
    }

    static variable_list backward(AutogradContext *ctx, const variable_list &grads)
    {
        const auto saved = ctx->get_saved_variables();
        variable_list out(10);
        if (!grads[0].defined())
            return out;
        const int64_t biases = ctx->saved_data["biases"].toInt();
        const bool wgrad = ctx->saved_data["wgrad"].toBool();
        const bool has1 = (biases & 1) != 0, has2 = (biases & 2) != 0;
        const Tensor &A1 = saved[1], &B1 = saved[2], &W1 = saved[3], &A2 = saved[4], &B2 = saved[5];
        const bool want_b1 = has1 && ctx->needs_input_grad(7), want_b2 = has2 && ctx->needs_input_grad(has1 ? 8 : 7);
        const bool want_w1 = ctx->needs_input_grad(3), want_w2 = ctx->needs_input_grad(6);
        const bool want_first = ctx->needs_input_grad(0) || ctx->needs_input_grad(1) || ctx->needs_input_grad(2);
        const bool want_dh = want_first || want_w1 || want_b1 || ctx->needs_input_grad(4) || ctx->needs_input_grad(5);
        const Tensor x = as_saved(saved[0], grads[0], saved[0].sizes());
        const int64_t D = x.size(-1), rows = x.numel() / D, hidden = W1.size(0);
        const Tensor W2 = as_saved(saved[6], x, {D, hidden});
        const Tensor dout = as_saved(grads[0].reshape({rows, D}), x, {rows, D});
        Tensor f1, h, f2;
        // With a graph of this pass wanted, the activations get their history back, and every gradient is formed by operations that
        // torch differentiates, each from the one behind it.  (torch::autograd::grad of the block formed again would not stop at the
        // block's inputs: on its way to a parameter it would walk their history too, and run their hooks.)
        const bool graph = at::GradMode::is_enabled();
        f2 = as_saved(saved[9], x, {rows, hidden});
        if (graph) {
            check_saved(x, x, A1, B1);
            f1 = Rational::apply(x, A1, B1, as_saved(saved[7], x, x.sizes())).view({rows, D});
            h = as_saved(saved[8], x, {rows, hidden});
            check_saved(h, h, A2, B2);
            h = Product::apply(f1, as_saved(W1, x, {hidden, D}),
                               has1 ? std::optional<Tensor>(ctx->saved_data["b1"].toTensor()) : std::nullopt, h);
            f2 = Rational::apply(h, A2, B2, f2);
        }
        // (both layers' weight gradients in one launch where both are wanted)
        const bool pair = want_w1 && want_w2 && wgrad && !graph;
        if (pair && want_first && coefficients_of(A1, B1, x, D) && coefficients_of(A2, B2, x, hidden)) {
            const Tensor W = as_saved(W1, x, {hidden, D});
            f1 = as_saved(saved[7], x, x.sizes());
            h = as_saved(saved[8], x, {rows, hidden});
            Scratches scratch{x.options().dtype(at::kByte), {}, nullptr};
            const Tensor dh = at::empty_like(h);
            out[0] = at::empty_like(x);
            out[1] = at::empty_like(A1);
            out[2] = at::empty_like(B1);
            out[3] = at::empty({hidden, D}, x.options());
            out[4] = at::empty_like(A2);
            out[5] = at::empty_like(B2);
            out[6] = at::empty({D, hidden}, x.options());
            if (want_b1)
                out[7] = at::empty({hidden}, x.options());
            if (want_b2)
                out[8] = at::empty({D}, x.options());
            const grkan_block_bwd_t b{rows, (int32_t)D, (int32_t)hidden, (int32_t)B1.size(0), (int32_t)B2.size(0), A1.dim() == 1, A2.dim() == 1,
                                      x.data_ptr(), f1.data_ptr(), h.data_ptr(), f2.data_ptr(), dout.data_ptr(), A1.data_ptr(), B1.data_ptr(),
                                      W.data_ptr(), A2.data_ptr(), B2.data_ptr(), W2.data_ptr(), out[0].data_ptr(), out[1].data_ptr(),
                                      out[2].data_ptr(), out[3].data_ptr(), want_b1 ? out[7].data_ptr() : nullptr, out[4].data_ptr(),
                                      out[5].data_ptr(), out[6].data_ptr(), want_b2 ? out[8].data_ptr() : nullptr, dh.data_ptr()};
            const grkan_status_t st = grkan_block_bwd(&b, &Scratches::alloc, &scratch, stream_of(x));
            if (scratch.error)
                std::rethrow_exception(scratch.error);
            check(st, "grkan_block_bwd");
            return out;
        }
        if (!pair)
            gradients_of(dout, f2, want_w2, want_b2, wgrad, out[6], out[8]);
        if (!want_dh)
            return out;
        if (!graph) {
            h = as_saved(saved[8], x, {rows, hidden});
            check_saved(h, h, A2, B2);
        }
        const int32_t G = (int32_t)B2.size(0);
        Tensor dh;
        // (as the kernel reads them: a saved-tensor hook may have made float32 of them, which the rational function takes)
        if (!graph && A2.scalar_type() == at::kBFloat16 && A2.size(-1) == 6 && B2.size(1) == 4 &&
            grkan_hidden_pays(rows, (int32_t)D, (int32_t)hidden, G, 1)) {
            dh = at::empty_like(h);
            out[4] = at::empty_like(A2);
            out[5] = at::empty_like(B2);
            const size_t need = grkan_hidden_workspace_bytes(rows, (int32_t)D, (int32_t)hidden, G);
            const Tensor ws = at::empty({(int64_t)need}, x.options().dtype(at::kByte));
            check(grkan_hidden_bwd(dout.data_ptr(), W2.data_ptr(), h.data_ptr(), A2.data_ptr(), B2.data_ptr(), dh.data_ptr(),
                                   out[4].data_ptr(), out[5].data_ptr(), ws.data_ptr(), need, rows, (int32_t)D, (int32_t)hidden, G,
                                   A2.dim() == 1, stream_of(x)),
                  "grkan_hidden_bwd");
        } else {
            const variable_list d = Rational::in_backward(h, graph ? dout.mm(W2) : product_of_rows(dout, W2, std::nullopt, true), A2, B2);
            dh = d[0];
            out[4] = d[1];
            out[5] = d[2];
        }
        if (want_w1 || want_b1) {
            if (!graph)
                f1 = as_saved(saved[7], x, x.sizes()).view({rows, D});
            if (!pair || !both_weight_gradients(dh, f1, want_b1, out[3], out[7], dout, f2, want_b2, out[6], out[8])) {
                gradients_of(dh, f1, want_w1, want_b1, wgrad, out[3], out[7]);
                if (pair)
                    gradients_of(dout, f2, want_w2, want_b2, wgrad, out[6], out[8]);
            }
        }
        if (want_first) {
            const Tensor df1 = graph ? dh.mm(W1) : product_of_rows(dh, as_saved(W1, x, {hidden, D}), std::nullopt, true);
            const variable_list d = Rational::in_backward(x, df1.view(x.sizes()), A1, B1);
            std::copy(d.begin(), d.end(), out.begin());
        }
        return out;
    }

    // Coefficients as grkan_block_bwd reads them (a saved-tensor hook may have made something else of them).
    static bool coefficients_of(const Tensor &A, const Tensor &B, const Tensor &x, int64_t channels)
    {
        return plain(A, x.device()) && plain(B, x.device()) && A.scalar_type() == at::kBFloat16 && B.scalar_type() == at::kBFloat16 &&
               A.is_contiguous() && B.is_contiguous() && B.dim() == 2 && B.size(1) == 4 && B.size(0) > 0 && channels % B.size(0) == 0 &&
               A.dim() >= 1 && A.dim() <= 2 && A.size(-1) == 6 && (A.dim() == 1 || A.size(0) == B.size(0));
    }

    static void gradients_of(const Tensor &dout, const Tensor &y, bool want_w, bool want_b, bool wgrad, Tensor &dW, Tensor &db)
    {
        if (want_w && wgrad && !at::GradMode::is_enabled() && weight_gradients(dout, y, want_b, dW, db))
            return;
        if (want_w)
            dW = dout.t().mm(y);
        if (want_b)
            db = dout.sum(0);
    }
};

// Shapes and types that grkan_fwd / grkan_bwd take; anything else is left to the Python route and its errors.
std::optional<Tensor> rational(const Tensor &x, const Tensor &A, const Tensor &B)
{
    if (!plain_context() || !on_current_gpu(x) || !plain(x, x.device()) || !plain(A, x.device()) || !plain(B, x.device()))
        return std::nullopt;
    if (!io_of(x) || A.scalar_type() != B.scalar_type() ||
        (A.scalar_type() != at::kFloat &&
         !(A.scalar_type() == at::kBFloat16 && x.scalar_type() == at::kBFloat16)) ||
        x.dim() < 1 || B.dim() != 2 || A.dim() < 1 || A.dim() > 2 || (A.dim() == 2 && A.size(0) != B.size(0)))
        return std::nullopt;
    const int64_t D = x.size(-1), G = B.size(0), m = A.size(-1) - 1, n = B.size(1);
    const bool degrees = (m == 5 && n == 4) || (m == 3 && n == 2) || (m == 7 && n == 6);
    if (!degrees || G <= 0 || D <= 0 || D > INT32_MAX || D % G != 0 || x.numel() == 0)
        return std::nullopt;
    return Rational::apply(x.contiguous(), A.contiguous(), B.contiguous(), std::nullopt);
}

// The product of a bfloat16 layer in training.  (Hooks and the like on the linear module are the caller's to check.)
std::optional<Tensor> product(const Tensor &y, const Tensor &W, const std::optional<Tensor> &bias)
{
    if (!plain_context() || !on_current_gpu(y) || !plain(y, y.device()) || !plain(W, y.device()) ||
        (bias && !plain(*bias, y.device())))
        return std::nullopt;
    if (y.scalar_type() != at::kBFloat16 || W.scalar_type() != at::kBFloat16 || (bias && bias->scalar_type() != at::kBFloat16) ||
        W.dim() != 2 || y.dim() < 1 || y.size(-1) != W.size(1) || !W.is_contiguous())
        return std::nullopt;
    return Product::apply(y, W, bias, std::nullopt);
}

// The MLP block in training, with a gradient wanted for its input and every parameter.  (Hooks and the like on its
// modules are the caller's to check.  In a pass without a graph nothing tells whether one is wanted for the input.)
std::optional<Tensor> block(const Tensor &x, const Tensor &A1, const Tensor &B1, const Tensor &W1, const std::optional<Tensor> &b1,
                            const Tensor &A2, const Tensor &B2, const Tensor &W2, const std::optional<Tensor> &b2, bool wgrad)
{
    if (!plain_context() || !on_current_gpu(x))
        return std::nullopt;
    for (const Tensor *t : {&x, &A1, &B1, &W1, &A2, &B2, &W2, b1 ? &*b1 : &W1, b2 ? &*b2 : &W2})
        if (!plain(*t, x.device()) || t->scalar_type() != at::kBFloat16 || (t != &x && !t->is_contiguous()) ||
            (!t->requires_grad() && (t != &x || at::GradMode::is_enabled())))
            return std::nullopt;
    if (x.dim() < 1 || x.numel() == 0 || W1.dim() != 2 || W2.dim() != 2 || x.size(-1) != W1.size(1) || W2.size(1) != W1.size(0) ||
        W2.size(0) != W1.size(1) || (b1 && (b1->dim() != 1 || b1->size(0) != W1.size(0))) || (b2 && (b2->dim() != 1 || b2->size(0) != W2.size(0))))
        return std::nullopt;
    auto coefficients = [](const Tensor &A, const Tensor &B, int64_t channels) {
        return B.dim() == 2 && B.size(1) == 4 && A.dim() >= 1 && A.dim() <= 2 && A.size(-1) == 6 &&
               (A.dim() == 1 || A.size(0) == B.size(0)) && B.size(0) > 0 && channels % B.size(0) == 0;
    };
    const int64_t D = W1.size(1), hidden = W1.size(0);
    if (D > INT32_MAX || hidden > INT32_MAX || !coefficients(A1, B1, D) || !coefficients(A2, B2, hidden) ||
        x.numel() / D > ((int64_t)1 << 30) || !grkan_hidden_supported((int32_t)D, (int32_t)hidden, (int32_t)B2.size(0)))
        return std::nullopt;
    for (const Tensor *t : {&W1, &W2, b1 ? &*b1 : &W1})
        if (reinterpret_cast<uintptr_t>(t->data_ptr()) % 16 != 0)
            return std::nullopt;
    // (contiguous: as for Rational)
    return Block::apply(x.contiguous(), A1, B1, W1, A2, B2, W2, b1, b2, wgrad);
}

// What layer_packed reads of a layer's parameters: the packed weights, the bias, and a row of coefficients for every
// group, in float32.
std::optional<std::tuple<Tensor, std::optional<Tensor>, Tensor, Tensor>>
pack_layer(const Tensor &W_in, const std::optional<Tensor> &bias, const Tensor &A, const Tensor &B)
{
    if (!plain_context() || !on_current_gpu(W_in))
        return std::nullopt;
    for (const Tensor *t : {&W_in, &A, &B, bias ? &*bias : &W_in})
        if (!plain(*t, W_in.device()))
            return std::nullopt;
    if (W_in.scalar_type() != at::kBFloat16 || W_in.dim() != 2 || A.dim() < 1 || A.dim() > 2 || B.dim() != 2 ||
        W_in.size(0) > INT32_MAX || W_in.size(1) > INT32_MAX)
        return std::nullopt;
    at::AutoGradMode no_grad(false);
    Tensor W = W_in.detach().contiguous();
    if (reinterpret_cast<uintptr_t>(W.data_ptr()) % 16 != 0) // a view into a larger buffer
        W = W.clone();
    const int32_t D_out = (int32_t)W.size(0), D_in = (int32_t)W.size(1);
    const size_t bytes = grkan_linear_packed_w_bytes(D_in, D_out);
    if (bytes == 0)
        return std::nullopt;
    const Tensor data = at::empty({(int64_t)bytes}, W.options().dtype(at::kByte));
    check(grkan_linear_pack_w(W.data_ptr(), data.data_ptr(), D_in, D_out, stream_of(W)), "grkan_linear_pack_w");
    // copies, not views of float32 parameters, which may be written to or resized behind them
    auto float32 = [](const Tensor &t, at::IntArrayRef shape) {
        Tensor out = at::empty(shape, t.options().dtype(at::kFloat));
        return out.copy_(t.detach().expand(shape));
    };
    std::optional<Tensor> b32;
    if (bias)
        b32 = float32(*bias, bias->sizes());
    return std::make_tuple(data, b32, float32(A, {B.size(0), A.size(-1)}), float32(B, B.sizes()));
}

// The one-kernel layer on packed weights (inference): all operands as the module keeps them.  `made_on`: the stream
// (its address) the kept copies were made on, -1 for copies that this call may read wherever it runs; on another stream,
// and under capture, the caller has something to do first and the call is not taken.
std::optional<Tensor> layer_packed(const Tensor &x_in, const Tensor &A, const Tensor &B, const Tensor &Wp, int64_t D_out,
                                   const std::optional<Tensor> &bias, int64_t made_on)
{
    if (made_on != -1 && on_current_gpu(x_in)) {
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        void *const stream = stream_of(x_in);
        if (reinterpret_cast<int64_t>(stream) != made_on ||
            hipStreamIsCapturing(static_cast<hipStream_t>(stream), &capture) != hipSuccess || capture != hipStreamCaptureStatusNone)
            return std::nullopt;
    }
    if (!plain_context() || !on_current_gpu(x_in) || !plain(x_in, x_in.device()) || x_in.scalar_type() != at::kBFloat16 ||
        x_in.numel() == 0 || !plain(A, x_in.device()) || !plain(B, x_in.device()) || !plain(Wp, x_in.device()) ||
        (bias && !plain(*bias, x_in.device())))
        return std::nullopt;
    const Tensor x = x_in.contiguous();
    if (reinterpret_cast<uintptr_t>(x.data_ptr()) % 16 != 0)
        return std::nullopt;
    const Sizes s = sizes_of(x, A, B);
    auto shape = x.sizes().vec();
    shape.back() = D_out;
    Tensor out = at::empty(shape, x.options());
    check(grkan_linear_fwd_packed(x.data_ptr(), A.data_ptr<float>(), B.data_ptr<float>(), Wp.data_ptr(),
                                  bias ? bias->data_ptr<float>() : nullptr, out.data_ptr(), s.rows, s.D, (int32_t)D_out, s.G, s.m,
                                  s.n, GRKAN_BF16, GRKAN_BF16, stream_of(x)),
          "grkan_linear_fwd_packed");
    return out;
}

// The one-kernel layer on a bfloat16 module's own parameters (inference): nothing is converted, packed or kept.
// Sizes, layouts and alignments that the kernel does not cover are not taken.
std::optional<Tensor> layer_model(const Tensor &x_in, const Tensor &A, const Tensor &B, const Tensor &W,
                                  const std::optional<Tensor> &bias)
{
    if (at::GradMode::is_enabled() || !plain_context() || !on_current_gpu(x_in))
        return std::nullopt;
    for (const Tensor *t : {&x_in, &A, &B, &W, bias ? &*bias : &x_in})
        if (!plain(*t, x_in.device()) || t->scalar_type() != at::kBFloat16 || (t != &x_in && !t->is_contiguous()))
            return std::nullopt;
    if (x_in.dim() < 1 || x_in.numel() == 0 || W.dim() != 2 || W.size(1) != x_in.size(-1) || B.dim() != 2 || B.size(1) != 4 ||
        A.dim() < 1 || A.dim() > 2 || A.size(-1) != 6 || (A.dim() == 2 && A.size(0) != B.size(0)) ||
        (bias && (bias->dim() != 1 || bias->size(0) != W.size(0))))
        return std::nullopt;
    const int64_t D = W.size(1), D_out = W.size(0), G = B.size(0);
    if (D > INT32_MAX || D_out > INT32_MAX || G <= 0 || D % 64 != 0 || D % G != 0 || D / G % 32 != 0 || D_out <= 0 || D_out % 4 != 0)
        return std::nullopt;
    auto misaligned = [](const Tensor &t, uintptr_t to) { return reinterpret_cast<uintptr_t>(t.data_ptr()) % to != 0; };
    const Tensor x = x_in.contiguous();
    if (misaligned(x, 16) || misaligned(W, 16) || misaligned(A, 4) || misaligned(B, 4) || (bias && misaligned(*bias, 8)))
        return std::nullopt;
    auto shape = x.sizes().vec();
    shape.back() = D_out;
    Tensor out = at::empty(shape, x.options());
    check(grkan_linear_fwd_model(x.data_ptr(), A.data_ptr(), B.data_ptr(), W.data_ptr(), bias ? bias->data_ptr() : nullptr,
                                 out.data_ptr(), x.numel() / D, (int32_t)D, (int32_t)D_out, (int32_t)G, 5, 4, A.dim() == 1,
                                 stream_of(x)),
          "grkan_linear_fwd_model");
    return out;
}

// The layer in inference as F(x) and the product, on a bfloat16 module's own parameters.
std::optional<Tensor> layer_product(const Tensor &x_in, const Tensor &A, const Tensor &B, const Tensor &W, const std::optional<Tensor> &bias)
{
    if (at::GradMode::is_enabled() || !plain_context() || !on_current_gpu(x_in))
        return std::nullopt;
    for (const Tensor *t : {&x_in, &A, &B, &W, bias ? &*bias : &x_in})
        if (!plain(*t, x_in.device()) || t->scalar_type() != at::kBFloat16 || (t != &x_in && !t->is_contiguous()))
            return std::nullopt;
    if (x_in.dim() < 1 || x_in.numel() == 0 || W.dim() != 2 || W.size(1) != x_in.size(-1) || B.dim() != 2 || B.size(1) != 4 ||
        A.dim() < 1 || A.dim() > 2 || A.size(-1) != 6 || (A.dim() == 2 && A.size(0) != B.size(0)) ||
        (bias && (bias->dim() != 1 || bias->size(0) != W.size(0))))
        return std::nullopt;
    const int64_t D = W.size(1), D_out = W.size(0), G = B.size(0), rows = x_in.numel() / D;
    if (D > INT32_MAX || D_out > INT32_MAX || G <= 0 || D % G != 0 || !grkan_product_supported(rows, (int32_t)D, (int32_t)D_out) ||
        !aligned(W, 16) || (bias && !aligned(*bias, 8)))
        return std::nullopt;
    const Tensor x = x_in.contiguous();
    auto shape = x.sizes().vec();
    shape.back() = D_out;
    const Tensor f = at::empty_like(x);
    Tensor out = at::empty(shape, x.options());
    check(grkan_fwd_model(x.data_ptr(), A.data_ptr(), B.data_ptr(), f.data_ptr(), rows, (int32_t)D, (int32_t)G, 5, 4, GRKAN_BF16, GRKAN_BF16,
                          A.dim() == 1, stream_of(x)),
          "grkan_fwd");
    check(grkan_product(f.data_ptr(), W.data_ptr(), bias ? bias->data_ptr() : nullptr, out.data_ptr(), rows, (int32_t)D, (int32_t)D_out, 0, nullptr,
                        nullptr, 1, 0, stream_of(x)),
          "grkan_product");
    return out;
}

// The MLP block in inference, on a bfloat16 module's own parameters: F1(x), the first product with the second layer's rational
// function on its rounded result, the second product.  Nothing is converted, packed or kept.
std::optional<Tensor> block_inference(const Tensor &x_in, const Tensor &A1, const Tensor &B1, const Tensor &W1, const std::optional<Tensor> &b1,
                                      const Tensor &A2, const Tensor &B2, const Tensor &W2, const std::optional<Tensor> &b2)
{
    if (at::GradMode::is_enabled() || !plain_context() || !on_current_gpu(x_in))
        return std::nullopt;
    for (const Tensor *t : {&x_in, &A1, &B1, &W1, &A2, &B2, &W2, b1 ? &*b1 : &x_in, b2 ? &*b2 : &x_in})
        if (!plain(*t, x_in.device()) || t->scalar_type() != at::kBFloat16 || (t != &x_in && !t->is_contiguous()))
            return std::nullopt;
    if (x_in.dim() < 1 || x_in.numel() == 0 || W1.dim() != 2 || W2.dim() != 2 || x_in.size(-1) != W1.size(1) || W2.size(1) != W1.size(0) ||
        (b1 && (b1->dim() != 1 || b1->size(0) != W1.size(0))) || (b2 && (b2->dim() != 1 || b2->size(0) != W2.size(0))))
        return std::nullopt;
    const int64_t D = W1.size(1), hidden = W1.size(0), D_out = W2.size(0), rows = x_in.numel() / D;
    auto coefficients = [](const Tensor &A, const Tensor &B, int64_t channels) {
        return B.dim() == 2 && B.size(1) == 4 && A.dim() >= 1 && A.dim() <= 2 && A.size(-1) == 6 &&
               (A.dim() == 1 || A.size(0) == B.size(0)) && B.size(0) > 0 && channels % B.size(0) == 0;
    };
    if (D > INT32_MAX || hidden > INT32_MAX || D_out > INT32_MAX || !coefficients(A1, B1, D) || !coefficients(A2, B2, hidden) ||
        hidden / B2.size(0) % 8 != 0 || !grkan_product_supported(rows, (int32_t)D, (int32_t)hidden) ||
        !grkan_product_supported(rows, (int32_t)hidden, (int32_t)D_out))
        return std::nullopt;
    const Tensor x = x_in.contiguous();
    if (!aligned(W1, 16) || !aligned(W2, 16) || (b1 && !aligned(*b1, 8)) || (b2 && !aligned(*b2, 8)))
        return std::nullopt;
    auto shape = x.sizes().vec();
    shape.back() = D_out;
    Tensor out = at::empty(shape, x.options());
    // (F1(x) has been read when the result is written)
    const Tensor f1 = D_out == D ? out : at::empty_like(x), f2 = at::empty({rows, hidden}, x.options());
    void *const stream = stream_of(x);
    check(grkan_fwd_model(x.data_ptr(), A1.data_ptr(), B1.data_ptr(), f1.data_ptr(), rows, (int32_t)D, (int32_t)B1.size(0), 5, 4, GRKAN_BF16,
                          GRKAN_BF16, A1.dim() == 1, stream),
          "grkan_fwd");
    check(grkan_product(f1.data_ptr(), W1.data_ptr(), b1 ? b1->data_ptr() : nullptr, f2.data_ptr(), rows, (int32_t)D, (int32_t)hidden, 0,
                        A2.data_ptr(), B2.data_ptr(), (int32_t)B2.size(0), A2.dim() == 1, stream),
          "grkan_product");
    check(grkan_product(f2.data_ptr(), W2.data_ptr(), b2 ? b2->data_ptr() : nullptr, out.data_ptr(), rows, (int32_t)hidden, (int32_t)D_out, 0,
                        nullptr, nullptr, 1, 0, stream),
          "grkan_product");
    return out;
}

// No function mode, or device contexts alone (torch.set_default_device: they act on factory functions only).
bool no_function_mode()
{
    if (!at::impl::torch_function_mode_enabled())
        return true;
    const pybind11::object device_context = pybind11::module_::import("torch.utils._device").attr("DeviceContext");
    for (const pybind11::handle mode : pybind11::module_::import("torch.overrides").attr("_get_current_function_mode_stack")())
        if (reinterpret_cast<PyObject *>(Py_TYPE(mode.ptr())) != device_context.ptr())
            return false;
    return true;
}

// The arguments of an entry as tensors; `taken` is false if one is a tensor subclass (or no tensor at all), or if a
// function mode would see the calls of the Python route.
struct Arguments {
    bool taken = no_function_mode();

    Tensor tensor(pybind11::handle h)
    {
        if (!taken || !THPVariable_CheckExact(h.ptr())) {
            taken = false;
            return Tensor();
        }
        return THPVariable_Unpack(h.ptr());
    }
    std::optional<Tensor> optional(pybind11::handle h)
    {
        return h.is_none() ? std::nullopt : std::optional<Tensor>(tensor(h));
    }
    template <typename Entry> auto call(Entry &&entry) const -> decltype(entry())
    {
        if (!taken)
            return std::nullopt;
        pybind11::gil_scoped_release no_gil;
        return entry();
    }
};

} // namespace

PYBIND11_MODULE(_native, mod)
{
    using pybind11::handle;
    mod.def("rational", [](handle x_, handle A_, handle B_) {
        Arguments args;
        const Tensor x = args.tensor(x_), A = args.tensor(A_), B = args.tensor(B_);
        return args.call([&] { return rational(x, A, B); });
    });
    mod.def("product", [](handle y_, handle W_, handle bias_) {
        Arguments args;
        const Tensor y = args.tensor(y_), W = args.tensor(W_);
        const std::optional<Tensor> bias = args.optional(bias_);
        return args.call([&] { return product(y, W, bias); });
    });
    mod.def("block", [](handle x_, handle A1_, handle B1_, handle W1_, handle b1_, handle A2_, handle B2_, handle W2_, handle b2_,
                        bool wgrad) {
        Arguments args;
        const Tensor x = args.tensor(x_), A1 = args.tensor(A1_), B1 = args.tensor(B1_), W1 = args.tensor(W1_);
        const std::optional<Tensor> b1 = args.optional(b1_);
        const Tensor A2 = args.tensor(A2_), B2 = args.tensor(B2_), W2 = args.tensor(W2_);
        const std::optional<Tensor> b2 = args.optional(b2_);
        return args.call([&] { return block(x, A1, B1, W1, b1, A2, B2, W2, b2, wgrad); });
    });
    mod.def("block_inference", [](handle x_, handle A1_, handle B1_, handle W1_, handle b1_, handle A2_, handle B2_, handle W2_, handle b2_) {
        Arguments args;
        const Tensor x = args.tensor(x_), A1 = args.tensor(A1_), B1 = args.tensor(B1_), W1 = args.tensor(W1_);
        const std::optional<Tensor> b1 = args.optional(b1_);
        const Tensor A2 = args.tensor(A2_), B2 = args.tensor(B2_), W2 = args.tensor(W2_);
        const std::optional<Tensor> b2 = args.optional(b2_);
        return args.call([&] { return block_inference(x, A1, B1, W1, b1, A2, B2, W2, b2); });
    });
    mod.def("layer_model", [](handle x_, handle A_, handle B_, handle W_, handle bias_) {
        Arguments args;
        const Tensor x = args.tensor(x_), A = args.tensor(A_), B = args.tensor(B_), W = args.tensor(W_);
        const std::optional<Tensor> bias = args.optional(bias_);
        return args.call([&] { return layer_model(x, A, B, W, bias); });
    });
    mod.def("layer_product", [](handle x_, handle A_, handle B_, handle W_, handle bias_) {
        Arguments args;
        const Tensor x = args.tensor(x_), A = args.tensor(A_), B = args.tensor(B_), W = args.tensor(W_);
        const std::optional<Tensor> bias = args.optional(bias_);
        return args.call([&] { return layer_product(x, A, B, W, bias); });
    });
    mod.def("pack_layer", [](handle W_, handle bias_, handle A_, handle B_) {
        Arguments args;
        const Tensor W = args.tensor(W_), A = args.tensor(A_), B = args.tensor(B_);
        const std::optional<Tensor> bias = args.optional(bias_);
        return args.call([&] { return pack_layer(W, bias, A, B); });
    });
    mod.def("layer_packed", [](handle x_, handle A_, handle B_, handle Wp_, int64_t D_out, handle bias_,
                                int64_t made_on) {
        Arguments args;
        const Tensor x = args.tensor(x_), A = args.tensor(A_), B = args.tensor(B_), Wp = args.tensor(Wp_);
        const std::optional<Tensor> bias = args.optional(bias_);
        return args.call([&] { return layer_packed(x, A, B, Wp, D_out, bias, made_on); });
    });
}
