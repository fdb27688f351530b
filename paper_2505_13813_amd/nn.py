"""PyTorch front end of the GR-KAN layer: an autograd function over the HIP
kernels, the group-wise rational module with the paper's model-level
conventions, the GR-KAN linear layer and the KAT MLP block.

The rational function runs in this package's kernels; the matrix products are
torch's (library GEMMs), except in bfloat16 on the GPU: the one-kernel layer
grkan_linear_fwd (GRKANLinear(fused=...)), the products of layers in inference
and of MLP blocks (grkan_product), and the weight and bias gradients of
training (grkan_linear_wgrad).  Plain calls run as native autograd
functions; what those do not take runs in the Python ones here.  Conventions taken from the FlashKAT paper:
  * GR-KAN(x) = W F(x): the rational function is applied to the INPUT of each
    linear layer (Eq. "GR_KAN").
  * the groups use one common set of numerator coefficients and have their own
    denominator coefficients (Sec. "Results"): one numerator row, read by the
    kernels as it is, dA summed over the groups (in the Python functions it is
    broadcast to [G, m+1] and autograd's expand sums).
  * the first rational of an MLP block starts as the identity, the second as a
    Swish (Sec. "Results").  The paper prints no Swish coefficients, so they
    are obtained here by a (linearised) least-squares fit on [-3, 3].
  * variance-preserving weights (Sec. "Kolmogorov-Arnold Transformer"):
    W ~ N(0, alpha / d_in).  The paper prints alpha = E[F(x)^2] / Var[x], which
    would not preserve the variance (Var[W F(x)] = d_in * Var[w] * E[F^2]); the
    stated purpose decides, so alpha = Var[x] / E[F(x)^2] here, with
    x ~ N(0, 1) -- the usual gain (2 for ReLU).  Both readings coincide for the
    identity initialisation.
"""
from __future__ import annotations

import math
import weakref
from functools import lru_cache
from typing import Tuple

import numpy as np
import torch
from torch import nn
from torch.nn.modules import module as every_module

from . import binding

M_DEGREE = binding.M_DEGREE
N_DEGREE = binding.N_DEGREE


_workspaces = {}


def _workspace(x, rows: int, D: int, G: int) -> torch.Tensor:
    """One backward workspace per (device, stream), grown on demand.  Calls on one
    stream run one after the other, so they can share it; the workspace's
    contents mean nothing between calls."""
    need = binding._workspace_bytes_cached(rows, D, G, binding._io_of(x), x.device.index or 0)
    key = (x.device.index or 0, torch.cuda.current_stream(x.device).cuda_stream)
    ws = _workspaces.get(key)
    if ws is None or ws.numel() < need:
        ws = torch.empty(max(need, 1 << 16), dtype=torch.uint8, device=x.device)
        _workspaces[key] = ws
    return ws


class _Undifferentiable(torch.autograd.Function):
    """Gradients of a backward pass that was asked for a graph of itself and has none: differentiating them with
    respect to what they depend on is an error instead of leaving it out."""

    @staticmethod
    def forward(ctx, dx, dA, dB, x, A, B, dy):
        return dx.view_as(dx), dA.view_as(dA), dB.view_as(dB)

    @staticmethod
    def backward(ctx, *_):
        raise RuntimeError("the group-wise rational function is not differentiable twice")


def _rational_gradients(x, dy, A, B):
    """(dx, dA, dB) of F in a backward pass."""
    D = int(x.shape[-1])
    ws = _workspace(x, int(x.numel() // D) if D else 0, D, int(A.shape[0]))
    grads = binding.grkan_bwd(x, dy.contiguous(), A, B, workspace=ws)
    return _Undifferentiable.apply(*grads, x, A, B, dy) if torch.is_grad_enabled() else grads


class GroupRationalFunction(torch.autograd.Function):
    """y = F(x) group-wise; backward through grkan_bwd (nothing but x, A, B is saved).  Of operands that are not contiguous it
    saves copies, which have no history: callers that may be differentiated twice pass contiguous ones."""

    @staticmethod
    def forward(ctx, x, A, B):
        x = x.contiguous()
        A = A.contiguous()
        B = B.contiguous()
        ctx.save_for_backward(x, A, B)
        return binding.grkan_fwd(x, A, B)

    @staticmethod
    def backward(ctx, dy):
        x, A, B = ctx.saved_tensors
        return _rational_gradients(x, dy, A, B)


def fused_layer_supported(x, A, weight) -> bool:
    """Shapes and types the one-kernel layer (grkan_linear_fwd) covers: bfloat16 x and W on the GPU,
    degrees (5, 4), D_in a multiple of 64, d_g a multiple of 32, D_out a multiple of 4."""
    return _fused_shapes(x, int(A.shape[0]), int(A.shape[1]), weight)


def _fused_shapes(x, G: int, numerator_columns: int, weight) -> bool:
    return (_fused_sizes(x.shape[-1], weight.shape[0], G, numerator_columns) and x.is_cuda and x.dtype == torch.bfloat16
            and weight.dtype == torch.bfloat16)


def _fused_sizes(D_in: int, D_out: int, G: int, numerator_columns: int) -> bool:
    return (D_in % 64 == 0 and D_in % G == 0 and (D_in // G) % 32 == 0 and D_out % 4 == 0
            and numerator_columns == M_DEGREE + 1)


def fused_layer_pays(rows: int, D_in: int, D_out: int) -> bool:
    """The sizes at which a GRKANLinear runs the one-kernel layer on a packed copy of its weights that it keeps between
    calls: the layer's 112-row tiles (of 768, 384 or 192 channels) fill the chip, or the contraction is short.  (At
    other sizes the module in evaluation mode takes the layer on its parameters as they are, where
    one_kernel_is_faster says so.)"""
    bn = 768 if D_out % 768 == 0 else (384 if D_out % 384 == 0 else 192)
    workgroups = -(-int(rows) // 112) * -(-int(D_out) // bn)
    return workgroups >= 200 or D_in <= 768


@lru_cache(maxsize=1024)
def one_kernel_is_faster(rows: int, D_in: int, D_out: int) -> bool:
    """Whether the one-kernel layer is the faster route in inference, by its own estimate and one of the two kernels:
    the elementwise pass at 5.5 TB/s and the library product in whole rounds of 256 x 256 or 128 x 128 tiles, and no
    less than the 27 us of host time that two launches take.  (Measured on MI355X, bfloat16, at 266 sizes: nineteen
    layer shapes, 1 - 25,216 rows.  Nowhere was the route that this takes more than 4 % slower than the two kernels;
    at fifteen sizes it passes by a gain of 5 % or more, most of them where the library's own choice of tile is a poor
    one.  3072 -> 768: 197 rows 10.1 us against 27.7, 1,576 30 against 28.1, 6,304 42.5 against 51, 25,216 128 against
    195; 768 -> 3072: 1,576 rows 15.5 against 28, 6,304 44 against 56, 12,608 85 against 71.)"""
    return binding.grkan_linear_estimate_us(rows, D_in, D_out) <= _two_kernels_us(rows, D_in, D_out)


def _two_kernels_us(rows: int, D_in: int, D_out: int) -> float:
    def product_us(tile, us_per_1k):
        rounds = -(-(-(-rows // tile) * -(-D_out // tile)) // 256)
        return rounds * (6.0 + us_per_1k * D_in / 1024)

    return max(27.0, rows * D_in * 4 / 5.5e6 + min(product_us(256, 24.0), product_us(128, 4.0)))


# Weights (D_in x D_out) up to which grkan_product's estimate was measured to hold beside the other routes (3072 x 3072).  With larger
# ones it is up to 1.8 times too low (256 rows of 16384 -> 4096: 55 us estimated, 98 taken; through torch's linear 62).
_MOST_PRODUCT_WEIGHTS = 10_000_000


@lru_cache(maxsize=1024)
def layer_product_is_faster(rows: int, D_in: int, D_out: int, one: bool, packed: bool) -> bool:
    """Whether a GRKANLinear in inference runs F and grkan_product.  F takes 3.3 us and 5.5 TB/s.

    Instead of the one-kernel layer, where that would be the route (`one`; on packed weights it is 4 % faster than it
    estimates), with 4 us to be gained.  (us of the one kernel / this: 512 -> 2048 at 12,608 rows 57 / 46, at 50,432 217 / 144.)

    Instead of F and torch's linear, which take 31 us of host time through the module: up to 512 channels always (no size of these was slower by more than
    1 %); above, where the estimate, with a margin that grows with D_in (it is 7 us too low for few rows of 3072), is below
    what one_kernel_is_faster counts for torch's.  The library reaches 1.1 - 1.35 PFLOP/s where its rounds of tiles are full, this 0.9 - 1.1.
    Where D_out is no multiple of 64 it reaches 0.5 - 0.9.  (Measured on MI355X at 32 pairs D_in, D_out, 16 - 40,000 rows; us of torch's / this:
    768 -> 3072 at 2,048 rows 29 / 21, at 5,000 31 / 33, at 16,384 81 / 93, at 25,216 139 / 138; 3072 -> 3072 at 5,000 84 / 92, at
    25,216 494 / 430; 1024 -> 1024 at 16,384 45 / 48, 1024 -> 1000 78 / 47.  Of 390 sizes two lose more than 3 % to the route without
    grkan_product, the most 1024 -> 4096 at 12,608 rows, 107 / 116; to the faster of both the rule loses 0.8 % in the mean.)"""
    product = binding.grkan_product_estimate_us(rows, D_in, D_out)
    if not product or D_in * D_out > _MOST_PRODUCT_WEIGHTS:
        return False
    this = 3.3 + rows * D_in * 4 / 5.5e6 + product
    if one:
        return this + 4.0 < binding.grkan_linear_estimate_us(rows, D_in, D_out) * (0.96 if packed else 1.0)
    if D_in <= 512:
        return True
    two = _two_kernels_us(rows, D_in, D_out)
    return this <= 1.35 * two if D_out % 64 else this * (1.0 + D_in / 12288) <= max(31.0, two)


@lru_cache(maxsize=1024)
def _layer_route(rows: int, D_in: int, D_out: int, G: int, numerator_columns: int, keep_packed: bool) -> str:
    """How a GRKANLinear on the GPU runs in evaluation mode: "product", "model" (the one kernel on the parameters), "packed" (the one
    kernel on the kept copy), or "other"."""
    if G <= 0 or rows <= 0 or D_in <= 0 or D_in % G or numerator_columns != M_DEGREE + 1:
        return "other"
    one = _fused_sizes(D_in, D_out, G, numerator_columns) and one_kernel_is_faster(rows, D_in, D_out)
    packed = keep_packed and one and fused_layer_pays(rows, D_in, D_out)
    if layer_product_is_faster(rows, D_in, D_out, one, packed):
        return "product"
    return "other" if not one else "packed" if packed else "model"


@lru_cache(maxsize=1024)
def block_products_are_faster(rows: int, D: int, hidden: int, D_out: int, G1: int, G2: int) -> bool:
    """Whether an MLP block in inference runs as F1, the first product with F2 on its result, and the second product
    (grkan_product), instead of its two layers.  F1 takes 3.3 us and 5.5 TB/s; three launches take no less than 15 us of host time, the
    layers' two 13 by themselves and 19 through the layers' calls, behind the look at this rule.  (Measured on MI355X, widths 128 - 4096,
    8 - 40,000 rows, us of the layers / this: 192 at 6,304 rows 45 / 22, 384 44 / 34, 512 69 / 54, 768 85 / 73; 768 at 25,216 270 / 265,
    1024 at 25,216 442 / 403; 768 -> 768 at 49 rows 18.9 / 15.9.  The layers win at few rows of a wide model, where each is one round of small
    tiles: 768 at 49 rows 15.8 / 18.8, at 197 18.7 / 22.3, 512 at 49 13.3 / 16.2, at 394 16.1 / 18.1, 1024 at 49 17.7 / 22.4; 768 at
    394 31 / 26.  With both contractions short the estimate is up to 7 us too low at 25,216 rows: 256 -> 256 34 / 36.  With weights past the measured ones this is too low, as for layers: 2048 at 394 rows 63 / 67, 4096 at 197 121 / 135.)"""
    def layer_us(D_in, D_out, G):
        two = _two_kernels_us(rows, D_in, D_out)
        return min(two, binding.grkan_linear_estimate_us(rows, D_in, D_out)) if _fused_sizes(D_in, D_out, G, M_DEGREE + 1) else two

    if G1 <= 0 or G2 <= 0 or D % G1 or hidden % G2 or max(D, D_out) * hidden > _MOST_PRODUCT_WEIGHTS:
        return False
    first, second = binding.grkan_product_estimate_us(rows, D, hidden, True), binding.grkan_product_estimate_us(rows, hidden, D_out, False)
    if not first or not second:
        return False
    products = 3.3 + rows * D * 4 / 5.5e6 + first + second + (rows / 3500 if max(D, hidden) <= 512 else 0.0)
    calls = (_layer_route(rows, D, hidden, G1, M_DEGREE + 1, False), _layer_route(rows, hidden, D_out, G2, M_DEGREE + 1, True))
    host = 13.0 if calls == ("model", "model") else 19.0
    return max(15.0, products) <= max(host, layer_us(D, hidden, G1) + layer_us(hidden, D_out, G2))


@lru_cache(maxsize=1024)
def _block_route(rows: int, D: int, hidden: int, D_out: int, G1: int, G2: int, columns1: int, columns2: int) -> str:
    """How a KATMlp on the GPU runs in evaluation mode: "products", "models" (the one kernel on the parameters for both layers: 256 wide at
    49 - 788 rows 15.4 - 16.5 us through the layers' calls, 11.8 - 12.8 without them; 512 at 49 16.4 / 13.4), or "layers" (each on its
    own)."""
    if D <= 0 or rows <= 0:
        return "layers"
    if block_products_are_faster(rows, D, hidden, D_out, G1, G2):
        return "products"
    both = (_layer_route(rows, D, hidden, G1, columns1, False), _layer_route(rows, hidden, D_out, G2, columns2, True))
    return "models" if both == ("model", "model") else "layers"


class GRKANLayerFunction(torch.autograd.Function):
    """out = F(x) W^T + bias with the forward pass in one kernel (F never written to memory) and
    nothing but x, A, B, W saved.  The backward pass recomputes F(x) for dW = dOut^T F(x)
    (grkan_fwd + a library product), forms dF = dOut W (library product) and runs grkan_bwd on it:
    one extra elementwise forward kernel in exchange for not keeping F(x) alive between the passes."""

    @staticmethod
    def forward(ctx, x, A, B, weight, bias):
        x = x.contiguous()
        A = A.contiguous()
        B = B.contiguous()
        weight = weight.contiguous()
        ctx.save_for_backward(x, A, B, weight)
        ctx.has_bias = bias is not None
        ctx.bias_dtype = bias.dtype if bias is not None else None
        b32 = bias.to(torch.float32).contiguous() if bias is not None else None
        return binding.grkan_linear_fwd(x, A, B, weight, b32, out_dtype=x.dtype)

    @staticmethod
    def backward(ctx, dout):
        x, A, B, weight = ctx.saved_tensors
        D_in, D_out = int(x.shape[-1]), int(weight.shape[0])
        dout2 = dout.contiguous().view(-1, D_out)
        # F(x), recomputed (with a graph of its own where one of this pass is wanted)
        y = (GroupRationalFunction.apply if torch.is_grad_enabled() else binding.grkan_fwd)(x, A, B).view(-1, D_in)
        dW = dout2.t().mm(y)
        dF = dout2.mm(weight).view(x.shape)
        dx, dA, dB = _rational_gradients(x, dF, A, B)
        dbias = dout2.sum(0).to(ctx.bias_dtype) if ctx.has_bias else None
        return dx, dA, dB, dW, dbias


def wgrad_pays(rows: int, D_in: int, D_out: int) -> bool:
    """Whether a bfloat16 product's gradients are grkan_linear_wgrad's rather than the library's product and column sum.  Tiles are 192 x 192,
    one per compute unit at a time; up to 128 of them the rows are split over the units, above they are not.

    Measured on MI355X at seventeen shapes of 1 - 256 tiles and 256 - 25,216 rows the kernel is the faster one at all of them: us of it / the
    library at 25,216 rows 384 x 1536 41 / 171, 768 x 3072 108 / 270, 2048 x 2048 187 / 373, 1024 x 4096 (132 tiles) 277 / 339, 3072 x 3072
    388 / 539; at 640 rows 16 / 29, 24 / 27, 25 / 30, 27 / 30, 30 / 37; at 512 rows 15 / 28, 23 / 27, 26 / 30, 26 / 30, 28 / 33.  The line is
    narrower than that: it was drawn for the kernel in an earlier form (eight wavefronts that loaded, read and multiplied in turn), which
    lost with 129 - 223 tiles at some row counts (1024 x 4096 413 / 340), and at 512 rows from 96 tiles on."""
    tiles = -(-D_in // 192) * -(-D_out // 192)
    return (D_in % 8 == 0 and D_out % 8 == 0 and rows >= (512 if tiles <= 64 else 640)
            and (tiles <= 128 or 224 <= tiles <= 256))


def _native_product(linear, y):
    """The linear layer on y with grkan_linear_wgrad in its backward pass, or None where that route is not
    taken: plain bfloat16 training on the GPU, at sizes it pays for, with nothing attached to the linear layer
    that its own call would run or change (hooks, parametrisations, autocast, tracing, tensor subclasses)."""
    if not _only_a(nn.Linear, linear):
        return None
    w, b = linear.weight, linear.bias
    if (y.dtype != torch.bfloat16 or not torch.is_grad_enabled() or not w.requires_grad
            or type(w) is not nn.Parameter or (b is not None and type(b) is not nn.Parameter) or type(y) is not torch.Tensor
            or torch.is_autocast_enabled()
            or torch.compiler.is_compiling() or not wgrad_pays(y.numel() // y.shape[-1], w.shape[1], w.shape[0])):
        return None
    return binding.load_native().product(y, w, b)


def _only_a(cls, module) -> bool:
    """Whether calling `module` runs cls.forward and nothing else, so that a route past the call changes nothing: no
    subclass (an adapter, a parametrisation), no forward of its own, no hooks on it or on every module."""
    return (type(module) is cls and "forward" not in module.__dict__
            and not (module._forward_hooks or module._forward_pre_hooks or module._backward_hooks
                     or module._backward_pre_hooks or every_module._global_forward_hooks
                     or every_module._global_forward_pre_hooks or every_module._global_backward_hooks
                     or every_module._global_backward_pre_hooks))


def _autocast_elsewhere() -> bool:
    """Whether autocast would have torch's linear compute in another type than bfloat16."""
    return torch.is_autocast_enabled() and torch.get_autocast_dtype("cuda") != torch.bfloat16


def group_rational(x, A, B):
    """Functional form: x [..., D] float32 / bfloat16 / float16 on the GPU, A [G, m+1], B [G, n] float32."""
    if not torch.compiler.is_compiling() and A.dim() == 2 and A.dtype == torch.float32 and B.dtype == torch.float32:
        y = binding.load_native().rational(x, A, B)
        if y is not None:
            return y
    return GroupRationalFunction.apply(x.contiguous(), A.contiguous(), B.contiguous())


def _rational_np(x, a, b):
    p = sum(a[i] * x ** i for i in range(len(a)))
    q = 1.0 + np.abs(sum(b[j] * x ** (j + 1) for j in range(len(b))))
    return p / q


@lru_cache(maxsize=None)
def swish_coefficients(m: int = M_DEGREE, n: int = N_DEGREE) -> Tuple[Tuple[float, ...], Tuple[float, ...]]:
    """(a_0..a_m, b_1..b_n) of a safe Pade unit fitted to Swish, x * sigmoid(x).

    Linearised least squares on a uniform grid over [-3, 3]: minimise
    |P(x) - t(x) * sum_j b_j x^j - t(x)| over (a, b), which is linear.  The
    solution has an even, non-negative denominator polynomial (odd b_j = 0,
    even b_j > 0), so the absolute value of the safe unit is inactive; for
    (5, 4) the fit error of F itself is below 1e-6 on the grid (8e-3 on
    [-6, 6]), for (3, 2) 5e-3, for (7, 6) 1e-10.  Deterministic: plain linear
    algebra in float64.
    """
    xs = np.linspace(-3.0, 3.0, 601)
    target = xs / (1.0 + np.exp(-xs))
    cols = [xs ** i for i in range(m + 1)] + [-target * xs ** (j + 1) for j in range(n)]
    theta, *_ = np.linalg.lstsq(np.stack(cols, axis=1), target, rcond=None)
    return tuple(float(v) for v in theta[:m + 1]), tuple(float(v) for v in theta[m + 1:])


def second_moment(a, b, points: int = 128) -> float:
    """E[F(x)^2] for x ~ N(0, 1) by Gauss-Hermite quadrature."""
    t, w = np.polynomial.hermite_e.hermegauss(points)
    f = _rational_np(t, np.asarray(a, dtype=np.float64), np.asarray(b, dtype=np.float64))
    return float(np.sum(w * f * f) / math.sqrt(2.0 * math.pi))


class GroupRational(nn.Module):
    """The group-wise rational function with learnable coefficients.

    `init`: "identity" (a = e_1, b = 0) or "swish".  With `shared_numerator`
    (the paper's setting) there is one numerator row for all groups.
    `degrees` = (m, n), one of the pairs the library is built for.
    """

    def __init__(self, groups: int = 8, init: str = "identity", shared_numerator: bool = True,
                 degrees: Tuple[int, int] = (M_DEGREE, N_DEGREE)):
        super().__init__()
        m, n = (int(v) for v in degrees)
        if (m, n) not in binding.DEGREES:
            raise ValueError("degrees must be one of %s" % (binding.DEGREES,))
        self.degrees = (m, n)
        if init == "identity":
            a = [0.0, 1.0] + [0.0] * (m - 1)
            b = [0.0] * n
        elif init == "swish":
            a, b = swish_coefficients(m, n)
        else:
            raise ValueError("init must be 'identity' or 'swish'")
        self.groups = int(groups)
        self.shared_numerator = bool(shared_numerator)
        a_t = torch.tensor(a, dtype=torch.float32)
        b_t = torch.tensor(b, dtype=torch.float32)
        self.numerator = nn.Parameter(a_t.clone() if shared_numerator else a_t.repeat(self.groups, 1))
        self.denominator = nn.Parameter(b_t.repeat(self.groups, 1))

    def coefficient_rows(self):
        A = self.numerator.expand(self.groups, self.degrees[0] + 1) if self.shared_numerator else self.numerator
        return A, self.denominator

    def second_moment(self) -> float:
        """E[F(x)^2], x ~ N(0,1), averaged over the groups (they start identical)."""
        A, B = self.coefficient_rows()
        A = A.detach().cpu().numpy()
        B = B.detach().cpu().numpy()
        return float(np.mean([second_moment(A[g], B[g]) for g in range(self.groups)]))

    def forward(self, x):
        if (not torch.compiler.is_compiling() and "coefficient_rows" not in self.__dict__
                and type(self).coefficient_rows is GroupRational.coefficient_rows):
            # the parameters as they are: one numerator row for all groups, float32 or bfloat16
            y = binding.load_native().rational(x, self.numerator, self.denominator)
            if y is not None:
                return y
        A, B = self.coefficient_rows()
        return group_rational(x, A.to(torch.float32), B.to(torch.float32))


class _Packed(tuple):
    """(PackedWeight, bias, A rows, B rows) of one state of a layer's parameters, with the stream it was made on and the
    event after which others may read it (made_on = -1: made during a capture, for the call that made it).  Not part of a
    copied or saved module."""

    made_on, stream, made = -1, None, None

    @classmethod
    def of(cls, params):
        """The copies, or None where the parameters are not plain tensors on the current GPU."""
        copies = binding.load_native().pack_layer(*params)
        if copies is None:
            return None
        data, b32, A32, B32 = copies
        self = cls((binding.PackedWeight(data, *params[0].shape), b32, A32, B32))
        self._made_of = tuple((None, 0, 0) if p is None else (weakref.ref(p), p.data_ptr(), p._version) for p in params)
        return self

    def is_of(self, params) -> bool:
        for p, (ref, address, version) in zip(params, self._made_of):
            if p is None or ref is None:
                if p is not None or ref is not None:
                    return False
            elif ref() is not p or p.data_ptr() != address or p._version != version:
                return False
        return True

    def tensors(self):
        return [t for t in (self[0].data, *self[1:]) if t is not None]

    def __deepcopy__(self, memo):
        return None

    def __reduce__(self):
        return type(None), ()


class GRKANLinear(nn.Module):
    """GR-KAN(x) = W F(x) + bias (Eq. "GR_KAN"), variance-preserving init."""

    def __init__(self, in_features: int, out_features: int, groups: int = 8, init: str = "identity",
                 bias: bool = True, shared_numerator: bool = True,
                 degrees: Tuple[int, int] = (M_DEGREE, N_DEGREE), fused: str = "inference"):
        """`fused`: when the one-kernel layer (F inside the matrix product) is used where it applies
        (bfloat16, see fused_layer_supported): "inference" = when no gradient is recorded (in training
        its backward pass has to recompute F(x)) and it is the faster route at this size
        (one_kernel_is_faster); "always" = wherever it applies; "never".

        At the sizes of fused_layer_pays it runs on a packed copy of the weights (with bias and coefficients
        in float32) that is kept until a parameter is written to or replaced, the module is moved, converted or
        switched between training and evaluation, or a state is loaded.  Writes through `.data` or a detached alias
        leave no trace that this could be told from: after one, call drop_packed_weights() (or train() / eval()).
        At all other sizes, in evaluation mode, it reads the parameters themselves and keeps nothing; so does the layer as F and
        a matrix product of this package, where that is the fastest of the three (layer_product_is_faster)."""
        super().__init__()
        if in_features % groups:
            raise ValueError("in_features must be a multiple of groups")
        if fused not in ("inference", "always", "never"):
            raise ValueError("fused must be 'inference', 'always' or 'never'")
        self.fused = fused
        self._packed = None  # _Packed
        self.rational = GroupRational(groups, init, shared_numerator, degrees)
        self.linear = nn.Linear(in_features, out_features, bias=bias)
        alpha = 1.0 / self.rational.second_moment()  # Var[x] / E[F(x)^2] with Var[x] = 1
        with torch.no_grad():
            self.linear.weight.normal_(0.0, math.sqrt(alpha / in_features))
            if bias:
                self.linear.bias.zero_()

    _keep_packed = True

    def drop_packed_weights(self):
        """Forgets the packed copy of the weights; the next call that needs one makes it anew."""
        self._packed = None

    def train(self, mode: bool = True):
        self.drop_packed_weights()
        return super().train(mode)

    def _apply(self, *args, **kwargs):
        self.drop_packed_weights()
        return super()._apply(*args, **kwargs)

    def _load_from_state_dict(self, *args, **kwargs):
        self.drop_packed_weights()
        return super()._load_from_state_dict(*args, **kwargs)

    def __setstate__(self, state):
        super().__setstate__(state)
        self._packed = None

    def _inference_weights(self, params):
        """Packed weights (the kernel then fetches them in whole cache lines), the bias and the coefficient rows in
        float32, kept until a parameter is written to or replaced; None where no copy can be kept: a tensor put in a
        parameter's place for one call may sit where the last one did, and inference tensors have no version."""
        packed = self._packed
        if packed is not None and packed.is_of(params):
            return packed
        if not all(type(p) is nn.Parameter and not p.is_inference() for p in params if p is not None):
            return None
        packed = _Packed.of(params)
        if packed is not None and not torch.cuda.is_current_stream_capturing():
            packed.stream = torch.cuda.current_stream(params[0].device)
            packed.made = packed.stream.record_event()
            packed.made_on = packed.stream.cuda_stream
            self._packed = packed
        return packed

    def _packed_layer(self, x, packed, params):
        """The layer on the packed weights; None where the native entry does not take the call."""
        entry = binding.load_native().layer_packed
        pw, b32, A32, B32 = packed
        out = entry(x, A32, B32, pw.data, pw.D_out, b32, packed.made_on)
        if out is None and packed.made_on != -1:
            packed = self._readable_here(packed, params)
            if packed is None:
                return None
            pw, b32, A32, B32 = packed
            out = entry(x, A32, B32, pw.data, pw.D_out, b32, -1)
        return out

    def _readable_here(self, packed, params):
        """The kept copy ordered behind its packing on whatever stream this is; under capture one that is part of the
        graph, so that a replay follows the parameters and its memory is the graph's own."""
        if torch.cuda.is_current_stream_capturing():
            return _Packed.of(params)
        stream = torch.cuda.current_stream(params[0].device)
        if stream != packed.stream:
            stream.wait_event(packed.made)
            for t in packed.tensors():
                t.record_stream(stream)
        return packed

    def forward(self, x):
        out = self._one_kernel(x)
        if out is not None:
            return out
        y = self.rational(x)
        out = _native_product(self.linear, y)
        return self.linear(y) if out is None else out

    def _one_kernel(self, x):
        """The layer's output from the one kernel, or None where that route is not taken.  (What the native entries
        do not take - alignment, forward-mode differentiation, function transforms - is left to the two kernels.)"""
        fused, grad = self.fused, torch.is_grad_enabled()
        always = fused == "always"
        if fused == "never" or (grad and not always) or x.dtype is not torch.bfloat16:
            return None
        linear, rational = self._modules.get("linear"), self._modules.get("rational")
        if not _only_a(nn.Linear, linear) or not _only_a(GroupRational, rational) or _autocast_elsewhere():
            return None
        weight, bias = linear._parameters.get("weight"), linear._parameters.get("bias")
        numerator, denominator = rational._parameters.get("numerator"), rational._parameters.get("denominator")
        if weight is None or numerator is None or denominator is None or "coefficient_rows" in rational.__dict__:
            return None
        if bias is None and "bias" not in linear._parameters:  # a buffer or a plain tensor
            return None
        if not x.dim() or not x.shape[-1]:
            return None
        D_in, D_out = x.shape[-1], weight.shape[0]
        rows = x.numel() // D_in
        if x.is_cuda and not (grad or always or self.training or torch.compiler.is_compiling()) and weight.shape[1] == D_in:
            route = _layer_route(rows, D_in, D_out, denominator.shape[0], numerator.shape[-1], self._keep_packed)
            if route == "packed" and weight.dtype is torch.bfloat16:
                params = (weight, bias, numerator, denominator)
                packed = self._inference_weights(params)
                if packed is not None:
                    return self._packed_layer(x, packed, params)
            elif route != "other":
                native = binding.load_native()
                out = (native.layer_product if route == "product" else native.layer_model)(x, numerator, denominator, weight, bias)
                if out is not None or route == "model":
                    return out
        if not _fused_shapes(x, denominator.shape[0], numerator.shape[-1], weight) or D_in != weight.shape[1]:
            return None
        if grad:
            A, B = rational.coefficient_rows()
            operands = (x, A.to(torch.float32), B.to(torch.float32), weight)
            return GRKANLayerFunction.apply(*(t.contiguous() for t in operands), bias)
        if not always and not one_kernel_is_faster(rows, D_in, D_out):
            return None
        compiling = torch.compiler.is_compiling()
        if self._keep_packed and (always or fused_layer_pays(rows, D_in, D_out)):
            params = (weight, bias, numerator, denominator)
            packed = self._inference_weights(params)
            if packed is not None:
                if compiling:
                    if packed.made_on != -1:
                        packed = self._readable_here(packed, params)
                    if packed is None:
                        return None
                    pw, b32, A32, B32 = packed
                    return binding.grkan_linear_fwd(x.contiguous(), A32, B32, pw, b32, out_dtype=x.dtype)
                return self._packed_layer(x, packed, params)
        # In training mode a pass without a gradient may be the first half of one with (reentrant checkpointing): both
        # take the same kernels.
        if compiling or (self.training and not always):
            return None
        return binding.load_native().layer_model(x, numerator, denominator, weight, bias)


class KATMlp(nn.Module):
    """The MLP of a KAT block: two GR-KAN layers, hidden width 4x by default;
    the first rational starts as the identity, the second as Swish.

    `fused`: of the second layer, as GRKANLinear has it (the first one is fused in evaluation mode only).  With the default,
    "inference", bfloat16 training on the GPU runs the whole block as one autograd function where that applies
    (_native_block), with the hidden activation's product and rational function in one kernel where that is faster, and inference
    as three kernels that write F2(h) instead of h, or its layers' two without the layers' calls, where that is
    (_native_inference); "never" and "always" leave both to the two
    layers."""

    def __init__(self, dim: int, hidden: int | None = None, groups: int = 8,
                 degrees: Tuple[int, int] = (M_DEGREE, N_DEGREE), fused: str = "inference"):
        super().__init__()
        hidden = 4 * dim if hidden is None else hidden
        # in training a product after the elementwise kernel is the faster route for fc1
        self.fc1 = GRKANLinear(dim, hidden, groups, init="identity", degrees=degrees,
                               fused="never" if fused == "never" else "inference")
        self.fc1._keep_packed = False
        self.fc2 = GRKANLinear(hidden, dim, groups, init="swish", degrees=degrees, fused=fused)

    def forward(self, x):
        out = self._native_block(x)
        if out is None:
            out = self._native_inference(x)
        return self.fc2(self.fc1(x)) if out is None else out

    def _layers_parameters(self):
        """Numerator, denominator, weight and bias of both layers, or None where a layer or a part of one is of another kind."""
        params = []
        for fc in (self._modules.get("fc1"), self._modules.get("fc2")):
            if type(fc) is not GRKANLinear:
                return None
            linear, rational = fc._modules.get("linear"), fc._modules.get("rational")
            if type(linear) is not nn.Linear or type(rational) is not GroupRational:
                return None
            params += [rational._parameters.get("numerator"), rational._parameters.get("denominator"),
                       linear._parameters.get("weight"), linear._parameters.get("bias")]
        return params

    def _plain_calls(self) -> bool:
        """Whether calling the two layers (of the usual kinds) would do nothing else than their parts do."""
        for fc in (self._modules["fc1"], self._modules["fc2"]):
            if not _only_a(GRKANLinear, fc) or fc.fused != "inference":
                return False
            linear, rational = fc._modules["linear"], fc._modules["rational"]
            if not _only_a(nn.Linear, linear) or not _only_a(GroupRational, rational) or "coefficient_rows" in rational.__dict__:
                return False
            if "bias" not in linear._parameters:  # a buffer or a plain tensor, that only linear's own forward reads
                return False
        return True

    def _native_inference(self, x):
        """The block in bfloat16 inference as F1, a product with F2 on its result and a product, or as its layers' two kernels (what
        the layers themselves would run, without their calls), on the parameters as they are; None where neither route is taken
        (as _native_block; in training mode a pass without a gradient takes that one's kernels or the layers, as the pass with
        one does)."""
        if x.dtype is not torch.bfloat16 or torch.is_grad_enabled() or self.training or not x.is_cuda:
            return None
        if torch.compiler.is_compiling() or _autocast_elsewhere():
            return None
        params = self._layers_parameters()
        if params is None:
            return None
        A1, B1, W1, b1, A2, B2, W2, b2 = params
        if A1 is None or B1 is None or W1 is None or A2 is None or B2 is None or W2 is None or not x.dim():
            return None
        # (the look at the sizes first: where the layers are called after all, it is all that this adds to them)
        # (what these are is the native entries' to check)
        dim = x.shape[-1]
        route = _block_route(x.numel() // dim if dim else 0, dim, W1.shape[0], W2.shape[0], B1.shape[0], B2.shape[0],
                             A1.shape[-1], A2.shape[-1])
        if route == "layers" or self._modules["fc1"].training or self._modules["fc2"].training or not self._plain_calls():
            return None
        native = binding.load_native()
        if route == "products":
            return native.block_inference(x, *params)
        h = native.layer_model(x, A1, B1, W1, b1)
        return None if h is None else native.layer_model(h, A2, B2, W2, b2)

    def _native_block(self, x):
        """The block in bfloat16 training as one native autograd function (the hidden activation's product and rational
        function in one kernel each way where that is the faster route), or None where that route is not taken: where calling
        the two layers would do anything else than their parts do, or a parameter or x takes no gradient.  A pass without a
        gradient in training mode may be the first half of one with (reentrant checkpointing): both take the same kernels, and
        in the first x has lost its gradient if anything came before the block.  (Only where x takes none in the second pass
        either, a block right behind an input of a checkpointed segment that needs none, do the two passes differ, by the
        rounding.)"""
        if x.dtype is not torch.bfloat16 or not (x.requires_grad if torch.is_grad_enabled() else self.training):
            return None
        if torch.is_autocast_enabled() or torch.compiler.is_compiling():
            return None
        params = self._layers_parameters()
        if params is None or not self._plain_calls():
            return None
        for i, p in enumerate(params):
            if type(p) is not nn.Parameter and not (p is None and i % 4 == 3):
                return None
        dim = x.shape[-1] if x.dim() else 0
        hidden = params[2].shape[0] if params[2].dim() else 0
        if not dim or not hidden:
            return None
        return binding.load_native().block(x, *params, wgrad_pays(x.numel() // dim, dim, hidden))
