"""GPU tests of grkan_linear_wgrad (dW = dOut^T Y, dbias = column sums of dOut) against float64, and of
the route the module takes to it in training."""
import numpy as np
import pytest

import grkan_inputs

pytestmark = pytest.mark.gpu

SHAPES = [
    # rows, D_in, D_out          what it exercises
    (1, 8, 8),                 # one row: a single, almost empty stage
    (63, 192, 192), (64, 192, 192), (65, 192, 200),   # around one stage; one tile and a sliver of a second
    (129, 184, 392),           # two and a bit stages, partial tiles in both directions
    (191, 24, 576),            # three stages, the last one partial
    (1030, 384, 192),          # several row ranges, two tiles, ragged end
    (4096, 200, 1000),         # whole stages only, partial tiles
    (2000, 1536, 384),         # 16 tiles
    (8200, 192, 192),          # one tile, many row ranges
]


def _bf16(rng, *shape):
    bits = grkan_inputs.round_to_bf16_bits(rng.standard_normal(shape).astype(np.float32))
    return bits, grkan_inputs.bf16_bits_to_f32(bits).astype(np.float64)


def _device(bits):
    import torch

    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).to("cuda:0").view(torch.bfloat16)


@pytest.mark.parametrize("bias", [True, False])
@pytest.mark.parametrize("rows,D_in,D_out", SHAPES)
def test_weight_gradient_shapes(rows, D_in, D_out, bias):
    """Every element: one rounding to bfloat16 (2^-9 of the value) plus float32 accumulation, whose error is
    about sqrt(rows) 2^-24 of the root-sum-square R of the summed terms; 16 of those are allowed."""
    import torch

    import paper_2505_13813_amd as grkan

    rng = np.random.default_rng(rows + 3 * D_in + 7 * D_out)
    db_bits, d = _bf16(rng, rows, D_out)
    y_bits, y = _bf16(rng, rows, D_in)
    dout, yt = _device(db_bits), _device(y_bits)
    first = grkan.grkan_linear_wgrad(dout, yt, bias)
    again = grkan.grkan_linear_wgrad(dout, yt, bias)
    torch.cuda.synchronize()
    assert torch.equal(first[0].view(torch.int16), again[0].view(torch.int16))
    acc = 16 * np.sqrt(rows) * 2.0 ** -24

    def close(got, want, R):
        got = got.to(torch.float32).cpu().numpy().astype(np.float64)
        assert got.shape == want.shape
        assert np.all(np.abs(got - want) <= 2.0 ** -8 * np.abs(want) + acc * R), np.max(np.abs(got - want) / R)

    close(first[0], d.T @ y, np.sqrt((d ** 2).T @ (y ** 2)))
    if bias:
        close(first[1], d.sum(0), np.sqrt((d ** 2).sum(0)))
        assert torch.equal(first[1].view(torch.int16), again[1].view(torch.int16))
    else:
        assert first[1] is None


def test_rows_past_the_end_and_non_finite_values_stay_where_they_are():
    """Rows after the last must not enter the sums (they are infinities here), and a NaN in one column of Y
    reaches that column of dW only."""
    import torch

    import paper_2505_13813_amd as grkan

    rng = np.random.default_rng(3)
    rows, D_in, D_out = 100, 40, 208
    d_all = torch.full((rows + 64, D_out), float("inf"), device="cuda:0", dtype=torch.bfloat16)
    y_all = torch.full((rows + 64, D_in), float("inf"), device="cuda:0", dtype=torch.bfloat16)
    d_all[:rows] = _device(_bf16(rng, rows, D_out)[0])
    y_all[:rows] = _device(_bf16(rng, rows, D_in)[0])
    y_all[7, 5] = float("nan")
    dW, db = grkan.grkan_linear_wgrad(d_all[:rows], y_all[:rows])
    torch.cuda.synchronize()
    nan = torch.isnan(dW)
    assert bool(nan[:, 5].all()) and int(nan.sum()) == D_out
    assert bool(torch.isfinite(db).all())
    empty_W, empty_b = grkan.grkan_linear_wgrad(d_all[:0], y_all[:0])
    assert not empty_W.any() and not empty_b.any()


def test_weight_gradient_rejects_what_it_does_not_cover():
    import torch

    import paper_2505_13813_amd as grkan

    z = lambda *s, dtype=torch.bfloat16: torch.zeros(*s, device="cuda:0", dtype=dtype)
    with pytest.raises(grkan.GrkanError) as e:
        grkan.grkan_linear_wgrad(z(16, 12), z(16, 64))     # D_out is not a multiple of 8
    assert e.value.status == 8
    with pytest.raises(ValueError):
        grkan.grkan_linear_wgrad(z(16, 64, dtype=torch.float32), z(16, 64))
    with pytest.raises(ValueError):
        grkan.grkan_linear_wgrad(z(16, 64), z(15, 64))
    with pytest.raises(ValueError):
        grkan.grkan_linear_wgrad(z(64, 16).t(), z(16, 64))


def test_module_training_route_matches_torchs_linear():
    """The layer's gradients through the native product against the same layer through torch's own linear (one
    rounding each); frozen parameters; a differentiable backward pass; hooks on the linear layer keep it called."""
    import torch

    from paper_2505_13813_amd import nn as gnn

    torch.manual_seed(4)
    layer = gnn.GRKANLinear(192, 392, 2, init="swish").to("cuda:0").to(torch.bfloat16)
    x = torch.randn(3, 200, 192, device="cuda:0").to(torch.bfloat16).requires_grad_()
    dy = torch.randn(3, 200, 392, device="cuda:0").to(torch.bfloat16)
    params = [x] + list(layer.parameters())
    out = layer(x)
    assert "Product" in out.grad_fn.name()
    got = torch.autograd.grad(out, params, dy)

    calls = []
    handle = layer.linear.register_forward_hook(lambda *a: calls.append(1))
    ref_out = layer(x)
    assert calls and "Product" not in ref_out.grad_fn.name()
    ref = torch.autograd.grad(ref_out, params, dy)
    handle.remove()
    assert torch.equal(out, ref_out)
    for g, r in zip(got, ref):
        assert g.dtype == r.dtype and g.shape == r.shape
        assert float((g.float() - r.float()).norm()) <= 2.0 ** -7 * float(r.float().norm()) + 1e-6

    # a graph of the backward pass: dW as a function of the upstream gradient
    up = dy.clone().requires_grad_()
    out = layer(x)
    (dW,) = torch.autograd.grad(out, [layer.linear.weight], up, create_graph=True)
    (second,) = torch.autograd.grad(dW.sum(), [up])
    assert second.shape == up.shape and bool(second.abs().sum() > 0)

    layer.linear.weight.requires_grad_(False)
    out = layer(x)
    (dx,) = torch.autograd.grad(out, [x], dy)
    assert torch.equal(dx, got[0])
