"""GPU tests of the C++ autograd route of the rational function: the same results as the Python functions over
the same kernels, the model's coefficients as they are kept, and what is left to the Python route."""
import pytest

pytestmark = pytest.mark.gpu


def _inputs(torch, rows, D, G, m, n, dtype, seed=0):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(seed + rows * 31 + D)
    x = torch.randn(rows, D, device="cuda:0", generator=gen).to(dtype)
    dy = torch.randn(rows, D, device="cuda:0", generator=gen).to(dtype)
    A = (2 * torch.rand(G, m + 1, device="cuda:0", generator=gen) - 1) / torch.arange(1, m + 2, device="cuda:0")
    B = torch.rand(G, n, device="cuda:0", generator=gen) - 0.5
    return x, dy, A, B


SHAPES = [(1, 8, 1), (197, 192, 8), (129, 3072, 8), (65, 35, 5), (300, 768, 64), (1000, 768, 1)]


@pytest.mark.parametrize("dtype", ["float32", "bfloat16", "float16"])
@pytest.mark.parametrize("rows,D,G", SHAPES)
def test_same_bits_as_the_python_function(rows, D, G, dtype):
    import torch

    from paper_2505_13813_amd import nn as gnn

    for m, n in ((5, 4), (7, 6)):
        x, dy, A, B = _inputs(torch, rows, D, G, m, n, getattr(torch, dtype))
        leaves = [t.requires_grad_() for t in (x, A, B)]
        y = gnn.group_rational(*leaves)
        ref = gnn.GroupRationalFunction.apply(*leaves)
        assert "GroupRationalFunction" not in y.grad_fn.name() and "GroupRationalFunction" in ref.grad_fn.name()
        assert torch.equal(y, ref)
        for g, r in zip(torch.autograd.grad(y, leaves, dy), torch.autograd.grad(ref, leaves, dy)):
            assert g.dtype == r.dtype and torch.equal(g, r)


@pytest.mark.parametrize("coef", ["float32", "bfloat16"])
@pytest.mark.parametrize("rows,D,G", SHAPES)
def test_shared_numerator_and_bfloat16_coefficients(rows, D, G, coef):
    """The module's parameters as they are against their expanded float32 rows through the Python function: the
    same outputs, the numerator's gradient summed over the groups (float32: in double, 2^-22 of the magnitudes'
    sum; bfloat16: of the groups' rounded gradients, rounded once more: 2^-8 of the value)."""
    import torch

    from paper_2505_13813_amd import nn as gnn

    unit = gnn.GroupRational(G).to("cuda:0")
    x, dy, A, B = _inputs(torch, rows, D, G, 5, 4, getattr(torch, coef))
    with torch.no_grad():
        unit.numerator.copy_(A[0])
        unit.denominator.copy_(B)
    unit = unit.to(getattr(torch, coef))
    x.requires_grad_()
    y = unit(x)
    got = torch.autograd.grad(y, [x, unit.numerator, unit.denominator], dy)
    rows_A, rows_B = (t.detach().to(torch.float32).contiguous().requires_grad_() for t in unit.coefficient_rows())
    ref = gnn.GroupRationalFunction.apply(x, rows_A, rows_B)
    dx, dA, dB = torch.autograd.grad(ref, [x, rows_A, rows_B], dy)
    assert torch.equal(y, ref) and torch.equal(got[0], dx)
    assert got[1].dtype == unit.numerator.dtype and got[1].shape == unit.numerator.shape
    assert torch.equal(got[2], dB.to(unit.denominator.dtype))
    want = dA.to(unit.numerator.dtype).double().sum(0)
    bound = 2.0 ** -22 * dA.abs().sum(0).double() + (2.0 ** -8 * want.abs() if coef == "bfloat16" else 0.0)
    assert bool(((got[1].double() - want).abs() <= bound + 1e-30).all())


def test_views_empty_inputs_and_hooks():
    import torch

    from paper_2505_13813_amd import nn as gnn

    x, dy, A, B = _inputs(torch, 64, 96, 4, 5, 4, torch.float32)
    # a strided input, and an upstream gradient without memory of its own (the sum's)
    wide = torch.randn(64, 192, device="cuda:0").requires_grad_()
    y = gnn.group_rational(wide[:, ::2], A, B)
    (g,) = torch.autograd.grad(y.sum(), [wide])
    (r,) = torch.autograd.grad(gnn.GroupRationalFunction.apply(wide[:, ::2], A, B).sum(), [wide])
    assert torch.equal(g, r)
    assert gnn.group_rational(x[:0], A, B).shape == (0, 96)
    # float32 activations with bfloat16 coefficients are converted first
    unit = gnn.GroupRational(4).to("cuda:0").to(torch.bfloat16)
    rows_A, rows_B = (t.detach().to(torch.float32).contiguous() for t in unit.coefficient_rows())
    assert torch.equal(unit(x), gnn.GroupRationalFunction.apply(x, rows_A, rows_B))
    # saved tensors go through the caller's hooks, and changing one before the backward pass is an error
    packed = []
    with torch.autograd.graph.saved_tensors_hooks(lambda t: (packed.append(t.shape), t)[1], lambda t: t):
        y = gnn.group_rational(x.clone().requires_grad_(), A, B)
    assert len(packed) == 3
    y.backward(dy)
    z = x.clone().requires_grad_()
    w = z * 1.0
    y = gnn.group_rational(w, A, B)
    w.add_(1.0)
    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        y.backward(dy)


def test_calls_left_to_the_python_route_are_refused_as_before():
    import torch

    from paper_2505_13813_amd import nn as gnn

    x, _, A, B = _inputs(torch, 16, 96, 4, 5, 4, torch.float32)
    with pytest.raises(TypeError):
        gnn.group_rational(x, A.to(torch.bfloat16), B.to(torch.bfloat16))
    with pytest.raises(ValueError):
        gnn.group_rational(x.cpu(), A, B)
    with pytest.raises(gnn.binding.GrkanError):
        gnn.group_rational(x[:, :95].contiguous(), A, B)
    with pytest.raises(RuntimeError):
        torch.func.vmap(lambda t: gnn.group_rational(t, A, B))(torch.stack([x, x]))
    with pytest.raises(Exception):
        torch.func.jvp(lambda t: gnn.group_rational(t, A, B), (x,), (x,))
