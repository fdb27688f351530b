"""Which calls of the MLP block and of its layers take the native routes, without a GPU: the native entries are replaced by ones
that note their arguments."""
import types

import pytest
import torch

from paper_2505_13813_amd import nn as gnn


@pytest.fixture
def entries(monkeypatch):
    """Calls of the native entries, as (name, arguments); all of them answer with the first argument."""
    calls = []

    def entry(name):
        def call(*args):
            calls.append((name, args))
            return args[0]
        return call

    native = types.SimpleNamespace(**{name: entry(name) for name in ("block", "rational", "product", "layer_model")})
    monkeypatch.setattr(gnn.binding, "load_native", lambda: native)
    return calls


def _block(**kwargs):
    return gnn.KATMlp(64, **kwargs).to(torch.bfloat16)


def _x(requires_grad=True):
    return torch.randn(16, 64).to(torch.bfloat16).requires_grad_(requires_grad)


def _foreign_bias(linear, kind):
    """A bias that linear.bias finds and that is no parameter."""
    bias = linear.bias.detach() + 1.0
    del linear.bias
    if kind == "buffer":
        linear.register_buffer("bias", bias)
    else:
        linear.bias = bias
    assert linear.bias is bias and "bias" not in linear._parameters


def test_block_with_parameters_alone(entries):
    block, x = _block(), _x()
    block(x)
    (name, args), = entries
    assert name == "block" and args[0] is x and args[4] is block.fc1.linear.bias and args[8] is block.fc2.linear.bias
    block.fc1.linear.bias = block.fc2.linear.bias = None  # layers without a bias
    del entries[:]
    block(x)
    (name, args), = entries
    assert name == "block" and args[4] is None and args[8] is None


@pytest.mark.parametrize("fc", ["fc1", "fc2"])
@pytest.mark.parametrize("kind", ["buffer", "tensor"])
def test_block_leaves_a_bias_that_is_no_parameter_to_its_layers(entries, fc, kind):
    block = _block()
    _foreign_bias(getattr(block, fc).linear, kind)
    assert block._native_block(_x()) is None and not entries


@pytest.mark.parametrize("kind", [None, "buffer", "tensor"])
@pytest.mark.parametrize("fused", ["inference", "always"])
def test_layer_leaves_a_bias_that_is_no_parameter_to_its_parts(entries, monkeypatch, fused, kind):
    monkeypatch.setattr(gnn, "_fused_shapes", lambda *_: True)  # (x is not on the GPU)
    monkeypatch.setattr(gnn, "one_kernel_is_faster", lambda *_: True)
    layer = gnn.GRKANLinear(64, 64, 2, fused=fused).to(torch.bfloat16).eval()
    layer._keep_packed = False
    if kind is not None:
        _foreign_bias(layer.linear, kind)
    x = _x(False)
    with torch.no_grad():
        out = layer(x)
    if kind is None:
        assert [name for name, _ in entries] == ["layer_model"] and entries[0][1][4] is layer.linear.bias
    else:
        assert [name for name, _ in entries] == ["rational"] and torch.equal(out, layer.linear(x))


def test_never_fused_is_never_fused(entries):
    """fused="never": neither layer's product is in one kernel with a rational function, in training as in inference."""
    block = _block(fused="never")
    for train in (True, False):
        for grad in (True, False):
            with torch.set_grad_enabled(grad):
                block.train(train)(_x())
    assert entries and {name for name, _ in entries} <= {"rational", "product"}
    block = _block()
    block.fc2.fused = "never"  # on one layer
    assert block._native_block(_x()) is None


def test_passes_without_a_gradient(entries):
    """In training mode they take the block, whether or not x has lost its gradient; in evaluation mode the layers."""
    block = _block()
    for requires_grad in (True, False):
        del entries[:]
        with torch.no_grad():
            block.train()(_x(requires_grad))
            assert [name for name, _ in entries] == ["block"]
            assert block.eval()._native_block(_x(requires_grad)) is None
    assert block.train()._native_block(_x(False)) is None  # with a graph, and no gradient wanted for x


def test_where_the_hidden_kernels_pay():
    """Small calls always (a launch less); large ones by the compute units that get a workgroup, 8 * (32 / slabs) * slabs."""
    from paper_2505_13813_amd import binding

    lib = binding.load_library()
    for rows, K, N, forward, backward in (
            (25216, 192, 768, 1, 1), (25216, 384, 1536, 1, 1), (50432, 256, 1024, 1, 1), (50432, 512, 2048, 1, 1),
            (50432, 640, 2560, 1, 1),                           # 240 units
            (6304, 768, 3072, 1, 1), (25216, 768, 3072, 1, 0),  # 192 units, which is enough for the forward kernel
            (50432, 768, 1536, 1, 1),                           # 240
            (12608, 768, 4352, 0, 0), (5000, 768, 4352, 1, 1),  # 136
            (12608, 512, 4352, 0, 0), (12608, 640, 5120, 0, 0), (12608, 256, 4352, 1, 0),
            (25216, 384, 7680, 1, 0), (25216, 192, 4608, 1, 1),
            (25216, 320, 1280, 0, 0)):                          # not built
        G = 8
        assert lib.grkan_hidden_supported(K, N, G) == (K != 320)
        assert (lib.grkan_hidden_pays(rows, K, N, G, 0), lib.grkan_hidden_pays(rows, K, N, G, 1)) == (forward, backward), (rows, K, N)
