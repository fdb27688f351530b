"""GPU tests of where the C++ autograd route meets Python: exceptions keep their types, saved-tensor hooks and
checkpointing see what they saw before, and what is not a plain tensor stays with the Python functions."""
import pytest

pytestmark = pytest.mark.gpu


def _unit(torch, dtype, D=96, G=4):
    from paper_2505_13813_amd import nn as gnn

    torch.manual_seed(0)
    unit = gnn.GroupRational(G, "swish").to("cuda:0").to(dtype)
    return unit, torch.randn(600, D, device="cuda:0").to(dtype).requires_grad_()


def _layer(torch):
    from paper_2505_13813_amd import nn as gnn

    torch.manual_seed(1)
    layer = gnn.GRKANLinear(192, 392, 2, init="swish").to("cuda:0").to(torch.bfloat16)
    return layer, torch.randn(3, 200, 192, device="cuda:0").to(torch.bfloat16).requires_grad_()


@pytest.mark.parametrize("early_stop", [True, False])
def test_checkpointing_with_saved_tensor_hooks(early_stop):
    """Non-reentrant checkpointing ends its recomputation with an exception of its own out of a saved-tensor hook,
    which has to come back as it is."""
    import torch
    from torch.utils.checkpoint import checkpoint, set_checkpoint_early_stop

    for part, x in (_unit(torch, torch.float32), _unit(torch, torch.bfloat16), _layer(torch)):
        leaves = [x] + list(part.parameters())
        want_y = part(x)
        dy = torch.randn_like(want_y)
        want = torch.autograd.grad(want_y, leaves, dy)
        with set_checkpoint_early_stop(early_stop):
            y = checkpoint(part, x, use_reentrant=False)
        got = torch.autograd.grad(y, leaves, dy)
        assert torch.equal(y, want_y) and all(torch.equal(g, w) for g, w in zip(got, want))


def test_exceptions_keep_their_types():
    import torch

    import paper_2505_13813_amd as grkan
    from paper_2505_13813_amd import binding

    class Refused(Exception):
        pass

    def refuse(t):
        raise Refused("no")

    for part, x in (_unit(torch, torch.float32), _layer(torch)):
        with pytest.raises(Refused), torch.autograd.graph.saved_tensors_hooks(refuse, lambda t: t):
            part(x)
        with torch.autograd.graph.saved_tensors_hooks(lambda t: t, refuse):
            y = part(x)
        with pytest.raises(Refused):
            y.sum().backward()

    unit, _ = _unit(torch, torch.float32, 3072, 8)
    big = torch.zeros(1 << 15, 3072, device="cuda:0")
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (64 << 20)) / total)
    try:
        with pytest.raises(torch.OutOfMemoryError):
            unit(big)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)


def test_a_status_of_the_library_is_a_grkan_error():
    import torch

    import paper_2505_13813_amd as grkan
    from paper_2505_13813_amd import binding

    x = torch.zeros(16, 64, device="cuda:0", dtype=torch.bfloat16)
    A, B = torch.zeros(2, 6, device="cuda:0"), torch.zeros(2, 4, device="cuda:0")
    pw = grkan.grkan_linear_pack_w(torch.zeros(64, 64, device="cuda:0", dtype=torch.bfloat16))
    with torch.no_grad(), pytest.raises(grkan.GrkanError) as e:
        binding.load_native().layer_packed(x, A, B, pw.data, 62, None, -1)   # not a multiple of 4: refused on the host
    assert e.value.status == 8


def test_subclasses_and_function_modes_stay_with_the_python_functions():
    """A tensor subclass comes back as one, a function mode sees the linear layer's call; a default device (which is
    a function mode too) changes nothing."""
    import torch
    from torch.overrides import TorchFunctionMode

    from paper_2505_13813_amd import nn as gnn

    class Tagged(torch.Tensor):
        pass

    class Log(TorchFunctionMode):
        def __init__(self):
            super().__init__()
            self.seen = []

        def __torch_function__(self, func, types, args=(), kwargs=None):
            self.seen.append(getattr(func, "__name__", str(func)))
            return func(*args, **(kwargs or {}))

    for dtype in (torch.float32, torch.bfloat16):
        unit, x = _unit(torch, dtype)
        tagged = x.detach().as_subclass(Tagged)
        A, B = (t.detach().float().contiguous() for t in unit.coefficient_rows())
        assert type(unit(tagged)) is Tagged and type(gnn.group_rational(tagged, A, B)) is Tagged
        assert torch.equal(unit(tagged), unit(x))
    layer, x = _layer(torch)
    want = layer(x)
    assert "Product" in want.grad_fn.name()
    with Log() as log:
        got = layer(x)
    assert "linear" in log.seen and torch.equal(got, want)
    layer.eval()
    with torch.no_grad(), Log() as log:
        got = layer(x)
    assert "linear" in log.seen and torch.equal(got, want)
    with torch.device("cuda:0"):
        assert "Product" in layer(x).grad_fn.name()


def test_what_saved_tensor_hooks_return_is_checked():
    """The backward pass reads what the caller's hooks give back by address: tensors of another layout, type, size or
    device are refused as the Python function refuses them (the product's are left to torch)."""
    import torch

    from paper_2505_13813_amd import binding
    from paper_2505_13813_amd import nn as gnn

    strided = lambda t: t.new_empty(*t.shape, 2)[..., 0].copy_(t)
    for change in (strided, lambda t: t.cpu(), lambda t: t.half(), lambda t: t[:1], lambda t: t.flatten(), lambda t: t[0]):
        x, A, B = (torch.randn(*s, device="cuda:0", requires_grad=True) for s in ((64, 96), (4, 6), (4, 4)))
        for which in range(3):
            def unpack(packed):
                i, t = packed
                return change(t) if i == which else t

            for route in (gnn.group_rational, gnn.GroupRationalFunction.apply):
                order = iter(range(3))
                with torch.autograd.graph.saved_tensors_hooks(lambda t: (next(order), t), unpack):
                    y = route(x, A, B)
                with pytest.raises((ValueError, TypeError, RuntimeError)):
                    y.sum().backward()

    y = torch.randn(600, 96, device="cuda:0").to(torch.bfloat16).requires_grad_()
    W = torch.randn(64, 96, device="cuda:0").to(torch.bfloat16).requires_grad_()
    dout = torch.randn(600, 64, device="cuda:0").to(torch.bfloat16)
    want = torch.autograd.grad(torch.nn.functional.linear(y, W), [W], dout)[0]
    for change in (lambda t: t, strided, lambda t: t.cpu(), lambda t: t.float(), lambda t: t[:8]):
        with torch.autograd.graph.saved_tensors_hooks(lambda t: t, lambda t: change(t) if t.shape == y.shape else t):
            out = binding.load_native().product(y, W, None)
        if change(y).shape == y.shape and change(y).is_cuda and change(y).dtype == y.dtype:
            (got,) = torch.autograd.grad(out, [W], dout)
            assert float((got.float() - want.float()).norm()) <= 2.0 ** -7 * float(want.float().norm())
        else:
            with pytest.raises(RuntimeError):
                torch.autograd.grad(out, [W], dout)


def test_the_product_saves_what_torchs_linear_saves():
    """A weight whose input takes no gradient may be written to between the passes (an optimizer step in between two
    backward passes); an expanded upstream gradient (a sum's) and each subset of wanted gradients."""
    import torch

    from paper_2505_13813_amd import binding

    y = torch.randn(4, 150, 96, device="cuda:0").to(torch.bfloat16)
    W = torch.randn(64, 96, device="cuda:0").to(torch.bfloat16).requires_grad_()
    b = torch.randn(64, device="cuda:0").to(torch.bfloat16).requires_grad_()
    near = lambda g, w: float((g.float() - w.float()).norm()) <= 2.0 ** -7 * float(w.float().norm())
    out = binding.load_native().product(y, W, b)
    want = torch.autograd.grad(torch.nn.functional.linear(y, W, b).sum(), [W, b])
    with torch.no_grad():
        W.add_(1.0)
    got = torch.autograd.grad(out.sum(), [W, b])
    assert all(near(g, w) for g, w in zip(got, want))

    leaves = [y.clone().requires_grad_(), W, b]
    for chosen in ([0], [1], [2], [0, 2], [0, 1, 2]):
        inputs = [leaves[i] for i in chosen]
        got = torch.autograd.grad(binding.load_native().product(*leaves).sum(), inputs)
        want = torch.autograd.grad(torch.nn.functional.linear(*leaves).sum(), inputs)
        assert all(g.shape == w.shape and near(g, w) for g, w in zip(got, want))
    out = binding.load_native().product(leaves[0], W.detach(), None)
    assert near(torch.autograd.grad(out.sum(), [leaves[0]])[0], torch.autograd.grad(
        torch.nn.functional.linear(leaves[0], W.detach()).sum(), [leaves[0]])[0])


def test_a_second_derivative_is_refused():
    """create_graph=True gives the first derivatives; differentiating them raises instead of leaving out their
    dependence on x and the coefficients (a gradient penalty through a layer, say)."""
    import torch

    from paper_2505_13813_amd import nn as gnn

    x, A, B = (torch.randn(*s, device="cuda:0", requires_grad=True) for s in ((64, 96), (4, 6), (4, 4)))
    dy = torch.randn(64, 96, device="cuda:0", requires_grad=True)
    for route in (gnn.group_rational, gnn.GroupRationalFunction.apply):
        first = torch.autograd.grad(route(x, A, B), [x, A, B], dy)
        again = torch.autograd.grad(route(x, A, B), [x, A, B], dy, create_graph=True)
        assert all(torch.equal(f, g) and not f.requires_grad for f, g in zip(first, again))
        for g in again:
            with pytest.raises(RuntimeError, match="not differentiable twice"):
                torch.autograd.grad(g.sum(), [x, dy], allow_unused=True, retain_graph=True)

    for fused in ("inference", "always"):
        layer, x = _layer(torch)
        layer.fused = fused
        out = layer(x)
        (dx,) = torch.autograd.grad(out.float().square().sum(), [x], create_graph=True)
        with pytest.raises(RuntimeError, match="not differentiable twice"):
            (out.float().sum() + dx.float().square().sum()).backward()
        # the weight's gradient is differentiable: out = F(x) W^T, dW = up^T F(x)
        up = torch.randn_like(out).requires_grad_()
        (dW,) = torch.autograd.grad(layer(x), [layer.linear.weight], up, create_graph=True)
        du, dx = torch.autograd.grad(dW.float().sum(), [up, x])
        f = layer.rational(x)
        want_u = f.float().sum(-1, keepdim=True).expand_as(up)
        (want_x,) = torch.autograd.grad(f, [x], up.detach().float().sum(-1, keepdim=True).expand_as(f).to(f.dtype))
        for got, want in ((du, want_u), (dx, want_x)):
            assert float((got.float() - want.float()).norm()) <= 2e-2 * float(want.float().norm())


def _step(torch, block, x, dy):
    y = block(x)
    return (y.detach(),) + torch.autograd.grad(y, [x] + list(block.parameters()), dy)


def test_streams_threads_and_capture():
    """A training step of the block on a stream of its own behind work that makes its input, in two threads at once,
    and captured in a graph: the bits of the eager step on the default stream."""
    import threading

    import torch

    from paper_2505_13813_amd import nn as gnn

    torch.manual_seed(2)
    block = gnn.KATMlp(256, groups=4).to("cuda:0").to(torch.bfloat16)
    inputs = [torch.randn(700, 256, device="cuda:0").to(torch.bfloat16) for _ in range(4)]
    dy = torch.randn(700, 256, device="cuda:0").to(torch.bfloat16)
    want = [_step(torch, block, t.clone().requires_grad_(), dy) for t in inputs]
    same = lambda got, ref: all(torch.equal(g, r) for g, r in zip(got, ref))
    torch.cuda.synchronize()

    results = [None] * len(inputs)

    def on_a_stream(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            x = torch.zeros_like(inputs[i])
            torch.cuda._sleep(5_000_000)
            x.copy_(inputs[i])
            results[i] = _step(torch, block, x.requires_grad_(), dy)
            torch.cuda.current_stream().synchronize()

    threads = [threading.Thread(target=on_a_stream, args=(i,)) for i in range(len(inputs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert all(same(got, ref) for got, ref in zip(results, want))

    x = inputs[0].clone().requires_grad_()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        _step(torch, block, x, dy)
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = _step(torch, block, x, dy)
    for t, ref in zip(inputs + inputs, want + want):
        with torch.no_grad():
            x.copy_(t)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert same(out, ref)
        assert same(_step(torch, block, t.clone().requires_grad_(), dy), ref)
