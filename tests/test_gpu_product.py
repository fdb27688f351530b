"""GPU tests of grkan_product (the products of an MLP block, with and without the rational function on the result) and of the
block's inference route that runs them."""
import pytest

pytestmark = pytest.mark.gpu

BF16 = 2.0 ** -8  # half a unit in the last place, relative

# rows, K, N, G, (tile, workgroups per unit): every tile; one row, ragged rows and channels, one stage of 64 and fewer stages than
# buffers, whole tiles, more than one round, a second launch for the last rows, groups of 8 channels
SIZES = [(1, 64, 8, 1, (64, 64, 1)), (130, 192, 200, 25, (64, 64, 1)), (3000, 128, 72, 3, (64, 64, 1)),
         (1570, 128, 1544, 193, (96, 128, 1)), (1570, 2048, 768, 8, (96, 128, 1)), (4700, 320, 768, 96, (160, 128, 1)),
         (4480, 1088, 776, 97, (160, 128, 1)), (3100, 128, 1000, 125, (160, 128, 2)), (9500, 192, 1000, 5, (160, 128, 2)),
         (30000, 64, 1544, 193, (160, 128, 2)), (4100, 960, 1544, 193, (160, 192, 1)), (9500, 192, 760, 1, (160, 192, 1)),
         (25209, 960, 384, 8, (224, 192, 1)), (12501, 256, 1544, 193, (224, 192, 1)), (4100, 128, 3072, 8, (256, 256, 1)),
         (12501, 256, 1000, 125, (256, 256, 1)), (6304, 768, 3072, 8, (320, 256, 1)), (25001, 704, 760, 5, (320, 256, 1)),
         (7001, 320, 3072, 8, (320, 256, 1, 6720)), (30000, 768, 760, 95, (320, 256, 1, 27200)),
         (30000, 1088, 384, 8, (224, 192, 1, 28672))]


def _operands(torch, rows, K, N, G):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(rows + K + N + G)

    def rand(*shape, std=1.0):
        return (torch.randn(*shape, device="cuda:0", generator=gen) * std).to(torch.bfloat16)

    A = rand(G, 6, std=0.3)
    return dict(x=rand(rows, K), W=rand(N, K, std=K ** -0.5), bias=rand(N, std=0.1), A=A,
                B=(torch.rand(G, 4, device="cuda:0", generator=gen) * 0.2).to(torch.bfloat16))


def _product(torch, x, W, bias, transposed=False, A=None, B=None, guard=3):
    """out, from a buffer whose rows behind it keep what was there."""
    from paper_2505_13813_amd import binding

    rows, K = x.shape
    N = W.shape[1 if transposed else 0]
    full = torch.full((rows + guard, N), 7.0, device=x.device, dtype=x.dtype)
    at = [t.data_ptr() if t is not None else None for t in (x, W, bias)]
    G, shared = (B.shape[0], A.dim() == 1) if A is not None else (1, 0)
    st = binding.load_library().grkan_product(*at, full.data_ptr(), rows, K, N, int(transposed), A.data_ptr() if A is not None else None,
                                              B.data_ptr() if B is not None else None, G, int(shared),
                                              torch.cuda.current_stream().cuda_stream)
    assert st == 0
    torch.cuda.synchronize()
    assert (full[rows:] == 7).all()
    return full[:rows]


@pytest.mark.parametrize("rows,K,N,G,tile", SIZES)
def test_product(rows, K, N, G, tile):
    """Both orders of W against 64 bits (one rounding to bfloat16, and sums in 32 bits: at most (K + 1) 2^-24 of the
    terms' magnitudes), bit for bit again; F element by element against 64 bits, and bit for bit against grkan_fwd on the rounded product
    where both run in the same tile."""
    import torch

    from paper_2505_13813_amd import binding

    assert binding.grkan_product_tile(rows, K, N) == tile + ((rows,) if len(tile) == 3 else ())
    d = _operands(torch, rows, K, N, G)
    x, W, bias = d["x"], d["W"], d["bias"]
    want = x.double() @ W.double().t() + bias.double()
    terms = x.double().abs() @ W.double().abs().t() + bias.double().abs()
    Wt = W.t().contiguous()
    out = _product(torch, x, W, bias)
    for got in (out, _product(torch, x, Wt, bias, True)):
        assert ((got.double() - want).abs() <= BF16 * want.abs() + (K + 1) * 2.0 ** -24 * terms).all()
    assert torch.equal(out, _product(torch, x, W, bias))
    bare = _product(torch, x, W, None)
    bound = BF16 * (want - bias.double()).abs() + (K + 1) * 2.0 ** -24 * terms
    assert ((bare.double() - (want - bias.double())).abs() <= bound).all()

    # F(h) for h within `off` of the exact product: off by no more than off times the slope's bound, with Q >= 1
    # |F'| <= sum i |a_i| m^(i-1) + sum |a_i| m^i sum j |b_j| m^(j-1) for |h| <= m, and one rounding
    off = BF16 * want.abs() + (K + 1) * 2.0 ** -24 * terms
    m = want.abs() + off

    def bound_of_f(A):
        a, b = (t.double().repeat_interleave(N // G, 0).t() for t in ((A if A.dim() == 2 else A.expand(G, 6)), d["B"]))
        num = sum(a[i] * want ** i for i in range(6))
        exact = num / (1 + sum(b[j] * want ** (j + 1) for j in range(4)).abs())
        slope = (sum(i * a[i].abs() * m ** (i - 1) for i in range(1, 6))
                 + sum(a[i].abs() * m ** i for i in range(6)) * sum((j + 1) * b[j].abs() * m ** j for j in range(4)))
        return exact, off * slope + 2 * BF16 * exact.abs() + 2.0 ** -20 * sum(a[i].abs() * m ** i for i in range(6))

    # (the tile may be another one with F, and its sums in another order: the same bits where it is the same)
    with_f = binding.grkan_product_tile(rows, K, N, True) == binding.grkan_product_tile(rows, K, N)
    for A in (d["A"], d["A"][0].contiguous()):
        f = _product(torch, x, W, bias, A=A, B=d["B"])
        exact, bound = bound_of_f(A)
        assert ((f.double() - exact).abs() <= bound).all()
        if with_f:
            rows_of_A = (A if A.dim() == 2 else A.expand(G, 6)).float().contiguous()
            import paper_2505_13813_amd as grkan

            assert torch.equal(f, grkan.grkan_fwd(out.contiguous(), rows_of_A, d["B"].float().contiguous()))


def _block(torch, dim, bias=True, shared=True):
    from paper_2505_13813_amd import nn as gnn

    torch.manual_seed(dim)
    block = gnn.KATMlp(dim)
    for fc, init in ((block.fc1, "identity"), (block.fc2, "swish")):
        if not shared:
            fc.rational = gnn.GroupRational(8, init, shared_numerator=False)
        if not bias:
            fc.linear.bias = None
    block = block.to("cuda:0").to(torch.bfloat16)
    with torch.no_grad():
        for p in block.parameters():
            p.add_(torch.randn_like(p) * 0.01)
    return block.eval()


@pytest.mark.parametrize("dim,rows,bias,shared", [(192, 197, True, True), (256, 1300, False, True), (384, 2500, True, False), (768, 6304, True, True)])
def test_block_inference(dim, rows, bias, shared, monkeypatch):
    """Taken at these sizes; bit for bit its parts (each with tests of its own values), and row by row near the layers one by one (the
    hidden activation's bfloat16 roundings may fall differently: a few units of bfloat16 over each row), no graph, strided input, and in a
    captured graph, replayed with the eager call between."""
    import torch

    from paper_2505_13813_amd import binding

    block = _block(torch, dim, bias, shared)
    x = torch.randn(2, rows // 2, dim, device="cuda:0").to(torch.bfloat16)
    native, calls = binding.load_native(), []

    class Counting:
        def __getattr__(self, name):
            entry = getattr(native, name)
            return entry if name != "block_inference" else lambda *args: calls.append(1) or entry(*args)

    monkeypatch.setattr(binding, "load_native", lambda: Counting())
    with torch.no_grad():
        out = block(x)
        assert len(calls) == 1
        want = block.fc2(block.fc1(x))
        assert out.shape == x.shape
        assert ((out.double() - want.double()).norm(dim=-1) <= 4 * BF16 * want.double().norm(dim=-1)).all()
        one, two = block.fc1, block.fc2
        f2 = _product(torch, one.rational(x).view(-1, dim), one.linear.weight, one.linear.bias, A=two.rational.numerator, B=two.rational.denominator)
        assert torch.equal(out.view(-1, dim), _product(torch, f2, two.linear.weight, two.linear.bias))
        strided = torch.stack((x, x), dim=-1)[..., 0]
        assert not strided.is_contiguous() and torch.equal(block(strided), out)
    with torch.inference_mode():
        assert torch.equal(block(x), out)
    graph, z = torch.cuda.CUDAGraph(), x.clone()
    with torch.no_grad(), torch.cuda.graph(graph):
        captured = block(z)
    for i in range(3):
        with torch.no_grad():
            z.copy_(torch.randn_like(x))
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(captured, block(z)), i


def test_block_inference_is_left_to_the_layers(monkeypatch):
    """Where calling the layers would do anything else: hooks, training, other types, a gradient wanted, fused='never'."""
    import torch

    from paper_2505_13813_amd import nn as gnn

    block = _block(torch, 192)
    x = torch.randn(300, 192, device="cuda:0").to(torch.bfloat16)
    with torch.no_grad():
        assert block._native_inference(x) is not None
        seen = []
        hook = block.fc1.register_forward_hook(lambda m, i, o: seen.append(o.shape))
        assert block._native_inference(x) is None
        block(x)
        hook.remove()
        assert seen == [(300, 768)]
        assert block._native_inference(x.float()) is None
        block.fc2.train()
        assert block._native_inference(x) is None
        block.eval()
        assert gnn.KATMlp(192, fused="never").to("cuda:0").to(torch.bfloat16).eval()._native_inference(x) is None
        assert gnn.KATMlp(192, degrees=(3, 2)).to("cuda:0").to(torch.bfloat16).eval()._native_inference(x) is None
        with torch.autocast("cuda", dtype=torch.float16):
            assert block._native_inference(x) is None
        assert block._native_inference(x[:0]) is None
    assert block._native_inference(x) is None


@pytest.mark.parametrize("D,rows", [(512, 1), (512, 394), (768, 197)])
def test_block_inference_as_its_layers_kernels(D, rows):
    """Few rows: bit for bit what the two layers give, with strided rows and in a captured graph too; what the kernel does not take is
    left to the layers."""
    import torch

    from paper_2505_13813_amd import nn as gnn

    assert gnn._block_route(rows, D, 4 * D, D, 8, 8, 6, 6) == "models"
    block = _block(torch, D)
    x = torch.randn(2, rows, D, device="cuda:0").to(torch.bfloat16)
    with torch.no_grad():
        want = block.fc2(block.fc1(x[0]))
        assert torch.equal(block._native_inference(x[0]), want) and torch.equal(block(x[0]), want)
        strided = torch.stack((x[0], x[1]), dim=-1)[..., 0]
        assert not strided.is_contiguous() and torch.equal(block(strided), want)
        graph, z = torch.cuda.CUDAGraph(), x[0].clone()
        with torch.cuda.graph(graph):
            captured = block(z)
        for i in range(3):
            z.copy_(torch.randn_like(z))
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(captured, block(z)), i
        block.fc2.linear.weight.data = torch.cat([block.fc2.linear.weight.data.flatten(), x.flatten()[:1]])[1:].view(D, 4 * D)
        assert block._native_inference(x[0]) is None and block(x[0]).shape == (rows, D)  # misaligned weights


@pytest.mark.parametrize("K,N,G,rows,bias,shared", [(192, 768, 8, 300, True, True), (512, 2048, 8, 9001, False, True), (320, 72, 8, 77, True, False)])
def test_layer_inference_through_the_product(K, N, G, rows, bias, shared, monkeypatch):
    """At sizes of this route: bit for bit the rational function and the product, which the layer's two modules agree with."""
    import torch

    from paper_2505_13813_amd import binding
    from paper_2505_13813_amd import nn as gnn

    assert gnn._layer_route(rows, K, N, G, 6, True) == "product"
    torch.manual_seed(K)
    layer = gnn.GRKANLinear(K, N, G, init="swish", bias=bias, shared_numerator=shared).to("cuda:0").to(torch.bfloat16).eval()
    x = torch.randn(rows, K, device="cuda:0").to(torch.bfloat16)
    with torch.no_grad():
        for p in layer.parameters():
            p.add_(torch.randn_like(p) * 0.01)
        out = layer(x)
        f = layer.rational(x)
        assert torch.equal(out, _product(torch, f, layer.linear.weight, layer.linear.bias))
        want = layer.linear(f)
        assert (out.double() - want.double()).norm() <= 2 * BF16 * want.double().norm()
        assert torch.equal(layer(x.view(1, rows, K)[0]), out) and layer(x.view(1, rows, K)).shape == (1, rows, N)
        hook = layer.linear.register_forward_hook(lambda m, i, o: o + 1)
        assert torch.equal(layer(x), want + 1)
        hook.remove()
    graph, z = torch.cuda.CUDAGraph(), x.clone()
    with torch.no_grad(), torch.cuda.graph(graph):
        captured = layer(z)
    for _ in range(3):
        with torch.no_grad():
            z.copy_(torch.randn_like(x))
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(captured, layer(z))
