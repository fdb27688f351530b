"""GPU tests of the hidden activation's kernels (product and rational function in one, each way) and of the MLP block's
native training route that runs them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

BF16 = 2.0 ** -8  # half a unit in the last place, relative

# rows, K, N, G: one token, ragged last tiles, one tile, fewer tiles than parts, two tiles per part; one and several slabs,
# groups of one and of several wavefronts, more than one group per wavefront's neighbours
SHAPES = [(1, 192, 768, 8), (33, 192, 384, 4), (4133, 192, 768, 2), (31, 256, 256, 8), (2100, 256, 1024, 8), (4111, 256, 768, 24),
          (32, 384, 384, 1), (47, 384, 1536, 8), (2090, 384, 1536, 48), (4001, 384, 768, 8), (75, 512, 512, 4),
          (1040, 640, 768, 8), (531, 768, 1024, 8)]


def _operands(torch, rows, K, N, G):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(rows + K + N + G)

    def rand(*shape, std=1.0):
        return (torch.randn(*shape, device="cuda:0", generator=gen) * std).to(torch.bfloat16)

    A = rand(G, 6, std=0.3)
    A[:, 1] += 0.5
    B = (torch.rand(G, 4, device="cuda:0", generator=gen) * 0.2).to(torch.bfloat16)
    return dict(y=rand(rows, K), W=rand(N, K, std=K ** -0.5), bias=rand(N, std=0.1), A=A, B=B, dout=rand(rows, K, std=0.01),
                W2=rand(K, N, std=N ** -0.5))


def _call(torch, d, rows, K, N, G, shared=False, bias=True):
    from paper_2505_13813_amd import binding

    lib = binding.load_library()
    stream = torch.cuda.current_stream().cuda_stream
    A = d["A"][0].contiguous() if shared else d["A"]
    h, f, dh = (torch.full((rows, N), float("nan"), device="cuda:0", dtype=torch.bfloat16) for _ in range(3))
    dA, dB = torch.empty_like(A), torch.empty_like(d["B"])
    need = lib.grkan_hidden_workspace_bytes(rows, K, N, G)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")
    assert lib.grkan_hidden_fwd(d["y"].data_ptr(), d["W"].data_ptr(), d["bias"].data_ptr() if bias else None, A.data_ptr(),
                                d["B"].data_ptr(), h.data_ptr(), f.data_ptr(), rows, K, N, G, int(shared), stream) == 0
    assert lib.grkan_hidden_bwd(d["dout"].data_ptr(), d["W2"].data_ptr(), h.data_ptr(), A.data_ptr(), d["B"].data_ptr(), dh.data_ptr(),
                                dA.data_ptr(), dB.data_ptr(), ws.data_ptr(), need, rows, K, N, G, int(shared), stream) == 0
    torch.cuda.synchronize()
    return h, f, dh, dA, dB


@pytest.mark.parametrize("rows,K,N,G", SHAPES)
def test_hidden_kernels(oracle, rows, K, N, G):
    """h against the product in 64 bits, f bit for bit against grkan_fwd on h, dh and the coefficient gradients against
    the oracle at h with dF from 64 bits; bit for bit again."""
    import torch

    import paper_2505_13813_amd as grkan

    d = _operands(torch, rows, K, N, G)
    h, f, dh, dA, dB = _call(torch, d, rows, K, N, G)
    w = {k: v.double().cpu().numpy() for k, v in d.items()}
    host = [t.double().cpu().numpy() for t in (h, dh, dA, dB)]
    assert all(np.all(np.isfinite(t)) for t in host)
    # a sum of K products in float32 (about sqrt(K) 2^-24 of the root of the terms' squares; 2^-18 bounds it), rounded once
    want = w["y"] @ w["W"].T + w["bias"]
    term = np.sqrt((w["y"] ** 2) @ (w["W"] ** 2).T + w["bias"] ** 2)
    assert np.all(np.abs(host[0] - want) <= BF16 * np.abs(want) + 2.0 ** -18 * term)
    assert torch.equal(f.view(torch.int16), grkan.grkan_fwd(h, d["A"].float(), d["B"].float()).view(torch.int16))
    # dF rounded to bfloat16; where the float32 sum lies on the other side of a rounding boundary than the one in 64 bits
    # (about one in a thousand: 2^-18 against 2^-8) it is one unit, 2^-7, off
    dF = torch.from_numpy(w["dout"] @ w["W2"]).float().to(torch.bfloat16).double().numpy()
    dF_term = np.sqrt((w["dout"] ** 2) @ (w["W2"] ** 2))
    dx, rA, rB = oracle.bwd(host[0], dF, w["A"], w["B"], threads=8)
    RA, RB = oracle.scales(host[0], dF, w["A"], w["B"], threads=8)[2:]
    Sdx = oracle.scales(host[0], np.abs(dF) + dF_term, w["A"], w["B"], threads=8)[1]
    # one rounding and such a unit; the float32 evaluation, and the float32 sum where it cancels, next to their scales
    assert np.all(np.abs(host[1] - dx) <= 3 * BF16 * np.abs(dx) + 2.0 ** -16 * Sdx)
    # one rounding; units in a thousandth of the terms, sqrt(1e-3) 2^-7 of their scale, six times
    for got, ref, R in ((host[2], rA, RA), (host[3], rB, RB)):
        assert np.all(np.abs(got - ref) <= BF16 * np.abs(ref) + 1.5e-3 * R)
    for one, two in zip((h, f, dh, dA, dB), _call(torch, d, rows, K, N, G)):
        assert torch.equal(one.view(torch.int16), two.view(torch.int16))


def test_shared_numerator_and_no_bias():
    """One numerator row for all groups: the gradient is the groups' rounded ones added in float32; and a product without
    a bias is the one with a bias of zeros."""
    import torch

    rows, K, N, G = 1000, 384, 1536, 8
    d = _operands(torch, rows, K, N, G)
    d["A"] = d["A"][:1].expand(G, 6).contiguous()
    d["bias"] = torch.zeros_like(d["bias"])
    each = _call(torch, d, rows, K, N, G)
    one = _call(torch, d, rows, K, N, G, shared=True, bias=False)
    for i in (0, 1, 2, 4):
        assert torch.equal(each[i], one[i])
    close = (each[3].float().sum(0) - one[3].float()).abs()
    assert bool((close <= BF16 * one[3].float().abs() + 2.0 ** -20 * each[3].float().abs().sum(0)).all())


# Seventeen slabs leave eight parts (one per XCD): four or five tiles for each, the last one ragged.  From the third tile of a part on
# a token buffer is written again after it has been read, and tiles are loaded two ahead.
LONG = [(34 * (16 if K == 768 else 32) + 7, K, 17 * slab, G) for K, slab, G in
        ((192, 384, 17), (256, 256, 34), (384, 384, 51), (512, 256, 17), (640, 256, 8), (768, 256, 34))]


@pytest.mark.parametrize("rows,K,N,G", LONG)
def test_several_tiles_per_part(oracle, rows, K, N, G):
    from paper_2505_13813_amd import binding

    wavefronts = N // G // 32  # of a part that share a group (32 channels each); one row of ten sums for each
    parts = binding.load_library().grkan_hidden_workspace_bytes(rows, K, N, G) // (G * wavefronts * 40)
    tiles = -(-rows // (16 if K == 768 else 32))
    assert parts == 8 and tiles == 35
    test_hidden_kernels(oracle, rows, K, N, G)


@pytest.mark.parametrize("rows,K", [(37, 384), (1, 192), (17, 768), (33, 768), (63, 256)])
def test_tokens_past_the_end_add_nothing(rows, K):
    """The last tile's missing tokens repeat the last one's h and dout in the loads.  With tokens of dout = 0 in their place,
    which add zeros to the same sums, every gradient has the same bits; the last token is the largest, so that each repeat of it
    would show."""
    import torch

    N, G = 4 * K, 8
    d = _operands(torch, rows, K, N, G)
    d["dout"][-1] *= 100.0
    whole = -(-rows // 32) * 32
    more = dict(d, y=torch.cat([d["y"], _operands(torch, whole - rows, K, N, G)["y"]]),
                dout=torch.cat([d["dout"], torch.zeros(whole - rows, K, device="cuda:0", dtype=torch.bfloat16)]))
    got, want = _call(torch, d, rows, K, N, G), _call(torch, more, whole, K, N, G)
    for i in range(3):
        assert torch.equal(got[i], want[i][:rows])
    assert torch.equal(got[3], want[3]) and torch.equal(got[4], want[4])
    # and an infinite token stays among its own outputs
    d["y"][-1], d["dout"][-1] = float("inf"), 0.0
    if rows > 1:
        less = {k: v[:-1].contiguous() if k in ("y", "dout") else v for k, v in d.items()}
        whole, part = _call(torch, d, rows, K, N, G), _call(torch, less, rows - 1, K, N, G)
        for i in range(3):
            assert torch.equal(whole[i][:-1], part[i])


def _block(torch, dim=192, rows=600, bias=True):
    from paper_2505_13813_amd import nn as gnn

    torch.manual_seed(dim)
    block = gnn.KATMlp(dim).to("cuda:0")
    if not bias:
        block.fc1.linear.bias = None
    with torch.no_grad():
        for p in block.parameters():
            p.add_(0.02 * torch.randn_like(p))
    return block.to(torch.bfloat16), torch.randn(2, rows // 2, dim, device="cuda:0").to(torch.bfloat16).requires_grad_()


def _layers(block, x):
    return block.fc2(block.fc1(x))


def _near(got, want):
    """The same function with its sums in another order: in the norm, a few roundings."""
    return float((got.detach().double() - want.detach().double()).norm()) <= 2.0 ** -6 * float(want.detach().double().norm())


@pytest.mark.parametrize("dim,rows,bias", [(192, 600, True), (256, 300, False), (384, 2100, True)])
def test_block_against_its_layers(dim, rows, bias):
    import torch

    block, x = _block(torch, dim, rows, bias)
    leaves = [x] + list(block.parameters())
    y = block(x)
    assert "Block" in y.grad_fn.name()
    dy = 0.01 * torch.randn_like(y)
    want_y = _layers(block, x)
    want = torch.autograd.grad(want_y, leaves, dy)
    got = torch.autograd.grad(y, leaves, dy, retain_graph=True)
    assert _near(y, want_y) and all(g.dtype == w.dtype and g.shape == w.shape and _near(g, w) for g, w in zip(got, want))
    for i, leaf in enumerate(leaves):  # gradients by themselves (a bias's then comes from torch's column sum)
        alone = torch.autograd.grad(y, leaf, dy, retain_graph=True)[0]
        assert torch.equal(alone, got[i]) or (leaf.dim() == 1 and _near(alone, got[i]))


def test_block_leaves_other_calls_to_its_layers():
    import torch

    block, x = _block(torch)
    assert "Block" in block(x).grad_fn.name()
    seen = []
    for part in (block.fc1, block.fc1.rational, block.fc2.linear):
        handle = part.register_forward_hook(lambda *_: seen.append(1))
        assert "Block" not in block(x).grad_fn.name()
        handle.remove()
    assert len(seen) == 3
    for p in (block.fc1.linear.weight, block.fc2.rational.denominator):
        p.requires_grad_(False)
        assert "Block" not in block(x).grad_fn.name()
        p.requires_grad_(True)
    assert "Block" not in block(x.detach()).grad_fn.name()
    with torch.autocast("cuda", dtype=torch.bfloat16):
        assert "Block" not in block(x).grad_fn.name()
    strided = torch.cat([x, x], -1)[..., :x.shape[-1]]
    assert _near(block(strided), _layers(block, x))


@pytest.mark.parametrize("reentrant", [True, False])
def test_block_under_checkpointing(reentrant):
    import torch
    from torch.utils.checkpoint import checkpoint

    block, x = _block(torch)
    leaves = list(block.parameters())
    want_y = block(x)
    dy = torch.randn_like(want_y)
    want = torch.autograd.grad(want_y, [x] + leaves, dy)
    y = checkpoint(block, x, use_reentrant=reentrant)
    assert torch.equal(y, want_y)
    y.backward(dy)
    assert all(torch.equal(p.grad, w) for p, w in zip([x] + leaves, want))


def test_block_saved_tensors_and_graphs_of_the_backward_pass():
    import torch

    block, x = _block(torch)
    leaves = [x] + list(block.parameters())
    y = block(x)
    dy = torch.randn_like(y)
    want = torch.autograd.grad(y, leaves, dy)
    with torch.autograd.graph.save_on_cpu():
        kept = block(x)
    assert all(torch.equal(g, w) for g, w in zip(torch.autograd.grad(kept, leaves, dy), want))
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t, lambda t: t.float()):
        kept = block(x)
    with pytest.raises(TypeError):
        torch.autograd.grad(kept, leaves, dy)
    # a gradient of a gradient that does not differentiate F's own: what the layers give
    W2, W1 = block.fc2.linear.weight, block.fc1.linear.weight

    def second(out):
        g, = torch.autograd.grad(out, W2, dy, create_graph=True)
        return torch.autograd.grad(g.float().pow(2).sum(), W1)[0]

    assert _near(second(block(x)), second(_layers(block, x)))
    # and one that does is refused
    g, = torch.autograd.grad(block(x), x, dy, create_graph=True)
    with pytest.raises(RuntimeError, match="not differentiable twice"):
        g.float().pow(2).sum().backward()


def test_block_in_a_captured_graph():
    import torch

    block, x = _block(torch, 384, 800)
    leaves = [x] + list(block.parameters())
    dy = torch.randn(x.shape, device="cuda:0").to(torch.bfloat16)

    def step():
        y = block(x)
        return (y,) + torch.autograd.grad(y, leaves, dy)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        for _ in range(3):
            step()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        kept = step()
    for seed in range(3):
        with torch.no_grad():
            torch.manual_seed(seed)
            x.copy_(torch.randn_like(x))
        want = [t.clone() for t in step()]
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(k, w) for k, w in zip(kept, want))
