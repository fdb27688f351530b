"""Performance cases of the GR-KAN layer: what a user of this package has it do,
through its public entry points.

Three kinds of case:
  rational  one forward and one backward pass of the group-wise rational
            function (the activation of a training step), through the module,
            the functional form or the binding on the caller's own buffers
  layer     one forward pass of a GR-KAN layer, out = W F(x) + bias, in bfloat16
            (inference), through the module or the binding
  mlp       the KAT MLP block, in inference or with all gradients

Sizes are those of the paper's model table (KAT-T / S / B: 192 / 384 / 768
channels, hidden width four times that, 197 tokens, 8 groups, 128 images per
GPU), its stress shape, and generic ones with other token counts, group sizes
and batches.  Inputs are standard normal activations, upstream gradients of
standard deviation 0.01, and coefficients away from the initialisation, as in a
trained model.
"""
import math

import torch

import paper_2505_13813_amd as grkan
from paper_2505_13813_amd import nn as gnn

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
DEVICE = "cuda:0"

# work of the largest listed cases: a drawn case stays below
MOST_RATIONAL_BYTES = 5 * 4 * 256 * 197 * 3072
MOST_LAYER_FLOPS = 2 * 128 * 197 * 3072 * 768
MOST_MLP_FLOPS = 6 * 2 * 128 * 197 * 384 * 1536


def _rational(name, dtype, batch, tokens, dim, groups, call, m=5, n=4):
    return {"name": name, "kind": "rational", "dtype": dtype, "batch": batch, "tokens": tokens, "dim": dim,
            "groups": groups, "m": m, "n": n, "call": call}


def _layer(name, batch, tokens, d_in, d_out, groups, call, out):
    return {"name": name, "kind": "layer", "dtype": "bf16", "batch": batch, "tokens": tokens, "d_in": d_in,
            "d_out": d_out, "groups": groups, "call": call, "out": out}


def _mlp(name, batch, tokens, dim, groups, train):
    return {"name": name, "kind": "mlp", "dtype": "bf16", "batch": batch, "tokens": tokens, "dim": dim,
            "groups": groups, "train": train}


def listed():
    return [
        # a debugging or fine-tuning step on a handful of images: launches and host time count
        _rational("tiny f32", "f32", 4, 197, 192, 8, "module"),
        # KAT-T, first layer of the MLP, mixed-precision training: groups of 24 channels (48-byte segments)
        _rational("kat_t fc1 bf16", "bf16", 128, 197, 192, 8, "functional"),
        # KAT-B, second layer, float32 training: the paper's headline tensor, on the caller's buffers
        _rational("kat_b fc2 f32", "f32", 128, 197, 3072, 8, "buffers"),
        # the same layer in mixed precision
        _rational("kat_b fc2 bf16", "bf16", 128, 197, 3072, 8, "functional"),
        # KAT-S, second layer, float16 training with the higher-degree unit
        _rational("kat_s fc2 f16 (7,6)", "f16", 128, 197, 1536, 8, "module", 7, 6),
        # twice the batch with many narrow groups: the largest tensors
        _rational("many groups f32", "f32", 256, 197, 3072, 64, "buffers"),
        # an input of another resolution and a width whose groups are not whole vectors (d_g = 75)
        _rational("ragged f16", "f16", 61, 257, 600, 8, "functional"),
        # KAT-B, second layer, throughput inference
        _layer("layer kat_b fc2 b128", 128, 197, 3072, 768, 8, "module", "bf16"),
        # the same layer on one image: latency inference
        _layer("layer kat_b fc2 b1", 1, 197, 3072, 768, 8, "module", "bf16"),
        # KAT-S, second layer, a serving batch, called through the binding with the model's own weights
        _layer("layer kat_s fc2 b32", 32, 197, 1536, 384, 8, "plain", "bf16"),
        # KAT-B, the whole MLP block on a serving batch
        _mlp("mlp kat_b infer b32", 32, 197, 768, 8, False),
        # KAT-S, the whole MLP block of a training step: output and all gradients
        _mlp("mlp kat_s train b128", 128, 197, 384, 8, True),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["rational"] * 5 + ["layer"] * 4 + ["mlp"] * 2)
    tokens = rng.choice([49, 50, 64, 65, 196, 197, 197, 256, 257, 577])
    batch = _log_int(rng, 1, 256)
    if kind == "rational":
        dtype = rng.choice(["f32", "f32", "bf16", "bf16", "f16"])
        groups = rng.choice([1, 2, 4, 8, 8, 8, 8, 16, 64])
        # channels: a model width in most draws, any group size (odd ones too) in the others
        if rng.random() < 0.65:
            dim = rng.choice([64, 96, 128, 192, 256, 320, 384, 512, 768, 1024, 1152, 1536, 2048, 3072])
            while dim % groups:
                groups //= 2
        else:
            dim = groups * _log_int(rng, 5, max(6, 3072 // groups))
        m, n = rng.choice([(5, 4), (5, 4), (5, 4), (3, 2), (7, 6)])
        size = 4 if dtype == "f32" else 2
        while batch > 1 and 5 * size * batch * tokens * dim > MOST_RATIONAL_BYTES:
            batch -= 1 + batch // 8
        case = _rational("", dtype, max(1, batch), tokens, dim, groups, rng.choice(["module", "functional", "buffers"]), m, n)
    elif kind == "layer":
        groups = rng.choice([1, 2, 4, 8, 8, 8, 8, 16])
        width = rng.choice([32, 64, 96, 96, 128, 192, 192, 256, 384])
        while groups * width > 3072 or (groups * width) % 64:
            groups, width = (groups // 2, width) if groups * width > 3072 else (groups * 2, width)
        d_in = groups * width
        d_out = rng.choice([d_in // 4, d_in // 4, d_in, 4 * d_in if d_in <= 768 else d_in, 192, 384, 768, 1000, 4 * rng.randint(16, 256)])
        d_out = max(16, d_out - d_out % 4)
        while batch > 1 and 2 * batch * tokens * d_in * d_out > MOST_LAYER_FLOPS:
            batch -= 1 + batch // 8
        case = _layer("", max(1, batch), tokens, d_in, d_out, groups, rng.choice(["module", "module", "plain", "packed"]), rng.choice(["bf16", "bf16", "f32"]))
        if case["call"] == "module":
            case["out"] = "bf16"
    else:
        train = rng.random() < 0.5
        dim = rng.choice([192, 256, 384, 512, 640, 768])
        while batch > 1 and (6 if train else 2) * 2 * batch * tokens * dim * 4 * dim > MOST_MLP_FLOPS:
            batch -= 1 + batch // 8
        case = _mlp("", max(1, batch), tokens, dim, 8, train)
    del case["name"]
    return case


# ---------------------------------------------------------------- inputs
def _coefficients(case, gen, groups, m, n, shared, base_a=None, base_b=None, spread_a=1.0, spread_b=0.5):
    """A [G, m+1] (one row when shared) and B [G, n] float32, around `base` or zero.  (Around the Swish base the
    denominators stay positive: a gradient that jumps with the sign of the denominator polynomial would make the
    rounding of the hidden activation, and not the arithmetic, the error of a block's coefficient gradients.)"""
    rows = 1 if shared else groups
    i = torch.arange(1, m + 2, device=DEVICE, dtype=torch.float32)
    j = torch.arange(1, n + 1, device=DEVICE, dtype=torch.float32)
    A = spread_a * (2.0 * torch.rand(rows, m + 1, device=DEVICE, generator=gen) - 1.0) / i
    B = spread_b * (2.0 * torch.rand(groups, n, device=DEVICE, generator=gen) - 1.0)
    if base_a is not None:
        A, B = A / i + base_a, B / (j * j) + base_b
    return (A[0] if shared else A).contiguous(), B.contiguous()


def _near_init(kind, m, n):
    """Coefficients of the two initialisations a trained rational starts from: identity, or a Swish-like unit
    (x / 2 + x^2 / 4 over 1 + x^2 / 12)."""
    a, b = [0.0] * (m + 1), [0.0] * n
    a[1] = 1.0
    if kind == "swish":
        a[1], a[2], b[1] = 0.5, 0.25, 0.085
    return torch.tensor(a, device=DEVICE), torch.tensor(b, device=DEVICE)


def _randn(gen, *shape, std=1.0, dtype=torch.float32):
    return (torch.randn(*shape, device=DEVICE, generator=gen) * std).to(dtype)


def _linear_inputs(gen, d_in, d_out, dtype):
    return {"weight": _randn(gen, d_out, d_in, std=1.0 / math.sqrt(d_in), dtype=dtype),
            "bias": _randn(gen, d_out, std=0.1, dtype=dtype)}


def _inputs(case, seed):
    """Every number the case computes with, from the seed alone."""
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed) * 7919 + 17)
    dtype = DTYPES[case["dtype"]]
    lead = (case["batch"], case["tokens"])
    if case["kind"] == "rational":
        m, n, G = case["m"], case["n"], case["groups"]
        A, B = _coefficients(case, gen, G, m, n, case["call"] == "module")
        return {"x": _randn(gen, *lead, case["dim"], dtype=dtype),
                "dy": _randn(gen, *lead, case["dim"], std=0.01, dtype=dtype), "A": A, "B": B}
    if case["kind"] == "layer":
        module = case["call"] == "module"
        a0, b0 = _near_init("swish", 5, 4)
        A, B = _coefficients(case, gen, case["groups"], 5, 4, module, a0, b0, 0.1, 0.02)
        d = {"x": _randn(gen, *lead, case["d_in"], dtype=dtype), "A": A, "B": B}
        d.update(_linear_inputs(gen, case["d_in"], case["d_out"], dtype))
        if module:  # a module in bfloat16 keeps its coefficients in bfloat16 too
            d["A"], d["B"] = d["A"].to(dtype), d["B"].to(dtype)
        else:
            d["bias"] = d["bias"].to(torch.float32)
        return d
    dim, hidden = case["dim"], 4 * case["dim"]
    d = {"x": _randn(gen, *lead, dim, dtype=dtype), "dy": _randn(gen, *lead, dim, std=0.01, dtype=dtype)}
    for name, start, d_in, d_out in (("fc1", "identity", dim, hidden), ("fc2", "swish", hidden, dim)):
        a0, b0 = _near_init(start, 5, 4)
        A, B = _coefficients(case, gen, case["groups"], 5, 4, True, a0, b0, 0.1, 0.02)
        d[name] = {"A": A.to(dtype), "B": B.to(dtype), **_linear_inputs(gen, d_in, d_out, dtype)}
    return d


def _fill_layer(layer, d):
    with torch.no_grad():
        layer.rational.numerator.copy_(d["A"])
        layer.rational.denominator.copy_(d["B"])
        layer.linear.weight.copy_(d["weight"])
        layer.linear.bias.copy_(d["bias"])


def prepare(case, seed):
    d = _inputs(case, seed)
    dtype = DTYPES[case["dtype"]]
    state = {"case": case, "x": d["x"]}
    if case["kind"] == "rational":
        state["dy"] = d["dy"]
        if case["call"] == "module":
            unit = gnn.GroupRational(case["groups"], degrees=(case["m"], case["n"])).to(DEVICE)
            with torch.no_grad():
                unit.numerator.copy_(d["A"])
                unit.denominator.copy_(d["B"])
            state["unit"], state["x"] = unit, d["x"].requires_grad_()
        elif case["call"] == "functional":
            state["x"] = d["x"].requires_grad_()
            state["A"], state["B"] = d["A"].requires_grad_(), d["B"].requires_grad_()
        else:
            rows, io = case["batch"] * case["tokens"], {"f32": grkan.GRKAN_F32, "bf16": grkan.GRKAN_BF16, "f16": grkan.GRKAN_F16}
            need = grkan.grkan_bwd_workspace_bytes(rows, case["dim"], case["groups"], io[case["dtype"]])
            state.update(A=d["A"], B=d["B"], y=torch.empty_like(d["x"]), dx=torch.empty_like(d["x"]),
                         dA=torch.empty_like(d["A"]), dB=torch.empty_like(d["B"]),
                         workspace=torch.empty(need, dtype=torch.uint8, device=DEVICE))
    elif case["kind"] == "layer":
        if case["call"] == "module":
            layer = gnn.GRKANLinear(case["d_in"], case["d_out"], case["groups"], init="swish").to(DEVICE).to(dtype).eval()
            _fill_layer(layer, d)
            state["layer"] = layer
        else:
            state.update(A=d["A"], B=d["B"], bias=d["bias"],
                         W=grkan.grkan_linear_pack_w(d["weight"]) if case["call"] == "packed" else d["weight"])
    else:
        block = gnn.KATMlp(case["dim"], groups=case["groups"]).to(DEVICE).to(dtype)
        _fill_layer(block.fc1, d["fc1"])
        _fill_layer(block.fc2, d["fc2"])
        state["block"] = block.train(case["train"])
        state["dy"] = d["dy"]
        if case["train"]:
            state["x"] = d["x"].requires_grad_()
            state["params"] = list(block.parameters())
    return state


def run(state):
    case, x = state["case"], state["x"]
    if case["kind"] == "rational":
        if case["call"] == "buffers":
            out = (state["dx"], state["dA"], state["dB"])
            grkan.grkan_fwd(x, state["A"], state["B"], out=state["y"])
            grkan.grkan_bwd(x, state["dy"], state["A"], state["B"], workspace=state["workspace"], out=out)
            return (state["y"],) + out
        if case["call"] == "module":
            y = state["unit"](x)
            return (y.detach(),) + torch.autograd.grad(y, [x, state["unit"].numerator, state["unit"].denominator], state["dy"])
        y = gnn.group_rational(x, state["A"], state["B"])
        return (y.detach(),) + torch.autograd.grad(y, [x, state["A"], state["B"]], state["dy"])
    if case["kind"] == "layer":
        if case["call"] == "module":
            with torch.no_grad():
                return state["layer"](x)
        return grkan.grkan_linear_fwd(x, state["A"], state["B"], state["W"], state["bias"],
                                      out_dtype=torch.float32 if case["out"] == "f32" else torch.bfloat16)
    if not case["train"]:
        with torch.no_grad():
            return state["block"](x)
    y = state["block"](x)
    return (y.detach(),) + torch.autograd.grad(y, [x] + state["params"], state["dy"])


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    rows = case["batch"] * case["tokens"]
    size = 4 if case["dtype"] == "f32" else 2
    if case["kind"] == "rational":
        m, n = case["m"], case["n"]
        elems = rows * case["dim"]
        # x in each direction, dy in, y and dx out; the paper's count forward, and powers, derivatives and sums backward
        return {"bytes": 5 * size * elems, "flops": elems * ((2 * m + 2 * n + 3) + (6 * m + 6 * n + 8))}
    if case["kind"] == "layer":
        d_in, d_out = case["d_in"], case["d_out"]
        return {"bytes": rows * d_in * 2 + d_in * d_out * 2 + rows * d_out * (4 if case["out"] == "f32" else 2),
                "flops": 2 * rows * d_in * d_out}
    dim = case["dim"]
    product = 2 * rows * dim * 4 * dim
    if not case["train"]:
        return {"bytes": 2 * (2 * rows * dim + 8 * dim * dim), "flops": 2 * product}
    # x, dy in, y, dx out, weights in, their gradients out; the hidden activation out and back in
    return {"bytes": 2 * (4 * rows * dim + 16 * dim * dim + 2 * 4 * rows * dim), "flops": 6 * product}


def tolerance(case):
    # about four times what is measured against 64 bits: sums in 32 bits, results rounded once to the storage type
    if case["kind"] == "rational":
        return {"f32": {"rel": 1e-5, "max": 1e-3}, "bf16": {"rel": 7e-3, "max": 0.1}, "f16": {"rel": 1e-3, "max": 0.02}}[case["dtype"]]
    if case["kind"] == "layer":
        return {"rel": 1e-2, "max": 0.1}
    return {"rel": 2e-2, "max": 0.3}


# ---------------------------------------------------------------- the same in 64 bits
def _exact_rational(x, dy, A, B, G):
    """F and, with dy, its gradients in float64: x [rows, D], A [G, m+1], B [G, n]; in blocks of rows."""
    rows, D = x.shape
    dg = D // G
    a = [A[:, i].double().repeat_interleave(dg) for i in range(A.shape[1])]
    b = [B[:, j].double().repeat_interleave(dg) for j in range(B.shape[1])]
    y = torch.empty(rows, D, dtype=torch.float64, device=x.device)
    dx = torch.empty_like(y) if dy is not None else None
    dA = torch.zeros(G, len(a), dtype=torch.float64, device=x.device)
    dB = torch.zeros(G, len(b), dtype=torch.float64, device=x.device)
    step = max(1, (1 << 24) // D)
    for lo in range(0, rows, step):
        t = x[lo:lo + step].double()
        p = torch.zeros_like(t) + a[-1]
        for c in reversed(a[:-1]):
            p = p * t + c
        h = torch.zeros_like(t) + b[-1]
        for c in reversed(b[:-1]):
            h = h * t + c
        h = h * t
        q = 1.0 + h.abs()
        y[lo:lo + step] = p / q
        if dy is None:
            continue
        d = dy[lo:lo + step].double()
        dp = sum(i * a[i] * t ** (i - 1) for i in range(1, len(a)))
        dh = sum((j + 1) * b[j] * t ** j for j in range(len(b)))
        w = torch.sign(h) * p / (q * q)
        dx[lo:lo + step] = d * (dp / q - w * dh)
        for i in range(len(a)):
            dA[:, i] += (d / q * t ** i).sum(0).view(G, dg).sum(1)
        for j in range(len(b)):
            dB[:, j] -= (d * w * t ** (j + 1)).sum(0).view(G, dg).sum(1)
    return y, dx, dA, dB


def exact(case, seed):
    d = _inputs(case, seed)
    lead = (case["batch"], case["tokens"])
    G = case["groups"]

    def rows_of(A):
        return A.expand(G, A.shape[-1]) if A.dim() == 1 else A

    if case["kind"] == "rational":
        D = case["dim"]
        y, dx, dA, dB = _exact_rational(d["x"].view(-1, D), d["dy"].view(-1, D), rows_of(d["A"]), d["B"], G)
        return y.view(*lead, D), dx.view(*lead, D), dA.sum(0) if d["A"].dim() == 1 else dA, dB
    if case["kind"] == "layer":
        f = _exact_rational(d["x"].view(-1, case["d_in"]), None, rows_of(d["A"]), d["B"], G)[0]
        return (f @ d["weight"].double().t() + d["bias"].double()).view(*lead, case["d_out"])
    dim, one, two = case["dim"], d["fc1"], d["fc2"]
    x = d["x"].view(-1, dim)
    W1, W2 = one["weight"].double(), two["weight"].double()
    f1 = _exact_rational(x, None, rows_of(one["A"]), one["B"], G)[0]
    h = f1 @ W1.t() + one["bias"].double()
    f2 = _exact_rational(h, None, rows_of(two["A"]), two["B"], G)[0]
    y = (f2 @ W2.t() + two["bias"].double()).view(*lead, dim)
    if not case["train"]:
        return y
    dy = d["dy"].view(-1, dim).double()
    _, dh, dA2, dB2 = _exact_rational(h, dy @ W2, rows_of(two["A"]), two["B"], G)
    _, dx, dA1, dB1 = _exact_rational(x, dh @ W1, rows_of(one["A"]), one["B"], G)
    # the order of the block's parameters: each layer's numerator, denominator, weight, bias
    return (y, dx.view(*lead, dim), dA1.sum(0), dB1, dh.t() @ f1, dh.sum(0), dA2.sum(0), dB2, dy.t() @ f2, dy.sum(0))
