"""The overlapped walk (groups that are not whole vectors): its cover on the host, and its results on the GPU
against the oracle and against the narrow walk that calls with shared memory take."""
import random

import pytest

import paper_2505_13813_amd as grkan
from paper_2505_13813_amd import GRKAN_BF16, GRKAN_F16, GRKAN_F32


def test_cover_of_random_shapes():
    """Every element stored by lanes of its own group, counted once, nothing outside: awkward group sizes, row
    counts and device sizes; and the rule takes every d_g that holds a 16-byte vector and is not a whole number of
    them (backward: of 8-byte vectors)."""
    rng = random.Random(75)
    taken = 0
    for trial in range(400):
        io = rng.choice([GRKAN_F32, GRKAN_BF16, GRKAN_F16])
        es = 4 if io == GRKAN_F32 else 2
        G = rng.choice([1, 2, 3, 5, 7, 8, 16, 33])
        dg = rng.choice([1, 2, 3, 5, 7, 8, 9, 10, 11, 13, 15, 17, 25, 31, 33, 50, 63, 75, 97, 125, 130, 145, 250, 383])
        rows = rng.choice([1, 2, 3, 17, 64, 65, 200, 301])
        if rows * G * dg > 300_000:
            rows = max(1, 300_000 // (G * dg))
        cu, wg = rng.choice([(256, 3), (256, 8), (8, 1), (1, 1), (64, 7)])
        forward = rng.random() < 0.5
        errors = grkan.binding.overlapped_cover_errors(rows, G * dg, G, io, cu, wg, forward)
        vec = 16 // es
        divides = next(v for v in (vec, vec // 2, vec // 4, 1) if v and dg % v == 0)
        if divides * es > (8 if forward else 4) or dg < vec:
            assert errors == -2, (rows, G, dg, io)
        else:
            assert errors in (0, -2), (trial, rows, G, dg, io, cu, wg, errors)  # -2: columns cannot be fixed
            taken += errors == 0
    assert taken > 80
    assert grkan.binding.overlapped_cover_errors(0, 600, 8, GRKAN_F16) == -2


SHAPES = [(1, 75, 1), (3, 600, 8), (197, 600, 8), (2000, 600, 8), (129, 9 * 33, 33), (300, 8 * 11, 8), (64, 2 * 383, 2), (501, 130, 1), (333, 8 * 12, 8), (90, 4 * 100, 4)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("rows,D,G", SHAPES)
def test_against_the_oracle_and_the_narrow_walk(oracle, rows, D, G, dtype):
    import torch

    from parity_util import assert_parity, run_gpu, run_oracle, to_device
    from test_gpu_parity import custom_case

    for m, n in ((5, 4), (7, 6)):
        case = custom_case(rows * 7919 + D + m, rows, D, G, dtype, m=m, n=n)
        gpu = run_gpu(case)
        assert_parity(gpu, run_oracle(oracle, case, threads=4), dtype, label="overlapped %dx%d G=%d %s" % (rows, D, G, dtype))

    # y over x and dx over dy share memory: the narrow walk.  Same elements, so the same y and dx; also from
    # tensors that start at an odd element
    from paper_2505_13813_amd import binding

    A, B = (torch.tensor(case[k], device="cuda:0") for k in ("A", "B"))
    for off in (0, 1):
        flat = {k: torch.empty(rows * D + off, device="cuda:0", dtype=getattr(torch, {"f32": "float32", "bf16": "bfloat16", "f16": "float16"}[dtype]))
                for k in ("x", "dy")}
        x, dy = (flat[k][off:].view(rows, D) for k in ("x", "dy"))
        x.copy_(torch.tensor(case["x"]))
        dy.copy_(torch.tensor(case["dy"]))
        y = binding.grkan_fwd(x, A, B)
        dx, dA, dB = binding.grkan_bwd(x, dy, A, B)
        x2, dy2 = x.clone(), dy.clone()
        narrow = binding.grkan_bwd(x2, dy2, A, B, out=(dy2, torch.empty_like(A), torch.empty_like(B)))
        binding.grkan_fwd(x2, A, B, out=x2)
        torch.cuda.synchronize()
        for got, want in ((y, x2), (dx, narrow[0])):
            if dtype == "f16":
                # one variant may convert and multiply in one instruction where the other uses two: a float32
                # result next to a rounding boundary falls to either side, one unit in the last place (2^-10, or
                # the subnormal spacing 2^-24)
                assert bool(((got.float() - want.float()).abs() <= 2.0 ** -10 * want.float().abs() + 2.0 ** -24).all())
            else:
                assert torch.equal(got, want)
        # the sums differ by their order only: 2^-20 of the magnitudes' root-sum-square is far above that
        again = binding.grkan_bwd(x, dy, A, B)
        assert all(torch.equal(p, q) for p, q in zip(again, (dx, dA, dB))) and torch.equal(binding.grkan_fwd(x, A, B), y)
        for g, r in ((dA, narrow[1]), (dB, narrow[2])):
            assert float((g - r).norm()) <= 1e-5 * float(r.norm()) + 1e-20


@pytest.mark.gpu
def test_non_finite_elements_are_counted_once():
    """An infinity or NaN among the repeated elements (64 .. 71 of 75 sit in two vectors) reaches the sums of its
    own group and only once: the other groups stay finite."""
    import torch

    from paper_2505_13813_amd import binding

    x = torch.randn(50, 600, device="cuda:0")
    dy = torch.randn(50, 600, device="cuda:0")
    A, B = torch.rand(8, 6, device="cuda:0"), torch.rand(8, 4, device="cuda:0")
    x[3, 2 * 75 + 73] = float("nan")
    x[9, 5 * 75 + 72] = float("inf")
    _, dA, dB = binding.grkan_bwd(x, dy, A, B)
    finite = torch.isfinite(dA).all(1) & torch.isfinite(dB).all(1)
    assert finite.tolist() == [g not in (2, 5) for g in range(8)]
