"""The sign of the denominator polynomial in the backward pass, at and next to its zeros: s = sign(Aden) is 0 exactly where
Aden is 0 (x = 0, and a root elsewhere) and +-1 at the smallest numbers on either side, also where they are subnormal."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# smallest positive number of each type
TINY = {"f32": 2.0 ** -149, "bf16": 2.0 ** -133, "f16": 2.0 ** -24}


@pytest.mark.parametrize("m,n", [(5, 4), (3, 2), (7, 6)])
@pytest.mark.parametrize("io", ["f32", "bf16", "f16"])
def test_sign_of_the_denominator_polynomial(io, m, n):
    import paper_2505_13813_amd as grkan

    dtype = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[io]
    tiny = TINY[io]
    # P = 1 + x / 4, Aden = x - x^2: zero at 0 and at 1
    values = np.array([0.0, -0.0, 1.0, tiny, -tiny, 5 * tiny, -5 * tiny, 2.0 ** -14, -2.0 ** -14, 0.5, 2.0])
    D = 16
    x64 = np.resize(values, (len(values), D))  # every value in every column position
    A = torch.zeros(1, m + 1)
    A[0, 0], A[0, 1] = 1.0, 0.25
    B = torch.zeros(1, n)
    B[0, 0], B[0, 1] = 1.0, -1.0
    x = torch.tensor(x64).to(dtype).cuda()
    assert np.array_equal(x.double().cpu().numpy(), x64)
    dx, dA, dB = grkan.grkan_bwd(x, torch.ones_like(x), A.cuda(), B.cuda())

    aden = x64 - x64 * x64
    s, q, p = np.sign(aden), 1.0 + np.abs(aden), 1.0 + 0.25 * x64
    ref = 0.25 / q - s * (1.0 - 2.0 * x64) * p / (q * q)
    got = dx.double().cpu().numpy()
    exact = (np.abs(x64) < 1e-9) | (x64 == 1.0)
    assert exact.sum() > D
    assert np.array_equal(got[exact], ref[exact])  # 0.25, -0.75 and 1.25: Q is 1 within float32
    # elsewhere: one rounding to the type (8 or 11 bits), some float32 roundings before it
    unit = {"f32": 2.0 ** -20, "bf16": 2.0 ** -8, "f16": 2.0 ** -10}[io]
    assert np.all(np.abs(got - ref) <= unit * np.maximum(np.abs(ref), 1.0))
    for j in range(1, n + 1):
        terms = -(x64 ** j) * s * p / (q * q)
        assert abs(float(dB[0, j - 1]) - terms.sum()) <= 2.0 ** -18 * np.abs(terms).sum()
