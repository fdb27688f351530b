"""GPU test of grkan_block_bwd: an MLP block's whole backward pass in one call."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

BF16 = 2.0 ** -8  # half a unit in the last place, relative

# rows, D, hidden, G1, G2, tile of the product that F1's backward pass runs in (None: apart, in groups that are not whole
# 16-byte pieces, or above ten million elements of dx)
CASES = [(1, 192, 384, 8, 4, (64, 64)), (1000, 192, 768, 8, 8, (64, 64)), (650, 192, 768, 64, 8, None), (9501, 256, 512, 4, 8, (96, 128)),
         (9501, 384, 1536, 8, 8, (160, 128)), (8207, 640, 2560, 16, 8, (160, 192)), (25001, 256, 1024, 32, 8, (160, 128)),
         (25000, 256, 2048, 8, 8, (160, 128)), (52000, 192, 384, 8, 4, (224, 192)), (52300, 192, 384, 3, 4, None),
         # F2 apart too, at the second both; at the first the product that makes its upstream gradient takes two launches
         (7901, 768, 3072, 8, 8, (160, 192)), (13100, 768, 3072, 8, 8, None)]


class Call(ctypes.Structure):
    _fields_ = ([("rows", ctypes.c_int64)] + [(n, ctypes.c_int32) for n in ("D", "hidden", "G1", "G2", "shared1", "shared2")]
                + [(n, ctypes.c_void_p) for n in ("x", "f1", "h", "f2", "dout", "A1", "B1", "W1", "A2", "B2", "W2", "dx", "dA1", "dB1",
                                                  "dW1", "db1", "dA2", "dB2", "dW2", "db2", "dh")])


def _run(torch, lib, d, sizes, shared, bias):
    rows, D, hidden, G1, G2 = sizes
    like = {"dx": d["x"], "dA1": d["A1"], "dB1": d["B1"], "dW1": d["W1"], "dA2": d["A2"], "dB2": d["B2"], "dW2": d["W2"], "dh": d["h"]}
    out = {k: torch.full_like(v, 7.0) for k, v in like.items()}
    out["db1"], out["db2"] = (torch.full((n,), 7.0, device="cuda:0", dtype=torch.bfloat16) for n in (hidden, D))
    kept = []

    @ctypes.CFUNCTYPE(ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p)
    def alloc(size, _):
        kept.append(torch.full((size,), 0xff, dtype=torch.uint8, device="cuda:0"))  # NaN, so that an unwritten row shows
        return kept[-1].data_ptr()

    address = {k: v.data_ptr() for k, v in {**d, **out}.items()}
    if not bias:
        address["db1"] = address["db2"] = None
    call = Call(rows, D, hidden, G1, G2, shared, shared, **{n: address[n] for n, _ in Call._fields_[7:]})
    lib.grkan_block_bwd.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p]
    assert lib.grkan_block_bwd(ctypes.byref(call), ctypes.cast(alloc, ctypes.c_void_p), None, torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    # beside the partial sums at most one tensor of rows x D: none of the hidden width
    assert sum(t.numel() for t in kept) < 2 * rows * D + 48_000_000
    return out


@pytest.mark.parametrize("rows,D,hidden,G1,G2,tile", CASES)
def test_block_backward(oracle, rows, D, hidden, G1, G2, tile):
    """dx and F1's gradients against the oracle at x with dh W1 from 64 bits, weight and bias gradients against 64 bits, with the
    bounds of the hidden kernels' and the weight gradients' own tests; F2's side bit for bit as from grkan_hidden_bwd where that
    runs, and as from grkan_product and grkan_bwd_model where they do; bit for bit again; one numerator row for all groups."""
    import torch

    from paper_2505_13813_amd import binding

    lib, gen = binding.load_library(), torch.Generator(device="cuda:0")
    gen.manual_seed(rows + D)
    if tile:
        assert binding.grkan_product_tile(rows, hidden, D, 2)[:2] == tile

    def rand(*shape, std=1.0):
        return (torch.randn(*shape, device="cuda:0", generator=gen) * std).to(torch.bfloat16)

    def coefficients(G):
        A = rand(G, 6, std=0.3)
        A[:, 1] += 0.5
        return A, (torch.rand(G, 4, device="cuda:0", generator=gen) * 0.2).to(torch.bfloat16)

    d = dict(x=rand(rows, D), f1=rand(rows, D), h=rand(rows, hidden), f2=rand(rows, hidden), dout=rand(rows, D, std=0.01),
             W1=rand(hidden, D, std=D ** -0.5), W2=rand(D, hidden, std=hidden ** -0.5))
    (d["A1"], d["B1"]), (d["A2"], d["B2"]) = coefficients(G1), coefficients(G2)
    sizes = (rows, D, hidden, G1, G2)
    out = _run(torch, lib, d, sizes, 0, True)
    assert all(torch.isfinite(v.float()).all() for v in out.values())

    dh, W1 = out["dh"].double(), d["W1"].double()
    host = {k: v.double().cpu().numpy() for k, v in {**out, "x": d["x"], "A1": d["A1"], "B1": d["B1"]}.items()}
    exact = (dh @ W1).cpu()
    dF = exact.float().to(torch.bfloat16).double().numpy()
    dF_term = (dh.square() @ W1.square()).sqrt().cpu().numpy()
    dx, rA, rB = oracle.bwd(host["x"], dF, host["A1"], host["B1"], threads=8)
    RA, RB = oracle.scales(host["x"], dF, host["A1"], host["B1"], threads=8)[2:]
    Sdx = oracle.scales(host["x"], np.abs(dF) + dF_term, host["A1"], host["B1"], threads=8)[1]
    assert np.all(np.abs(host["dx"] - dx) <= 3 * BF16 * np.abs(dx) + 2.0 ** -16 * Sdx)
    for got, ref, R in ((host["dA1"], rA, RA), (host["dB1"], rB, RB)):
        assert np.all(np.abs(got - ref) <= BF16 * np.abs(ref) + 1.5e-3 * R)
    for dout, y, dW, db in ((dh, d["f1"].double(), out["dW1"], out["db1"]), (d["dout"].double(), d["f2"].double(), out["dW2"], out["db2"])):
        for got, want, R in ((dW, dout.t() @ y, (dout.square().t() @ y.square()).sqrt()), (db, dout.sum(0), dout.square().sum(0).sqrt())):
            assert ((got.double() - want).abs() <= BF16 * want.abs() + 16 * rows ** 0.5 * 2.0 ** -24 * R).all()

    if lib.grkan_hidden_pays(rows, D, hidden, G2, 1):
        need = lib.grkan_hidden_workspace_bytes(rows, D, hidden, G2)
        ws, each = torch.empty(need, dtype=torch.uint8, device="cuda:0"), [torch.empty_like(out[k]) for k in ("dh", "dA2", "dB2")]
        assert lib.grkan_hidden_bwd(*(d[k].data_ptr() for k in ("dout", "W2", "h", "A2", "B2")), *(t.data_ptr() for t in each), ws.data_ptr(),
                                    need, rows, D, hidden, G2, 0, torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        assert all(torch.equal(t, out[k]) for t, k in zip(each, ("dh", "dA2", "dB2")))

    else:
        dF2, each = torch.empty_like(d["h"]), [torch.empty_like(out[k]) for k in ("dh", "dA2", "dB2")]
        stream, kept = torch.cuda.current_stream().cuda_stream, []

        @ctypes.CFUNCTYPE(ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p)
        def alloc(size, _):
            kept.append(torch.empty(size, dtype=torch.uint8, device="cuda:0"))
            return kept[-1].data_ptr()

        assert lib.grkan_product(d["dout"].data_ptr(), d["W2"].data_ptr(), None, dF2.data_ptr(), rows, D, hidden, 1, None, None, 1, 0, stream) == 0
        exact = d["dout"].double() @ d["W2"].double()
        terms = d["dout"].double().abs() @ d["W2"].double().abs()
        assert ((dF2.double() - exact).abs() <= BF16 * exact.abs() + (D + 1) * 2.0 ** -24 * terms).all()
        del exact, terms
        at = [ctypes.c_void_p(t.data_ptr()) for t in (d["h"], dF2, d["A2"], d["B2"], *each)]
        assert lib.grkan_bwd_model(*at, ctypes.cast(alloc, ctypes.c_void_p), None, ctypes.c_int64(rows), hidden, G2, 5, 4, binding.GRKAN_BF16,
                                   binding.GRKAN_BF16, 0, ctypes.c_void_p(stream)) == 0
        torch.cuda.synchronize()
        for t, k in zip(each, ("dh", "dA2", "dB2")):
            assert torch.equal(t, out[k]), k

    again = _run(torch, lib, d, sizes, 0, False)
    assert all(torch.equal(v, again[k]) for k, v in out.items() if k not in ("db1", "db2"))
    assert (again["db1"] == 7).all() and (again["db2"] == 7).all()

    for k in ("A1", "A2"):
        d[k] = d[k][:1].expand_as(d[k]).contiguous()
    each = _run(torch, lib, d, sizes, 0, True)
    one = _run(torch, lib, {**d, "A1": d["A1"][0].contiguous(), "A2": d["A2"][0].contiguous()}, sizes, 1, True)
    for k in out:
        if k not in ("dA1", "dA2"):
            assert torch.equal(each[k], one[k])
        else:
            sums = each[k].float()
            assert ((sums.sum(0) - one[k].float()).abs() <= BF16 * one[k].float().abs() + 2.0 ** -20 * sums.abs().sum(0)).all()
