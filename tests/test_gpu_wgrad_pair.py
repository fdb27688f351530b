"""GPU test of grkan_linear_wgrad_pair: the weight and bias gradients of two products over the same rows."""
import pytest

pytestmark = pytest.mark.gpu

# rows, (D_in, D_out) of both: one row; around one stage; the last stage partial and alone behind whole ones (buffers wrap);
# more and fewer tiles in the second, partial tiles, one range of rows and many
CASES = [(1, (8, 8), (200, 16)), (65, (192, 200), (192, 192)), (257, (64, 768), (768, 64)), (320, (192, 192), (8, 400)),
         (3001, (384, 1536), (1536, 384)), (8199, (200, 8), (192, 192)), (640, (1536, 1536), (1536, 1600)),
         (10001, (1536, 1632), (1632, 1536)), (16001, (1896, 1096), (1632, 1536))]  # each in a launch of its own


@pytest.mark.parametrize("bias", [(True, True), (False, True), (True, False)])
@pytest.mark.parametrize("rows,first,second", CASES)
def test_pair(rows, first, second, bias):
    """Against 64 bits, with the bound of grkan_linear_wgrad's own test: one rounding to bfloat16, and sums in 32 bits, 16
    sqrt(rows) 2^-24 of the root-sum-square of the terms; bit for bit again; nothing written past the ends."""
    import torch

    from paper_2505_13813_amd import binding

    lib, gen = binding.load_library(), torch.Generator(device="cuda:0")
    gen.manual_seed(rows)
    sizes, args, outs, pairs = (first, second), [], [], []
    for (D_in, D_out), want_b in zip(sizes, bias):
        dout, y = (torch.randn(rows, d, device="cuda:0", generator=gen).to(torch.bfloat16) for d in (D_out, D_in))
        dW, db = (torch.full((n + 8,), 7.0, device="cuda:0", dtype=torch.bfloat16) for n in (D_in * D_out, D_out))
        args += [dout.data_ptr(), y.data_ptr(), dW.data_ptr(), db.data_ptr() if want_b else None, D_in, D_out]
        outs += [dW, db]
        pairs.append((dout, y))
    need = lib.grkan_linear_wgrad_pair_workspace_bytes(rows, *first, *second)
    each = [lib.grkan_linear_wgrad_workspace_bytes(rows, *size) for size in sizes]
    apart = need == sum(each)
    if rows > 9000:
        assert apart
    ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")

    def run():
        assert lib.grkan_linear_wgrad_pair(*args, ws.data_ptr(), need, rows, torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        return [t.clone() for t in outs]

    got = run()
    assert all(torch.equal(a, b) for a, b in zip(got, run()))
    for k, ((dout, y), (D_in, D_out)) in enumerate(zip(pairs, sizes)):
        d, v = dout.double(), y.double()
        for g, want, R, wanted in ((got[2 * k][:-8].view(D_out, D_in), d.t() @ v, (d.square().t() @ v.square()).sqrt(), True),
                                   (got[2 * k + 1][:-8], d.sum(0), d.square().sum(0).sqrt(), bias[k])):
            if wanted:
                assert ((g.double() - want).abs() <= 2.0 ** -8 * want.abs() + 16 * rows ** 0.5 * 2.0 ** -24 * R).all()
            else:
                assert (g == 7).all()
        assert (got[2 * k][-8:] == 7).all() and (got[2 * k + 1][-8:] == 7).all()
    assert lib.grkan_linear_wgrad_pair(*args, ws.data_ptr(), need - 16, rows, None) == 5
    if apart:  # the same row ranges as each by itself: the same bits
        for k, (D_in, D_out) in enumerate(sizes):
            at = args[6 * k:6 * k + 4]
            outs[2 * k].fill_(7.0)
            assert lib.grkan_linear_wgrad(*at, ws.data_ptr(), each[k], rows, D_in, D_out, binding.GRKAN_BF16,
                                          torch.cuda.current_stream().cuda_stream) == 0
            assert torch.equal(outs[2 * k], got[2 * k]) and torch.equal(outs[2 * k + 1], got[2 * k + 1])
