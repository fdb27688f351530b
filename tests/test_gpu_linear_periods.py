"""GPU tests of the small tiles of the fused layer at the lengths of the contraction where their loop can go wrong: every
number of periods around the depth the token operand is loaded ahead, odd and even numbers of 64-k blocks per period,
groups of wavefronts with unequal shares, coefficient groups that end inside a block, and a last channel tile that
starts before its place."""
import pytest

from test_gpu_linear import check, custom_linear_case

pytestmark = pytest.mark.gpu

PERIODS = [
    # rows, D_in, D_out, G, tile
    (16, 512, 260, 2, (16, 64)),      # eight blocks for sixteen wavefronts
    (16, 1024, 64, 32, (16, 64)),     # one each; d_g = 32
    (9, 1088, 132, 17, (16, 64)),     # two for the first; d_g = 64
    (15, 2240, 68, 5, (16, 64)),      # 35 blocks: three for the first three
    (31, 2624, 52, 41, (16, 64)),     # 41 blocks; d_g = 64
    (770, 576, 776, 6, (32, 128)),   # nine blocks for four groups, d_g = 96
    (801, 1280, 500, 40, (32, 128)),  # 20 blocks: five whole periods, d_g = 32
    (3072, 960, 396, 10, (64, 192)),  # 15 blocks: eight periods, the last for one of two groups; d_g = 96
    (3009, 576, 580, 2, (64, 192)),   # nine blocks: five periods, d_g = 288
    (6240, 192, 772, 2, (64, 384)),   # three blocks: a period of two and one of one; d_g = 96
    (6241, 640, 768, 4, (64, 384)),   # ten blocks: five periods; d_g = 160
    (6250, 832, 768, 26, (64, 384)),  # 13 blocks: seven periods, the last of one block; d_g = 32
]


@pytest.mark.parametrize("rows,D_in,D_out,G,tile", PERIODS)
def test_small_tile_periods(oracle, rows, D_in, D_out, G, tile):
    """Every output against the oracle (the gates of the layer's other tests), bit for bit again, and the packed weights
    bit for bit against the plain ones."""
    import torch

    import grkan_inputs
    import paper_2505_13813_amd as grkan

    assert grkan.binding.grkan_linear_tile(rows, D_in, D_out) == tile
    case = custom_linear_case(rows + 7 * D_in + D_out + G, rows, D_in, D_out, G, bias=bool(G % 2))
    check(oracle, case, "bf16" if rows % 2 else "f32", "periods %dx%d -> %d G=%d" % (rows, D_in, D_out, G), threads=8,
          full=True)
    dev = grkan_inputs.upload_linear(case)
    packed_w = grkan.grkan_linear_pack_w(dev["W"])
    plain, again, packed = (grkan.grkan_linear_fwd(dev["x"], dev["A"], dev["B"], w, dev["bias"], out_dtype=torch.float32)
                            for w in (dev["W"], dev["W"], packed_w))
    torch.cuda.synchronize()
    assert torch.equal(plain, again) and torch.equal(plain, packed)
