"""The rule of grkan_linear_wgrad_pair without a GPU: one launch for both products, or one for each."""
import pytest

from paper_2505_13813_amd import binding


def _apart(rows, dim, hidden):
    """Whether both products get the row ranges, and so the workspace, that each has by itself where one launch would have fewer."""
    lib = binding.load_library()
    each = [lib.grkan_linear_wgrad_workspace_bytes(rows, *size) for size in ((dim, hidden), (hidden, dim))]
    both = lib.grkan_linear_wgrad_pair_workspace_bytes(rows, dim, hidden, hidden, dim)
    assert both and both <= sum(each)
    return both == sum(each)


@pytest.mark.parametrize("rows,dim,hidden", [(25216, 512, 4096), (25216, 640, 3328), (25216, 768, 3328), (25216, 768, 3584), (12608, 768, 3840),
                                             (25216, 384, 7680), (12608, 256, 6400), (50432, 256, 4096), (50432, 768, 2048)])
def test_two_launches_where_one_would_leave_units_idle(rows, dim, hidden):
    """Tiles of 192 x 192 of one product: 44 at the last two (two ranges of rows for both, five for each), 66 - 80 at the others (one
    for both, three for each)."""
    assert _apart(rows, dim, hidden) and not _apart(1600, dim, hidden)


@pytest.mark.parametrize("dim,hidden", [(192, 768), (384, 1536), (512, 2048)])
def test_one_launch_where_both_fill_the_chip(dim, hidden):
    assert not _apart(25216, dim, hidden)


def test_one_launch_for_the_same_ranges():
    """768 -> 3072: 64 tiles each, two ranges for both and four for each: as many stages in a row either way."""
    lib = binding.load_library()
    both = lib.grkan_linear_wgrad_pair_workspace_bytes(50432, 768, 3072, 3072, 768)
    assert both == lib.grkan_linear_wgrad_workspace_bytes(50432, 768, 3072)


def test_rows_that_a_range_can_count():
    """2^36 rows are 2^31 stages of 32: one range of them is one too many, 256 ranges are not."""
    lib = binding.load_library()
    assert lib.grkan_linear_wgrad_workspace_bytes(1 << 36, 8, 8) and not lib.grkan_linear_wgrad_workspace_bytes(1 << 36, 3072, 3072)
    assert lib.grkan_linear_wgrad_workspace_bytes(1 << 35, 3072, 3072) and not lib.grkan_linear_wgrad_workspace_bytes((1 << 36) + 1, 8, 8)
    assert not lib.grkan_linear_wgrad_pair_workspace_bytes(1 << 36, 2048, 2048, 2048, 2048)
    assert lib.grkan_linear_wgrad(16, 16, 16, None, 16, 1 << 40, 1 << 36, 3072, 3072, binding.GRKAN_BF16, None) == 8
