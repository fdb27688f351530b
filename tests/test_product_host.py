"""grkan_product without a GPU: what it refuses, and the rule for its tile."""
import ctypes

import pytest

from paper_2505_13813_amd import binding
from paper_2505_13813_amd import nn as gnn


def test_product_rejects_on_the_host():
    lib = binding.load_library()
    names = ("x", "W", "bias", "out", "rows", "K", "N", "transposed", "A", "B", "G", "shared", "stream")
    good = [16, 16, 8, 16, 4, 192, 64, 0, 2, 2, 8, 1, None]

    def status(**changes):
        return lib.grkan_product(*[changes.get(n, v) for n, v in zip(names, good)])

    assert status(rows=0) == 0 and status(rows=0, x=None, out=None, bias=None) == 0
    assert all(status(**{p: None}) == 1 for p in ("x", "W", "out", "A", "B"))
    assert all(status(**{p: v}) == 4 for p, v in (("x", 8), ("W", 8), ("out", 8), ("bias", 4), ("A", 1), ("B", 1)))
    assert status(rows=-1) == 2 and status(K=0) == 2 and status(G=0) == 2 and status(G=3) == 2
    assert status(K=96) == 8 and status(N=68, G=1) == 8 and status(G=16) == 8 and status(transposed=1) == 8
    assert status(rows=(1 << 30) + 1) == 8 and status(K=(1 << 20) + 64) == 8
    assert not lib.grkan_product_supported(4, 100, 64) and lib.grkan_product_supported(4, 64, 8)
    assert binding.grkan_product_estimate_us(4, 100, 64) == 0 and binding.grkan_product_estimate_us(0, 64, 64) == 0
    with pytest.raises(binding.GrkanError):
        binding.grkan_product_tile(0, 64, 64)
    one = ctypes.c_int32()
    assert lib.grkan_product_tile(4, 64, 64, 0, ctypes.byref(one), None, ctypes.byref(one), ctypes.byref(ctypes.c_int64())) == 1


def test_tiles_grow_with_the_call():
    tile = binding.grkan_product_tile
    assert tile(197, 1536, 384) == (64, 64, 1, 197)
    assert tile(3152, 3072, 768) == (96, 128, 1, 3152)
    assert tile(6304, 3072, 768) == (160, 128, 1, 6304)
    assert tile(25216, 1536, 384) == (224, 192, 1, 25216)
    assert tile(6304, 768, 3072) == (320, 256, 1, 6304) and tile(25216, 3072, 768) == (320, 256, 1, 25216)
    assert tile(12593, 2048, 2048) == (320, 256, 1, 10240)  # one whole round of 32 x 8 tiles, and the rest in another


def test_tiles_of_the_backward_pass_of_f():
    """Every tile that grkan_block_bwd may take is one that a block it takes reaches: not the two largest, at any size."""
    tiles = {binding.grkan_product_tile(rows, K, N, 2)[:3] for rows in (1, 197, 3000, 6304, 12608, 25216, 52000)
             for K in (384, 1536, 3072) for N in (192, 256, 384, 768, 3072)}
    assert tiles == {(64, 64, 1), (96, 128, 1), (160, 128, 1), (160, 128, 2), (160, 192, 1), (224, 192, 1)}


def test_rule_of_the_blocks_inference_route():
    faster = gnn.block_products_are_faster
    assert faster(6304, 768, 3072, 768, 8, 8) and faster(197, 192, 768, 192, 8, 8)
    assert not faster(49, 768, 3072, 768, 8, 8) and not faster(197, 768, 3072, 768, 8, 8)
    assert not faster(400, 96, 384, 96, 8, 8)  # K = 96 is no multiple of 64
    assert not faster(400, 192, 768, 192, 0, 8) and not faster(400, 192, 768, 192, 5, 8) and not faster(0, 192, 768, 192, 8, 8)
    # where the layers are called one by one (the second on its packed copy) their calls' host time counts; weights past the measured ones
    assert faster(49, 768, 768, 768, 8, 8) and faster(1576, 256, 256, 256, 8, 8) and not faster(25216, 256, 256, 256, 8, 8)
    assert not faster(394, 2048, 8192, 2048, 8, 8) and not faster(197, 4096, 16384, 4096, 8, 8)


def test_rule_of_a_layers_inference_route():
    route = gnn._layer_route
    assert route(50432, 512, 2048, 8, 6, True) == route(3152, 768, 3072, 8, 6, True) == "product"
    assert route(197, 3072, 768, 8, 6, True) == route(6304, 1536, 384, 8, 6, True) == "model"
    assert route(25216, 3072, 768, 8, 6, True) == "packed" and route(25216, 3072, 768, 8, 6, False) == "model"
    assert route(300, 192, 768, 8, 6, True) == "product"       # groups of 24: not the one kernel's
    assert route(300, 768, 192, 8, 4, True) == "other"         # other degrees
    assert route(300, 100, 192, 4, 6, True) == "other" and route(0, 768, 192, 8, 6, True) == "other"


def test_layers_that_torchs_product_is_faster_for():
    """Sizes at which F and torch's linear were measured 5 - 57 % faster than F and this product, and neighbours at which they are not."""
    route = gnn._layer_route
    for size in ((16384, 768, 3072), (16384, 768, 2048), (5000, 3072, 3072), (2048, 3072, 768), (16384, 1024, 1024), (25216, 2048, 512),
                 (500, 4096, 4096), (500, 8192, 8192), (8192, 4096, 16384), (1000, 16384, 4096)):
        assert route(*size, 8, 6, True) == "other", size
    for size in ((25216, 2048, 1000), (16384, 1024, 1000), (40000, 512, 2048), (25216, 192, 768), (2048, 640, 2560), (256, 320, 1000), (2048, 1024, 4096)):
        assert route(*size, 8, 6, True) == "product", size
