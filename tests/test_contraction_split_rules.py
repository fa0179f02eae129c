"""Which layers take the contraction kernels that split the reduction over waves, shift lines of four planes or form the
product inside the inverse transform: the library's own rules asked on the CPU, on both sides of each line."""
import importlib.util
import os

import pytest

import contraction_rules


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    return contraction_rules.build(tmp_path_factory.mktemp("rules"))


def _layer(S, f, fo, h, k):
    return S, f, fo, h, h, k, k


def test_split_reduction(rules):
    split = lambda p, *layer: rules.single(p, *_layer(*layer))[0] == "direct"
    assert split("accgrad", 122, 6, 16, 104, 7)                  # 16 x 6, thousands of samples and tiles
    assert split("bprop", 2, 32, 277, 8, 3) and split("fprop", 15, 353, 12, 11, 3)
    assert split("fprop", 8, 256, 256, 27, 5)                    # 3392 tiles, 256 steps
    assert not split("fprop", 5, 8, 32, 13, 3)                   # one chunk
    assert not split("fprop", 128, 64, 64, 27, 5)                # wide
    assert not split("fprop", 128, 384, 384, 13, 3) and not split("fprop", 108, 290, 112, 8, 4)      # bf16
    assert split("fprop", 3, 48, 320, 32, 3) and not split("fprop", 20, 24, 384, 32, 3)             # 128 tiles to a step
    assert split("fprop", 16, 24, 384, 32, 3) and not split("fprop", 17, 24, 384, 32, 3)            # ... at sides above 16
    assert not split("fprop", 5, 176, 248, 40, 3)                # lines of four bins
    assert not split("fprop", 128, 3, 96, 128, 11)               # thin


def test_split_reduction_of_full_tiles(rules):
    """Sides of 33 .. 64 that fill their 64x64 tiles, where those give every compute unit one: with more than 32 steps in whole quads."""
    split = lambda p, *layer: rules.single(p, *_layer(*layer))[0] == "direct"
    assert split("fprop", 40, 63, 130, 10, 3) and not split("fprop", 40, 63, 300, 10, 3)          # 192, 320 tiles
    assert not split("bprop", 44, 399, 29, 11, 2) and not split("bprop", 34, 208, 27, 13, 5)
    assert not split("bprop", 50, 256, 182, 14, 3) and split("bprop", 35, 198, 228, 10, 2)
    assert split("accgrad", 188, 144, 39, 13, 5) and not split("accgrad", 17, 53, 288, 13, 2)
    assert split("accgrad", 179, 38, 72, 15, 3) and split("bprop", 92, 36, 66, 15, 3)             # three 32x32 tiles to one


def test_split_reduction_possible_at_any_alignment_of_4_bytes(rules):
    for off in (0, 4, 8, 12, 16):
        assert rules.single("fprop", *_layer(15, 353, 12, 11, 3), offset=off)[0] == "direct"
        assert (rules.single("fprop", *_layer(33, 37, 75, 40, 3), offset=off)[0] == "shifted") == (off % 16 == 0)
    assert not rules.possible("fprop", *_layer(4, 40, 40, 120, 31))[0]        # single planes


def test_shifted_lines(rules):
    shifted = lambda p, *layer: rules.single(p, *_layer(*layer))[0] == "shifted"
    assert shifted("fprop", 50, 37, 75, 56, 5)
    assert rules.single("fprop", *_layer(50, 36, 76, 56, 5))[0] == "bin4"     # multiples of four
    assert not shifted("fprop", 50, 37, 75, 27, 5)                            # runs of sixteen
    assert not shifted("bprop", 40, 51, 14, 50, 3)                            # 40 x 51: a whole 64x64 tile
    assert shifted("accgrad", 26, 229, 175, 50, 3)                            # full tiles, many of them


def test_shifted_lines_only_where_they_are_faster(rules):
    """By the 32x32 tiles to a 64x64 one, the reduction, and whether the 64x64 tiles are one round of workgroups."""
    shifted = lambda p, *layer: rules.single(p, *_layer(*layer))[0] == "shifted"
    assert not shifted("fprop", 9, 7, 30, 36, 3) and shifted("fprop", 9, 18, 30, 36, 3)             # one tile, one round
    assert shifted("fprop", 9, 7, 30, 40, 3)                                                        # ... more than one round
    assert not shifted("fprop", 20, 65, 47, 36, 3) and shifted("accgrad", 65, 20, 47, 36, 3)        # two tiles, one round
    assert not shifted("fprop", 20, 6, 47, 40, 3) and shifted("fprop", 20, 18, 47, 40, 3)           # ... and few terms
    assert shifted("fprop", 20, 6, 47, 48, 3) and not shifted("fprop", 20, 6, 47, 56, 3) and shifted("fprop", 20, 6, 47, 64, 3)
    assert not shifted("fprop", 46, 6, 134, 40, 3) and not shifted("bprop", 41, 217, 29, 38, 3)     # nearly full tiles
    assert shifted("bprop", 41, 217, 70, 38, 3) and not shifted("fprop", 40, 30, 90, 40, 3)
    assert shifted("bprop", 64, 91, 14, 48, 3) and not shifted("bprop", 152, 41, 2, 55, 3)          # ... and odd columns
    assert shifted("fprop", 66, 6, 130, 40, 3) and shifted("accgrad", 14, 81, 108, 51, 2)           # three by four
    assert not shifted("accgrad", 17, 128, 167, 40, 3) and shifted("accgrad", 34, 128, 167, 40, 3)  # ... in whole quads of columns
    assert not shifted("accgrad", 3, 80, 102, 36, 3) and shifted("accgrad", 3, 81, 102, 36, 3)


def test_shared_launches(rules):
    pair = lambda *layer: rules.pair(*_layer(*layer))
    assert pair(22, 16, 311, 14, 7) == "direct" and pair(7, 16, 6, 75, 3) == "direct"
    assert pair(34, 33, 35, 28, 3) == "scalar" and pair(34, 130, 131, 32, 3) == "scalar"
    assert pair(6, 16, 304, 14, 3) == "direct" and pair(5, 368, 24, 14, 7) == "tiles"      # 24 steps
    assert pair(128, 64, 64, 27, 5) == "tiles" and pair(16, 4, 16, 13, 3) == "tiles"
    assert pair(4, 6, 5, 27, 5) == "scalar"                      # reductions of one chunk


def test_a_lone_gradient_on_the_waves_of_the_shared_launch(rules):
    """... unless that costs it more than a kernel of its own: full tiles, few steps or large grids."""
    lone = lambda p, *layer: rules.lone(p, *_layer(*layer))
    for p, layer in (("bprop", (512, 317, 4, 11, 5)), ("bprop", (362, 387, 25, 11, 4)), ("accgrad", (3, 288, 347, 9, 3)),
                     ("bprop", (275, 121, 16, 9, 4)), ("accgrad", (40, 399, 184, 13, 3)), ("bprop", (453, 12, 32, 17, 3)),
                     ("bprop", (4, 21, 339, 34, 3)), ("bprop", (70, 9, 13, 13, 3)), ("bprop", (34, 18, 15, 34, 3)),
                     ("accgrad", (13, 201, 31, 20, 3)), ("bprop", (900, 17, 4, 20, 3))):
        assert rules.pair(*_layer(*layer)) == "direct" and lone(p, *layer) != "direct+", (p, layer)
    for p, layer in (("bprop", (70, 5, 6, 13, 3)), ("accgrad", (70, 5, 6, 13, 3)), ("bprop", (33, 13, 140, 20, 3)),
                     ("accgrad", (4, 72, 68, 9, 3)), ("accgrad", (129, 16, 20, 13, 3)), ("bprop", (65, 65, 64, 13, 3)),
                     ("bprop", (75, 14, 7, 32, 3)), ("bprop", (163, 5, 4, 112, 5)), ("bprop", (8, 7, 16, 65, 3)),
                     ("bprop", (70, 9, 13, 8, 3)), ("bprop", (66, 18, 15, 34, 3)), ("bprop", (2, 7, 328, 35, 3)),
                     ("bprop", (128, 7, 32, 38, 3))):
        assert rules.pair(*_layer(*layer)) == "direct" and lone(p, *layer) == "direct+", (p, layer)
    assert rules.pair(*_layer(20, 33, 70, 20, 3)) == "scalar" and lone("bprop", 20, 33, 70, 20, 3) == "tile"


def test_product_inside_the_inverse_transform(rules):
    product = lambda p, *layer: rules.single(p, *_layer(*layer))[0] == "product"
    assert product("fprop", 64, 3, 384, 13, 3) and product("fprop", 16, 4, 16, 20, 3) and product("fprop", 128, 3, 96, 128, 11)
    assert product("bprop", 64, 384, 3, 28, 5) and product("fprop", 64, 1, 32, 56, 7)
    assert not product("fprop", 8, 3, 16, 56, 7) and not product("fprop", 128, 4, 64, 56, 5)
    assert not product("fprop", 128, 3, 64, 64, 7) and not product("fprop", 128, 5, 64, 13, 3)


def test_four_terms_and_full_grids_outside_the_inverse_transform(rules):
    """Where two kernels are the faster way: a fourth term's gathers on bases 16 .. 24, weights with many rows first, and the
    four-lane inverse of basis 28 on large grids."""
    product = lambda p, *layer: rules.single(p, *_layer(*layer))[0] == "product"
    for layer in ((52, 4, 28, 24, 2), (33, 4, 72, 23, 3), (54, 4, 4, 24, 7), (1, 4, 368, 16, 3), (233, 4, 316, 16, 3),
                  (280, 4, 128, 18, 3), (34, 4, 8, 18, 3), (10, 4, 28, 20, 3), (384, 4, 64, 20, 3), (491, 4, 112, 24, 3)):
        assert not product("fprop", *layer), layer
    assert not product("fprop", 1108, 4, 120, 13, 3) and product("fprop", 128, 4, 96, 13, 3)
    for layer in ((64, 4, 64, 16, 3), (16, 4, 16, 20, 3), (301, 4, 4, 18, 3), (40, 4, 64, 20, 3), (416, 4, 4, 24, 3), (1, 4, 4, 24, 3)):
        assert product("fprop", *layer), layer
    for layer in ((11, 12, 4, 23, 7), (4, 308, 4, 23, 3), (106, 4, 4, 24, 3)):
        assert not product("bprop", *layer), layer
    for layer in ((64, 16, 4, 22, 3), (30, 216, 4, 24, 3), (416, 4, 4, 22, 3), (42, 112, 4, 20, 3)):
        assert product("bprop", *layer), layer
    assert not product("bprop", 480, 36, 3, 27, 3) and product("bprop", 196, 52, 3, 27, 3)
    assert not product("fprop", 300, 3, 64, 28, 3) and product("fprop", 300, 1, 64, 28, 3) and not product("bprop", 64, 304, 3, 27, 3)


def test_the_gpu_test_forms_products_inside_every_inverse_transform(rules):
    """Every basis that has the kernel, one to four terms of either operand's layout (above basis 24 three at most)."""
    path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "test_gpu_contraction.py")
    spec = importlib.util.spec_from_file_location("gpu_contraction_layers", path)
    gpu = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gpu)
    for side in gpu.PRODUCT_SIDES:
        got = {(p, l[1 if p == "fprop" else 2]) for l in gpu.product_layers(side) for p in ("fprop", "bprop")
               if rules.single(p, l[0], l[1], l[2], side, side, 3, l[3])[0] == "product"}
        want = {("fprop", 1), ("fprop", 3), ("bprop", 2)}
        if side <= 24:
            want |= {("fprop", 2), ("fprop", 4), ("bprop", 3), ("bprop", 4)}
        assert want <= got, (side, want - got)
