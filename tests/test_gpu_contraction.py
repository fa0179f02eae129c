"""The per-bin contraction at the edges of its kernels (GPU, C ABI): sides around the matrix-core
tiles (32, 64, 128) and K tile (16), and the vector-unit kernels for sides of 1 .. 4, on layouts with
runs of 4, 8, 16, 32 and 64 planes.  tests/test_contraction_rules.py checks on the CPU that these layers reach
every kernel, kind of gather and remainder.

Reference: the convolution in fp64 (torch, CPU).  Bound on max|err| / max|ref|: the transforms
make about 12 roundings of 2^-24 a value and the sum one per 2 terms (fp32) or 5 (bf16, three per 16),
80 at most here, each against the largest partial sum and of either sign; 4e-6 is 67 roundings in one
direction, seven times the root of 92."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
TOL = 4e-6


@pytest.fixture(scope="module")
def hd(lib):
    h = lib.Handle(0)
    yield h
    h.close()


def _relerr(got, ref):
    return float((got.cpu().double() - ref).abs().max() / ref.abs().max())


def _check(hd, S, f, fo, h, w, kh, kw, gx=True):
    import torch
    import torch.nn.functional as F
    g = torch.Generator().manual_seed(S * 7 + f * 11 + fo * 13 + h)
    x, wt = torch.randn(S, f, h, w, generator=g), torch.randn(fo, f, kh, kw, generator=g)
    gy = torch.randn(S, fo, h - kh + 1, w - kw + 1, generator=g)
    xd, wd, gd = x.double(), wt.double(), gy.double()
    ry = F.conv2d(xd, wd)
    rx = F.conv_transpose2d(gd, wd)
    rw = F.conv2d(xd.transpose(0, 1), gd.transpose(0, 1)).transpose(0, 1)
    dx, dw, dg = x.cuda(), wt.cuda(), gy.cuda()
    got = {"fprop": (hd.fft_conv_fprop(dx, dw), ry), "bprop": (hd.fft_conv_bprop(dg, dw, h, w), rx),
           "accgrad": (hd.fft_conv_accgrad(dx, dg), rw)}
    saved = torch.empty(hd.saved_bytes(S, f, fo, h, w, kh, kw) // 4, device="cuda")
    got["fprop_save"] = (hd.fft_conv_fprop_save(dx, dw, saved), ry)
    bx, bw = hd.fft_conv_backward(dg, saved, f, h, w, kh, kw, want_gx=gx)
    if gx:
        got["backward.gx"] = (bx, rx)
    got["backward.gw"] = (bw, rw)
    wf = hd.fft_conv_transform_weights(dw, h, w)
    got["weights"] = (hd.fft_conv_fprop_weights(dx, wf, fo, kh, kw), ry)
    torch.cuda.synchronize()
    for k, (a, b) in got.items():
        assert a.shape == b.shape
        assert _relerr(a, b) <= TOL, (k, _relerr(a, b))


# images whose bases have runs of 64, 32, 16, 8 and 4 planes
SIDES = {"run64": 8, "run32": 13, "run16": 20, "run8": 32, "run4": 40}


@pytest.mark.parametrize("side", SIDES.values(), ids=SIDES.keys())
@pytest.mark.parametrize("S,f,fo", [(1, 3, 4), (5, 3, 96), (9, 1, 12), (6, 2, 20), (33, 4, 8), (5, 16, 1), (7, 12, 3),
                                    (1, 4, 4), (2, 3, 6), (66, 3, 16)])
def test_thin_sides(hd, S, f, fo, side):
    _check(hd, S, f, fo, side, side, 3, 3)


@pytest.mark.parametrize("S,f,fo,side,gx", [(3, 3, 8, 150, False), (2, 3, 12, 70, True), (1, 1, 4, 150, True)])
def test_thin_sides_tiled(hd, S, f, fo, side, gx):
    _check(hd, S, f, fo, side, side - 9, 5, 4, gx)


@pytest.mark.parametrize("side", [8, 13, 20, 32], ids=["run64", "run32", "run16", "run8"])
@pytest.mark.parametrize("S,f,fo", [(8, 64, 128), (31, 16, 64), (32, 32, 32), (33, 48, 160), (64, 64, 64), (65, 17, 33),
                                    (129, 5, 31), (16, 63, 129), (7, 20, 68)])
def test_tile_edges(hd, S, f, fo, side):
    _check(hd, S, f, fo, side, side, 3, 2)


# Layers that reach what the ones above do not.  (S, f, fo, image side)
EDGES = [
    (257, 48, 32, 13), (129, 48, 32, 20), (129, 36, 20, 20), (130, 20, 36, 20), (33, 20, 132, 20),      # 128x32
    (31, 48, 144, 20), (31, 144, 48, 20), (40, 144, 32, 20), (5, 36, 132, 20), (7, 132, 36, 20), (33, 132, 20, 20),  # 32x128
    (33, 64, 128, 8), (65, 64, 64, 8), (70, 96, 160, 13), (33, 32, 64, 13),                             # bf16, fast addressing
    (130, 128, 144, 20), (130, 120, 136, 32), (100, 120, 136, 32),
    (65, 36, 44, 13), (70, 100, 68, 8), (130, 124, 132, 20), (129, 124, 132, 32), (20, 68, 132, 13),    # bf16, general
    (130, 123, 127, 13), (130, 123, 127, 20), (131, 125, 129, 8),                                       # bf16, 4-byte gathers
    (160, 4, 8, 40), (90, 3, 96, 40), (90, 96, 3, 40), (260, 4, 4, 8), (20, 4, 12, 20), (12, 40, 4, 13),  # thin sides
    (1, 36, 44, 20), (1, 64, 64, 40), (33, 64, 64, 40),
    (20, 32, 128, 28), (20, 128, 32, 28), (33, 128, 32, 28), (32, 32, 256, 16), (20, 36, 132, 28), (36, 132, 28, 28),   # 32x128
    (130, 32, 32, 28), (33, 32, 128, 28), (130, 36, 28, 28), (130, 28, 36, 28), (36, 28, 132, 28),           # 128x32
    (150, 4, 96, 40), (150, 96, 4, 40), (40, 12, 2, 20),                                                # thin sides
]


@pytest.mark.parametrize("S,f,fo,side", EDGES)
def test_edges_of_every_kernel(hd, S, f, fo, side):
    _check(hd, S, f, fo, side, side, 3, 2)


def test_rectangular_basis(hd):
    _check(hd, 20, 37, 75, 30, 19, 7, 4)
    _check(hd, 9, 3, 16, 30, 19, 5, 4)


# powers of two on x, wt and gy
ENDS = {"small_x": (-124, 0, 0), "small_wt": (0, -124, 0), "small_gy": (0, 0, -124), "large_x": (None, -30, -30),
        "large_gy": (-30, -30, None), "apart_x": (116, -120, -120), "apart_wt": (-120, 116, -120),
        "apart_gy": (-120, -120, 116), "product": (58, 52, 48)}


@pytest.mark.parametrize("powers", ENDS.values(), ids=ENDS.keys())
def test_ends_of_the_range(hd, powers):
    """A layer of the bf16 form with operands at the ends of fp32's range, results inside it.
    small: spectra of about 2^-120, whose bf16 remainders of the third order, 2^-137 and less, lie under
    the smallest bf16 subnormal (2^-133).  large: planes of one value each with their sum, the zero
    bin, between bf16's largest finite value (3.3895e38) and fp32's (3.4028e38); the other bins lie far
    enough below it for the sum of a real and an imaginary part.  apart: one operand large, the other
    small.  product: ordinary operands whose products are large.  The bound is the file's: every
    step is a rounding of 2^-24 here, too (subnormals start 2^-6 below the small spectra's size, and
    what they round is 2^-29 of it)."""
    import torch
    import torch.nn.functional as F
    S = f = fo = 64
    h, k = 13, 3
    g = torch.Generator().manual_seed(3)
    t = [torch.randn(S, f, h, h, generator=g), torch.randn(fo, f, k, k, generator=g),
         torch.randn(S, fo, h - k + 1, h - k + 1, generator=g)]
    for i, p in enumerate(powers):
        if p is None:
            n = t[i].shape[2] * t[i].shape[3]
            t[i] = torch.sign(t[i][:, :, :1, :1]).expand_as(t[i]).contiguous() * (3.3995e38 / n)
        else:
            t[i] = t[i] * 2.0 ** p
    (dx, dw, dg), (x, w, gy) = (o.cuda() for o in t), (o.double() for o in t)
    passes = {"fprop": (0, 1, lambda: hd.fft_conv_fprop(dx, dw), lambda: F.conv2d(x, w)),
              "bprop": (2, 1, lambda: hd.fft_conv_bprop(dg, dw, h, h), lambda: F.conv_transpose2d(gy, w)),
              "accgrad": (0, 2, lambda: hd.fft_conv_accgrad(dx, dg),
                          lambda: F.conv2d(x.transpose(0, 1), gy.transpose(0, 1)).transpose(0, 1))}
    for p, (a, b, got, ref) in passes.items():
        pa, pb = powers[a], powers[b]
        if pa is not None and pb is not None and not -128 < pa + pb < 118:
            continue                                        # the result itself would leave the range
        r = ref()
        assert r.abs().max() < 1e38 and r.abs().max() > 1e-36
        assert _relerr(got(), r) <= TOL, (p, powers)


def test_values_that_are_not_finite_stay_in_their_sample(hd):
    import torch
    import torch.nn.functional as F
    g = torch.Generator().manual_seed(4)
    x, w = torch.randn(64, 64, 13, 13, generator=g), torch.randn(64, 64, 3, 3, generator=g)
    ref = F.conv2d(x.double(), w.double())
    x[5, 7, 3, 3] = float("inf")
    x[9, 1, 0, 0] = float("nan")
    got = hd.fft_conv_fprop(x.cuda(), w.cuda()).cpu()
    other = [s for s in range(64) if s not in (5, 9)]
    assert not torch.isfinite(got[5]).any() and not torch.isfinite(got[9]).any()
    assert float((got[other].double() - ref[other]).abs().max() / ref.abs().max()) <= TOL


@pytest.mark.parametrize("side", [10, 12, 20], ids=["bins60of64", "bins84of88", "bins220of224"])
def test_bf16_kernel_leaves_the_padding_bins_alone(hd, lib, side):
    """They hold whatever the memory held: NaN there would have the kernel repeat their tiles for nothing."""
    import torch
    import torch.nn.functional as F
    S, f, fo = 136, 128, 128
    d = lib.describe_plan(lib.FPROP, S, f, fo, side, side, 3, 3)
    live, bins, T = d["Nr"] * (d["Nr"] // 2 + 1), d["bins"], 1 << d["tile_log2"]
    assert live < bins
    g = torch.Generator().manual_seed(6)
    x, w = torch.randn(S, f, side, side, generator=g), torch.randn(fo, f, 3, 3, generator=g)
    ws = torch.full((d["total"] // 4,), float("nan"), device="cuda")
    got = hd.fft_conv_fprop(x.cuda(), w.cuda(), ws=ws)
    assert _relerr(got, F.conv2d(x.double(), w.double())) <= TOL
    product = ws[d["offC"] // 4:][:-(-d["planesC"] // T) * T * bins * 2].view(-1, bins, 2, T)
    assert torch.isfinite(product[:, :live]).all()
    ws.fill_(7.0)
    hd.fft_conv_fprop(x.cuda(), w.cuda(), ws=ws)
    assert (product[:, live:] == 7.0).all()


# Channel counts that are no multiple of four on runs of four planes (bases 36 .. 64): sides around the 32x32 tile and the
# K tile of 16, rows that start on every place of a line.  (S, f, fo, image side)
@pytest.mark.parametrize("S,f,fo,side", [(33, 5, 7, 40), (31, 17, 33, 40), (5, 33, 65, 40), (66, 37, 70, 40), (1, 6, 9, 40),
                                         (17, 1, 5, 40), (9, 15, 31, 35), (34, 18, 47, 46), (3, 66, 130, 55), (6, 31, 14, 63)])
def test_any_channel_counts_on_runs_of_four(hd, S, f, fo, side):
    _check(hd, S, f, fo, side, side, 3, 2)


# Long reductions with a narrow side or few tiles: one chunk of eight steps more or less than the waves, every layout's
# run, both gradients in one launch, strides on and off the quad and the run.  (S, f, fo, image side)
SPLIT = [(300, 5, 6, 8), (140, 8, 12, 8), (9, 132, 31, 8), (131, 7, 9, 13), (129, 16, 20, 13), (6, 16, 304, 14), (33, 13, 140, 20),
         (4, 200, 6, 20), (200, 16, 12, 20), (17, 18, 17, 20), (25, 24, 30, 20), (5, 6, 150, 32), (160, 8, 16, 32), (33, 31, 97, 32),
         (1, 69, 2, 13), (65, 65, 64, 13), (7, 16, 6, 40), (40, 33, 5, 13)]


@pytest.mark.parametrize("S,f,fo,side", SPLIT)
def test_reduction_split_over_waves(hd, S, f, fo, side):
    _check(hd, S, f, fo, side, side, 3, 2)


# Sides of at most 16 on either matrix: one row, 15 and 16 rows, a second strip that is empty, part of one or full (columns 16,
# 17, 33, 47, 64), reductions that end within a chunk of 16 and, at odd counts, within four steps.
@pytest.mark.parametrize("side", [8, 13, 20, 32], ids=["run64", "run32", "run16", "run8"])
@pytest.mark.parametrize("S,f,fo", [(1, 40, 33), (15, 36, 64), (16, 64, 47), (5, 37, 81), (9, 256, 17), (40, 16, 28), (70, 12, 100),
                                    (3, 19, 16), (17, 90, 15)])
def test_sides_of_at_most_sixteen(hd, S, f, fo, side):
    _check(hd, S, f, fo, side, side, 3, 2)


@pytest.mark.parametrize("S,f,fo,side", EDGES + SPLIT[::3])
def test_the_kernels_that_these_replace_on_some_layers(lib, S, f, fo, side, monkeypatch):
    """With the split reductions switched off their layers run on the tiles that other layers still take."""
    monkeypatch.setenv("FFTCONV_GEMM_NO_DIRECT", "1")
    h = lib.Handle(0)
    try:
        _check(h, S, f, fo, side, side, 3, 2)
    finally:
        h.close()


@pytest.mark.parametrize("S,f,fo,side,k", [(70, 5, 6, 13, 3), (33, 13, 140, 20, 3), (129, 16, 20, 13, 3), (4, 72, 68, 9, 3), (20, 33, 70, 20, 3)])
def test_a_gradient_alone_is_the_same_bits(hd, S, f, fo, side, k):
    """Asking for one gradient only gives what asking for both gives, whatever launch both share."""
    import torch
    g = torch.Generator().manual_seed(8)
    o = side - k + 1
    x, w = torch.randn(S, f, side, side, generator=g).cuda(), torch.randn(fo, f, k, k, generator=g).cuda()
    gy = torch.randn(S, fo, o, o, generator=g).cuda()
    saved = torch.empty(hd.saved_bytes(S, f, fo, side, side, k, k) // 4, device="cuda")
    hd.fft_conv_fprop_save(x, w, saved)
    gx, gw = hd.fft_conv_backward(gy, saved, f, side, side, k, k)
    assert torch.equal(hd.fft_conv_backward(gy, saved, f, side, side, k, k, want_gw=False)[0], gx)
    assert torch.equal(hd.fft_conv_backward(gy, saved, f, side, side, k, k, want_gx=False)[1], gw)


# Where a lone gradient takes a kernel of its own: a thin side, bf16 in the shared launch only, more than nine 32x32 tiles to four, 9 .. 16
# steps, a grid too large for the steps, and the inverse transforms of bases 16 and 28.  (S, f, fo, image side)
@pytest.mark.parametrize("S,f,fo,side", [(16, 4, 16, 13), (16, 144, 144, 13), (128, 93, 4, 11), (70, 9, 13, 13), (300, 12, 32, 17),
                                         (4, 21, 120, 34), (43, 42, 70, 15), (9, 16, 44, 15), (26, 10, 16, 26), (3, 60, 61, 26)])
def test_a_gradient_alone_is_right_on_a_kernel_of_its_own(hd, S, f, fo, side):
    import torch
    import torch.nn.functional as F
    g = torch.Generator().manual_seed(10)
    x, w = torch.randn(S, f, side, side, generator=g), torch.randn(fo, f, 3, 3, generator=g)
    gy = torch.randn(S, fo, side - 2, side - 2, generator=g)
    saved = torch.empty(hd.saved_bytes(S, f, fo, side, side, 3, 3) // 4, device="cuda")
    hd.fft_conv_fprop_save(x.cuda(), w.cuda(), saved)
    gx = hd.fft_conv_backward(gy.cuda(), saved, f, side, side, 3, 3, want_gw=False)[0]
    old = torch.randn(fo, f, 3, 3, generator=g)
    gw = old.cuda()
    hd.fft_conv_backward(gy.cuda(), saved, f, side, side, 3, 3, gw=gw, want_gx=False, scale=0.5, accumulate=True)
    xd, wd, gd = x.double(), w.double(), gy.double()
    assert _relerr(gx, F.conv_transpose2d(gd, wd)) <= TOL
    assert _relerr(gw, old.double() + 0.5 * F.conv2d(xd.transpose(0, 1), gd.transpose(0, 1)).transpose(0, 1)) <= TOL


# Both inverse transforms of a backward pass in one launch on every basis: few channels (odd counts, a ragged last tile) and a
# shared contraction, then both contractions of their own; windows and padding; scale and accumulate stay with their product.
@pytest.mark.parametrize("side", [8, 10, 12, 14, 18, 20, 24, 32, 36, 40, 48, 56, 64, 80, 96, 112, 128])
def test_both_inverse_transforms_in_one_launch(hd, side):
    import torch
    import torch.nn.functional as F
    g = torch.Generator().manual_seed(9)
    k = 33 if side > 64 else 3
    o = side - k + 1
    for S, f, fo in ((7, 5, 9), (6, 3, 16)) if side <= 64 else ((3, 2, 5),):
        x, w = torch.randn(S, f, side, side, generator=g).cuda(), torch.randn(fo, f, k, k, generator=g).cuda()
        gy = torch.randn(S, fo, o, o, generator=g).cuda()
        saved = torch.empty(hd.saved_bytes(S, f, fo, side, side, k, k) // 4, device="cuda")
        hd.fft_conv_fprop_save(x, w, saved)
        old = torch.randn(fo, f, k, k, generator=g).cuda()
        gw = old.clone()
        hd.set_profiling(True)
        try:
            gx, _ = hd.fft_conv_backward(gy, saved, f, side, side, k, k, gw=gw, scale=0.5, accumulate=True)
            assert hd.last_kernel_labels()[-1] == "ifft.pair"
        finally:
            hd.set_profiling(False)
        assert torch.equal(hd.fft_conv_backward(gy, saved, f, side, side, k, k, want_gw=False)[0], gx)
        alone = old.clone()
        hd.fft_conv_backward(gy, saved, f, side, side, k, k, gw=alone, want_gx=False, scale=0.5, accumulate=True)
        assert torch.equal(alone, gw)
        xd, wd, gd = x.cpu().double(), w.cpu().double(), gy.cpu().double()
        assert _relerr(gx, F.conv_transpose2d(gd, wd)) <= TOL
        assert _relerr(gw, old.cpu().double() + 0.5 * F.conv2d(xd.transpose(0, 1), gd.transpose(0, 1)).transpose(0, 1)) <= TOL


# Products of at most four terms formed inside the inverse transform: every basis that has the kernel, one .. four terms
# from either operand's layout, quads of columns that start in the middle of a run, a ragged last tile, windows.
PRODUCT_SIDES = [8, 10, 12, 14, 16, 18, 20, 24, 28, 32, 36, 40, 48, 56]


def product_layers(side):
    if side > 24:
        return [(53, 3, 20, 2), (86, 1, 12, 2), (260, 12, 2, 2)]
    return [(43, 3, 20, 2), (9, 2, 12, 2), (6, 20, 2, 2), (5, 1, 4, 2), (3, 4, 24, 2), (5, 28, 3, 3),
            (43, 4, 24, 2), (5, 4, 16, 2), (241, 4, 4, 2), (7, 32, 4, 2)]


@pytest.mark.parametrize("side", PRODUCT_SIDES)
def test_product_inside_the_inverse_transform(hd, side):
    for S, f, fo, kw in product_layers(side):
        _check(hd, S, f, fo, side, side, 3, kw)


@pytest.mark.parametrize("S,f,fo,side", [(2, 3, 12, 150), (1, 12, 3, 150), (19, 3, 64, 70)])
def test_product_inside_the_inverse_transform_of_windows(hd, S, f, fo, side):
    _check(hd, S, f, fo, side, side - 9, 5, 4)
