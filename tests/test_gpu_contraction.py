"""The per-bin contraction at the edges of its kernels (GPU, C ABI): sides around the matrix-core
tiles (32, 64, 128) and K tile (16), and the vector-unit kernels for sides of 1 .. 4, on layouts with
runs of 4, 8, 16, 32 and 64 planes.

Reference: the convolution in fp64 (torch, CPU).  Bound on max|err| / max|ref|: the transforms
make about 12 roundings of 2^-24 a value and the sum one per 16 terms, at most 64 here, each against
the largest partial sum; 4e-6 is 67 such roundings, all in one direction."""
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


def test_rectangular_basis(hd):
    _check(hd, 20, 37, 75, 30, 19, 7, 4)
    _check(hd, 9, 3, 16, 30, 19, 5, 4)
