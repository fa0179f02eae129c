"""Representative workloads of the library: what its users have it do, as plain data, with the
inputs, the one pass through the public entry points, the least work and the accuracy of each.

A case is a dict.  `kind` says which calls make up a pass:

  train    one layer of a training step: fft_conv_fprop_save, then fft_conv_backward with the
           transforms it saved (gx is left out for a net's first layer; gw may be accumulated)
  padded   the same through the zero-padded entry points
  passes   the three independent passes fft_conv_fprop, _bprop, _accgrad
  infer    fft_conv_fprop_weights on weights transformed once, ahead
  fft1d    a batch of 1-D real transforms, forward and back, inputs zero-padded to the basis
  fft2d    the same in 2-D

Everything is fp32, the only data type of the library.
"""
from __future__ import annotations

import math

import torch

import paper_1412_7580_amd as pkg

BASES_2D = (8, 10, 12, 14, 16, 18, 20, 24, 28, 32, 36, 40, 48, 56, 64, 80, 96, 112, 128)
BASES_1D = BASES_2D + (160, 192, 224, 256)


def _conv(name, kind, S, f, fo, h, w, kh, kw, ph=0, pw=0, gx=True, acc=False):
    return {"name": name, "kind": kind, "S": S, "f": f, "fo": fo, "h": h, "w": w, "kh": kh, "kw": kw,
            "ph": ph, "pw": pw, "gx": gx, "acc": acc}


def _fft(name, kind, n, n_in, batch):
    return {"name": name, "kind": kind, "n": n, "n_in": n_in, "batch": batch}


def listed():
    return [
        # the smallest call in earnest: one small layer served on weights transformed ahead
        _conv("infer_13_f16", "infer", 16, 16, 16, 13, 13, 3, 3),
        # serving a batch of a few images through a wide layer: the weights dominate
        _conv("infer_27_s8_f256", "infer", 8, 256, 256, 27, 27, 5, 5),
        # the small layer's three passes by themselves: launches and latency
        _conv("passes_13_f16", "passes", 16, 16, 16, 13, 13, 3, 3),
        # odd channel counts, non-square image and kernel (a net whose widths nobody rounded)
        _conv("passes_30x19_odd", "passes", 50, 37, 75, 30, 19, 7, 4),
        # second layer of an AlexNet-like net: the ordinary training layer
        _conv("train_27_f64", "train", 128, 64, 64, 27, 27, 5, 5),
        # deep layer, many channels, small images: the contraction dominates
        _conv("train_13_f384", "train", 128, 384, 384, 13, 13, 3, 3),
        # large kernels, the regime the method is best at: transforms and memory dominate
        _conv("train_64_k31", "train", 32, 128, 128, 64, 64, 31, 31),
        # first layer of a net: three input channels, large kernel, no input gradient
        _conv("train_first_128_k11", "train", 128, 3, 96, 128, 128, 11, 11, gx=False),
        # margin-padded 3x3 layer, gradient accumulated over micro-batches
        _conv("padded_56_k3", "padded", 32, 64, 128, 56, 56, 3, 3, 1, 1, acc=True),
        # images larger than any basis: tiled
        _conv("train_224_k5", "train", 16, 64, 64, 224, 224, 5, 5),
        # stand-alone batches of transforms at a small and at the largest 2-D size
        _fft("fft1d_32", "fft1d", 32, 29, 1 << 21),
        _fft("fft2d_128", "fft2d", 128, 125, 4096),
    ]


# ------------------------------------------------------------------ drawn cases
def _logint(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _channels(rng):
    """A width as nets have them: mostly multiples of 16, sometimes 3 or any number."""
    c = _logint(rng, 3, 384)
    return max(16, (c + 8) // 16 * 16) if rng.random() < 0.6 else c


def _draw_any(rng):
    kind = rng.choice(("train", "train", "passes", "padded", "infer", "fft1d", "fft2d"))
    if kind == "fft1d":
        n = rng.choice(BASES_1D)
        return _fft("", kind, n, rng.randint(n // 2 + 1, n), _logint(rng, 256, (1 << 26) // n))
    if kind == "fft2d":
        n = rng.choice(BASES_2D)
        return _fft("", kind, n, rng.randint(n // 2 + 1, n), _logint(rng, 16, (1 << 26) // (n * n)))
    h = _logint(rng, 7, 224)
    w = h if rng.random() < 0.6 else _logint(rng, max(7, h // 2), min(224, 2 * h))
    kh = min(rng.choice((3, 3, 3, 5, 5, 7, 9, 11, 15, 31)), h // 2)
    kw = kh if rng.random() < 0.7 else min(rng.choice((2, 3, 4, 5, 7, 9, 11)), w // 2)
    kw = min(kw, w // 2)
    ph, pw = (kh // 2, kw // 2) if kind == "padded" else (0, 0)
    S = _logint(rng, 1, 128) if kind == "infer" else _logint(rng, 8, 128)
    gx = not (kind == "train" and rng.random() < 0.15)
    return _conv("", kind, S, _channels(rng), _channels(rng), h, w, kh, kw, ph, pw, gx,
                 kind == "padded" and rng.random() < 0.5)


def _frequency_bytes(c):
    """Upper estimate of the frequency-domain data of a pass (bases are at most 15 % wider)."""
    if c["kind"].startswith("fft"):
        return 0
    area = 8 * (c["h"] + 2 * c["ph"] + 8) * ((c["w"] + 2 * c["pw"] + 8) / 2 + 1)
    return area * (c["S"] * c["f"] + c["S"] * c["fo"] + c["f"] * c["fo"])


def _cost(c):
    k = work(c)
    return k["bytes"] / 4e12 + k["flops"] / 6e13 + 6 * _frequency_bytes(c) / 4e12


def draw(rng):
    limit = max(_cost(c) for c in listed())
    while True:
        c = _draw_any(rng)
        if _cost(c) <= limit:
            return {k: v for k, v in c.items() if k != "name"}


# ------------------------------------------------------------------ inputs and the pass
_handle = None


def _library():
    global _handle
    if _handle is None:
        _handle = pkg.Handle(torch.cuda.current_device())   # one per process, as a program keeps it
    return _handle


def prepare(case, seed):
    hd = _library()
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape, std=1.0):
        return torch.empty(shape, device="cuda").normal_(0.0, std, generator=gen)

    st = {"hd": hd, "case": dict(case)}
    if case["kind"].startswith("fft"):
        n, n_in, B = case["n"], case["n_in"], case["batch"]
        if case["kind"] == "fft1d":
            st["x"] = normal(B, n_in)
            st["X"] = torch.empty((B, n // 2 + 1, 2), device="cuda")
        else:
            st["x"] = normal(B, n_in, n_in)
            st["X"] = torch.empty((B, n, n // 2 + 1, 2), device="cuda")
        st["back"] = torch.empty_like(st["x"])
        return st
    S, f, fo, h, w, kh, kw, ph, pw = (case[k] for k in ("S", "f", "fo", "h", "w", "kh", "kw", "ph", "pw"))
    oh, ow = h + 2 * ph - kh + 1, w + 2 * pw - kw + 1
    st["x"] = torch.relu(normal(S, f, h, w))                              # rectified activations
    wt = normal(fo, f, kh, kw, std=math.sqrt(2.0 / (f * kh * kw)))       # weights of a rectifier net
    st["y"] = torch.empty((S, fo, oh, ow), device="cuda")
    if case["kind"] == "infer":
        st["wf"] = hd.fft_conv_transform_weights(wt, h, w, ph, pw)
        return st
    st["wt"] = wt
    st["gy"] = normal(S, fo, oh, ow, std=0.01)
    st["gx"] = torch.empty_like(st["x"])
    st["gw"] = torch.zeros_like(wt)
    if case["kind"] == "train":
        st["saved"] = torch.empty(hd.saved_bytes(S, f, fo, h, w, kh, kw) // 4, device="cuda")
    elif case["kind"] == "padded":
        st["saved"] = torch.empty(hd.saved_bytes_padded(S, f, fo, h, w, kh, kw, ph, pw) // 4, device="cuda")
        st["gw0"] = normal(fo, f, kh, kw)                                 # sum of the earlier micro-batches
    return st


def run(st):
    hd, c = st["hd"], st["case"]
    kind = c["kind"]
    if kind == "fft1d":
        hd.fft_r2c_1d(st["x"], c["n"], out=st["X"])
        hd.fft_c2r_1d(st["X"], c["n"], c["n_in"], out=st["back"])
        return st["X"], st["back"]
    if kind == "fft2d":
        hd.fft_r2c_2d(st["x"], c["n"], out=st["X"])
        hd.fft_c2r_2d(st["X"], c["n"], c["n_in"], c["n_in"], out=st["back"])
        return st["X"], st["back"]
    f, h, w, kh, kw = c["f"], c["h"], c["w"], c["kh"], c["kw"]
    if kind == "infer":
        return hd.fft_conv_fprop_weights(st["x"], st["wf"], c["fo"], kh, kw, c["ph"], c["pw"], y=st["y"])
    if kind == "passes":
        return (hd.fft_conv_fprop(st["x"], st["wt"], y=st["y"]),
                hd.fft_conv_bprop(st["gy"], st["wt"], h, w, gx=st["gx"]),
                hd.fft_conv_accgrad(st["x"], st["gy"], gw=st["gw"]))
    if kind == "train":
        hd.fft_conv_fprop_save(st["x"], st["wt"], st["saved"], y=st["y"])
        hd.fft_conv_backward(st["gy"], st["saved"], f, h, w, kh, kw, gx=st["gx"] if c["gx"] else None, gw=st["gw"],
                             want_gx=c["gx"])
        return (st["y"], st["gx"], st["gw"]) if c["gx"] else (st["y"], st["gw"])
    if c["acc"]:
        st["gw"].copy_(st["gw0"])
    hd.fft_conv_fprop_save_padded(st["x"], st["wt"], c["ph"], c["pw"], st["saved"], y=st["y"])
    hd.fft_conv_backward_padded(st["gy"], st["saved"], f, h, w, kh, kw, c["ph"], c["pw"], gx=st["gx"], gw=st["gw"],
                                accumulate=c["acc"])
    return st["y"], st["gx"], st["gw"]


# ------------------------------------------------------------------ least work and accuracy
def work(case):
    """Bytes: every input once in, every output once out.  Flops: per pass the smaller of the
    direct sum and the product of half spectra of the padded image's own size (three real
    products per complex one), plus the transforms at 5/2 n log2 n."""
    def transform(points):
        return 2.5 * points * math.log2(max(points, 2))

    if case["kind"].startswith("fft"):
        n, n_in, B = case["n"], case["n_in"], case["batch"]
        d = 1 if case["kind"] == "fft1d" else 2
        half = (n // 2 + 1) * n ** (d - 1)
        return {"bytes": 2 * B * (4 * n_in ** d + 8 * half), "flops": 2 * B * transform(n ** d)}
    S, f, fo, h, w, kh, kw, ph, pw = (case[k] for k in ("S", "f", "fo", "h", "w", "kh", "kw", "ph", "pw"))
    hp, wp = h + 2 * ph, w + 2 * pw
    oh, ow = hp - kh + 1, wp - kw + 1
    x, y, g = S * f * h * w, S * fo * oh * ow, fo * f * kh * kw
    spectrum = hp * (wp // 2 + 1)
    product = min(2 * S * f * fo * kh * kw * oh * ow, 6 * S * f * fo * spectrum)
    planes = S * f, S * fo, f * fo
    if case["kind"] == "infer":     # the weights' half spectra are the operand in hand
        return {"bytes": 4 * (x + y) + 8 * f * fo * spectrum,
                "flops": product + (planes[0] + planes[1]) * transform(hp * wp)}
    passes = 2 + (1 if case["gx"] else 0)
    if case["kind"] == "passes":    # each call reads its two operands and writes its result
        moved, transforms = 3 * (x + y + g), 3 * sum(planes)
    else:                           # x, weights and gy in; y, gx and gw out
        moved, transforms = (2 if case["gx"] else 1) * x + 2 * y + 2 * g + (g if case["acc"] else 0), 2 * sum(planes)
    return {"bytes": 4 * moved, "flops": passes * product + transforms * transform(hp * wp)}


def tolerance(case):
    """Relative 2-norm error, about four times the largest measured against the same sums in 64
    bits: transforms 0.8e-7 .. 2.1e-7; convolutions 1.6e-7 .. 4.9e-7, and 7e-7 .. 1e-6 for the weight
    gradients of tiled layers, which sum over samples and tiles."""
    return {"rel": 1e-6 if case["kind"].startswith("fft") else 4e-6}
