"""Which layers take the contraction kernels that split the reduction over waves, shift lines of four planes or form the
product inside the inverse transform: the library's own rules asked on the CPU, on both sides of each line."""
import ctypes
import os
import subprocess

import pytest

import paper_1412_7580_amd as pkg

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
PASSES = {"fprop": pkg.FPROP, "bprop": pkg.BPROP, "accgrad": pkg.ACCGRAD}


class Rules:
    def __init__(self, path):
        self._lib = ctypes.CDLL(path)

    @staticmethod
    def _matrix(d):
        return (ctypes.c_long * 11)(d["M"], d["N"], d["K"], d["bins"], d["tile_log2"], d["a_rs"], d["a_cs"], d["b_rs"],
                                    d["b_cs"], d["c_rs"], d["c_cs"])

    def single(self, pass_, S, f, fo, h, k, offset=0):
        d = pkg.describe_plan(PASSES[pass_], S, f, fo, h, h, k, k)
        out = (ctypes.c_int * 4)()
        assert self._lib.split_single(self._matrix(d), ctypes.c_long(offset), d["Nr"], out) == 0
        return dict(zip(("shifted", "possible", "split", "product"), map(bool, out)))

    def pair(self, S, f, fo, h, k):
        b, a = (self._matrix(pkg.describe_plan(p, S, f, fo, h, h, k, k)) for p in (pkg.BPROP, pkg.ACCGRAD))
        out = (ctypes.c_int * 2)()
        assert self._lib.split_pair(b, a, out) == 0
        return "split" if out[0] else "scalar" if out[1] else None


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    path = str(tmp_path_factory.mktemp("rules") / "split_rules.so")
    subprocess.check_call([os.path.join(ROCM, "llvm", "bin", "clang++"), "-std=c++17", "-O1", "-fPIC", "-shared", "-x", "c++",
                           "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROCM, "include"), "-Wno-unused-function",
                           os.path.join(HERE, "contraction_rules", "split_rules.cpp"), "-o", path])
    return Rules(path)


def test_split_reduction(rules):
    split = lambda p, *layer: rules.single(p, *layer)["split"]
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


def test_split_reduction_possible_at_any_alignment_of_4_bytes(rules):
    for off in (0, 4, 8, 12, 16):
        got = rules.single("fprop", 15, 353, 12, 11, 3, offset=off)
        assert got["possible"] and got["split"]
        assert rules.single("fprop", 33, 37, 75, 40, 3, offset=off)["shifted"] == (off % 16 == 0)
    assert not rules.single("fprop", 4, 40, 40, 120, 31)["possible"]          # single planes


def test_shifted_lines(rules):
    assert rules.single("fprop", 50, 37, 75, 56, 5)["shifted"]
    assert not rules.single("fprop", 50, 36, 76, 56, 5)["shifted"]            # multiples of four: the four-bin kernel
    assert not rules.single("fprop", 50, 37, 75, 27, 5)["shifted"]            # runs of sixteen
    assert not rules.single("bprop", 40, 51, 14, 50, 3)["shifted"]            # 40 x 51: a whole 64x64 tile
    assert rules.single("accgrad", 26, 229, 175, 50, 3)["shifted"]            # full tiles, many of them


def test_shared_launches(rules):
    assert rules.pair(22, 16, 311, 14, 7) == "split" and rules.pair(7, 16, 6, 75, 3) == "split"
    assert rules.pair(34, 33, 35, 28, 3) == "scalar" and rules.pair(34, 130, 131, 32, 3) == "scalar"
    assert rules.pair(6, 16, 304, 14, 3) == "split" and rules.pair(5, 368, 24, 14, 7) is None
    assert rules.pair(128, 64, 64, 27, 5) is None and rules.pair(16, 4, 16, 13, 3) is None
    assert rules.pair(4, 6, 5, 27, 5) == "scalar"                # reductions of one chunk


def test_product_inside_the_inverse_transform(rules):
    product = lambda p, *layer: rules.single(p, *layer)["product"]
    assert product("fprop", 64, 3, 384, 13, 3) and product("fprop", 16, 4, 16, 20, 3) and product("fprop", 128, 3, 96, 128, 11)
    assert product("bprop", 64, 384, 3, 28, 5) and product("fprop", 64, 1, 32, 56, 7)
    assert not product("fprop", 8, 3, 16, 56, 7) and not product("fprop", 128, 4, 64, 56, 5)
    assert not product("fprop", 128, 3, 64, 64, 7) and not product("fprop", 128, 5, 64, 13, 3)
