"""Which kernel runs a contraction, asked of the library's own rules on the CPU: a small program around the header that
holds them, for the matrices that the planner gives each pass of a layer."""
import ctypes
import os
import subprocess

import paper_1412_7580_amd as pkg

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
PASSES = {"fprop": pkg.FPROP, "bprop": pkg.BPROP, "accgrad": pkg.ACCGRAD}
KERNELS = ("product", "thin", "direct", "bin4", "shifted", "bf16", "tile")


def build(folder):
    path = os.path.join(str(folder), "rules.so")
    subprocess.check_call([os.path.join(ROCM, "llvm", "bin", "clang++"), "-std=c++17", "-O1", "-fPIC", "-shared", "-x", "c++",
                           "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROCM, "include"), "-Wno-unused-function",
                           os.path.join(HERE, "rules.cpp"), "-o", path])
    return Rules(path)


class Rules:
    """A layer is (S, f, fo, h, w, kh, kw) and, if not the library's choice, the tile basis."""

    def __init__(self, path):
        self._lib = ctypes.CDLL(path)

    @staticmethod
    def _plan(pass_, S, f, fo, h, w, kh, kw, basis=-1):
        return pkg.describe_plan(PASSES[pass_], S, f, fo, h, w, kh, kw, basis)

    @classmethod
    def _matrix(cls, pass_, layer):
        d = cls._plan(pass_, *layer)
        return (ctypes.c_long * 11)(d["M"], d["N"], d["K"], d["bins"], d["tile_log2"], d["a_rs"], d["a_cs"], d["b_rs"],
                                    d["b_cs"], d["c_rs"], d["c_cs"])

    @staticmethod
    def _switches(tile=-1, no_pair=False, no_direct=False):
        return (ctypes.c_long * 3)(tile, no_pair, no_direct)

    def _ask(self, pass_, layer, offset=0, **switches):
        d = self._plan(pass_, *layer)
        out = (ctypes.c_int * 8)()
        assert self._lib.rules_single(self._matrix(pass_, layer), ctypes.c_long(offset), 0 if d["rect"] else d["Nr"],
                                      self._switches(**switches), out) == 0
        return list(out)

    def rows(self, pass_, *layer):
        return self._ask(pass_, layer)[5]

    def possible(self, pass_, *layer, offset=0):
        """Whether (the direct kernel, the shifted lines) can run."""
        return tuple(map(bool, self._ask(pass_, layer, offset)[6:8]))

    def single(self, pass_, *layer, offset=0, **switches):
        """(kernel, gathers): kernel one of product, thin_k, thin_n, thin_acc, direct, bin4, shifted, bf16, tile<shape>;
        gathers one of fast, vec, scalar."""
        kernel, vec, fast, thin, shape = self._ask(pass_, layer, offset, **switches)[:5]
        name = KERNELS[kernel]
        if name == "thin":
            name = ("thin_k", "thin_n", "thin_acc")[thin - 1]
        return name + (str(shape) if name == "tile" else ""), "fast" if fast else "vec" if vec else "scalar"

    def pair(self, *layer, **switches):
        got = self._lib.rules_pair(self._matrix("bprop", layer), self._matrix("accgrad", layer), self._switches(**switches))
        return ("two launches", "direct", "tiles", "bf16", "scalar")[got]

    def lone(self, pass_, *layer, **switches):
        """The kernel of one gradient alone; direct+ is the direct kernel on the waves of the launch that both share."""
        other = "accgrad" if pass_ == "bprop" else "bprop"
        out = (ctypes.c_int * 2)()
        assert self._lib.rules_lone(self._matrix(pass_, layer), self._matrix(other, layer), self._switches(**switches), out) == 0
        return KERNELS[out[0]] + ("+" if out[1] else "")
