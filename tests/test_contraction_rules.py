"""Which kernel runs a contraction, asked of the library's own rules on the CPU, and that the GPU tests' layers reach every
kernel."""
import importlib.util
import os

import pytest

import contraction_rules
import paper_1412_7580_amd as pkg
from contraction_rules import PASSES

HERE = os.path.dirname(os.path.abspath(__file__))


def _module(path):
    spec = importlib.util.spec_from_file_location(os.path.basename(path)[:-3], path)
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    return contraction_rules.build(tmp_path_factory.mktemp("rules"))


def _layer(S, f, fo, h, k):
    return S, f, fo, h, h, k, k


def test_ordinary_layers(rules):
    assert rules.single("fprop", *_layer(128, 64, 64, 27, 5)) == ("tile3", "fast")
    assert rules.single("fprop", *_layer(128, 384, 384, 13, 3)) == ("bf16", "fast")
    assert rules.single("fprop", *_layer(32, 128, 128, 64, 31)) == ("bin4", "fast")
    assert rules.single("fprop", *_layer(128, 3, 96, 128, 11)) == ("product", "scalar")
    assert rules.single("accgrad", *_layer(128, 3, 96, 128, 11)) == ("thin_acc", "scalar")
    assert rules.single("fprop", *_layer(8, 256, 256, 27, 5)) == ("direct", "fast")
    assert rules.single("fprop", *_layer(8, 256, 256, 27, 5), no_direct=True) == ("tile6", "fast")
    assert rules.single("fprop", *_layer(20, 32, 128, 28, 3)) == ("tile6", "fast")
    assert rules.single("bprop", *_layer(50, 37, 75, 30, 7)) == ("tile3", "scalar")
    assert rules.pair(*_layer(128, 64, 64, 27, 5)) == "tiles"
    assert rules.pair(*_layer(128, 384, 384, 13, 3)) == "bf16"
    assert rules.pair(*_layer(128, 64, 64, 27, 5), no_pair=True) == "two launches"
    assert rules.pair(*_layer(32, 128, 128, 64, 31)) == "two launches"


@pytest.mark.parametrize("layer", [(130, 123, 127, 13, 3), (130, 123, 127, 20, 3), (128, 255, 255, 27, 5), (128, 385, 383, 8, 3)],
                         ids=lambda l: "S{}f{}fo{}_{}k{}".format(*l))
def test_4_byte_gathers_along_the_reduction_stay_in_fp32(rules, layer):
    """The bf16 kernel's 4-byte gathers cost a pass up to 30 % there; along the rows they gain 8 %."""
    assert rules.single("fprop", *_layer(*layer)) == ("tile3", "scalar")
    assert rules.single("bprop", *_layer(*layer)) == ("tile3", "scalar")
    assert rules.single("accgrad", *_layer(*layer)) == ("bf16", "scalar")
    assert rules.pair(*_layer(*layer)) == "two launches"


def test_general_addressing(rules):
    """Channel counts that are a multiple of 4 and not of a run: the bf16 kernel as under fast addressing,
    but for accGrad's grids that only the fp32 kernel holds in one round and shared launches of few tiles."""
    for layer, pair in (((128, 48, 48, 7, 3), "tiles"), ((128, 32, 96, 7, 3), "tiles"), ((64, 32, 384, 7, 3), "bf16"),
                        ((128, 100, 100, 13, 3), "bf16"), ((128, 196, 204, 27, 5), "bf16")):
        for p in PASSES:
            assert rules.single(p, *_layer(*layer)) == ("bf16", "vec"), (p, layer)
        assert rules.pair(*_layer(*layer)) == pair
    for layer in ((128, 196, 204, 10, 3), (16, 144, 144, 13, 3)):
        assert rules.single("bprop", *_layer(*layer)) == ("bf16", "vec")
        assert rules.single("accgrad", *_layer(*layer)) == ("tile3", "vec")
        assert rules.pair(*_layer(*layer)) == "bf16"
    assert rules.single("accgrad", *_layer(128, 32, 96, 10, 3)) == ("bf16", "fast")
    assert rules.single("fprop", *_layer(128, 100, 100, 27, 5)) == ("tile3", "vec")          # 36 products an element


SHARED = {   # backward passes with a thin side: where the shared launch measured faster, and where two did
    "tiles": [(16, 4, 16, 13, 3), (16, 4, 384, 28, 5), (128, 4, 64, 20, 3), (128, 4, 16, 28, 5), (64, 4, 128, 28, 5),
              (128, 4, 384, 13, 3), (64, 4, 384, 20, 3), (256, 4, 384, 8, 3), (128, 4, 4, 13, 3), (64, 16, 4, 32, 5),
              (256, 64, 4, 32, 5), (128, 64, 4, 112, 5), (16, 384, 4, 28, 5), (1, 64, 64, 13, 3), (1, 64, 128, 32, 5),
              (1, 512, 512, 8, 3), (1, 256, 256, 13, 3), (1, 128, 256, 20, 3), (512, 4, 4, 8, 3), (512, 4, 4, 13, 3)],
    "two launches": [(128, 4, 64, 28, 5), (128, 4, 128, 28, 5), (128, 4, 384, 20, 5), (256, 4, 128, 20, 5),
                     (1024, 4, 16, 32, 5), (32, 4, 16, 224, 5), (128, 4, 4, 32, 5), (256, 384, 4, 20, 5),
                     (1, 256, 256, 20, 3), (1, 512, 512, 13, 3), (1, 128, 256, 32, 5)],
}


@pytest.mark.parametrize("form,layer", [(f, l) for f, ls in SHARED.items() for l in ls], ids=lambda v: str(v).replace(" ", ""))
def test_shared_launch_of_a_backward_pass_with_a_thin_side(rules, form, layer):
    assert rules.pair(*_layer(*layer)) == form


def test_rows_a_lane_of_a_thin_product(rules):
    """As few as leave 8192 waves or fewer, 1 .. 8."""
    assert rules.rows("fprop", *_layer(64, 4, 384, 28, 5)) == 2          # 10752 waves at one
    assert rules.rows("fprop", *_layer(128, 4, 64, 56, 3)) == 2
    assert rules.rows("fprop", *_layer(16, 4, 64, 28, 5)) == 1
    assert rules.rows("fprop", *_layer(128, 3, 96, 128, 11)) == 8
    assert rules.rows("bprop", *_layer(64, 384, 4, 32, 5)) == 2


def test_thin_products_that_another_kernel_does_faster(rules):
    """Few rows for the n form, wide layers of four channels for the k form, one sample's gradient about
    the last-level cache's size, the widest layers at basis 64 for the acc form."""
    for layer in ((4, 4, 8, 40, 5), (16, 4, 256, 40, 5), (32, 4, 16, 56, 7), (64, 4, 64, 40, 5), (128, 4, 256, 64, 5)):
        assert rules.single("bprop", *_layer(*layer))[0] == "bin4", layer
    for layer in ((128, 4, 64, 56, 5), (256, 4, 16, 64, 5), (8, 3, 64, 40, 5), (64, 3, 384, 56, 5), (128, 3, 384, 40, 5)):
        assert rules.single("bprop", *_layer(*layer))[0] == "thin_n", layer
    assert rules.single("bprop", *_layer(64, 3, 384, 40, 5)) == ("shifted", "scalar")
    for layer in ((32, 4, 256, 56, 5), (64, 4, 256, 48, 5), (256, 4, 256, 40, 5)):
        assert rules.single("fprop", *_layer(*layer))[0] == "bin4", layer
    for layer in ((16, 4, 256, 64, 5), (128, 4, 64, 56, 5), (128, 4, 16, 40, 5)):
        assert rules.single("fprop", *_layer(*layer))[0] == "thin_k", layer
    assert rules.single("fprop", *_layer(128, 3, 384, 56, 5))[0] == "product"
    assert rules.single("bprop", *_layer(128, 256, 4, 56, 5))[0] == "thin_k"
    assert rules.single("fprop", *_layer(128, 4, 4, 8, 3))[0] == "tile3"
    assert rules.single("fprop", *_layer(128, 4, 4, 20, 3))[0] == "product"
    assert rules.single("fprop", *_layer(512, 4, 4, 8, 3))[0] == "product"
    for layer, kernel in (((1, 64, 64, 56, 3), "product"), ((1, 128, 256, 56, 3), "bin4"), ((1, 256, 256, 40, 5), "bin4"),
                          ((1, 256, 256, 56, 5), "product"), ((1, 128, 129, 48, 5), "product"), ((256, 4, 256, 64, 5), "bin4"),
                          ((256, 4, 64, 64, 5), "thin_acc"), ((256, 4, 256, 56, 5), "thin_acc")):
        assert rules.single("accgrad", *_layer(*layer))[0] == kernel, layer


def test_a_named_tile_shape_takes_every_layer_of_the_fp32_kernel(rules):
    for layer in ((128, 3, 96, 128, 11), (128, 384, 384, 13, 3), (8, 256, 256, 27, 5), (128, 64, 64, 27, 5)):
        for p in PASSES:
            for tile in (0, 3, 7):
                assert rules.single(p, *_layer(*layer), tile=tile)[0] == f"tile{tile}", (p, layer)


def test_the_benchmark_counts_the_products_of_the_kernel_that_runs(rules):
    bench = _module(os.path.join(os.path.dirname(HERE), "bench.py"))
    from paper_1412_7580_amd import synth
    units = {}
    for name in ("C2", "C3", "C4"):
        cfg = synth.CONV_CONFIGS[name]
        layer = tuple(cfg[k] for k in ("S", "f", "fo", "h", "w", "kh", "kw"))
        for basis in (cfg["N"], -1):
            used = dict(cfg, N=cfg["N"] if basis > 0 else bench.library_basis(cfg))
            for p in PASSES:
                model = bench.stage_model(used, p)["contraction"]
                bf16 = rules.single(p, *layer, basis)[0] == "bf16"
                assert model["unit"] == ("bf16" if bf16 else "fp32"), (name, p, basis)
                units.setdefault(name, set()).add(model["unit"])
                M, Nn, K = {"fprop": (cfg["S"], cfg["fo"], cfg["f"]), "bprop": (cfg["S"], cfg["f"], cfg["fo"]),
                            "accgrad": (cfg["fo"], cfg["f"], cfg["S"])}[p]
                bins = used["N"] * (used["N"] // 2 + 1)
                assert model["flops"] == (48 if bf16 else 6) * M * Nn * K * bins
            if name != "C4":
                shared = bench.kernel_model(used, "backward.contraction")
                assert rules.pair(*layer, basis) == {"bf16": "bf16", "fp32": "tiles"}[shared["unit"]]
                ent = bench.roofline_entry(0.2, shared)
                assert ent["frac_mfma"] == round(shared["flops"] / 0.2e-3 / 1e12 / bench.MFMA_PEAK_TFLOPS[shared["unit"]], 4)
    assert units == {"C2": {"fp32"}, "C3": {"bf16"}, "C4": {"fp32"}}


def test_the_gpu_test_reaches_every_kernel(rules):
    """Every kernel that a contraction can take, with every kind of gather and operand order it is built
    for, with rows, columns and reduction that leave a remainder, on short and on long runs."""
    gpu = _module(os.path.join(HERE, "test_gpu_contraction.py"))
    params = lambda test, names="S,f,fo": next(m.args[1] for m in test.pytestmark if m.name == "parametrize" and m.args[0] == names)
    layers = [(S, f, fo, h, h, 3, 2) for S, f, fo, h in gpu.EDGES + gpu.SPLIT + params(gpu.test_any_channel_counts_on_runs_of_four, "S,f,fo,side")]
    layers += [(*c, h, h, 3, 3) for c in params(gpu.test_thin_sides) for h in gpu.SIDES.values()]
    layers += [(*c, h, h, 3, 2) for t in (gpu.test_tile_edges, gpu.test_sides_of_at_most_sixteen) for c in params(t) for h in (8, 13, 20, 32)]
    got, ragged, pairs, walks = set(), set(), set(), set()
    for layer in layers:
        for p in PASSES:
            d = pkg.describe_plan(PASSES[p], *layer)
            kernel, gathers = rules.single(p, *layer)
            runs = "long" if d["tile_log2"] >= 5 else "short"
            if kernel == "direct":
                kernel += "16" if min(d["M"], d["N"]) <= 16 else "32"
            got.add((kernel, gathers, p, runs))
            tm, tn = {"tile6": (32, 128), "tile7": (128, 32), "direct16": (16, 16), "direct32": (32, 32), "shifted": (32, 32)}.get(kernel, (64, 64))
            for side, v in (("M", d["M"] % tm), ("N", d["N"] % tn), ("K", d["K"] % (8 if kernel == "direct32" else 16))):
                if v:
                    ragged.add((kernel, side))
            if kernel == "thin_k":
                walks.add((p, rules.rows(p, *layer) > 1, min(d["K"], 4)))
            if kernel == "product":
                walks.add((p, "product", d["K"]))
        pairs.add((rules.pair(*layer), rules.single("bprop", *layer)[1],
                   rules.single("accgrad", *layer)[0].startswith("thin") or rules.single("bprop", *layer)[0].startswith("thin")))
    missing = []
    for p in PASSES:
        for runs in ("long", "short"):
            missing += [k for k in (("bf16", "fast", p, runs), ("tile3", "vec", p, runs), ("tile3", "scalar", p, runs)) if k not in got]
            # (fprop and bprop with fast addressing on long runs have a reduction of 32 and more: what the bf16 kernel leaves of
            # them is the direct kernel's or the narrow tiles')
            if runs == "short" or p == "accgrad":
                missing += [("tile3", "fast", p, runs)] * (("tile3", "fast", p, runs) not in got)
        for g in ("fast", "vec"):
            missing += [("narrow", g, p)] * (not any((t, g, p, r) in got for t in ("tile6", "tile7") for r in ("long", "short")))
        missing += [(d, g, p) for d in ("direct16", "direct32") for g in ("fast", "vec", "scalar")
                    if not any((d, g, p, r) in got for r in ("long", "short"))]
        missing += [("bin4", p)] * (("bin4", "fast", p, "short") not in got)
        missing += [("shifted", p)] * (("shifted", "scalar", p, "short") not in got)
        missing += [("bf16", "vec", p)] * (("bf16", "vec", p, "long") not in got or ("bf16", "vec", p, "short") not in got)
    missing += [("bf16", "scalar", r) for r in ("long", "short") if ("bf16", "scalar", "accgrad", r) not in got]
    missing += [(t, g) for t in ("tile6", "tile7") for g in ("fast", "vec") if not any(k[:2] == (t, g) for k in got)]
    missing += [(k, s) for k in ("tile3", "tile6", "tile7", "bf16", "direct16", "direct32", "shifted") for s in "MNK" if (k, s) not in ragged]
    missing += [t for t in ("thin_n", "thin_acc") if not any(k[0] == t for k in got)]
    missing += [w for w in (("fprop", True, 4), ("bprop", True, 4), ("fprop", False, 3), ("bprop", False, 3), ("bprop", False, 1),
                            ("fprop", "product", 1), ("fprop", "product", 3), ("fprop", "product", 4), ("bprop", "product", 2),
                            ("bprop", "product", 3), ("bprop", "product", 4), ("accgrad", "product", 1)) if w not in walks]
    missing += [q for q in (("bf16", "fast", False), ("bf16", "vec", False), ("tiles", "fast", False), ("tiles", "vec", False),
                            ("tiles", "vec", True), ("two launches", "scalar", True), ("direct", "scalar", False), ("direct", "vec", False),
                            ("direct", "fast", False), ("scalar", "scalar", False)) if q not in pairs]
    assert not missing, missing
