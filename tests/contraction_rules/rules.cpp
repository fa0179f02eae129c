// The contraction's rules (paper_1412_7580_amd/csrc/gemm_rules.hpp) for a CPU program: no GPU, no launch.
#include "../../paper_1412_7580_amd/csrc/gemm_rules.hpp"

using namespace fc;

// v: M N K bins tile_log2 a_rs a_cs b_rs b_cs c_rs c_cs; operands at aligned addresses.
static bool problem(const long *v, const GemmSwitches &sw, Prepared *q) {
    const FreqLayout lay{(int)v[4], (int)v[3]};
    float *at = reinterpret_cast<float *>((size_t)1 << 20);
    const GemmProblem g{GemmOperand{at, lay, v[5], v[6], false}, GemmOperand{at, lay, v[7], v[8], false}, at, lay, v[9], v[10],
                        (int)v[0], (int)v[1], (int)v[2], (int)v[3], (int)v[3]};
    return prepare(g, sw, q) == hipSuccess;
}
// sw: tile shape (-1: none), then no_pair
static GemmSwitches switches(const long *sw) {
    GemmSwitches s;
    s.tile = (int)sw[0];
    s.no_pair = sw[1] != 0;
    return s;
}

extern "C" {
// out: k contiguous in A, in B, 16-byte gathers, fast addressing, thin form, four-bin kernel, bf16 kernel, tile shape,
// quads of rows a lane of the thin k form walks over
int rules_single(const long *v, const long *sw, int *out) {
    Prepared q;
    const GemmSwitches s = switches(sw);
    if (!problem(v, s, &q)) return -1;
    out[0] = q.akf; out[1] = q.bkf; out[2] = q.vec; out[3] = q.prm.fast;
    out[4] = (int)q.thin; out[5] = q.bingroup; out[6] = q.split_alone; out[7] = pick_tile(s, q.prm, q.vec);
    out[8] = q.thin == Thin::k ? thin_k_rows(q.prm) : 0;
    return 0;
}
// 0: two launches, 1: one launch of 64x64 tiles, 2: one launch of the bf16 kernel
int rules_pair(const long *bprop, const long *accgrad, const long *sw) {
    Prepared b, a;
    const GemmSwitches s = switches(sw);
    if (!problem(bprop, s, &b) || !problem(accgrad, s, &a)) return -1;
    return (int)pair_form(b, a, s);
}
}
