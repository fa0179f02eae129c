// Rules of the contraction kernels that split the reduction or shift lines (paper_1412_7580_amd/csrc/gemm_rules.hpp) for a
// CPU program: no GPU, no launch.
#include "../../paper_1412_7580_amd/csrc/gemm_rules.hpp"

using namespace fc;

// v: M N K bins tile_log2 a_rs a_cs b_rs b_cs c_rs c_cs; operands `off` bytes past an aligned address.
static bool problem(const long *v, long off, Prepared *q) {
    const FreqLayout lay{(int)v[4], (int)v[3]};
    float *at = reinterpret_cast<float *>(((size_t)1 << 20) + off);
    const GemmProblem g{GemmOperand{at, lay, v[5], v[6], false}, GemmOperand{at, lay, v[7], v[8], false}, at, lay, v[9], v[10],
                        (int)v[0], (int)v[1], (int)v[2], (int)v[3], (int)v[3]};
    return prepare(g, GemmSwitches(), q) == hipSuccess;
}

extern "C" {
// out: shifted lines, split reduction possible, split reduction alone, product inside the inverse transform of `basis`
int split_single(const long *v, long off, int basis, int *out) {
    Prepared q;
    if (!problem(v, off, &q)) return -1;
    out[0] = q.shifted; out[1] = q.direct; out[2] = q.direct_alone; out[3] = product_inverse_pays(q, basis);
    return 0;
}
// out: the split reduction's shared launch, 64x64 tiles with 4-byte gathers
int split_pair(const long *bprop, const long *accgrad, int *out) {
    Prepared b, a;
    if (!problem(bprop, 0, &b) || !problem(accgrad, 0, &a)) return -1;
    out[0] = direct_pair_pays(b, a); out[1] = scalar_pair_pays(b, a);
    return 0;
}
}
