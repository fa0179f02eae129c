// The contraction's rules (paper_1412_7580_amd/csrc/gemm_rules.hpp) for a CPU program: no GPU, no launch.
#include "../../paper_1412_7580_amd/csrc/gemm_rules.hpp"

using namespace fc;

// v: M N K bins tile_log2 a_rs a_cs b_rs b_cs c_rs c_cs; operands `off` bytes past an aligned address.
static bool problem(const long *v, long off, const GemmSwitches &sw, Prepared *q) {
    const FreqLayout lay{(int)v[4], (int)v[3]};
    float *at = reinterpret_cast<float *>(((size_t)1 << 20) + off);
    const GemmProblem g{GemmOperand{at, lay, v[5], v[6], false}, GemmOperand{at, lay, v[7], v[8], false}, at, lay, v[9], v[10],
                        (int)v[0], (int)v[1], (int)v[2], (int)v[3], (int)v[3]};
    return prepare(g, sw, q) == hipSuccess;
}
// sw: tile shape (-1: none), no_pair, no_direct
static GemmSwitches switches(const long *sw) {
    GemmSwitches s;
    s.tile = (int)sw[0];
    s.no_pair = sw[1] != 0;
    s.no_direct = sw[2] != 0;
    return s;
}

extern "C" {
// out: kernel of the pass (0 product inside the inverse of `basis`, 1 thin, 2 direct, 3 four bins, 4 shifted lines, 5 bf16, 6
// tiles), 16-byte gathers, fast addressing, thin form, tile shape, quads of rows a lane of the thin k form walks over,
// whether the direct kernel and the shifted lines are possible
int rules_single(const long *v, long off, int basis, const long *sw, int *out) {
    Prepared q;
    const GemmSwitches s = switches(sw);
    if (!problem(v, off, s, &q)) return -1;
    out[0] = (int)kernel_of_pass(q, basis); out[1] = q.vec; out[2] = q.prm.fast; out[3] = (int)q.thin;
    out[4] = pick_tile(s, q.prm, q.vec); out[5] = q.thin == Thin::k ? thin_k_rows(q.prm) : 0;
    out[6] = q.direct; out[7] = q.shifted;
    return 0;
}
// 0: two launches, 1: the direct kernel, 2: 64x64 tiles, 3: bf16, 4: 64x64 tiles with 4-byte gathers
int rules_pair(const long *bprop, const long *accgrad, const long *sw) {
    Prepared b, a;
    const GemmSwitches s = switches(sw);
    if (!problem(bprop, 0, s, &b) || !problem(accgrad, 0, s, &a)) return -1;
    return (int)shared_launch(b, a, s);
}
// The kernel of one gradient alone, the other being its partner in the shared launch: out[1] = 1 on the shared launch's waves.
int rules_lone(const long *one, const long *partner, const long *sw, int *out) {
    Prepared q, o;
    const GemmSwitches s = switches(sw);
    if (!problem(one, 0, s, &q) || !problem(partner, 0, s, &o)) return -1;
    const Lone l = lone_gradient(q, o, s);
    out[0] = (int)l.kernel; out[1] = l.as_shared;
    return 0;
}
}
