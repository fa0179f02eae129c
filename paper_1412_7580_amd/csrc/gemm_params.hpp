// Parameters shared by the contraction kernels.
#pragma once
#include "kernels.hpp"

namespace fc {

typedef float floatx16 __attribute__((ext_vector_type(16)));

struct GemmParams {
    const float *A, *B;
    float *C;
    FreqLayout layA, layB, layC;
    long a_rs, a_cs, b_rs, b_cs, c_rs, c_cs;
    int M, N, K, bins, live;   // bins from `live` on are padding
    int tiles_m, tiles_n;
    unsigned a_sign, b_sign;   // 0x80000000 to conjugate the operand (flips Im on the way to the MFMA)
    unsigned split_from;       // cgemm_tail_kernel: first workgroup index of the quadrant workgroups
    int fast;                  // addresses split into a uniform and a per-lane part (fast_addressing())
};

__device__ __forceinline__ float flip(float v, unsigned sign) {
    return __builtin_bit_cast(float, __builtin_bit_cast(unsigned, v) ^ sign);
}

// Contractions on the bf16 matrix cores (cgemm_split.hip).  vec: 16-byte gathers are possible.  A pair is
// bprop (A along the reduction) and accGrad (A along the rows), akf1 saying which comes first.
hipError_t launch_cgemm_split(GemmParams prm, bool akf, bool bkf, bool vec, LaunchCtx st);
hipError_t launch_cgemm_split_pair(const GemmParams &p1, bool akf1, const GemmParams &p2, LaunchCtx st);

// Contractions with a narrow side or few tiles (cgemm_direct.hip).  partner: the other product of the shared launch that
// this one is to agree with bit for bit.
hipError_t launch_cgemm_direct(GemmParams prm, bool akf, bool bkf, LaunchCtx st, const GemmParams *partner = nullptr);
hipError_t launch_cgemm_direct_pair(const GemmParams &bprop, const GemmParams &accgrad, LaunchCtx st);

// Contractions with a side of at most four (cgemm_thin.hip), in one of three forms (thin_form()).
enum class Thin { none, k, n, acc };
hipError_t launch_cgemm_thin(const GemmParams &prm, Thin form, LaunchCtx st);
// The k form's product as the input of the inverse transform (fft_thin_inv.hip).
hipError_t launch_fft2d_c2r_product(const GemmParams &g, float *out, int N, int h_out, int w_out, float scale,
                                    bool accumulate, LaunchCtx st, const PlaneView *view);

constexpr int kXcds = 8;   // workgroup i is placed on XCD i % kXcds

}  // namespace fc
