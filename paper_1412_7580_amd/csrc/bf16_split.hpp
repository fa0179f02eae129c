// fp32 products on the bf16 matrix cores: the cut of a value into three bf16 terms (Dekker's splitting),
// the six-product complex multiply-accumulate, and bounds-checked buffer loads for the gathers.
#pragma once
#include "gemm_params.hpp"

namespace fc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ unsigned pack_bf16(float a, float b) {        // v_cvt_pk_bf16_f32: to nearest even
    const floatx2 v = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ float low_of(unsigned p) { return __builtin_bit_cast(float, p << 16); }
__device__ __forceinline__ float high_of(unsigned p) { return __builtin_bit_cast(float, p & 0xffff0000u); }

// (a, b) = h + m + l: rounding to 8 bits leaves a remainder of at most 16 significant bits, rounding
// that one of at most 8, and both subtractions are exact.  So the cut is, where h stays finite
// (below 3.39e38) and l, which may end 23 bits under h, does not fall under bf16's smallest
// subnormal, 2^-133: for sizes from 2^-110 on.  Conversion and matrix cores keep subnormals.
__device__ __forceinline__ void split2(float a, float b, unsigned &h, unsigned &m, unsigned &l) {
    h = pack_bf16(a, b);
    const float ra = a - low_of(h), rb = b - high_of(h);
    m = pack_bf16(ra, rb);
    l = pack_bf16(ra - low_of(m), rb - high_of(m));
}
__device__ __forceinline__ void split4(float a, float b, float c, float d, uint2 &h, uint2 &m, uint2 &l) {
    split2(a, b, h.x, m.x, l.x);
    split2(c, d, h.y, m.y, l.y);
}

__device__ __forceinline__ bf16x8 negated(bf16x8 v) {
    uint4 u = __builtin_bit_cast(uint4, v);
    u.x ^= 0x80008000u; u.y ^= 0x80008000u; u.z ^= 0x80008000u; u.w ^= 0x80008000u;
    return __builtin_bit_cast(bf16x8, u);
}

// The upper lane half of a and the lower one of b trade places: a = (a.low, b.low), b = (a.high, b.high).
__device__ __forceinline__ void swap_halves(float &a, float &b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
    const unsigned x = r[0], y = r[1];
    a = __builtin_bit_cast(float, x);
    b = __builtin_bit_cast(float, y);
}

// One 32x32 tile, 16 of K: c += ar br + ai bi (the caller negates what the component asks for);
// [0..2] = h, m, l.  The five small products of each term meet in a sum of their own, so that a
// long reduction rounds at its full magnitude three times per 16 terms and not twelve.
__device__ __forceinline__ void multiply_split(floatx16 &c, const bf16x8 (&ar)[3], const bf16x8 (&br)[3],
                                               const bf16x8 (&ai)[3], const bf16x8 (&bi)[3]) {
    constexpr int ta[5] = {2, 0, 1, 1, 0}, tb[5] = {0, 2, 1, 0, 1};
    floatx16 low = {};
#pragma unroll
    for (int t = 0; t < 5; ++t) {
        low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ar[ta[t]], br[tb[t]], low, 0, 0, 0);
        low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ai[ta[t]], bi[tb[t]], low, 0, 0, 0);
    }
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ar[0], br[0], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ai[0], bi[0], c, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 16; ++v) c[v] += low[v];
}

// fp32 spans more than that, so the operands are cut at a power of two of their own.  2^16 makes the
// cut exact for everything below 2^111, subnormals too (all are whole numbers of 2^-149).  What is larger,
// and products whose sums pass 2^96, leave an infinity or a NaN in the sums; then one operand,
// the other, and last both are halved instead.  (Halved, the cut is exact from 2^-109 on: 2^-205
// of what made it necessary, or less.)
constexpr float kScaleUp = 65536.f, kScaleDown = 0.5f;
constexpr int kScalings = 4;
__device__ __forceinline__ float scale_a(int attempt) { return attempt & 1 ? kScaleDown : kScaleUp; }
__device__ __forceinline__ float scale_b(int attempt) { return attempt & 2 ? kScaleDown : kScaleUp; }

// 0 for finite sums, else NaN.
__device__ __forceinline__ float non_finite(const floatx16 &c, float t) {
#pragma unroll
    for (int v = 0; v < 16; ++v) t = fmaf(c[v], 0.f, t);
    return t;
}

// Loads from a base that is uniform over the wave at per-lane byte offsets below 2^31; an offset
// with the top bit set is out of range and reads as zero.
struct BufferView {
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ __forceinline__ explicit BufferView(const float *base)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0, 0x80000000u, 4u << 15)) {}   // format: 32
    __device__ __forceinline__ float load1(unsigned voff, unsigned soff) const {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, voff, soff, 0));
    }
    __device__ __forceinline__ void load4(float (&d)[4], unsigned voff, unsigned soff) const {
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, soff, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) { const unsigned w = v[i]; d[i] = __builtin_bit_cast(float, w); }
    }
};

}  // namespace fc
