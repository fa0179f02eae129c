// Pieces of the products with a side of at most four: quads of planes at one bin, and rows of W planes.
#pragma once
#include "gemm_params.hpp"

namespace fc {

struct Quad { float4 re, im; };

__device__ __forceinline__ float at4(const float4 &v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }
__device__ __forceinline__ void put4(float4 &v, int i, float f) { (i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w) = f; }

// Planes 4 q .. 4 q + 3 at one bin; planes from `planes` on (rounded up to four) read as zero.
__device__ __forceinline__ Quad load_quad(const float *base, const FreqLayout &lay, long q, long planes, int bin) {
    Quad v;
    if (4 * q < planes) {
        const float *p = base + lay.index(4 * q, bin, 0);
        v.re = *reinterpret_cast<const float4 *>(p);
        v.im = *reinterpret_cast<const float4 *>(p + (1 << lay.tsh));
    } else {
        v.re = v.im = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    return v;
}
__device__ __forceinline__ void store_quad(float *base, const FreqLayout &lay, long q, int bin, const Quad &v) {
    float *p = base + lay.index(4 * q, bin, 0);
    *reinterpret_cast<float4 *>(p) = v.re;
    *reinterpret_cast<float4 *>(p + (1 << lay.tsh)) = v.im;
}
__device__ __forceinline__ void flip4(float4 &v, unsigned s) { v.x = flip(v.x, s); v.y = flip(v.y, s); v.z = flip(v.z, s); v.w = flip(v.w, s); }

// Four rows of an operand whose row r lives at planes r * W .. r * W + W - 1: rows 4 q .. 4 q + 3
// are W whole quads, and element (r, c) of them is number r * W + c.
template <int W>
struct Rows {
    Quad v[W];
    __device__ __forceinline__ void load(const float *base, const FreqLayout &lay, long q, long planes, int bin) {
#pragma unroll
        for (int i = 0; i < W; ++i) v[i] = load_quad(base, lay, q * W + i, planes, bin);
    }
    __device__ __forceinline__ float re(int r, int c) const { return at4(v[(r * W + c) / 4].re, (r * W + c) % 4); }
    __device__ __forceinline__ float im(int r, int c) const { return at4(v[(r * W + c) / 4].im, (r * W + c) % 4); }
    __device__ __forceinline__ void conj(unsigned s) {
#pragma unroll
        for (int i = 0; i < W; ++i) flip4(v[i].im, s);
    }
};

__device__ __forceinline__ void mac(float &cr, float &ci, float ar, float ai, float br, float bi) {
    cr = fmaf(ar, br, cr); cr = fmaf(-ai, bi, cr);
    ci = fmaf(ar, bi, ci); ci = fmaf(ai, br, ci);
}

}  // namespace fc
