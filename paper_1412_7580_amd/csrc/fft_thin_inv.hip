// Inverse transforms whose input never stood in memory: the product of a contraction with a reduction
// of at most four, formed where the transform would read it.
//
// A net's first layer (fprop of three channels into f') multiplies little and writes a lot: its spectra
// Y are the largest tensor of the layer, written by one kernel only to be read by the next.  Here the
// workgroup that inverts T planes of Y forms them itself, bin by bin, in the LDS image that the
// inverse starts from (Section 6 of the fbfft paper plans such an integration of the products with
// the transforms).  What it reads instead are the K input planes of its sample and the weights' K
// planes per output channel, small tensors that stay in the caches.
#include "fft_kernels_impl.hpp"
#include "thin.hpp"

namespace fc {

// C(m, n) = sum_k A(m, k) B(k, n) for the planes p = m cols + n of a tile; A's planes are m K + k, B's n K + k
// (BKF) or k b_rs + n.  A lane takes four columns n of one row m, the layout's unit of 16 bytes, at bin after bin;
// the same operations in the same order as cgemm_thin_k_kernel.
struct ProductTile {
    const float *A, *B;
    FreqLayout lay;
    long b_rs;
    int terms, cols;
    bool bkf;
    unsigned a_sign, b_sign;

    template <int K, bool BKF, int BINS, int T, int BT>
    __device__ __forceinline__ void form(float *dst, long p0, int np, int tid) const {
        constexpr int Q = T / 4;
        static_assert(BT % Q == 0, "a lane keeps its quad of the run");
        const int q = tid % Q;
        if (4 * q >= np) return;
        const unsigned p = (unsigned)p0 + 4 * q, m = p / (unsigned)cols, n = p - m * cols;
        const float *pa[K], *pb[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            pa[k] = A + lay.index((long)m * K + k, 0, 0);
            pb[k] = B + (BKF ? lay.index((long)n * K + 4 * k, 0, 0) : lay.index(k * b_rs + n, 0, 0));
        }
#pragma unroll 4
        for (int bin = tid / Q; bin < BINS; bin += BT / Q) {
            const int o = bin * 2 * T;
            float ar[K], ai[K];
            Rows<K> b;                                     // BKF: rows n .. n + 3; else v[k] is row k
#pragma unroll
            for (int k = 0; k < K; ++k) {
                ar[k] = pa[k][o]; ai[k] = flip(pa[k][o + T], a_sign);
                b.v[k].re = *reinterpret_cast<const float4 *>(pb[k] + o);
                b.v[k].im = *reinterpret_cast<const float4 *>(pb[k] + o + T);
            }
            b.conj(b_sign);
            Quad c;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float cr = 0.f, ci = 0.f;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    if constexpr (BKF) mac(cr, ci, ar[k], ai[k], b.re(e, k), b.im(e, k));
                    else mac(cr, ci, ar[k], ai[k], at4(b.v[k].re, e), at4(b.v[k].im, e));
                }
                put4(c.re, e, cr); put4(c.im, e, ci);
            }
            *reinterpret_cast<float4 *>(dst + o + 4 * q) = c.re;
            *reinterpret_cast<float4 *>(dst + o + T + 4 * q) = c.im;
        }
    }
    template <int N, int T, int BT>
    __device__ __forceinline__ void fill(float *dst, long p0, int np, int tid) const {
        constexpr int BINS = N * (N / 2 + 1);
        if (bkf) {
            if (terms == 3) form<3, true, BINS, T, BT>(dst, p0, np, tid);
            else if (terms == 1) form<1, true, BINS, T, BT>(dst, p0, np, tid);
            else if (terms == 4) form<4, true, BINS, T, BT>(dst, p0, np, tid);
            else form<2, true, BINS, T, BT>(dst, p0, np, tid);
        } else {
            if (terms == 3) form<3, false, BINS, T, BT>(dst, p0, np, tid);
            else if (terms == 4) form<4, false, BINS, T, BT>(dst, p0, np, tid);
            else form<2, false, BINS, T, BT>(dst, p0, np, tid);
        }
    }
};

struct ProductInverse {
    Inv2dParams inv;
    ProductTile src;
};
template <int L, int G, int T>
__global__ void __launch_bounds__(T *(L * G / 2) * G) fft2d_c2r_product_kernel(ProductInverse prm) {
    fft2d_c2r_body<L, G, T, true, true, false, ProductTile>(prm.inv, blockIdx.x, nullptr, -1, prm.src);
}

template <int L, int G, int T>
static hipError_t run_product(const ProductTile &src, float *out, long planes, int h_out, int w_out, float scale, bool accumulate,
                              LaunchCtx st, const PlaneView *view) {
    constexpr int N = L * G, BT = T * (N / 2) * G;
    size_t lds;
    bool istage;
    ProductInverse prm{make_inv2d<L, G, T>(nullptr, out, planes, h_out, w_out, true, scale, accumulate, view, &lds, &istage, true), src};
    lds = with_twiddle_table<L, G>(lds, &prm.inv.tw_off);
    auto k = fft2d_c2r_product_kernel<L, G, T>;
    if (hipError_t e = allow_big_lds((const void *)k, lds); e != hipSuccess) return e;
    launch_kernel(k, dim3((unsigned)((planes + T - 1) / T)), dim3(BT), lds, st, prm);
    return hipGetLastError();
}

// Lanes per line as the ordinary inverse takes them, but at least two: one lane per line leaves a
// quarter of the waves, which the products' loads need.
static hipError_t dispatch_product(int N, const ProductTile &src, float *out, long planes, int h, int w, float scale, bool acc,
                                   LaunchCtx st, const PlaneView *view) {
    switch (N) {
        case 8: return run_product<4, 2, 64>(src, out, planes, h, w, scale, acc, st, view);
        case 10: return run_product<5, 2, 32>(src, out, planes, h, w, scale, acc, st, view);
        case 12: return run_product<6, 2, 32>(src, out, planes, h, w, scale, acc, st, view);
        case 14: return run_product<7, 2, 32>(src, out, planes, h, w, scale, acc, st, view);
        case 16: return run_product<8, 2, 32>(src, out, planes, h, w, scale, acc, st, view);
        case 18: return run_product<9, 2, 16>(src, out, planes, h, w, scale, acc, st, view);
        case 20: return run_product<10, 2, 16>(src, out, planes, h, w, scale, acc, st, view);
        case 24: return run_product<6, 4, 16>(src, out, planes, h, w, scale, acc, st, view);
        case 28: return run_product<7, 4, 16>(src, out, planes, h, w, scale, acc, st, view);
        case 32: return run_product<8, 4, 8>(src, out, planes, h, w, scale, acc, st, view);
        case 36: return run_product<9, 4, 4>(src, out, planes, h, w, scale, acc, st, view);
        case 40: return run_product<10, 4, 4>(src, out, planes, h, w, scale, acc, st, view);
        case 48: return run_product<12, 4, 4>(src, out, planes, h, w, scale, acc, st, view);
        case 56: return run_product<14, 4, 4>(src, out, planes, h, w, scale, acc, st, view);
        default: return hipErrorNotSupported;
    }
}

hipError_t launch_fft2d_c2r_product(const GemmParams &g, float *out, int N, int h_out, int w_out, float scale,
                                    bool accumulate, LaunchCtx st, const PlaneView *view) {
    const long planes = (long)g.M * g.N;
    if (g.K < 1 || g.K > 4 || g.N % 4 || g.c_rs != g.N || g.a_rs != g.K || planes <= 0) return hipErrorInvalidValue;
    const bool bkf = g.b_cs != 1 || g.K == 1;
    const ProductTile src{g.A, g.B, g.layA, g.b_rs, g.K, g.N, bkf, g.a_sign, g.b_sign};
    return dispatch_product(N, src, out, planes, h_out, w_out, scale, accumulate, st, view);
}

}  // namespace fc
