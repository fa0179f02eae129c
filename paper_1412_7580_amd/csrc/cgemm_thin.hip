// Per-bin complex contractions with a side of at most four: the layers that meet the image's own
// one, three or four channels (a net's first layer, all three passes) or produce as few.
//
// Same operation as cgemm_kernels.hip (the Cgemm row of Table 1 of the fbfft paper).  With a side
// of 3 the matrix cores would multiply mostly padding, and at 96 output channels the layer is
// 5 flop a byte: the one large tensor has to stream.  So lanes run along the bins (the
// frequency tensors' contiguous direction), a lane works on four consecutive planes as one
// 16-byte access a component, and the products are fp32 on the vector units.  Runs of the layout
// longer than four put neighbouring quads of a run on neighbouring lanes.
#include "gemm_rules.hpp"
#include "thin.hpp"

namespace fc {

// Lane position: quad qi of a run and bin, from a flat index along (bin, quad of the run).
struct Lane { int qi, bin; };
__device__ __forceinline__ Lane lane_of(unsigned u, int tsh) {
    const int qs = tsh - 2;
    return Lane{(int)(u & ((1u << qs) - 1)), (int)(u >> qs)};
}

// K of at most four (fprop of a layer with few input channels, bprop of one with few output
// channels): C(m, n) = sum_k A(m, k) B(k, n).  A lane holds four columns of B and walks over
// `chunk` quads of rows, writing one quad of C a row.  Bound by the writes of C: 1632 bins of
// 1152 x 96 x 3 (first layer, 128x128 images on basis 56, 1.44 GB of C) 980 -> 325 us against the
// matrix-core kernel, whose 4-byte gathers and stores of runs of four fill a quarter of their lines.
// Workgroups of one (bins, rows) region, which share A, are numbered so that they run on one XCD.
template <int K, bool BKF>
__global__ void __launch_bounds__(256) cgemm_thin_k_kernel(GemmParams prm, int groups, int bin_blocks, int chunk) {
    const unsigned x = blockIdx.x % kXcds, s = blockIdx.x / kXcds;
    const unsigned region = s / groups * kXcds + x, g = s % groups;
    const unsigned bb = region % bin_blocks, mc = region / bin_blocks;
    const Lane ln = lane_of(bb * 256 + threadIdx.x, prm.layC.tsh);
    const long q = ((long)g << (prm.layC.tsh - 2)) + ln.qi;               // quad of columns
    if (ln.bin >= prm.bins || 4 * q >= prm.N) return;
    // B(k, n): planes n K + k (KF), or k * b_rs + n
    Rows<K> b;
    if constexpr (BKF) b.load(prm.B, prm.layB, q, (long)prm.N * K, ln.bin);
    else {
#pragma unroll
        for (int k = 0; k < K; ++k) b.v[k] = load_quad(prm.B, prm.layB, (k * prm.b_rs) / 4 + q, (long)K * prm.b_rs, ln.bin);
    }
    b.conj(prm.b_sign);
    const int mq_end = min((prm.M + 3) / 4, (int)(mc + 1) * chunk);
    for (int mq = mc * chunk; mq < mq_end; ++mq) {
        Rows<K> a;
        a.load(prm.A, prm.layA, mq, (long)prm.M * K, ln.bin);
        a.conj(prm.a_sign);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (4 * mq + r >= prm.M) break;
            Quad c;
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                float cr = 0.f, ci = 0.f;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    if constexpr (BKF) mac(cr, ci, a.re(r, k), a.im(r, k), b.re(n, k), b.im(n, k));
                    else mac(cr, ci, a.re(r, k), a.im(r, k), at4(b.v[k].re, n), at4(b.v[k].im, n));
                }
                put4(c.re, n, cr); put4(c.im, n, ci);
            }
            store_quad(prm.C, prm.layC, ((long)(4 * mq + r) * prm.c_rs) / 4 + q, ln.bin, c);
        }
    }
}

// N of at most four, reduction along the contiguous index of A (bprop of a layer with few input
// channels): a lane takes four rows at one bin and walks over K in quads; B's planes k N + n stay
// in the caches.  Bound by reading A.
template <int N>
__global__ void __launch_bounds__(256) cgemm_thin_n_kernel(GemmParams prm, int bin_blocks) {
    const unsigned bb = blockIdx.x % bin_blocks, rb = blockIdx.x / bin_blocks;
    const int bin = bb * 64 + (threadIdx.x & 63), mq = rb * 4 + (threadIdx.x >> 6);
    if (bin >= prm.bins || 4 * mq >= prm.M) return;
    float cr[4][N], ci[4][N];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int n = 0; n < N; ++n) cr[r][n] = ci[r][n] = 0.f;
    for (int kq = 0; 4 * kq < prm.K; ++kq) {
        Rows<N> b;
        b.load(prm.B, prm.layB, kq, (long)prm.K * N, bin);
        b.conj(prm.b_sign);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            Quad a = load_quad(prm.A, prm.layA, ((4 * mq + r) * prm.a_rs) / 4 + kq, prm.M * prm.a_rs, bin);
            flip4(a.im, prm.a_sign);
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int n = 0; n < N; ++n) mac(cr[r][n], ci[r][n], at4(a.re, k), at4(a.im, k), b.re(k, n), b.im(k, n));
        }
    }
    // rows 4 mq .. + 3 are planes 4 mq N ..: whole quads, but for the last row group
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int n = 0; n < N; ++n)
            if (4 * mq + r < prm.M) {
                float *p = prm.C + prm.layC.index((4 * mq + r) * prm.c_rs + n, bin, 0);
                p[0] = cr[r][n];
                p[1 << prm.layC.tsh] = ci[r][n];
            }
}

// N of at most four, reduction along the strided index of both operands (accGrad of a layer with
// few input channels): a lane takes four rows (output channels) at one bin, the eight waves of
// a workgroup split the reduction (samples and tiles) and meet in LDS.  Bound by reading A:
// 96 x 3 x 1152 on 1632 bins (1.44 GB) 1110 -> 347 us.
constexpr int kThinWaves = 8;
template <int N>
__global__ void __launch_bounds__(64 * kThinWaves) cgemm_thin_acc_kernel(GemmParams prm, int bin_blocks) {
    __shared__ float red[kThinWaves][8 * N][64];
    const unsigned bb = blockIdx.x % bin_blocks, g = blockIdx.x / bin_blocks;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const Lane ln = lane_of(bb * 64 + lane, prm.layA.tsh);
    const long q = ((long)g << (prm.layA.tsh - 2)) + ln.qi;               // quad of rows of C
    const bool live = ln.bin < prm.bins && 4 * q < prm.M;
    float cr[4][N], ci[4][N];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int n = 0; n < N; ++n) cr[r][n] = ci[r][n] = 0.f;
    if (live)
        for (int kq = wave; 4 * kq < prm.K; kq += kThinWaves) {
            Rows<N> b;
            b.load(prm.B, prm.layB, kq, (long)prm.K * N, ln.bin);
            b.conj(prm.b_sign);
            Quad a[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)                                    // a row past the last reads as zero ...
                a[k] = load_quad(prm.A, prm.layA, ((4 * kq + k) * prm.a_cs) / 4 + q, prm.K * prm.a_cs, ln.bin);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (4 * kq + k >= prm.K) break;                            // ... and what B's last quad holds past K is not used
                flip4(a[k].im, prm.a_sign);
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int n = 0; n < N; ++n) mac(cr[r][n], ci[r][n], at4(a[k].re, r), at4(a[k].im, r), b.re(k, n), b.im(k, n));
            }
        }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int n = 0; n < N; ++n) {
            red[wave][2 * (r * N + n)][lane] = cr[r][n];
            red[wave][2 * (r * N + n) + 1][lane] = ci[r][n];
        }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < N; ++e) {                                          // 8 N values over 8 waves
        const int v = wave * N + e, r = v / 2 / N, n = v / 2 % N, c = v % 2;
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < kThinWaves; ++w) sum += red[w][v][lane];
        if (live) prm.C[prm.layC.index((4 * q + r) * prm.c_rs + n, ln.bin, c)] = sum;
    }
}

template <class... P, class... Q>
static hipError_t launch_thin(void (*k)(P...), long grid, int block, LaunchCtx st, Q... q) {
    if (grid > 0x7fffffffL) return hipErrorInvalidValue;
    if (st.start || st.stop) hipExtLaunchKernelGGL(k, dim3((unsigned)grid), dim3(block), 0, st.stream, st.start, st.stop, 0, q...);
    else hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(block), 0, st.stream, q...);
    return hipGetLastError();
}

template <int W>
static hipError_t run_thin(Thin form, const GemmParams &p, LaunchCtx st) {
    const int per_run = 1 << (p.layC.tsh - 2);                             // quads of a run
    if (form == Thin::k) {
        const int groups = (p.N / 4 + per_run - 1) / per_run, bin_blocks = (p.bins * per_run + 255) / 256;
        const int mquads = (p.M + 3) / 4, chunk = thin_k_rows(p);
        const long regions = (long)bin_blocks * ((mquads + chunk - 1) / chunk);
        const long grid = (regions + kXcds - 1) / kXcds * kXcds * groups;
        if (p.b_cs != 1 || W == 1) return launch_thin(cgemm_thin_k_kernel<W, true>, grid, 256, st, p, groups, bin_blocks, chunk);
        return launch_thin(cgemm_thin_k_kernel<W, false>, grid, 256, st, p, groups, bin_blocks, chunk);
    }
    if (form == Thin::n) {
        const int bin_blocks = (p.bins + 63) / 64;
        return launch_thin(cgemm_thin_n_kernel<W>, (long)bin_blocks * (((p.M + 3) / 4 + 3) / 4), 256, st, p, bin_blocks);
    }
    const int bin_blocks = (p.bins * per_run + 63) / 64;
    return launch_thin(cgemm_thin_acc_kernel<W>, (long)bin_blocks * ((p.M / 4 + per_run - 1) / per_run), 64 * kThinWaves, st, p, bin_blocks);
}

hipError_t launch_cgemm_thin(const GemmParams &p, Thin form, LaunchCtx st) {
    switch (form == Thin::none ? 0 : form == Thin::k ? p.K : p.N) {
        case 1: return run_thin<1>(form, p, st);
        case 2: return run_thin<2>(form, p, st);
        case 3: return run_thin<3>(form, p, st);
        case 4: return run_thin<4>(form, p, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace fc
