// Per-bin complex contraction on the bf16 matrix cores, for layers whose channels and samples are
// many enough that the fp32 ones would be the bound (see split_pays()).
//
// Same operation as cgemm_kernels.hip (the Cgemm row of Table 1 of the fbfft paper), same layout,
// same order of workgroups.  Every fp32 operand value is cut, without loss, into three bf16 terms
// (x = h + m + l: each is the rounded value of what the ones before it leave, and 8 + 8 + 8 bits
// hold the whole significand; bf16_split.hpp has the range and what widens it to all of fp32), and
// a real product is the six bf16 products hh, hm, mh, mm, hl, lh, which are exact and are summed in
// fp32 by v_mfma_f32_32x32x16_bf16.  What is left out (ml, lm, ll) is at most 2^-23 of |a b| and of
// either sign, 2^-26 on average: below the rounding of the fp32 sum itself.  The fp32 MFMA does 2 of
// K in 64 cycles, the six products do 16 of K in 192.
//     Cr += Ar Br - Ai Bi,   Ci += Ar Bi + Ai Br      (four real products, no cancellation)
// Relative 2-norm error of the passes against 64 bits, three-product fp32 form -> this: 128 samples,
// 384 -> 384 channels, 13x13: 4.5e-7 / 4.9e-7 / 2.9e-7 -> 2.1e-7 / 2.3e-7 / 1.8e-7.
//
// Workgroup = 4 waves, a 64x64 tile, each wave one MFMA tile of 32x32 (re and im accumulators).  K is
// walked in tiles of 16 through one LDS image of both operands, cut on the way from the staging
// registers; the next tile's global loads are in flight while the current one is multiplied, and
// the barriers around the image are covered by the compute unit's other workgroups: four at 128
// registers under fast addressing (a build that spilled to stay there was 10 % slower on the
// backward pair), three or four under general.  The matrix cores are 55 .. 62 % busy, and the vector
// units with the cuts beside them about half the cycles.  128x64 tiles and two tiles of staging
// measured no faster, K tiles of 32 slower.  That layer's training step 485 -> 422 .. 440 us by the card;
// 128 x 256 -> 256 240 -> 219, 128 x 192 -> 192 163 -> 144, 8x8 images, 256 x 128 -> 128 88 -> 74.
#include "gemm_params.hpp"
#include "bf16_split.hpp"

namespace fc {

constexpr unsigned kOutside = 0x80000000u;       // byte offset past every buffer range

constexpr int ROWS = 64, TK = 16, KQ = TK / 4;

// How an operand's tile is addressed.  Fast: see prepare().  General: any strides, and along the rows
// any extents, by index arithmetic for each gather.
enum : int { kFast = 0, kGeneral = 1 };

// FreqLayout::index for a plane number of 32 bits, which every plane of a plan has: one wide product.
__device__ __forceinline__ size_t element(const FreqLayout &lay, unsigned plane, int bin, int c) {
    const unsigned pt = plane >> lay.tsh, pl = plane & ((1u << lay.tsh) - 1);
    return ((((size_t)pt * (unsigned)lay.bins + (unsigned)bin) * 2 + c) << lay.tsh) + pl;
}

// Loader of one operand tile (ROWS x TK) with the "row" index being m (or n) and the
// reduction index k.  KF: k is the contiguous plane index, and a unit of work is four
// consecutive k of one row, as one 16-byte gather; else the row index is contiguous, lanes run
// along the rows and a unit is four 4-byte gathers (as many cache lines a byte as wider loads
// would touch, and the four k that one LDS word pair holds meet in one lane).
// LDS image: [6 = (re, im) x (h, m, l)][k / 8][row][k % 8] of bf16: a fragment is one 16-byte load at a
// constant offset from the lane's address (8-byte pieces by k / 4 cost an address each, 11 of 159 vector
// instructions a K tile), and both kinds of unit store 8 bytes of it.  Octets padded so that the stores
// along k do not meet in the banks (48 cycles a wave and K tile) measured no different.
template <bool KF, int MODE>
struct SplitLoader {
    static constexpr int OCTET = ROWS * 16, PLANE = TK / 8 * OCTET, BYTES = 6 * PLANE;
    float re[4], im[4];
    unsigned off;        // byte offset of this lane's unit from the tile's base, which is uniform

    static __device__ __forceinline__ int row_of(int tid) { return KF ? tid / KQ : tid % ROWS; }
    static __device__ __forceinline__ int kq_of(int tid) { return KF ? tid % KQ : tid / ROWS; }

    // The strided index moves in whole plane tiles (fast_addressing() in gemm_rules.hpp), so an
    // address is a uniform base that changes with the K tile and an offset that never does.
    __device__ __forceinline__ void prepare(const FreqLayout &lay, long rs, long cs, int r0, int R, int tid) {
        if constexpr (MODE != kFast) return;
        const int rr = row_of(tid), kk = 4 * kq_of(tid);
        const size_t o = KF ? (size_t)rr * rs * lay.bins * 2 + lay.part(kk)
                            : lay.part(rr) + (size_t)kk * cs * lay.bins * 2;
        off = r0 + rr < R ? (unsigned)(o * sizeof(float)) : kOutside;
    }

    __device__ __forceinline__ void load(const float *base, const FreqLayout &lay, long rs, long cs, int bin, int r0,
                                         int k0, int R, int K, int tid) {
        if constexpr (MODE != kFast) {
            load_general(base, lay, rs, cs, bin, r0 + row_of(tid), k0 + 4 * kq_of(tid), R, K);
            return;
        }
        size_t o = (size_t)bin * (2u << lay.tsh);
        if constexpr (KF) o += (size_t)r0 * rs * lay.bins * 2 + lay.part(k0);
        else o += lay.part(r0) + (size_t)k0 * cs * lay.bins * 2;
        const BufferView buf(base + o);
        const unsigned im_bytes = 4u << lay.tsh;
        const int kk = k0 + 4 * kq_of(tid);
        if constexpr (KF) {                               // K is a multiple of 4
            const unsigned v = kk < K ? off : kOutside;
            buf.load4(re, v, 0);
            buf.load4(im, v, im_bytes);
        } else {
            const unsigned kstep = (unsigned)(cs * lay.bins * 8);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const unsigned v = kk + j < K ? off : kOutside;
                re[j] = buf.load1(v, j * kstep);
                im[j] = buf.load1(v, j * kstep + im_bytes);
            }
        }
    }

    __device__ __forceinline__ void load_general(const float *base, const FreqLayout &lay, long rs, long cs, int bin,
                                                 int r, int kk, int R, int K) {
        const unsigned im_off = 1u << lay.tsh;
#pragma unroll
        for (int j = 0; j < 4; ++j) { re[j] = 0.f; im[j] = 0.f; }
        if (r >= R) return;
        if constexpr (KF) {                               // cs is 1 ...
            if (kk < K) {                                 // K is a multiple of 4
                const float *q = base + element(lay, (unsigned)r * (unsigned)rs + kk, bin, 0);
                const float4 a = *reinterpret_cast<const float4 *>(q), b = *reinterpret_cast<const float4 *>(q + im_off);
                re[0] = a.x; re[1] = a.y; re[2] = a.z; re[3] = a.w;
                im[0] = b.x; im[1] = b.y; im[2] = b.z; im[3] = b.w;
            }
        } else {                                          // ... or rs is
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (kk + j < K) {
                    const float *q = base + element(lay, r + (unsigned)(kk + j) * (unsigned)cs, bin, 0);
                    re[j] = q[0];
                    im[j] = q[im_off];
                }
        }
    }

    // Terms of the staged values, times `scale`, into the LDS image; `sign` conjugates.
    __device__ __forceinline__ void store(char *img, float scale, unsigned sign, int tid) const {
        const int kq = kq_of(tid);
        char *q = img + (kq >> 1) * OCTET + row_of(tid) * 16 + (kq & 1) * 8;
        uint2 h, m, l;
        split4(scale * re[0], scale * re[1], scale * re[2], scale * re[3], h, m, l);
        *reinterpret_cast<uint2 *>(q) = h;
        *reinterpret_cast<uint2 *>(q + PLANE) = m;
        *reinterpret_cast<uint2 *>(q + 2 * PLANE) = l;
        const float si = flip(scale, sign);
        split4(si * im[0], si * im[1], si * im[2], si * im[3], h, m, l);
        *reinterpret_cast<uint2 *>(q + 3 * PLANE) = h;
        *reinterpret_cast<uint2 *>(q + 4 * PLANE) = m;
        *reinterpret_cast<uint2 *>(q + 5 * PLANE) = l;
    }

    // MFMA fragment of plane c: lane half lk holds k 8 lk .. 8 lk + 7.
    static __device__ __forceinline__ bf16x8 fragment(const char *img, int c, int row, int lk) {
        return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(img + c * PLANE + lk * OCTET + row * 16));
    }
};

// This lane's number, computed anew at each place that asks, so that neither it nor what follows
// from it takes registers in between.
__device__ __forceinline__ int lane_number() {
    unsigned zero = 0;
    asm volatile("" : "+v"(zero));
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, zero));
}

// One workgroup's share of the contraction, workgroup number wg of prm's grid, with the operands cut at
// the given powers of two.  False, for all of the workgroup, if that left a sum that is not finite:
// nothing is stored then, unless it is the last attempt.  (The question after the stores instead
// waits for them at its barrier: accGrad of 128 x 64 -> 64, 8x8 22.7 -> 25.0 us.)
template <bool AKF, bool BKF, int MODE>
__device__ __forceinline__ bool cgemm_split_attempt(const GemmParams &prm, const unsigned wg, const int wave, const float scale_a,
                                                    const float scale_b, const bool last, char *smem) {
    using LoadA = SplitLoader<AKF, MODE>;
    using LoadB = SplitLoader<BKF, MODE>;
    char *As = smem, *Bs = As + LoadA::BYTES;

    const int lane = lane_number(), tid = wave * 64 + lane;
    const int wm = wave >> 1, wn = wave & 1;

    // XCD-aware decomposition of the flat workgroup index (see the head of cgemm_kernels.hip).
    const int tiles = prm.tiles_m * prm.tiles_n;
    const int xcd = wg % kXcds, slot = wg / kXcds;
    const int bins_per_xcd = prm.bins / kXcds;
    const int bin = xcd * bins_per_xcd + slot / tiles;
    const int tile = slot % tiles;
    const int tm = tile / prm.tiles_n, tn = tile % prm.tiles_n;
    const int m0 = tm * ROWS, n0 = tn * ROWS;
    const int M = prm.M, N = prm.N, K = prm.K;

    floatx16 acc_r, acc_i;
#pragma unroll
    for (int v = 0; v < 16; ++v) { acc_r[v] = 0.f; acc_i[v] = 0.f; }

    LoadA la;
    LoadB lb;
    la.prepare(prm.layA, prm.a_rs, prm.a_cs, m0, M, tid);
    lb.prepare(prm.layB, prm.b_cs, prm.b_rs, n0, N, tid);     // B(k, n): the loader's row index is n
    auto issue = [&](int k0) {
        la.load(prm.A, prm.layA, prm.a_rs, prm.a_cs, bin, m0, k0, M, K, tid);
        lb.load(prm.B, prm.layB, prm.b_cs, prm.b_rs, bin, n0, k0, N, K, tid);
    };
    const int lrow = lane & 31, lk = lane >> 5;
    issue(0);
    for (int k0 = 0; k0 < K; k0 += TK) {
        if (k0) __syncthreads();                 // every wave has read the previous tile
        la.store(As, scale_a, prm.a_sign, tid);
        __builtin_amdgcn_sched_barrier(0);       // ... without waiting for B's gathers
        lb.store(Bs, scale_b, prm.b_sign, tid);
        __syncthreads();
        if (k0 + TK < K) issue(k0 + TK);
        __builtin_amdgcn_sched_barrier(0);       // ... and the gathers stay in front of the products
        bf16x8 ar[3], ai[3], br[3], bi[3];
#pragma unroll
        for (int u = 0; u < 3; ++u) {            // the terms in the order of the products' first use
            constexpr int fa[3] = {2, 0, 1}, fb[3] = {0, 2, 1};
            ar[fa[u]] = LoadA::fragment(As, fa[u], wm * 32 + lrow, lk);
            bi[fb[u]] = LoadB::fragment(Bs, 3 + fb[u], wn * 32 + lrow, lk);
            ai[fa[u]] = LoadA::fragment(As, 3 + fa[u], wm * 32 + lrow, lk);
            br[fb[u]] = LoadB::fragment(Bs, fb[u], wn * 32 + lrow, lk);
            __builtin_amdgcn_sched_barrier(0);
        }
        // one component after the other: registers for one sum of small products, and the
        // negated terms take the place of the others
        multiply_split(acc_i, ar, bi, ai, br);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < 3; ++t) bi[t] = negated(bi[t]);
        multiply_split(acc_r, ar, br, ai, bi);
    }

    if (!last) {
        // one flag a wave, beside the image: the next attempt writes it after barriers of its own
        int *redo = reinterpret_cast<int *>(Bs + LoadB::BYTES);
        const bool bad = __ballot(non_finite(acc_i, non_finite(acc_r, 0.f)) != 0.f) != 0;
        if (lane_number() == 0) redo[wave] = bad;
        __syncthreads();                         // ... and every wave has read the image
        if (redo[0] | redo[1] | redo[2] | redo[3]) return false;
    }
    const float unscale = 1.f / (scale_a * scale_b);                      // a power of two

    // D layout of the 32x32 MFMA: lane l, register v -> row 8*(v/4) + 4*(l/32) + v%4, col l%32.
    // The lane halves trade places between the components, so that one store covers a row's real
    // parts (lanes 0 .. 31) and its imaginary parts (32 .. 63): whole runs of the layout, half the
    // write requests.
    const int out = lane_number(), comp = out >> 5, nl = wn * 32 + (out & 31), ml = wm * 32;
    const bool n_ok = n0 + nl < N;
    if constexpr (MODE != kFast) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int m = m0 + ml + 8 * (v / 4) + (v % 4);
            float q0 = unscale * acc_r[v], q1 = unscale * acc_i[v];
            swap_halves(q0, q1);
            const unsigned plane = (unsigned)m * (unsigned)prm.c_rs + (n0 + nl);
            if (n_ok && m < M) prm.C[element(prm.layC, plane, bin, comp)] = q0;
            if (n_ok && m + 4 < M) prm.C[element(prm.layC, plane + 4 * (unsigned)prm.c_rs, bin, comp)] = q1;
        }
    } else {
        const size_t row = (size_t)prm.c_rs * prm.layC.bins * 2;          // floats per step of m
        char *cb = reinterpret_cast<char *>(prm.C + (size_t)bin * (2u << prm.layC.tsh) + prm.layC.part(n0) + (size_t)m0 * row);
        const unsigned lo = (unsigned)((prm.layC.part(nl) + ((size_t)comp << prm.layC.tsh)) * sizeof(float));
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int mv = ml + 8 * (v / 4) + (v % 4);
            float q0 = unscale * acc_r[v], q1 = unscale * acc_i[v];
            swap_halves(q0, q1);                                          // rows mv and mv + 4
            if (n_ok && m0 + mv < M) *reinterpret_cast<float *>(cb + (size_t)mv * row * sizeof(float) + lo) = q0;
            if (n_ok && m0 + mv + 4 < M) *reinterpret_cast<float *>(cb + (size_t)(mv + 4) * row * sizeof(float) + lo) = q1;
        }
    }
    return true;
}

// The attempts, of which all but the rarest data take one: not the layout's padding bins, which hold what
// the memory held.  The empty asm keeps the compiler from
// holding what the attempts have in common in registers through the K loop.
template <bool AKF, bool BKF, int MODE>
__device__ __forceinline__ void cgemm_split_body(const GemmParams &prm, const unsigned wg, char *smem) {
    const unsigned bins_per_xcd = prm.bins / kXcds, tiles = prm.tiles_m * prm.tiles_n;
    if (wg % kXcds * bins_per_xcd + wg / kXcds / tiles >= (unsigned)prm.live) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll 1
    for (int i = 0; i < kScalings; ++i) {
        unsigned w = wg;
        asm volatile("" : "+s"(w));
        if (cgemm_split_attempt<AKF, BKF, MODE>(prm, w, wave, scale_a(i), scale_b(i), i == kScalings - 1, smem)) return;
    }
}

constexpr int kSplitLds = SplitLoader<true, kFast>::BYTES + SplitLoader<false, kFast>::BYTES + 4 * (int)sizeof(int);

template <bool AKF, bool BKF, int MODE>
__global__ void __launch_bounds__(256, MODE == kFast ? 4 : 3) cgemm_split_kernel(GemmParams prm) {
    __shared__ __align__(16) char smem[kSplitLds];
    cgemm_split_body<AKF, BKF, MODE>(prm, blockIdx.x, smem);
}

// Both contractions of the backward pass in one launch (see cgemm_pair_kernel in
// cgemm_kernels.hip): workgroups [0, n1) work on p1, the rest on p2.
struct SplitPairParams {
    GemmParams p1, p2;
    unsigned n1;
};
template <bool AKF1, bool AKF2, int MODE>
__global__ void __launch_bounds__(256, MODE == kFast ? 4 : 3) cgemm_split_pair_kernel(SplitPairParams pp) {
    __shared__ __align__(16) char smem[kSplitLds];
    if (blockIdx.x < pp.n1) cgemm_split_body<AKF1, false, MODE>(pp.p1, blockIdx.x, smem);
    else cgemm_split_body<AKF2, false, MODE>(pp.p2, blockIdx.x - pp.n1, smem);
}

static long tile_grid(GemmParams &p) {
    p.tiles_m = (p.M + ROWS - 1) / ROWS;
    p.tiles_n = (p.N + ROWS - 1) / ROWS;
    return (long)p.bins * p.tiles_m * p.tiles_n;
}

hipError_t launch_cgemm_split(GemmParams p, bool akf, bool bkf, bool vec, LaunchCtx st) {
    const long grid = tile_grid(p);
    // (4-byte gathers: along the rows of both operands only, see split_pays())
    if (grid > 0x7fffffffL || (!akf && bkf) || (akf && !p.fast && !vec)) return hipErrorInvalidValue;
    auto k = !akf ? (p.fast ? cgemm_split_kernel<false, false, kFast> : cgemm_split_kernel<false, false, kGeneral>)
             : bkf ? (p.fast ? cgemm_split_kernel<true, true, kFast> : cgemm_split_kernel<true, true, kGeneral>)
                   : (p.fast ? cgemm_split_kernel<true, false, kFast> : cgemm_split_kernel<true, false, kGeneral>);
    launch_kernel(k, dim3((unsigned)grid), dim3(256), 0, st, p);
    return hipGetLastError();
}

// Both with 16-byte gathers (shared_launch()).
hipError_t launch_cgemm_split_pair(const GemmParams &p1, bool akf1, const GemmParams &p2, LaunchCtx st) {
    SplitPairParams pp{p1, p2, 0};
    const long n1 = tile_grid(pp.p1), n2 = tile_grid(pp.p2);
    if (n1 + n2 > 0x7fffffffL) return hipErrorInvalidValue;
    pp.n1 = (unsigned)n1;     // a multiple of the XCD count, as bins is
    auto k = p1.fast && p2.fast ? (akf1 ? cgemm_split_pair_kernel<true, false, kFast> : cgemm_split_pair_kernel<false, true, kFast>)
                                : (akf1 ? cgemm_split_pair_kernel<true, false, kGeneral> : cgemm_split_pair_kernel<false, true, kGeneral>);
    launch_kernel(k, dim3((unsigned)(n1 + n2)), dim3(256), 0, st, pp);
    return hipGetLastError();
}

}  // namespace fc
