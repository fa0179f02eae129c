// Per-bin complex contraction for matrices with a narrow side or few tiles: tiles of 32 or 16 rows whose reduction is
// split over the waves of a workgroup, operands straight from memory into the matrix cores' registers.
//
// Same operation as cgemm_kernels.hip (the Cgemm row of Table 1 of the fbfft paper).  A 64x64 tile on a 16 x 6
// matrix is nine tenths padding, and one tile a bin leaves a workgroup a compute unit or less, each walking alone over
// the whole reduction one K tile's latency at a time.  Here a workgroup of up to eight waves holds the 32x32
// tile of `group` neighbouring bins (those that share 128-byte lines) and wave w works on bin w % group and on
// every (waves / group)-th chunk of eight reduction steps; the partial tiles meet in LDS once, at the end.  A value
// loaded serves one tile only, so nothing is gained by a detour over LDS, and without one no wave waits for another.
#include "gemm_params.hpp"

namespace fc {

constexpr int kChunk = 8;       // reduction steps of a chunk: four of the matrix instruction, two halves of a wave
constexpr int kChunk16 = 16;    // the same with 16-row tiles: four of the matrix instruction, four quarters of a wave

typedef float floatx4 __attribute__((ext_vector_type(4)));

// How an operand's planes are addressed.  x: plane number from the start of the uniform base's plane tile.
struct Planes {
    unsigned tile_floats;       // floats of a plane tile, all bins
    int tsh;
    __device__ __forceinline__ unsigned offset(unsigned x) const { return (x >> tsh) * tile_floats + (x & ((1u << tsh) - 1)); }
};

// One operand's chunk: lane (row = lane % ROWS, h = lane / ROWS) holds k0 + 4 h + 0 .. 3 of its row.  The matrix
// instruction's step i then multiplies k0 + 4 h + i for every h; which of them are a step's does not matter as long
// as both operands agree.  KF: the reduction index is the contiguous plane index, else the row is.
// Along the reduction a lane gathers 16 bytes, MODE 0 at any alignment; across it 4 bytes a step.  MODE 2: a lane's
// part of the address never changes.
template <bool KF, int MODE, int ROWS = 32>
struct Strip {
    const float *base;          // bin's real parts, plane tile 0
    Planes pl;
    long rs, cs;                // plane strides of row and reduction index
    unsigned im;                // floats from real to imaginary part
    int r0, row, h;
    unsigned lane;              // MODE 2: the lane's part of the offset

    __device__ __forceinline__ void init(const float *ptr, const FreqLayout &lay, int bin, long row_stride, long k_stride, int first,
                                         int rows, int lane_id) {
        base = ptr + lay.index(0, bin, 0);
        pl.tsh = lay.tsh; pl.tile_floats = (unsigned)lay.bins * 2u << lay.tsh;
        rs = row_stride; cs = k_stride;
        im = 1u << lay.tsh;
        r0 = first;
        row = lane_id % ROWS; h = lane_id / ROWS;
        if (r0 + row >= rows) row = rows - 1 - r0;         // (its results are not stored)
        if constexpr (MODE == 2) {
            if constexpr (KF) lane = pl.offset((unsigned)row * (unsigned)rs) + pl.offset(4u * h);
            else lane = pl.offset((unsigned)((r0 & ((1 << pl.tsh) - 1)) + row)) + pl.offset((unsigned)(4 * h) * (unsigned)cs);
        }
    }
    // Uniform base of the plane tile of plane p0, and p0's place in it.
    __device__ __forceinline__ const float *tile_of(long p0) const { return base + (size_t)(p0 >> pl.tsh) * pl.tile_floats; }
    __device__ __forceinline__ unsigned within(long p0) const { return (unsigned)p0 & ((1u << pl.tsh) - 1); }

    __device__ __forceinline__ void load(float (&re)[4], float (&imag)[4], int k0, int K) const {
        const int k = k0 + 4 * h;
#pragma unroll
        for (int i = 0; i < 4; ++i) re[i] = imag[i] = 0.f;
        if constexpr (KF && MODE == 0) {
            // Four planes of a run, or the last of one and the first of the next, at any alignment: the 16 bytes that end
            // with the run hold the former (a 4-byte aligned access is allowed), the next run's first 16 the latter.
            typedef float unaligned4 __attribute__((ext_vector_type(4), aligned(4)));
            const long p0 = (long)r0 * rs;
            const unsigned T = 1u << pl.tsh, x = within(p0) + (unsigned)row * (unsigned)rs + k, at = x & (T - 1);
            const float *u = tile_of(p0);
            const unsigned over = at + 4 > T ? at + 4 - T : 0;           // planes that lie in the next run
            if (k < K) {
                const float *p = u + pl.offset(x - over);
                const unaligned4 a = *reinterpret_cast<const unaligned4 *>(p), b = *reinterpret_cast<const unaligned4 *>(p + im);
                unaligned4 c = unaligned4(0.f), d = unaligned4(0.f);
                if (over && k + 4 - (int)over < K) {
                    p = u + pl.offset(x + 4 - over);
                    c = *reinterpret_cast<const unaligned4 *>(p);
                    d = *reinterpret_cast<const unaligned4 *>(p + im);
                }
                // (a, c) shifted down by `over`
                const bool one = over & 1, two = over & 2;
                float s[6], t[6];
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    s[i] = one ? (i < 3 ? a[i + 1] : c[i - 3]) : (i < 4 ? a[i] : c[i - 4]);
                    t[i] = one ? (i < 3 ? b[i + 1] : d[i - 3]) : (i < 4 ? b[i] : d[i - 4]);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    re[i] = k + i < K ? (two ? s[i + 2] : s[i]) : 0.f;
                    imag[i] = k + i < K ? (two ? t[i + 2] : t[i]) : 0.f;
                }
            }
        } else if constexpr (KF) {
            const float *p;
            if constexpr (MODE == 2) p = tile_of((long)r0 * rs + k0) + within(k0) + lane;   // (r0 rs in whole tiles; k0 + 4 h + 3 in one run)
            else p = tile_of((long)r0 * rs) + pl.offset(within((long)r0 * rs) + (unsigned)row * (unsigned)rs + k);
            if (k < K) {
                const float4 a = *reinterpret_cast<const float4 *>(p), b = *reinterpret_cast<const float4 *>(p + im);
                re[0] = a.x; re[1] = a.y; re[2] = a.z; re[3] = a.w;
                imag[0] = b.x; imag[1] = b.y; imag[2] = b.z; imag[3] = b.w;
            }
        } else {
            const long p0 = r0 + (long)k0 * cs;
            const float *u = MODE == 2 ? tile_of((long)k0 * cs) + (size_t)(r0 >> pl.tsh) * pl.tile_floats : tile_of(p0);
            const unsigned first = within(p0) + row + (unsigned)(4 * h) * (unsigned)cs;
            const size_t fstep = MODE == 2 ? (size_t)(cs >> pl.tsh) * pl.tile_floats : 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float *p = MODE == 2 ? u + i * fstep + lane : u + pl.offset(first + (unsigned)i * (unsigned)cs);
                if (k + i < K) { re[i] = p[0]; imag[i] = p[im]; }
            }
        }
    }
};

// Workgroup number wg of prm's grid.
template <bool AKF, bool BKF, int MODE>
__device__ __forceinline__ void cgemm_direct_body(const GemmParams &prm, const int group, const unsigned wg) {
    extern __shared__ float red[];                  // [wave][component][register][lane]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int waves = blockDim.x >> 6, slices = waves / group, slice = wave / group;
    const int tiles = prm.tiles_m * prm.tiles_n, groups_per_xcd = prm.bins / group / kXcds;
    const int xcd = wg % kXcds, slot = wg / kXcds;
    const int bin = (xcd * groups_per_xcd + slot / tiles) * group + wave % group;
    const int tile = slot % tiles;
    const int m0 = (tile / prm.tiles_n) * 32, n0 = (tile % prm.tiles_n) * 32;

    // Gauss's three products, as in cgemm_bins_kernel
    floatx16 p1, p2, p3;
#pragma unroll
    for (int v = 0; v < 16; ++v) { p1[v] = 0.f; p2[v] = 0.f; p3[v] = 0.f; }
    // Slices with a chunk: the waves of a shared launch follow the longer reduction, and a slice without one neither stores
    // zeros nor has them added (a gradient alone, up to 8 terms on runs of 8 and more 0.96 of the time in the mean, 485 x 4 -> 5, 79x79 349 ->
    // 309 us; both gradients 0.99).
    const int chunks = (prm.K + kChunk - 1) / kChunk, used = chunks < slices ? chunks : slices;
    if (bin < prm.live && slice < used) {
        Strip<AKF, MODE> a;
        Strip<BKF, MODE> b;
        a.init(prm.A, prm.layA, bin, prm.a_rs, prm.a_cs, m0, prm.M, lane);
        b.init(prm.B, prm.layB, bin, prm.b_cs, prm.b_rs, n0, prm.N, lane);
        struct Chunk { float ar[4], ai[4], br[4], bi[4]; } now, next;
        const int K = prm.K, step = slices * kChunk;
        auto fetch = [&](Chunk &x, int k0) { a.load(x.ar, x.ai, k0, K); b.load(x.br, x.bi, k0, K); };
        int k0 = slice * kChunk;
        fetch(next, k0);                              // (past the end: zeros)
        while (k0 < K) {                              // the next chunk's loads are in flight while one is multiplied
            now = next;
            k0 += step;
            fetch(next, k0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float ai = flip(now.ai[i], prm.a_sign), bi = flip(now.bi[i], prm.b_sign);
                p1 = __builtin_amdgcn_mfma_f32_32x32x2f32(now.ar[i], now.br[i], p1, 0, 0, 0);
                p2 = __builtin_amdgcn_mfma_f32_32x32x2f32(ai, bi, p2, 0, 0, 0);
                p3 = __builtin_amdgcn_mfma_f32_32x32x2f32(now.ar[i] + ai, now.br[i] + bi, p3, 0, 0, 0);
            }
        }
    }
    if (slice < used) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            red[((wave * 2 + 0) * 16 + v) * 64 + lane] = p1[v] - p2[v];
            red[((wave * 2 + 1) * 16 + v) * 64 + lane] = p3[v] - p1[v] - p2[v];
        }
    }
    __syncthreads();
    // D layout of the 32x32x2 instruction: register v of lane l is row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32.  The
    // slices of a bin share its registers out.
    if (bin >= prm.live) return;
    const int n = n0 + (lane & 31), per = 16 / slices;
    const long pc = (long)m0 * prm.c_rs + n0;
    Planes pl{(unsigned)prm.layC.bins * 2u << prm.layC.tsh, prm.layC.tsh};
    float *cb = prm.C + prm.layC.index(0, bin, 0) + (size_t)(pc >> pl.tsh) * pl.tile_floats;
    const unsigned within = (unsigned)pc & ((1u << pl.tsh) - 1);
    for (int v = slice * per; v < (slice + 1) * per; ++v) {
        float cr = 0.f, ci = 0.f;
        for (int s = 0; s < used; ++s) {
            const float *r = red + (((s * group + wave % group) * 2) * 16 + v) * 64 + lane;
            cr += r[0];
            ci += r[16 * 64];
        }
        const int mm = 8 * (v / 4) + 4 * (lane >> 5) + v % 4;
        if (m0 + mm < prm.M && n < prm.N) {
            float *q = cb + pl.offset(within + (unsigned)mm * (unsigned)prm.c_rs + (lane & 31));
            q[0] = cr;
            q[1u << pl.tsh] = ci;
        }
    }
}

// A side of at most 16 (a few images served through a wide layer): 16x16x4 instructions, GA x GB of them a step, one
// of the two 1 and the other 2.  Half of a 32-row tile's products and registers would be padding, and its waves wait for
// memory: a chunk of 16 steps reads 64 bytes of a row at once (a whole run of 16 planes), keeps twice as many bytes in flight and
// halves the chain of chunks; half the partial tiles let more workgroups in.  us a pass on weights ahead, 32-row tiles / these:
// 8 x 256 -> 256, 27x27 87 / 61 (fprop and bprop; the contraction alone 236 MB, 76 / 50), 2 x 64 -> 256, 32x32 40 / 30, 7 x 130 -> 301,
// 27x27 bprop 90 / 60, 11 x 64 -> 256, 10x10 15.4 / 13.6; accGrad of 128 x 16 -> 304, 32x32 141 / 121.  Over 105 passes of random
// layers nothing was slower.
template <bool AKF, bool BKF, int MODE, int GA, int GB>
__device__ __forceinline__ void cgemm_direct16_body(const GemmParams &prm, const int group, const unsigned wg) {
    constexpr int P = GA * GB;
    extern __shared__ float red[];                  // [wave][component][product][register][lane]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int waves = blockDim.x >> 6, slices = waves / group, slice = wave / group;
    const int tiles = prm.tiles_m * prm.tiles_n, groups_per_xcd = prm.bins / group / kXcds;
    const int xcd = wg % kXcds, slot = wg / kXcds;
    const int bin = (xcd * groups_per_xcd + slot / tiles) * group + wave % group;
    const int tile = slot % tiles;
    const int m0 = (tile / prm.tiles_n) * 32, n0 = (tile % prm.tiles_n) * 32;

    // Gauss's three products, as in cgemm_bins_kernel
    floatx4 p1[P], p2[P], p3[P];
#pragma unroll
    for (int j = 0; j < P; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) { p1[j][v] = 0.f; p2[j][v] = 0.f; p3[j][v] = 0.f; }
    if (bin < prm.live) {
        Strip<AKF, MODE, 16> a[GA];
        Strip<BKF, MODE, 16> b[GB];
        // (a second strip past the end repeats the first; its results are not stored)
#pragma unroll
        for (int j = 0; j < GA; ++j)
            a[j].init(prm.A, prm.layA, bin, prm.a_rs, prm.a_cs, m0 + 16 * j < prm.M ? m0 + 16 * j : m0, prm.M, lane);
#pragma unroll
        for (int j = 0; j < GB; ++j)
            b[j].init(prm.B, prm.layB, bin, prm.b_cs, prm.b_rs, n0 + 16 * j < prm.N ? n0 + 16 * j : n0, prm.N, lane);
        struct Chunk { float ar[GA][4], ai[GA][4], br[GB][4], bi[GB][4]; } now, next;
        const int K = prm.K, step = slices * kChunk16;
        auto fetch = [&](Chunk &x, int k0) {
#pragma unroll
            for (int j = 0; j < GA; ++j) a[j].load(x.ar[j], x.ai[j], k0, K);
#pragma unroll
            for (int j = 0; j < GB; ++j) b[j].load(x.br[j], x.bi[j], k0, K);
        };
        int k0 = slice * kChunk16;
        fetch(next, k0);                              // (past the end: zeros)
        while (k0 < K) {                              // the next chunk's loads are in flight while one is multiplied
            now = next;
            k0 += step;
            fetch(next, k0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < P; ++j) {
                    const float ar = now.ar[j / GB][i], ai = flip(now.ai[j / GB][i], prm.a_sign);
                    const float br = now.br[j % GB][i], bi = flip(now.bi[j % GB][i], prm.b_sign);
                    p1[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(ar, br, p1[j], 0, 0, 0);
                    p2[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(ai, bi, p2[j], 0, 0, 0);
                    p3[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(ar + ai, br + bi, p3[j], 0, 0, 0);
                }
        }
    }
#pragma unroll
    for (int j = 0; j < P; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            red[(((wave * 2 + 0) * P + j) * 4 + v) * 64 + lane] = p1[j][v] - p2[j][v];
            red[(((wave * 2 + 1) * P + j) * 4 + v) * 64 + lane] = p3[j][v] - p1[j][v] - p2[j][v];
        }
    __syncthreads();
    // D layout of the 16x16x4 instruction: register v of lane l is row 4 (l / 16) + v, column l % 16.  The slices of a
    // bin share its registers out.
    if (bin >= prm.live) return;
    const long pc = (long)m0 * prm.c_rs + n0;
    Planes pl{(unsigned)prm.layC.bins * 2u << prm.layC.tsh, prm.layC.tsh};
    float *cb = prm.C + prm.layC.index(0, bin, 0) + (size_t)(pc >> pl.tsh) * pl.tile_floats;
    const unsigned within = (unsigned)pc & ((1u << pl.tsh) - 1);
    const int per = P * 4 / slices;                 // (slices: at most eight, a power of two)
    for (int r = slice * per; r < (slice + 1) * per; ++r) {
        float cr = 0.f, ci = 0.f;
        for (int s = 0; s < slices; ++s) {
            const float *q = red + (((s * group + wave % group) * 2) * P * 4 + r) * 64 + lane;
            cr += q[0];
            ci += q[P * 4 * 64];
        }
        const int j = r / 4, mm = 16 * (j / GB) + 4 * (lane >> 4) + r % 4, nn = 16 * (j % GB) + (lane & 15);
        if (m0 + mm < prm.M && n0 + nn < prm.N) {
            float *q = cb + pl.offset(within + (unsigned)mm * (unsigned)prm.c_rs + nn);
            q[0] = cr;
            q[1u << pl.tsh] = ci;
        }
    }
}

template <bool AKF, bool BKF, int MODE, int GA, int GB>
__global__ void __launch_bounds__(512, 4) cgemm_direct16_kernel(GemmParams prm, int group) {
    cgemm_direct16_body<AKF, BKF, MODE, GA, GB>(prm, group, blockIdx.x);
}

template <bool AKF, bool BKF, int MODE>
__global__ void __launch_bounds__(512, 4) cgemm_direct_kernel(GemmParams prm, int group) {
    cgemm_direct_body<AKF, BKF, MODE>(prm, group, blockIdx.x);
}

// bprop and accGrad of a layer in one launch: one ramp-up and one tail, and a shared inverse transform behind them.
struct DirectPair {
    GemmParams b, a;
    unsigned first;            // workgroups of the one that goes first: bprop's, or accGrad's if a_first
    int group, a_first;
};
template <int MODE>
__global__ void __launch_bounds__(512, 4) cgemm_direct_pair_kernel(DirectPair dp) {
    const bool second = blockIdx.x >= dp.first;
    const unsigned wg = second ? blockIdx.x - dp.first : blockIdx.x;
    if (second == (dp.a_first != 0)) cgemm_direct_body<true, false, MODE>(dp.b, dp.group, wg);
    else cgemm_direct_body<false, false, MODE == 0 ? 1 : MODE>(dp.a, dp.group, wg);
}

// MODE of an operand pair.  16-byte gathers: whole quads along the reduction.  Fast addressing: whole plane tiles
// between rows or reduction steps, of 8 planes and more (a chunk's halves lie in one run).
static int direct_mode(const GemmParams &p, bool akf, bool bkf) {
    const long T = 1L << p.layA.tsh, sa = akf ? p.a_rs : p.a_cs, sb = bkf ? p.b_cs : p.b_rs;
    auto quads = [&](bool kf, long stride, const float *q) { return !kf || (p.K % 4 == 0 && stride % 4 == 0 && ((size_t)q & 15) == 0); };
    if (!quads(akf, sa, p.A) || !quads(bkf, sb, p.B)) return 0;
    return T >= 8 && sa % T == 0 && sb % T == 0 ? 2 : 1;
}

// Bins that share 128-byte lines.
static int direct_group(const GemmParams &p) {
    int group = p.layA.tsh >= 4 ? 1 : 16 >> p.layA.tsh;
    while (p.bins / kXcds % group) group >>= 1;
    return group;
}
static long direct_tiles(const GemmParams &p) { return (long)((p.M + 31) / 32) * ((p.N + 31) / 32); }
// Slices of the reduction, of at least one chunk each, until two waves a SIMD are there: over 630 products of random layers as fast as
// any other number (1024 .. 2560 waves within 2 %), where 8192 with up to 16 waves a workgroup, whose partial tiles leave one workgroup a
// compute unit, cost 8 % on runs of 16 planes.  Up to eight waves (64 KB of partial tiles, two workgroups a compute unit).
static int direct_waves(int K, int group, long bin_tiles, int chunk = kChunk) {
    int slices = 1;
    while (slices * group < 8 && slices * chunk < K && (slices * group < 4 || bin_tiles * slices < 2048)) slices *= 2;
    return slices * group;
}

template <class P, class... Q>
static hipError_t launch_direct(void (*k)(P, Q...), long grid, int waves, int regs, LaunchCtx st, const P &prm, Q... q) {
    if (grid > 0x7fffffffL) return hipErrorInvalidValue;
    const size_t lds = (size_t)waves * 2 * regs * 64 * sizeof(float);
    if (hipError_t e = allow_big_lds((const void *)k, lds); e != hipSuccess) return e;
    if (st.start || st.stop) hipExtLaunchKernelGGL(k, dim3((unsigned)grid), dim3(64 * waves), (unsigned)lds, st.stream, st.start, st.stop, 0, prm, q...);
    else hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(64 * waves), lds, st.stream, prm, q...);
    return hipGetLastError();
}

template <bool AKF, bool BKF>
static hipError_t dispatch_direct(const GemmParams &prm, int group, int waves, LaunchCtx st) {
    const long grid = (long)(prm.bins / group) * prm.tiles_m * prm.tiles_n;
    const int mode = direct_mode(prm, AKF, BKF);
    if (mode == 2) return launch_direct(cgemm_direct_kernel<AKF, BKF, 2>, grid, waves, 16, st, prm, group);
    if constexpr (AKF || BKF) {
        if (mode == 0) return launch_direct(cgemm_direct_kernel<AKF, BKF, 0>, grid, waves, 16, st, prm, group);
    }
    return launch_direct(cgemm_direct_kernel<AKF, BKF, 1>, grid, waves, 16, st, prm, group);
}

// (direct_fits() bounds eight reduction steps to 2^32 bytes; offsets count floats, so sixteen fit, too)
static bool direct_16(const GemmParams &p) { return p.M <= 16 || p.N <= 16; }

template <bool AKF, bool BKF, int GA, int GB>
static hipError_t dispatch_direct16(const GemmParams &prm, int group, LaunchCtx st) {
    const long grid = (long)(prm.bins / group) * prm.tiles_m * prm.tiles_n;
    const int mode = direct_mode(prm, AKF, BKF), waves = direct_waves(prm.K, group, prm.bins * direct_tiles(prm), kChunk16);
    if (mode == 2) return launch_direct(cgemm_direct16_kernel<AKF, BKF, 2, GA, GB>, grid, waves, 8, st, prm, group);
    if constexpr (AKF || BKF) {
        if (mode == 0) return launch_direct(cgemm_direct16_kernel<AKF, BKF, 0, GA, GB>, grid, waves, 8, st, prm, group);
    }
    return launch_direct(cgemm_direct16_kernel<AKF, BKF, 1, GA, GB>, grid, waves, 8, st, prm, group);
}
template <bool AKF, bool BKF>
static hipError_t dispatch_direct16(const GemmParams &prm, int group, LaunchCtx st) {
    return prm.M <= 16 ? dispatch_direct16<AKF, BKF, 1, 2>(prm, group, st) : dispatch_direct16<AKF, BKF, 2, 1>(prm, group, st);
}

// Waves of the shared launch of two products.
static int direct_pair_waves(const GemmParams &p, const GemmParams &q, int group) {
    return direct_waves(p.K > q.K ? p.K : q.K, group, p.bins * (direct_tiles(p) + direct_tiles(q)));
}

hipError_t launch_cgemm_direct(GemmParams prm, bool akf, bool bkf, LaunchCtx st, const GemmParams *partner) {
    prm.tiles_m = (prm.M + 31) / 32;
    prm.tiles_n = (prm.N + 31) / 32;
    const int group = direct_group(prm);
    if (!partner && direct_16(prm)) {
        if (akf && bkf) return dispatch_direct16<true, true>(prm, group, st);
        if (akf && !bkf) return dispatch_direct16<true, false>(prm, group, st);
        if (!akf && !bkf) return dispatch_direct16<false, false>(prm, group, st);
        return dispatch_direct16<false, true>(prm, group, st);
    }
    const int waves = partner ? direct_pair_waves(prm, *partner, group) : direct_waves(prm.K, group, prm.bins * direct_tiles(prm));
    if (akf && bkf) return dispatch_direct<true, true>(prm, group, waves, st);
    if (akf && !bkf) return dispatch_direct<true, false>(prm, group, waves, st);
    if (!akf && !bkf) return dispatch_direct<false, false>(prm, group, waves, st);
    return dispatch_direct<false, true>(prm, group, waves, st);
}

hipError_t launch_cgemm_direct_pair(const GemmParams &bprop, const GemmParams &accgrad, LaunchCtx st) {
    DirectPair dp{bprop, accgrad, 0, direct_group(bprop), accgrad.K >= bprop.K};
    for (GemmParams *p : {&dp.b, &dp.a}) { p->tiles_m = (p->M + 31) / 32; p->tiles_n = (p->N + 31) / 32; }
    const long tb = direct_tiles(bprop), ta = direct_tiles(accgrad), groups = bprop.bins / dp.group;
    const int waves = direct_pair_waves(bprop, accgrad, dp.group);
    const long first = groups * (dp.a_first ? ta : tb), grid = groups * (ta + tb);
    if (grid > 0x7fffffffL) return hipErrorInvalidValue;
    dp.first = (unsigned)first;
    const int mb = direct_mode(bprop, true, false), ma = direct_mode(accgrad, false, false);
    if (mb == 2 && ma == 2) return launch_direct(cgemm_direct_pair_kernel<2>, grid, waves, 16, st, dp);
    if (mb == 0) return launch_direct(cgemm_direct_pair_kernel<0>, grid, waves, 16, st, dp);
    return launch_direct(cgemm_direct_pair_kernel<1>, grid, waves, 16, st, dp);
}

}  // namespace fc
