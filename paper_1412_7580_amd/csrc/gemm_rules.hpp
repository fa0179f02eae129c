// Which kernel runs a contraction: the rules, by sizes, layout and alignment, on the host alone (no
// launch, no device call), so that a CPU program can ask them.
#pragma once
#include "gemm_params.hpp"

#include <initializer_list>

namespace fc {

// Fast addressing of an operand (see TileLoader::prepare_fast): one index of the matrix is the
// contiguous plane index, the other moves `stride` planes per step.  When that stride is a
// whole number of plane tiles, a step of the strided index adds a constant to the element index,
// whatever the contiguous index is, so addresses split into a uniform part and a per-lane
// part.  The per-lane part must fit an unsigned 32-bit byte offset: 64 steps of the strided index.
inline bool fast_addressing(const FreqLayout &lay, long stride, int bins) {
    const long T = 1L << lay.tsh;
    if (stride <= 0 || stride % T != 0) return false;
    return (double)stride * bins * 2 * 4 * 65 < 2147483648.0;
}

// A side of at most 32 against one of at least 128 (a few images served through a wide layer, a
// layer of few channels): 32x128 or 128x32 tiles, as half of every 64x64 tile and of its products
// would be padding: 8 images, 256 -> 256 channels, 27x27, weights ahead 120 -> 100 us a pass (118 -> 91 on
// the same inputs again and again), bprop 155 -> 123; 128 images, 32 -> 32 channels bprop 40 -> 36.
// Not where that leaves compute units without a workgroup (112 workgroups: 33 -> 35), nor with gathers
// of 4 bytes or runs of four planes, where the gathers are the bound, nor for less than two whole K
// tiles (16 images 160x160, 16 -> 48 channels: 129 -> 131).  Under fast addressing the longer tile's
// per-lane offsets must fit, too.  What the split reduction takes (direct_pays: the first of these layers is at 75 us with it)
// does not come here, but for a lone gradient that sums in the order of a shared launch of 64x64 tiles (lone_gradient()).
inline bool narrow_tile(const GemmParams &prm, bool vec) {
    if (!vec || prm.layA.tsh < 3 || prm.K < 32) return false;
    if (!((prm.M <= 32 && prm.N >= 128) || (prm.N <= 32 && prm.M >= 128))) return false;
    const int longer = prm.M > prm.N ? prm.M : prm.N;
    if ((long)prm.bins * ((longer + 127) / 128) < 256) return false;
    if (!prm.fast) return true;
    long stride = prm.a_rs > prm.a_cs ? prm.a_rs : prm.a_cs;
    for (long s : {prm.b_rs, prm.b_cs, prm.c_rs}) stride = s > stride ? s : stride;
    return (double)stride * prm.bins * 2 * 4 * 129 < 2147483648.0;
}

// A bin's M N K products against its M K + K N + M N elements, by the layout's runs.  With runs of 32
// or 64 planes (bases up to 16) gathers are whole lines and the products bound a layer early (fp32
// form -> this, training step, us): 15 products an element (16 samples, 512 -> 512 channels, 8x8) 168 ->
// 147, 16 (32 x 64 -> 64, 13x13) 46 -> 42, 43 (128 x 128 -> 128) 95 -> 86, 55 163 -> 144.  With runs of 8 or
// 16 the gathers do, and the bf16 form's power costs the transforms behind it clock: 26 (128 x 64 ->
// 64, 27x27) 120 -> 114 on one card and 124 on another, 32 (56x56, padded) 305 -> 310; 43 (64 x 256 ->
// 256, 28x28 / 32x32) 545 -> 504 / 717 -> 679, 45 (128 x 96 -> 256, 27x27) 456 -> 407.  Runs of four and
// single planes are the gathers' alone (64 x 63 -> 129, 45x45: 491 -> 513).
// 4-byte gathers: where they run along the rows of both operands (accGrad) this loader is as good as the
// fp32 kernel's and the products count (128 x 255 -> 255, 13x13 / 27x27: 103 -> 95, 430 -> 397; 130 x 123 ->
// 127: 45 -> 41); along the reduction its four values a lane take four times the lines (fprop of the
// same layers 111 -> 133, 412 -> 504, 53 -> 56, bprop 109 -> 113, 407 -> 429, 52 -> 52).
// General addressing (16-byte gathers whose strides are no multiple of a run) follows the same rule: 128 x 100 ->
// 100, 13x13 fprop 40.2 -> 35.9, bprop 41.0 -> 37.9, 128 x 196 -> 204, 27x27 277 -> 244, 277 -> 259 and accGrad 323 -> 313.
inline long tiles_64(const GemmParams &p) { return (long)p.bins * ((p.M + 63) / 64) * ((p.N + 63) / 64); }
inline double products_per_element(const GemmParams &p) {
    const double m = p.M, n = p.N, k = p.K;
    return m * n * k / (m * k + k * n + m * n);
}
// General addressing of accGrad leaves three workgroups a compute unit, not four: by itself it does not take grids
// that the fp32 kernel holds in one round and this one would not (128 x 196 -> 204, 10x10 52 / 56).
inline bool split_alone_pays(const GemmParams &p, bool akf, bool vec) {
    return akf || p.fast || !vec || tiles_64(p) <= 3 * 256 || tiles_64(p) > 4 * 256;
}
inline bool split_pays(const GemmParams &p, bool akf, bool bkf, bool vec) {
    const int tsh = p.layA.tsh;
    if (tsh < 3 || (!vec && (akf || bkf || p.a_rs != 1 || p.b_cs != 1))) return false;
    return products_per_element(p) >= (tsh >= 5 && vec ? 12 : 40);
}

// The three forms, with A, B and C as the passes lay them out: rows of W planes side by side, the
// wide index in whole quads.
inline Thin thin_form(const GemmParams &p) {
    const bool akf = p.a_rs != 1, bkf = p.b_cs != 1;      // reduction index contiguous (row index, if both are)
    auto whole = [](const FreqLayout &l, const float *ptr) { return l.tsh >= 2 && ((size_t)ptr & 15) == 0; };
    if (!whole(p.layA, p.A) || !whole(p.layB, p.B) || !whole(p.layC, p.C) || p.layA.tsh != p.layC.tsh ||
        p.c_cs != 1) return Thin::none;
    if (akf || p.K == 1) {
        if (p.K <= 4 && p.a_rs == p.K && p.N % 4 == 0 && p.c_rs % 4 == 0 &&
            (p.K == 1 || bkf ? p.b_cs == p.K || (p.K == 1 && p.b_cs == 1) : p.b_rs % 4 == 0 && p.b_cs == 1))
            return Thin::k;
    }
    // (n only where runs are four planes: with longer ones a lane's 16 bytes are a part of each line and
    // the matrix-core kernel is ahead, e.g. 128 samples, 64 -> 3 channels, 28x28 57 us a pass against 49;
    // with runs of four 64x64 images 251 -> 181 us)
    if (akf && !bkf && p.layA.tsh == 2 && p.N <= 4 && p.K % 4 == 0 && p.a_rs % 4 == 0 && p.b_rs == p.N && p.b_cs == 1) return Thin::n;
    if (!akf && !bkf && p.N <= 4 && p.M % 4 == 0 && p.a_cs % 4 == 0 && p.b_rs == p.N && p.b_cs == 1) return Thin::acc;
    return Thin::none;
}

// Whether a thin product is the faster one, where another kernel takes the same matrices.  fourbin: the
// four-bins-per-line kernel would (16-byte gathers, runs of four planes); else it is 64x64 tiles.
//   n: a workgroup walks over K for 64 bins and 16 rows, so few rows leave the chip idle: 16 samples, 4 -> 256
//      channels, 40x40 51 us a pass in the four-bin kernel and 107 here, 128 x 4 -> 64, 56x56 101 and 92.  Against 64x64
//      tiles with 4-byte gathers only long reductions in a single round of workgroups lose: 64 x 3 ->
//      384, 40x40 191 and 204, 128 x 3 -> 384 328 and 267.
//   k: four wide rows of B are as much to read as to write (64 x 4 -> 256, 56x56 82.6 / 88.4 at 32 samples,
//      fewer rows or columns win: 16 samples, 64x64 91 / 82, 128 x 4 -> 64 equal).  Four columns on runs of 32
//      or 64 planes leave most of each line unused (128 x 4 -> 4, 8x8 13.9 / 14.5, 13x13 16.0 / 16.6; 512 samples
//      16.7 / 15.3, 20.2 / 17.5).
//      One sample's gradient, K = 1: equal or ahead, but for results somewhat larger than the 256 MB
//      last-level cache (256 -> 256, 40x40, 453 MB 216 / 233; 28 MB 39 / 37, 855 MB 428 / 401).
//   acc: behind only for wide layers of the largest such basis (256 x 4 -> 256, 64x64 829 / 860).
inline bool thin_pays(const GemmParams &p, Thin form, bool bkf, bool vec, bool fourbin) {
    const double result = (double)p.bins * p.M * p.N;
    if (form == Thin::n) {
        const long workgroups = (p.bins + 63) / 64 * (((p.M + 3) / 4 + 3) / 4);
        if (fourbin) return workgroups >= 128 && p.K <= 64;
        return p.K <= 256 || (long)p.bins * ((p.M + 63) / 64) > 1024;
    }
    if (!fourbin) return form != Thin::k || !vec || p.layC.tsh < 5 || p.N > 4 || p.M >= 256;
    if (form == Thin::k && p.K == 1) return result < 3.4e7 || result > 8e7;
    if (form == Thin::k) return p.K < 4 || !bkf || p.M < 32 || p.N < 128 || result < 7e6;
    return p.bins <= 2048 || p.M < 256 || p.K < 128;
}

// Quads of rows that a lane of the k form walks over with its columns of B: the fewest, up to 8, that
// leave 8192 waves or fewer (one a lane beyond that reads B anew for every quad it writes: 64 x 4 -> 384
// channels, 28x28, 10752 waves 76.7 us a pass, with two 70.0; 128 x 4 -> 64, 56x56 86.5 -> 80.6).
inline int thin_k_rows(const GemmParams &p) {
    const int per_run = 1 << (p.layC.tsh - 2);                             // quads of a run
    const long groups = (p.N / 4 + per_run - 1) / per_run, bin_blocks = (p.bins * per_run + 255) / 256;
    const long rows = ((p.M + 3) / 4 * groups * bin_blocks * 4 + 8191) / 8192;
    return rows < 1 ? 1 : rows > 8 ? 8 : (int)rows;
}

// Whether the four-bins-per-line kernel's form for any channel counts (cgemm_bingroup.hip) can run: runs of four
// planes, and 32-bit offsets that reach 32 rows or 16 reduction steps.
inline bool shifted_lines(const GemmParams &p, bool akf, bool bkf) {
    auto reach = [&](double planes) { return planes * p.bins * 2 * sizeof(float) < 4294967296.0; };
    auto whole = [](const FreqLayout &l, const float *ptr) { return l.tsh == 2 && ((size_t)ptr & 15) == 0; };
    return whole(p.layA, p.A) && whole(p.layB, p.B) && whole(p.layC, p.C) && p.bins % (4 * kXcds) == 0 && p.c_cs == 1 &&
           (akf || p.a_rs == 1) && (bkf || p.b_cs == 1) && reach(akf ? 32.0 * p.a_rs + 20 : 16.0 * p.a_cs + 36) &&
           reach(bkf ? 32.0 * p.b_cs + 20 : 16.0 * p.b_rs + 36);
}

// It is behind where its 32x32 tiles save no padding of 64x64 ones and there are few (40 x 51 x 16 on 1632 bins 21.6 / 27.8
// us, 256 x 46 x 12 53.8 / 61.8; 97 x 112 x 123 129 / 128, 176 x 229 x 26 403 / 330).
inline bool shifted_pays(const GemmParams &p) {
    return ((p.M + 31) / 32) * ((p.N + 31) / 32) < 4 * ((p.M + 63) / 64) * ((p.N + 63) / 64) || (p.M > 64 && p.N > 64);
}

// In a launch of its own, over 8000 products of random layers (whole passes, 64x64 tiles / this).  Its 32x32 tiles save padding while
// there are fewer than two to a 64x64 one (1.04 .. 1.57x), but few of them leave compute units without a workgroup where the others are one
// round, three a compute unit, and a reduction of one K tile then has nothing to make up for it (704 tiles 0.93 .. 1.0, 864 1.0 .. 1.1).  Two to
// one save little, and half as many workgroups fill their last round worse: behind in one round (fprop 0.92 .. 0.98; accGrad's longest
// 1.04 .. 1.14) and, up to one K tile, about two (1632 and 1728 tiles 0.93 .. 0.97; 1216 and 1408 1.0 .. 1.08, from 2048 1.0 .. 1.1, up to four terms
// from 2304).  Three and more to one, with a side of 33 .. 64, read the operands twice for little padding: up to two K tiles only where the
// others' results are single planes of every line (odd columns) and the tiles well filled (64 x 91 x 16 1.24, 60 x 65 x 8 1.27; 41 x 152 x 2,
// six tenths, 0.93, 58 x 80 x 5 0.95, 34 x 78 x 1 0.90); with both sides above 64 1.0 .. 1.37x, but for short reductions whose results
// are whole quads of planes (128 x 112 x 6 0.91, 167 x 128 x 17 0.87, 102 x 80 x 3 0.95).
inline bool shifted_alone_pays(const GemmParams &p, bool akf) {
    const long m = (p.M + 31) / 32, n = (p.N + 31) / 32, t32 = m * n, t64 = ((m + 1) / 2) * ((n + 1) / 2), tiles = p.bins * t64;
    const bool one_round = tiles <= 3 * 256;
    if (t32 < 2 * t64) return p.K > 16 || !one_round;
    if (t32 == 2 * t64) {
        if (one_round) return !akf && p.K > 64;
        return p.K > 16 || (tiles > 1024 && (tiles < 1536 || tiles >= (p.K <= 4 ? 2304 : 2048)));
    }
    if (t32 < 3 * t64) return true;
    if (m > 2 && n > 2) return p.N % 4 != 0 || p.K > (t32 == 4 * t64 ? 32 : 16);
    return p.K > 32 || (p.N % 2 == 1 && 8L * p.M * p.N >= 5 * 1024 * t32);
}

// Whether the kernel that splits the reduction over waves (cgemm_direct.hip) can run: runs of at least a quad, and
// 32-bit offsets that reach 32 rows and the reduction of an operand whose reduction index is contiguous, 64 rows and
// eight reduction steps of the others, 32 rows of the result.
inline bool direct_fits(const GemmParams &p, bool akf, bool bkf) {
    auto reach = [&](double planes) { return planes * p.bins * 2 * sizeof(float) < 4294967296.0; };
    const long T = 1L << p.layA.tsh;
    return p.layA.tsh >= 2 && p.layA.tsh == p.layB.tsh && p.layA.tsh == p.layC.tsh && p.c_cs == 1 && (akf || p.a_rs == 1) &&
           (bkf || p.b_cs == 1) && reach(akf ? 32.0 * p.a_rs + p.K + T : 64 + 8.0 * p.a_cs + T) &&
           reach(bkf ? 32.0 * p.b_cs + p.K + T : 64 + 8.0 * p.b_rs + T) && reach(32.0 * p.c_rs + 32 + T);
}

// Kernel parameters of one contraction and the kernel variant it can use.
struct Prepared {
    GemmParams prm;
    bool akf, bkf;     // the reduction index is the contiguous plane index of A / B
    bool vec;          // 16-byte gathers are possible
    bool bingroup;     // the four-bins-per-line kernel applies
    bool shifted;      // its form for any channel counts does ...
    bool shifted_alone; // ... and is the fastest in a launch of its own
    bool direct;       // the kernel that splits the reduction over waves can run ...
    bool direct_alone; // ... and is the fastest in a launch of its own
    bool split;        // bound by the fp32 matrix cores: the bf16 kernel applies (cgemm_split.hip) ...
    bool split_alone;  // ... and in a launch of its own, too
    Thin thin;         // a side of at most four: the vector-unit kernels apply (cgemm_thin.hip)
};

// 32x32 tiles with the reduction split over waves (cgemm_direct.hip) in a launch of its own, over 1100 products of random layers
// against 64x64 and narrow tiles, whose few workgroups each walk alone over a long reduction: 16 x 6 x 6832 on 544 bins 1486 -> ~130 us, 2 x 32 x
// 277 on 40 bins 28.9 -> 9.2, 16 x 16 x 192 on 112 bins 18.5 -> 7.6.  Not for two chunks of reduction or less (5 x 32 x
// 8: 4.0 / 9.5), nor with runs of four planes, where whole lines are worth more (5 x 248 x 176 on 864 bins 82 / 124), nor
// what the bf16 cores do.  A tile of 32 reads its operands for half as many products, so a side above 32 (64 on runs of 32
// and more, whose lines a strip uses whole) stays with 64x64 tiles (48 x 304 x 57 on 544 bins 50 / 68), and so does one of 33 .. 64 whose tiles
// of 64 are nearly full and give every compute unit one, with 32 steps and less or gathers that cross runs (whole passes 44 x 399 x 29 on 88 bins
// 25.6 / 29.8, 391 x 63 x 63 42.0 / 47.3, 50 x 256 x 182 50.1 / 55.2; but 35 x 198 x 228 1.15x, accGrad's 39 x 144 x 188 51 / 42), and so do, unless the
// tile of 64 would be half padding, grids of 32 tiles and more to a reduction step (9 x 256 x 32 on 312 bins 12.3 / 16.8), of 128
// where the other kernel's gathers are of 4 bytes or runs of eight planes (1134 x 8 x 32 on 544 bins 63 / 83).  Sides of at most 16,
// which have tiles of their own, are ahead on those grids, too (fprop of 8 x 32 -> 301, 21x21 27.9 / 24.7, 4 x 32 -> 130 21.3 / 19.1, 12 x 32 ->
// 256, 17x17 20.0 / 19.4; 13 such passes of random layers 1.03 .. 1.36x, none slower).
inline long tiles_32(const GemmParams &p) { return (long)p.bins * ((p.M + 31) / 32) * ((p.N + 31) / 32); }
inline bool direct_pays(const Prepared &q) {
    const GemmParams &p = q.prm;
    if (q.split || p.layA.tsh < 3 || p.K <= 16) return false;
    const int side = p.M < p.N ? p.M : p.N;
    if (side > (p.layA.tsh >= 5 ? 64 : 32)) return false;
    if (side > 32 && 3 * tiles_32(p) >= 10 * tiles_64(p) && tiles_64(p) >= 256 && (p.K < 32 || (q.akf && (p.K == 32 || p.K % 4 != 0)))) return false;
    return p.M <= 16 || p.N <= 16 || tiles_32(p) == tiles_64(p) || tiles_32(p) < (q.vec && p.layA.tsh >= 4 ? 32L : 128L) * p.K;
}

inline hipError_t prepare(const GemmProblem &g, const GemmSwitches &sw, Prepared *out) {
    const GemmOperand &A = g.A, &B = g.B;
    const int M = g.M, N = g.N, K = g.K, bins = g.bins;
    if (bins % kXcds != 0) return hipErrorInvalidValue;   // N*(N/2+1) with N >= 8 always is
    GemmParams &prm = out->prm;
    prm.A = A.ptr; prm.B = B.ptr; prm.C = g.C;
    prm.layA = A.lay; prm.layB = B.lay; prm.layC = g.layC;
    prm.a_rs = A.rs; prm.a_cs = A.cs; prm.b_rs = B.rs; prm.b_cs = B.cs;
    prm.c_rs = g.C_rs; prm.c_cs = g.C_cs;
    prm.M = M; prm.N = N; prm.K = K; prm.bins = bins; prm.live = g.live;
    prm.tiles_m = prm.tiles_n = 0;
    prm.split_from = 0xffffffffu;
    prm.a_sign = A.conj ? 0x80000000u : 0u;
    prm.b_sign = B.conj ? 0x80000000u : 0u;
    const bool akf = (A.cs == 1), bkf = (B.rs == 1);
    // 16-byte gathers need: runs of >= 4 planes, the contiguous index a multiple of 4 at every
    // vector start (tile origins are), its extent a multiple of 4, and the other stride too.
    auto vec_ok = [](const FreqLayout &l, long contiguous_extent, long other_stride, const float *p) {
        return l.tsh >= 2 && contiguous_extent % 4 == 0 && other_stride % 4 == 0 && ((size_t)p & 15) == 0;
    };
    const bool va = akf ? vec_ok(A.lay, K, A.rs, A.ptr) : (A.rs == 1 && vec_ok(A.lay, M, A.cs, A.ptr));
    const bool vb = bkf ? vec_ok(B.lay, K, B.cs, B.ptr) : (B.cs == 1 && vec_ok(B.lay, N, B.rs, B.ptr));
    out->akf = akf; out->bkf = bkf; out->vec = va && vb;
    prm.fast = (out->vec && fast_addressing(A.lay, akf ? A.rs : A.cs, bins) &&
                fast_addressing(B.lay, bkf ? B.cs : B.rs, bins) && g.C_cs == 1 && fast_addressing(g.layC, g.C_rs, bins) &&
                !sw.no_fast) ? 1 : 0;
    // Layouts with runs of 4 planes (basis 64) put four bins in every 128-byte line: the
    // bin-group kernel loads whole lines and multiplies the four bins side by side.
    out->bingroup = out->vec && !sw.no_bingroup && A.lay.tsh == 2 && B.lay.tsh == 2 && g.layC.tsh == 2 &&
                    bins % (4 * kXcds) == 0 && (akf || A.rs == 1) && (bkf || B.cs == 1) && g.C_cs == 1 &&
                    g.C_rs % 4 == 0 && N % 4 == 0 && ((size_t)g.C & 15) == 0;
    out->shifted = !out->vec && !sw.no_bingroup && sw.tile < 0 && shifted_lines(prm, akf, bkf) && shifted_pays(prm);
    out->shifted_alone = out->shifted && shifted_alone_pays(prm, akf);
    const Thin form = thin_form(prm);
    out->thin = sw.no_thin || sw.tile >= 0 || !thin_pays(prm, form, bkf, out->vec, out->bingroup) ? Thin::none : form;
    out->split = !out->bingroup && (akf || !bkf) && !sw.no_split && sw.tile < 0 && split_pays(prm, akf, bkf, out->vec) && !narrow_tile(prm, out->vec);
    out->split_alone = out->split && split_alone_pays(prm, akf, out->vec);
    out->direct = direct_fits(prm, akf, bkf) && sw.tile < 0 && !sw.no_direct;
    out->direct_alone = out->direct && out->thin == Thin::none && direct_pays(*out);
    return hipSuccess;
}

// The k form's product formed inside the inverse transform of its result (fft_thin_inv.hip): the result is neither written
// nor read back, its operands are read from the caches once per four planes.  us of fprop, two kernels / one: up to basis 24,
// where a launch counts, 64 x 3 -> 384, 13x13 27.5 / 17.6, 16 x 4 -> 16, 8x8 13.7 / 11.1; above with three terms or fewer and a
// few rounds of workgroups, 128 x 3 -> 64, 28x28 39.2 / 30.8, 56x56 75.8 / 72.8, 64 x 2 -> 20, 56x56 36.8 / 31.5, but 8 x 3 -> 16,
// 56x56 22.8 / 24.0; a fourth term's loads cost more than the trip (128 x 4 -> 64, 56x56 79.7 / 87.7, 16 x 4 -> 16, 28x28 22.2 /
// 25.5), and basis 64's tile leaves the fewest workgroups to hide them (128 x 3 -> 64 100 / 135).
// On basis 28 the ordinary inverse has a lane a line, which with three terms is ahead on full grids (bprop 480 x 36 -> 3, 27x27 46.2 / 52.3, 64 x 304
// -> 3 47.5 / 53.3, fprop 300 x 3 -> 64, 28x28 47.4 / 56.8), but for bprop's wide results in whole pairs of tiles (64 x 384 -> 3, 28x28 56.6 / 55.1).
// Four terms on bases up to 24, over 450 layers (weights ahead, fprop / bprop).  fprop, whose columns are four planes apart, gathers whole
// lines of the weights for each: only small results above basis 14 (233 x 4 -> 316, 16x16 46.3 / 56.5; 280 x 4 -> 128, 18x18 43.1 / 51.5;
// 379 x 4 -> 68, 24x24 54.9 / 70.9), on basis 16 not the smallest (1 x 4 -> 368 12.7 / 13.5), on 18 and 20 the smallest where a tile holds whole
// quads or rows of columns (34 x 4 -> 8, 18x18 15.2 / 15.7, 301 x 4 -> 4 16.7 / 15.4; 10 x 4 -> 28, 20x20 14.3 / 16.5), on 24 with four columns (52 x 4
// -> 28 19.2 / 23.1, 416 x 4 -> 4 20.8 / 18.9, 1 x 4 -> 4 13.6 / 12.3).  bprop is behind on basis 24 alone, where columns do not fill a tile (11 x 12 -> 4, 23x23 15.6 / 16.9).
inline bool product_inverse_pays(const Prepared &q, int basis) {
    if (q.thin != Thin::k || basis > 56) return false;
    const int N = q.prm.N;
    const long planes = (long)q.prm.M * N;
    if (q.prm.K <= 3) {
        if (basis == 28 && q.prm.K == 3 && planes >= 16384) return !q.bkf && N >= 192 && N % 32 == 0;
        return basis <= 24 || planes >= 1024;
    }
    if (basis > 24) return false;
    const bool four = N == 4 && (planes == 4 || planes >= 960);
    if (!q.bkf) return basis <= 20 || N % 16 == 0 || planes >= 3000 || four;
    if (basis <= 12) return true;
    if (basis == 14) return planes < 65536;
    if (basis == 16) return planes >= 1024 && planes < 65536;
    if (basis == 24) return four;
    return N == 4 || (planes < 12000 && (N == 16 || planes >= 2400));
}

// The kernel that a contraction takes in a launch of its own.
enum class Kernel { product, thin, direct, bingroup, shifted, split, tiles };
inline Kernel kernel_alone(const Prepared &q) {
    if (q.thin != Thin::none) return Kernel::thin;
    if (q.direct_alone) return Kernel::direct;
    if (q.bingroup) return Kernel::bingroup;
    if (q.shifted_alone) return Kernel::shifted;
    return q.split_alone ? Kernel::split : Kernel::tiles;
}
// With the inverse transform behind it; basis: the square basis of the pass, 0 for a rectangular one.
inline Kernel kernel_of_pass(const Prepared &q, int basis) {
    return basis && product_inverse_pays(q, basis) ? Kernel::product : kernel_alone(q);
}

// But for narrow sides, 64x64 tiles on four waves with one tile of register staging ahead (shape 3)
// measured fastest of the fp32 kernel's shapes for every layer tried (more workgroups in flight beat
// the larger tiles' operand reuse and the deeper staging's registers).
inline int pick_tile(const GemmSwitches &sw, const GemmParams &prm, bool vec) {
    if (sw.tile >= 0) return sw.tile;
    return narrow_tile(prm, vec) ? (prm.M <= 32 ? 6 : 7) : 3;
}

// What a contraction loses, in us, as a part of the shared launch's 64x64 tiles against the kernel that
// it has by itself: fits of the differences measured over 60 layers of 1, 4, 16 .. 384 channels.
inline double lost_in_shared_tiles(const Prepared &q) {
    const GemmParams &p = q.prm;
    const double steps = (double)p.bins * p.K * ((p.M + 63) / 64) * ((p.N + 63) / 64);
    if (q.thin == Thin::acc) {
        const double chain = 0.041 * p.K, lost = chain > 1.9e-4 * steps ? chain : 1.9e-4 * steps;
        return 4 * p.M < 1 << p.layA.tsh ? 0.3 * lost : lost;     // (few rows on a long run: a few lanes work)
    }
    if (q.thin != Thin::none) return 3 + 5e-4 * steps;
    return narrow_tile(p, q.vec) ? 1e-4 * steps : 0;
}

// bprop and accGrad of a layer with four or fewer channels on a side, or of one sample.  Constants of a time when two launches
// for the products meant two for the inverse transforms, too; since then separate products share an inverse launch while they
// are small, and one of at most four terms may need no launch of its own, so that two launches cost less than this charges.
// It charged 12 us and more with bprop's reduction: 16 samples,
// 4 -> 16 channels, 13x13 15 us a backward pass in the shared launch against 30; 128 x 4 -> 384, 20x20 119 / 114, 128 x
// 4 -> 128, 28x28 92 / 78.  With the thin side in bprop alone accGrad decides (256 x 64 -> 4, 32x32 91 /
// 109; 256 x 384 -> 4, 20x20 194 / 172).  One sample: by the size of the gradient's spectrum (64 -> 128 channels,
// 20x20, 58 MB 33 / 44; 256 -> 256, 115 MB 110 / 100).
inline bool shared_launch_pays(const Prepared &b, const Prepared &a) {
    if (b.thin == Thin::none && a.thin == Thin::none) return true;
    if (a.prm.K == 1) return (double)a.prm.bins * a.prm.M * a.prm.N < 1.4e7;
    const double lost = lost_in_shared_tiles(a);
    return lost == 0 || lost + lost_in_shared_tiles(b) < 12 + 0.03 * b.prm.K;
}

// bprop and accGrad as one launch of the kernel that splits the reduction, where 64x64 tiles would be about half padding (over
// 700 random layers, against the best of the other ways; us a backward pass).  Channel counts that are no multiple of four, with a
// reduction of more than two chunks: 22 samples, 16 -> 311, 14x14 39.8 / 30.0, 1 x 86 -> 14, 65x65 38.1 / 28.5; fuller tiles
// are behind (3 x 304 -> 207, 21x21 179 / 218) but with runs of 32 and more, whose lines a strip uses whole.  With runs of four planes up to
// 6000 tiles (7 x 16 -> 6, 75x75 41.2 / 37.9; 8 x 359 -> 13, 87x87 256 / 345).  Multiples of four: from 48 steps on (6 x 16 -> 304,
// 14x14 40.2 / 26.5; 5 x 368 -> 24, 14x14, 24 steps 29.0 / 31.4).
inline bool direct_pair_pays(const Prepared &b, const Prepared &a) {
    if (!b.direct || !a.direct || b.thin != Thin::none || a.thin != Thin::none) return false;
    if (!b.akf || b.bkf || a.akf || a.bkf) return false;
    const int tsh = b.prm.layA.tsh, K = b.prm.K > a.prm.K ? b.prm.K : a.prm.K;
    const long t64 = tiles_64(b.prm) + tiles_64(a.prm);
    const bool padded = tiles_32(b.prm) + tiles_32(a.prm) <= 2.2 * t64;
    if (tsh == 2) return b.shifted && a.shifted && padded && t64 < 6000;
    if (!b.vec || !a.vec) return K > 16 && (padded || (tsh >= 5 && !a.split));
    return K >= 48 && padded && !a.split && !b.split;
}

// The two as one launch of 64x64 tiles with 4-byte gathers: 50 random layers a quarter faster in the mean than two launches for
// the products and two for the inverse transforms (9 samples, 80 -> 38, 15x15 35.8 / 24.1 us a backward pass, 14 x 41 -> 112, 81x81
// 193 / 158).
inline bool scalar_pair_pays(const Prepared &b, const Prepared &a) {
    return !(b.vec && a.vec) && b.akf && !b.bkf && !a.akf && !a.bkf && b.prm.layA.tsh >= 3 && !a.split && !b.split &&
           b.thin == Thin::none && a.thin == Thin::none;
}

// Two contractions in one launch: bprop and accGrad of a layer, which share operand A and neither of
// which waits for the other.
enum class Shared { none, direct, tiles, split, scalar };
inline Shared shared_launch(const Prepared &q1, const Prepared &q2, const GemmSwitches &sw) {
    if (sw.tile >= 0 || sw.no_pair) return Shared::none;     // A/B runs of single-kernel shapes
    const Prepared &b = q1.akf ? q1 : q2, &a = q1.akf ? q2 : q1;
    const bool apart = q1.akf != q2.akf;
    if (apart && direct_pair_pays(b, a)) return Shared::direct;
    if (q1.vec && q2.vec && !q1.bingroup && !q2.bingroup && shared_launch_pays(b, a)) {
        if (b.thin != Thin::none || a.thin != Thin::none) return Shared::tiles;
        if (q1.bkf || q2.bkf || !apart) return Shared::tiles;
        if (!b.split || !a.split) return Shared::tiles;
        // Under general addressing small grids are behind (128 x 48 -> 48, 7x7, 40 tiles 27.6 / 29.0; 128 x 32 -> 96, 80 28.5 /
        // 29.6; 64 x 96 -> 96, 160 26.3 / 26.3; 64 x 32 -> 384, 240 53.0 / 51.3).
        return a.prm.fast || tiles_64(a.prm) >= 100 ? Shared::split : Shared::tiles;
    }
    return apart && scalar_pair_pays(b, a) ? Shared::scalar : Shared::none;
}

// Whether one gradient alone takes the waves of the shared direct launch, so that its product is the same bits with and without the
// other, or a kernel of its own.  10000 lone gradients of random layers, 64x64 tiles / shared waves (whole backward calls): 1.0 .. 2x where
// a tile of 32 is one of 64, but with runs of four planes for long reductions of many planes (4 x 21 x 339 on 704 bins 87 / 99, 46 x 4 x 298
// 103 / 117; 2 x 7 x 328 64 / 57), not with more
// than 9 tiles to 4 (512 x 317 x 4, 13x13 74.8 / 100.3 us), and between them with runs of eight (1.05 .. 1.2x).  With more than 16 steps
// otherwise up to the grids that the split reduction alone stops at; with fewer, where the shared launch leaves most of its waves without a
// chunk, while there are few tiles (runs of 16 and up to 8 steps: 1.05x below 4096, 0.90 .. 0.98 above; 9 .. 16: 1.0 below 1024, 0.91 .. 0.97; longer
// runs 1.02 .. 1.09x below 1024, 0.95; 9 .. 16 steps 0.97 from one tile a compute unit to two), and with runs of four and 9 .. 16 steps not for
// two tiles to one of 64 (704 bins 0.91, 864 0.97).
inline bool lone_as_shared_pays(const Prepared &q) {
    const GemmParams &p = q.prm;
    const long t32 = tiles_32(p), t64 = tiles_64(p);
    const int tsh = p.layA.tsh;
    if (tsh == 2 && p.K > 48 && (double)p.bins * p.K * (p.M + p.N) >= 2.5e6) return false;
    if (t32 == t64) return true;
    if (4 * t32 > 9 * t64) return false;
    if (tsh == 3) return true;
    if (tsh == 2) return p.K <= 8 || p.K > 16 || t32 < 2 * t64 || t64 > p.bins;
    if (p.K > 16) return t32 < (q.vec ? 32L : 128L) * p.K;
    if (tsh == 4) return t32 < (p.K <= 8 ? 4096 : 1024);
    return t32 < 1024 && (p.K <= 8 || t32 < 256 || t32 >= 512);
}

// One gradient of a backward pass asked for alone: the kernel that it takes, and whether that is the direct kernel on the
// waves of the shared launch.
struct Lone {
    Kernel kernel;
    bool as_shared;
};
inline Lone lone_gradient(const Prepared &q, const Prepared &partner, const GemmSwitches &sw) {
    const Shared how = shared_launch(q, partner, sw);
    if (how == Shared::direct && lone_as_shared_pays(q)) return {Kernel::direct, true};
    Prepared own = q;
    if (how != Shared::none && how != Shared::direct) own.direct_alone = false;
    return {kernel_alone(own), false};
}

}  // namespace fc
