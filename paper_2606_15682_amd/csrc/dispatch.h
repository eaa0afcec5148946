// Which kernel a call runs: rules on sizes, formats and strides alone, in plain C++
// (no HIP), so that a CPU test can ask them for any shape.
#pragma once
#include <stdint.h>

namespace reqat {

// Format selector shared by the launchers (same values as the C ABI enum).
enum Fmt : int { kNV = 0, kMX = 1 };

// NVFP4 with a computed global scale: tensors of at most this many elements are small
// enough for every workgroup to read whole (from L2) for the maximum, so that codes and
// scale take one launch (kGLocal) instead of a pass and a fix-up.
// Dense rows are walked as one run of vectors: 384 KB.  One launch / two, us in a graph:
// 16 x 1536 3.3 / -, 33 x 2048 4.5 / 6.7, 64 x 1536 4.5 / 6.6, 16 x 8960 5.8 / 6.8, 10 x 18944
// 6.4 / 6.8; it grows by 0.6 to 0.3 us per 2^15 elements, the two launches hardly.
// Rows with a stride cost a division and a filter of non-finite values per vector in every
// workgroup: 16 x 4096 6.1 / -, 33 x 2048 7.8 / 6.8, 24 x 5120 9.5 / 6.8, 96 x 2048 12.8 / 6.9.
constexpr int64_t kLocalMaxElems = int64_t(3) << 16;
constexpr int64_t kLocalMaxElemsStrided = int64_t(1) << 16;

inline bool nv_one_launch(int64_t elems, bool dense) {
    return elems <= (dense ? kLocalMaxElems : kLocalMaxElemsStrided);
}

// A launch holds fewer than 2^32 threads along x, and a tile has up to 512: where a kernel with one
// workgroup per tile would need more of them, the rules below leave it out.
constexpr int64_t kMaxTiles = (int64_t(1) << 23) - 1;

// ---------------------------------------------------------------- W4A4 product

// Tiles of gemm_ksplit.hip.  The deep ones have twice the waves and a longer ring (128 x 128:
// MXFP4 alone).  The last four serve up to 64 rows and take the packed decode image too.
enum KsplitTile : int {
    kTile64x64, kTile64x128, kTile128x128, kTile64x128Deep, kTile128x128Deep,
    kTile32x32, kTile32x128, kTile64x32, kTile64x64Few
};
constexpr int kTileLarge = 5;                   // of pick_product_tile: 256 x 256 tiles (gemm_tile256.hip)
constexpr int64_t kKsplitMaxK = int64_t(1) << 26;

// Which kernel runs a product of M > 64 rows: the one with the least estimated
// time, c + rounds (e + t K) with rounds = tiles / 256 CUs, rounded up, and a
// time per K that one round alone does not fall below (too few waves per CU
// to keep the matrix cores or the loads busy).  The numbers (nanoseconds; t per
// element of K) are a fit to measurements over M = 65 .. 2048 and (N, K) =
// (4608, 3584), (3584, 18944), (37888, 3584), (17920, 1536), (5120, 1280),
// (1792, 5120), (5120, 3456), (7168, 5120), one HIP graph, weights from HBM.
// Over 998 other shapes the pick took 1.006 of the fastest kernel's time (geometric mean),
// more than 10% over it in 17 of them, and never more than 5% over the 256 x 256 tiles'.
// For example, in us, for 64 x 64 / 64 x 128 / 128 x 128 / 256 x 256:
//   NVFP4  256 x 3584 x 18944: 45 / 85 / 131 / 331     1024 x 37888 x 3584: 386 / 277 / 259 / 237
//   MXFP4  128 x 4608 x 3584: 8.2 / 12.7 / 15.4 / 28   777 x 7168 x 5120: 46 / 41 / 29 / 40
//          2048 x 4608 x 3584: 55 / 38 / 35 / 29
// The rule uses sizes alone (big_ok also takes ldy, beyond 2^26), so a shape runs the same kernel.
//
// The deep tiles (eight waves, one workgroup per CU, three or four stages on their
// way) are for a single round: alone on a CU the plain 64 x 128 and 128 x 128 tiles
// wait a microsecond for each stage of 256 elements, shared by two workgroups they
// do not.  Plain / deep, in us: MXFP4 777 x 3584 x 18944 75 / 47, 777 x 1792 x 5120 16.5 / 12.9,
// NVFP4 256 x 5120 x 13824 63 / 52; in two rounds 1536 x 5120 x 1280 (MXFP4) 13.6 / 15.4.
struct ProductCost {
    int tm, tn;
    bool single;                                // for one round alone
    double c, e, t, alone;
};
constexpr ProductCost kProductCost[2][6] = {              // by KsplitTile, then 256 x 256
    // NVFP4
    {{64, 64, false, 3000, 1800, 2.15, 0}, {64, 128, false, 4000, 0, 3.6, 4.2}, {128, 128, false, 4000, 0, 6.9, 7.6},
     {64, 128, true, 4500, 0, 3.6, 0}, {0, 0, true, 0, 0, 0, 0}, {256, 256, false, 4000, 0, 22, 20}},
    // MXFP4
    {{64, 64, false, 3000, 1200, 1.3, 0}, {64, 128, false, 3000, 700, 2.0, 3.4}, {128, 128, false, 3000, 700, 2.9, 4.0},
     {64, 128, true, 3500, 0, 2.4, 0}, {128, 128, true, 4000, 0, 2.7, 0}, {256, 256, false, 3000, 700, 7.7, 0}},
};

// Small tiles have to promise this much: where the estimates are closer they
// err, mostly for many rounds of long rows (3855 x 5120 x 27648, five rounds of 128 x 128
// against two: 4% under the 256 x 256 tiles by the estimate, 4% over them measured).
constexpr double kLargeBias = 0.88;

// The KsplitTile, or kTileLarge: 256 x 256 tiles; -1 (the general kernel) where neither can run
inline int pick_product_tile(Fmt fmt, int64_t M, int64_t N, int64_t K, bool big_ok) {
    int best = -1;
    double least = 0;
    for (int i = 0; i < (big_ok ? kTileLarge + 1 : kTileLarge); ++i) {
        const ProductCost &q = kProductCost[fmt == kMX][i];
        if (q.tm == 0) continue;
        const int64_t tiles = ((M + q.tm - 1) / q.tm) * ((N + q.tn - 1) / q.tn);
        if (i < kTileLarge && tiles > kMaxTiles) continue;
        const double rounds = (double)((tiles + 255) / 256);
        if (q.single && rounds > 1) continue;
        const double t = rounds == 1 && q.alone > 0 ? q.alone : q.t;
        const double est = q.c + rounds * (q.e + t * (double)K);
        if (best < 0 || (i == kTileLarge ? kLargeBias : 1.0) * est < least) {
            best = i;
            least = est;
        }
    }
    return best;
}

// 17 to 64 rows: the skinny kernel (16 rows of W per workgroup, which reads all of X from L2
// in 16-byte pieces, M rows of it), or a tile that takes X through LDS once for 32 to 128 rows
// of W.  Up to 16 rows the skinny kernel is the faster one nearly everywhere.  The estimate, in
// us with K in thousands:
//   c + a K + rounds (e + b K + m K M / 64) + d K tiles / 256,   rounds = tiles / 256, rounded up:
// workgroups beyond one per CU share its load path, so a round costs, and part of the time
// goes with the tiles alone.  Fitted over 3500 shapes, N up to 56000, K up to 27648, both
// layouts of W, from HBM; a tile has to promise 4%.  Over those shapes the pick takes 0.836 of
// the skinny kernel's time (geometric mean) and 1.008 of the fastest one's; it is more than 5% over
// the skinny kernel in 1% of them (at most 18%), where packed and row-major weights differ.
// For example, in us, skinny / 64 x 32 / 64 x 64, packed weights:
//   MXFP4  62 x 5120 x 5120 19.4 / 10.0 / 11.4    64 x 27648 x 5120 65 / 35 / 24    58 x 17 x 1152 3.6 / 5.4 / 5.5
//   NVFP4  45 x 17776 x 640 9.5 / 15.8 / 9.1      54 x 2005 x 8576 14.9 / 17.1 / 25
struct DecodeCost {
    int rows, tn, tile;                         // rows of X it serves; tile -1: the skinny kernel
    double c, a, e, b, d, m;
};
constexpr DecodeCost kDecodeCost[2][7] = {
    // NVFP4
    {{32, 16, -1, 2.19, 0.28, 0.59, 0.16, 0.31, 0.69}, {48, 16, -1, 2.32, 0.40, 0.81, 0.20, 0.37, 0.63},
     {64, 16, -1, 1.50, 0.15, 1.86, 0.46, 0.47, 0.76},
     {32, 32, kTile32x32, 2.82, 0.25, 1.43, 0.63, 0.28, 0}, {32, 128, kTile32x128, 2.89, 1.11, 1.65, 1.86, 1.02, 0},
     {64, 32, kTile64x32, 1.15, 0.13, 3.79, 1.13, 0.36, 0}, {64, 64, kTile64x64Few, 2.78, 0.63, 1.90, 1.65, 0.59, 0}},
    // MXFP4
    {{32, 16, -1, 2.13, 0.16, 0.38, 0.09, 0.29, 0.75}, {48, 16, -1, 1.33, 0.13, 1.33, 0.20, 0.33, 0.76},
     {64, 16, -1, 1.31, 0.10, 1.49, 0.18, 0.36, 0.85},
     {32, 32, kTile32x32, 2.74, 0.21, 1.06, 0.21, 0.52, 0}, {32, 128, kTile32x128, 2.99, 0.48, 0.84, 0.87, 2.07, 0},
     {64, 32, kTile64x32, 1.31, 0.17, 2.92, 0.44, 0.61, 0}, {64, 64, kTile64x64Few, 3.08, 0.21, 0.98, 0.70, 1.02, 0}},
};
constexpr double kSkinnyBias = 0.96;            // the promise

// -1: the skinny kernel; else the KsplitTile.  Sizes alone, so that packed and
// row-major weights of a shape give the same result.
inline int pick_decode_tile(Fmt fmt, int64_t M, int64_t N, int64_t K) {
    if (M <= 16 || K > kKsplitMaxK) return -1;
    int best = -1;
    double least = 0;
    bool skinny = true;                         // the first skinny entry that holds M counts
    for (const DecodeCost &q : kDecodeCost[fmt == kMX]) {
        if (q.tile < 0 ? !skinny || M > q.rows : q.rows != (M <= 32 ? 32 : 64)) continue;
        const int64_t tiles = (N + q.tn - 1) / q.tn;
        if (q.tile >= 0 && tiles > kMaxTiles) continue;
        const double k = 1e-3 * (double)K, rounds = (double)((tiles + 255) / 256), full = (double)tiles / 256;
        const double est = (q.tile < 0 ? kSkinnyBias : 1.0) *
                           (q.c + q.a * k + rounds * (q.e + q.b * k + q.m * k * (double)M / 64) + q.d * k * full);
        if (q.tile < 0 || est < least) {
            best = q.tile;
            least = est;
        }
        if (q.tile < 0) skinny = false;
    }
    return best;
}

// ---------------------------------------------------------------- W4A16 product

#ifndef REQAT_W16_NT
#define REQAT_W16_NT 1
#endif
#ifndef REQAT_W16_KSMAX
#define REQAT_W16_KSMAX 12
#endif
#ifndef REQAT_W16_TARGET
#define REQAT_W16_TARGET 1024
#endif

// Tiles of gemm_w4a16_tile.hip (M > 32), and the two kernels of gemm_w4a16.hip.
enum W16Tile : int {
    kW16Decode = -2, kW16Split = -1, kW16Tile64x64, kW16Tile64x128, kW16Tile128x128, kW16Tile128x128x8
};
constexpr int64_t kW16TileMaxLd = int64_t(1) << 23;

inline int w4a16_row_tile(int64_t M) { return M <= 16 ? 1 : (M <= 32 ? 2 : 4); }

// K splits, when the weight rows alone give fewer workgroups than CUs: the
// fewest splits (fewest FP32 partials to add) that give about two workgroups
// per CU, spread evenly (the average CU has at least 90% of the busiest CU's
// count, so no CU runs a round alone); when no split count up to
// REQAT_W16_KSMAX does, enough to reach REQAT_W16_TARGET workgroups.  At most
// REQAT_W16_KSMAX splits and one pair of chunks each (splits start at even
// chunks).  On 16 x 5120 x 27648 (80 row groups) the first rule picks 6:
// 20.3 us against 21.6 for 12 and 24.5 for 4, which leaves a quarter of the
// CUs with one workgroup more than the rest.  The split depends on the shape
// alone, never on the device, so results are deterministic.
inline int gemm_w4a16_splits(int64_t M, int64_t N, int64_t K) {
    constexpr int64_t kCUs = 256;
    const int64_t rows = 64 * REQAT_W16_NT;
    const int64_t base = ((N + rows - 1) / rows) * ((M + 16 * w4a16_row_tile(M) - 1) / (16 * w4a16_row_tile(M)));
    const int64_t npair = K / 256;
    if (base >= kCUs || npair <= 1) return 1;
    const int64_t kmax = REQAT_W16_KSMAX < npair ? REQAT_W16_KSMAX : npair;
    for (int64_t ks = 2; ks <= kmax; ++ks) {
        const int64_t wg = base * ks, busiest = (wg + kCUs - 1) / kCUs;
        if (10 * wg >= 18 * kCUs && 10 * wg >= 9 * busiest * kCUs) return (int)ks;
    }
    int64_t ks = (REQAT_W16_TARGET + base - 1) / base;
    return (int)(ks < kmax ? ks : kmax);
}

// From 33 rows on: gemm_w4a16_kernel (64 rows of x and of W per workgroup, K split over
// workgroups) or the tile with the least estimated time, where it promises 12% or more.
// That kernel: 9 us and 16 ns per 64 x 64 block and 1000 elements of K.  Tiles: c + rounds
// t K; a workgroup alone on its CU and two sharing one finish at the same rate per tile,
// so rounds = tiles / 256, half way to the next whole number.  Fitted over M = 64 .. 1024 and
// twelve (N, K) from (2048, 1536) to (55296, 5120), weights from HBM.  For example, in us,
// that kernel / 64 x 64 / 64 x 128 / 128 x 128 of 4 waves / of 8 waves:
//   512 x 27648 x 5120: 221 / 181 / 131 / 130 / 142    512 x 5120 x 13824: 121 / 103 / 85 / 93 / 73
//   64 x 5120 x 13824: 26 / 44 / 52 / 91 / 63          128 x 2048 x 1536: 11.6 / 7.1 / 9.1 / 13.7 / 12.4
// Sizes alone decide, so packed and row-major weights give the same result.
struct W16Cost {
    int tm, tn;
    double c, t;                                // ns, ns per element of K and round
};
constexpr W16Cost kW16Cost[4] = {{64, 64, 3200, 2.9}, {64, 128, 3200, 3.7}, {128, 128, 4000, 6.5}, {128, 128, 4500, 5.3}};

// M <= 16: whether gemm_w4a16_decode_kernel, which reads x once for 16 rows of W, is faster
// than gemm_w4a16_kernel, which reads it once for 64 and splits K over workgroups where those
// are fewer than the CUs.  Estimates in us, K in thousands, 5% has to be promised: fitted over
// 3500 shapes, (N, K) up to (56000, 27648), M = 1 .. 16, both layouts, weights from HBM.  Over
// those the pick takes 0.74 of gemm_w4a16_kernel's time (geometric mean); it is more than 5%
// over it in 1% of them (row-major weights with K > 10000, at most 26%).  The time per round
// keeps many rounds of short rows off it (3 x 47888 x 768: 7.9 / 10.4).  For example, in us,
// gemm_w4a16_kernel / this one, packed weights:
//   4 x 3584 x 3584 7.1 / 3.9    4 x 37888 x 3584 17.3 / 15.3    16 x 1536 x 1536 5.8 / 3.3
//   7 x 7168 x 5120 11.1 / 7.7   7 x 5120 x 13824 12.4 / 14.7    16 x 27648 x 5120 19 / 36
inline bool w4a16_decode_pays(int64_t M, int64_t N, int64_t K) {
    if (M > 16 || K <= 0 || (N + 15) / 16 > kMaxTiles) return false;
    const double k = 1e-3 * (double)K, w = 1e-6 * (double)N * (double)K, wg = (double)((N + 15) / 16) / 256;
    const double split = N <= 64 * 255 ? 5.6 + 0.11 * w : 3.2 + 0.118 * w;
    const double rate = M <= 4 ? 0.38 : (M <= 8 ? 0.5 : 0.85);
    const double rounds = wg <= 1 ? 0.6 + 0.4 * wg : (double)(((N + 15) / 16 + 255) / 256);
    return 2.3 + rounds * (0.15 + rate * k) < 0.95 * split;
}

// kW16Split: gemm_w4a16_kernel; else the tile.
inline int pick_w4a16_tile(int64_t M, int64_t N, int64_t K, int64_t ldx) {
    if (M <= 32 || K <= 0 || K > kW16TileMaxLd || ldx > kW16TileMaxLd) return kW16Split;
    int best = kW16Split;
    double least = 0.88 * (9000 + 0.016 * (double)((N + 63) / 64) * (double)((M + 63) / 64) * (double)K);
    for (int i = 0; i < 4; ++i) {
        const W16Cost &q = kW16Cost[i];
        const int64_t tiles = ((M + q.tm - 1) / q.tm) * ((N + q.tn - 1) / q.tn);
        if (tiles > kMaxTiles) continue;
        if (i == kW16Tile128x128x8 && tiles > 256) continue;    // one workgroup per CU: for a single round
        const double full = (double)tiles / 256, rounds = tiles <= 256 ? 1.0 : 0.5 * (full + (double)((tiles + 255) / 256));
        const double est = q.c + rounds * q.t * (double)K;
        if (est < least) {
            best = i;
            least = est;
        }
    }
    return best;
}

// The W4A16 kernel of a product: a W16Tile.
inline int pick_w4a16(int64_t M, int64_t N, int64_t K, int64_t ldx) {
    const int tile = pick_w4a16_tile(M, N, K, ldx);
    return tile < 0 && w4a16_decode_pays(M, N, K) ? kW16Decode : tile;
}

}  // namespace reqat
