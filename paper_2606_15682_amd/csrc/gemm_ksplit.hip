// W4A4 GEMM for gfx950 where 256 x 256 tiles leave the chip idle: batches and
// prompt chunks of 65 to a few thousand rows, and every K that is a multiple
// of 128.
//
// Tiles of 64 x 64, 64 x 128 or 128 x 128, whole K each (splitting K over
// workgroups would need a workspace, which the product's callers do not pass).
// Inside a workgroup the waves stand side by side and, in the two smaller
// tiles, share out K as well: every wave works on a 64 x 64 block, so that
// NVFP4's decode (8 VALU per fragment) costs no more than its MFMAs, and a
// small tile still has two waves per SIMD.  The partial sums meet in LDS at
// the end and are added in the order of the waves: the result does not depend
// on timing.
//
// Each K stage of the tile's rows goes global -> LDS once, in whole 128-byte
// lines of codes, through a ring of NBUF buffers.  The load path of a CU takes
// about 2.5 cycles per row piece and 128-byte line, so the scale bytes go in
// groups of several stages (a line per row and 1024 MXFP4 elements).  Loads,
// LDS reads and MFMAs are interleaved instruction by instruction: one after the
// other (loads, then reads, then MFMAs) a stage of 34 KB took 1.03 us on
// MXFP4 instead of 0.45.
//
// 17 to 64 rows take tiles of 32 or 64 rows of X, from row-major weights or from
// the packed decode image (gemm_skinny.hip), which lies in LDS as it lies in
// memory; the operands are the same, and so is the result, bit for bit.
//
// What bounds each tile: NVFP4 the matrix cores and the decode beside them
// (64 x 64: 2.1 us per 1000 elements of K with one tile per CU, 0.93 us would be
// the MFMAs alone; counters: matrix pipe busy on 0.34 of the cycles, VALU issue on 0.49).
// MXFP4 (64 x 64: 1.3 us; 128 x 128: 4 us, 5 for two tiles per CU): issue and waits,
// with the matrix pipe busy on 0.05 (64 x 32, 40 to 50 scalar instructions per MFMA) to 0.25 of the
// cycles (128 x 128, 5 of them) and waves waiting for a counter or barrier on 0.36 to 0.52 of theirs.  Measured against the 256 x 256 kernel, one graph, weights
// from HBM: NVFP4 256 x 3584 x 18944 331 -> 45 us, 256 x 4608 x 3584 69 -> 19 us;
// MXFP4 777 x 6912 x 5120 37 -> 27 us, 777 x 1792 x 5120 36 -> 17 us; NVFP4
// 777 x 5120 x 3456 (K % 256 = 128, where the general kernel ran) 437 -> 43 us.
//
// LDS layout: 16-byte chunk c of row r sits at chunk c ^ f(r), scale dword j at
// j ^ g(r), so that 32 consecutive rows read at one logical column spread over
// the banks.  Lane (r, h) takes chunk 2 v + h of row r for slice v (64 elements)
// of a stage: 32 consecutive codes, which is one MXFP4 block
// (v_mfma_scale_f32_32x32x64, its E8M0 byte to the matrix core) or two NVFP4
// blocks (four v_mfma_f32_32x32x16_f16 on operands decoded exactly to FP16).
#include <type_traits>

#include "fp4_device.h"
#include "g2l.h"
#include "internal.h"

namespace reqat {

namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef __bf16 v4bf __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t pick(const uint4 &q, int s) {
    return s == 0 ? q.x : s == 1 ? q.y : s == 2 ? q.z : q.w;
}

// Eight codes (one dword) times a block scale (FP16, in both halves) -> FP16 (exact).
__device__ __forceinline__ v8h decode8(uint32_t c, v2h s) {
    const v2h p0 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(c, 1.0f, 0) * s;
    const v2h p1 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(c, 1.0f, 1) * s;
    const v2h p2 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(c, 1.0f, 2) * s;
    const v2h p3 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(c, 1.0f, 3) * s;
    return v8h{p0[0], p0[1], p1[0], p1[1], p2[0], p2[1], p3[0], p3[1]};
}

// RM x RN MFMA tiles of 32 x 32 per wave; WM x WN waves cover the workgroup's
// tile, WK such sets share out K: of the KS elements of a stage each takes SUB
// slices of 64.
template <int FMT, int RM_, int RN_, int WM_, int WN_, int WK_, int SUB_, int NBUF_, int SROW_>
struct Cfg {
    static constexpr int RM = RM_, RN = RN_, WM = WM_, WN = WN_, WK = WK_, SUB = SUB_, NBUF = NBUF_, SROW = SROW_;
    static constexpr int B = FMT == kMX ? 32 : 16;
    static constexpr int WAVES = WM * WN * WK, THREADS = 64 * WAVES;
    static constexpr int TM = 32 * RM * WM, TN = 32 * RN * WN, ROWS = TM + TN;
    static constexpr int KS = 64 * WK * SUB;
    static constexpr int ROW = KS / 2, CH = ROW / 16;       // code bytes, 16-byte chunks per row
    static constexpr int RPI = 1024 / ROW;                  // rows per 1 KB load
    static constexpr int SB = KS / B;                       // scale bytes per row and stage
    // Scale groups: SROW bytes per row (GS stages), a GS-th of a group loaded with
    // each stage's codes.  That piece belongs to the group after the stage's (GS >
    // 1) and goes out up to NBUF stages before the stage is read: NGRP buffers
    // keep it off a group that is still read.
    static constexpr int SD = SROW / 4, GS = SROW / SB;
    static constexpr int NGRP = GS == 1 ? NBUF : 2 + (NBUF + GS - 2) / GS;
    static constexpr int SRPI = 64 / SD;                    // rows per 256-byte scale load
    static constexpr int STAGE = ROWS * ROW, GROUP = ROWS * SROW;
    static constexpr int CL = STAGE / 1024 / WAVES;         // code loads per wave and stage
    static constexpr int SPP = ROWS / SRPI / GS;            // scale loads per stage, and per wave and stage
    static constexpr int SL = (SPP + WAVES - 1) / WAVES;    // (where they do not split evenly, the last one is repeated)
    static constexpr int LPS = CL + SL;
    // packed weights (units of 16 rows x 256 elements, see gemm_skinny.hip): units per row
    // group and stage, a unit's scale bytes, a row group's scale bytes per scale group
    static constexpr int CPS = KS / 256, SU = 16 * 256 / B, RUN = 16 * SROW;
    static constexpr int PART = WAVES * RN * 16 * 64 * 4;   // bytes of one round of the epilogue
    static constexpr int RING = NBUF * STAGE + NGRP * GROUP;
    static constexpr int LDS = RING > PART ? RING : PART;
    static_assert(STAGE % (1024 * WAVES) == 0 && ROWS % (SRPI * GS) == 0, "whole loads, code loads split evenly");
    static_assert(TM % RPI == 0 && TM % SRPI == 0, "a load's rows are all of A or all of B");
    static_assert(LDS <= 160 * 1024 && (CH == 8 || CH == 16) && (SD == 4 || SD == 8) && SROW % SB == 0, "LDS layout");
    static_assert(NBUF >= 2 && NBUF <= 4 && NBUF * LPS + GS * SL <= 63, "vmcnt range");
    static_assert(GS <= 2, "a stage's piece of a scale group goes by its parity");
    // both repeat every 32 rows: MFMA tile i of a wave lies 32 rows further at the same columns
    static __device__ __forceinline__ int fc(int r) { return CH == 16 ? (r & 15) : ((r & 7) ^ ((r >> 3) & 1)); }
    static __device__ __forceinline__ int fs(int r) { return SD == 8 ? ((r >> 3) & 3) : ((r >> 4) & 1); }
};

// A wave's operands of one slice: 32 codes and their scale bytes per MFMA tile.
template <class C> struct Raw {
    uint4 a[C::RM], b[C::RN];
    uint32_t sa[C::RM], sb[C::RN];
};

template <int FMT, class C, bool kPacked>
__global__ __launch_bounds__(C::THREADS, C::LDS <= 80 * 1024 ? C::WAVES / 2 : C::WAVES / 4) void gemm_ksplit_kernel(
    int64_t M, int64_t N, int64_t K, const uint8_t *__restrict__ a_codes, const uint8_t *__restrict__ a_scales,
    const float *__restrict__ ga, const uint8_t *__restrict__ b_codes, const uint8_t *__restrict__ b_scales,
    const float *__restrict__ gb, void *__restrict__ y, int y_bf16, int y_vec, int64_t ldy) {
    constexpr int RM = C::RM, RN = C::RN, WM = C::WM, WN = C::WN, WK = C::WK, SUB = C::SUB, NBUF = C::NBUF;
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave / (WM * WN), wm = wave / WN % WM, wn = wave % WN;
    const int64_t cpr = K / 2, spr = K / C::B;

    // Tile of this workgroup: workgroups are dealt round-robin to the 8 XCDs, so
    // each XCD takes a contiguous run of tiles, M fastest within groups of tile
    // rows: neighbours share a panel of W in their L2.
    const int64_t tm_n = (M + C::TM - 1) / C::TM, tn_n = (N + C::TN - 1) / C::TN, T = tm_n * tn_n;
    const int64_t xcd = blockIdx.x % 8, local = blockIdx.x / 8, per = T / 8, rem = T % 8;
    const int64_t t = xcd * per + (xcd < rem ? xcd : rem) + local;
    constexpr int GROUP_M = 1024 / C::TM;
    const int64_t width = GROUP_M * tn_n, first_m = (t / width) * GROUP_M;
    const int64_t gsz = (tm_n - first_m) < GROUP_M ? (tm_n - first_m) : GROUP_M;
    const int64_t m0 = (first_m + (t % width) % gsz) * C::TM, n0 = ((t % width) / gsz) * C::TN;

    // This wave's loads, each of rows of A or of B (rows past the edge re-read the last one)
    const uint8_t *ac = a_codes + m0 * cpr, *bc = b_codes + n0 * cpr;
    const uint8_t *as = a_scales + m0 * spr, *bs = b_scales + n0 * spr;
    const int left_a = (int)(M - m0 < C::TM ? M - m0 : C::TM) - 1, left_b = (int)(N - n0 < C::TN ? N - n0 : C::TN) - 1;
    // Packed weights: this tile's first unit, its row groups (past the last: the last)
    const int64_t nch = (K + 255) / 256;
    const uint8_t *pc = b_codes + (n0 >> 4) * nch * 2048, *ps = b_scales + (n0 >> 4) * nch * C::SU;
    const int left_g = (int)((N - n0 < C::TN ? N - n0 : C::TN) - 1) >> 4;
    const int nst = (int)((K + C::KS - 1) / C::KS), ngrp = (nst + C::GS - 1) / C::GS;
    uint8_t *const groups = smem + NBUF * C::STAGE;
    // Code load i: its rows' first byte, the lane's offset from it, and the lane's column in a
    // stage.  Packed weights: half a unit, 1 KB, as it lies in the image; column 0, and the
    // unit in the stage (cunit; units past the last: the last).
    const uint8_t *cbase[C::CL];
    uint32_t crow[C::CL];
    int ccol[C::CL], cunit[C::CL], cper[C::CL], cstep[C::CL];
    // (unrolled by templates: the bases have to end up in scalar registers at every
    // optimisation level, and a loop over the arrays can leave them in memory)
    static_for<0, C::CL>([&](auto I) __attribute__((always_inline)) {
        constexpr int i = decltype(I)::value;
        const int j = wave * C::CL + i, row = j * C::RPI + lane / C::CH;
        const bool a = j * C::RPI < C::TM, pk = kPacked && !a;
        const int jb = j - C::TM / C::RPI, rg = jb / (2 * C::CPS), half = jb % (2 * C::CPS);
        const int r = pk ? rg : a ? row : row - C::TM, last = pk ? left_g : a ? left_a : left_b;
        cbase[i] = pk ? pc : a ? ac : bc;
        crow[i] = (uint32_t)(r < last ? r : last) * (pk ? (uint32_t)nch * 2048u : (uint32_t)cpr) +
                  (pk ? (uint32_t)(half * 1024 + lane * 16) : 0u);
        ccol[i] = pk ? 0 : ((lane % C::CH) ^ C::fc(row)) * 16;
        cunit[i] = pk ? half >> 1 : 0;
        cper[i] = pk ? C::CPS : 1;
        cstep[i] = pk ? 2048 : C::ROW;
    });
    const int clast = kPacked ? (int)nch - 1 : 0;
    // Scale load i of piece p of a scale group, likewise (packed: 256 bytes of a row group's run).
    const uint8_t *sbase[C::GS][C::SL];
    uint32_t srow[C::GS][C::SL];
    int scol[C::GS][C::SL], sstep[C::GS][C::SL], send[C::GS][C::SL];
    static_for<0, C::GS>([&](auto PP) __attribute__((always_inline)) {
        static_for<0, C::SL>([&](auto I) __attribute__((always_inline)) {
            constexpr int p = decltype(PP)::value, i = decltype(I)::value;
            const int w = wave * C::SL + i, j = p * C::SPP + (w < C::SPP ? w : C::SPP - 1);
            const bool a = j * C::SRPI < C::TM, pk = kPacked && !a;
            const int jb = j - C::TM / C::SRPI, row = j * C::SRPI + lane / C::SD;
            const int r = pk ? jb * 256 / C::RUN : a ? row : row - C::TM, last = pk ? left_g : a ? left_a : left_b;
            const int per = pk ? (int)nch * C::SU : (int)spr;
            sbase[p][i] = pk ? ps : a ? as : bs;
            srow[p][i] = (uint32_t)(r < last ? r : last) * (uint32_t)per;
            scol[p][i] = pk ? jb * 256 % C::RUN + lane * 4 : ((lane % C::SD) ^ C::fs(row)) * 4;
            sstep[p][i] = pk ? C::RUN : C::SROW;
            send[p][i] = per - 4;
        });
    });
    // Scale load i of piece p of scale group g (past the last group: of the last, into
    // a buffer nobody reads).  Columns past K re-read the row's last ones, here and
    // below: they belong to slices that are skipped.
    auto load_scale = [&](int g, int p, int i) __attribute__((always_inline)) {
        const int w = wave * C::SL + i, j = p * C::SPP + (w < C::SPP ? w : C::SPP - 1);
        const int step = sstep[p][i], at = (g < ngrp ? g : ngrp - 1) * step;
        const int left = send[p][i] - at, lim = left < step ? left : step;
        g2l4(sbase[p][i] + at, srow[p][i] + (uint32_t)(scol[p][i] < lim ? scol[p][i] : lim),
             groups + (g % C::NGRP) * C::GROUP + j * 256);
    };
    // Load L of this wave's share of stage s (of parity PAR): its piece of a scale
    // group, then the code loads.
    auto load_one = [&](int s, int buf, auto LL, auto PAR) __attribute__((always_inline)) {
        constexpr int L = decltype(LL)::value;
        if constexpr (L < C::SL) {
            load_scale(C::GS == 1 ? s : s / C::GS + 1, C::GS == 1 ? 0 : decltype(PAR)::value, L);
        } else {
            constexpr int i = L - C::SL;
            const int j = wave * C::CL + i;
            const int64_t left = cpr - 16 - (int64_t)s * C::ROW;
            const int lim = left < C::ROW ? (int)left : C::ROW;
            int at = s;
            if constexpr (kPacked) {
                at = s * cper[i] + cunit[i];
                at = (at < clast ? at : clast) - cunit[i];
            }
            g2l16(cbase[i] + (int64_t)at * cstep[i], crow[i] + (uint32_t)(ccol[i] < lim ? ccol[i] : lim),
                  smem + buf * C::STAGE + j * 1024);
        }
    };
    auto load_all = [&](int s, int buf, auto PAR) {
        static_for<0, C::LPS>([&](auto L) { load_one(s, buf, L, PAR); });
    };

    // Slice u of a stage is the wave's 64 elements SUB wk + u of it; lane (r, h) takes
    // their half h of row r.
    const int lr = lane & 31, h = lane >> 5;
    constexpr int SPL = FMT == kMX ? 1 : 2;                 // scale bytes per lane and slice
    const int arow = wm * RM * 32 + lr, brow = C::TM + wn * RN * 32 + lr;
    // Tile t of slice u of stage s (in buffer buf) into registers: A tiles, then B tiles.
    auto read_tile = [&](Raw<C> &r, int s, int u, int buf, auto TT) {
        constexpr int t = decltype(TT)::value;
        const int unit = 2 * (SUB * wk + u) + h;
        const int chunk = (unit ^ C::fc(lr)) << 4;
        const int byte = (s % C::GS) * C::SB + unit * SPL;  // of the lane's scales in its row of the group
        const int so = (((byte >> 2) ^ C::fs(lr)) << 2) + (byte & 3);
        const int row = t < RM ? arow + 32 * t : brow + 32 * (t - RM);
        const uint8_t *cp = smem + buf * C::STAGE + row * C::ROW + chunk;
        const uint8_t *sp = groups + (s / C::GS) % C::NGRP * C::GROUP + row * C::SROW + so;
        if constexpr (kPacked && t >= RM) {
            const int rg = 2 * (wn * RN + t - RM) + (lr >> 4), sl = SUB * wk + u, l = (lr & 15) + 16 * (sl & 3);
            cp = smem + buf * C::STAGE + C::TM * C::ROW + (rg * C::CPS + (sl >> 2)) * 2048 + h * 1024 + 16 * l;
            sp = groups + (s / C::GS) % C::NGRP * C::GROUP + C::TM * C::SROW + rg * C::RUN +
                 ((s % C::GS) * C::CPS + (sl >> 2)) * C::SU + 2 * SPL * l + SPL * h;
        }
        const uint4 c = *reinterpret_cast<const uint4 *>(cp);
        uint32_t sc;
        if constexpr (FMT == kMX) sc = *sp;
        else sc = *reinterpret_cast<const uint16_t *>(sp);
        if constexpr (t < RM) { r.a[t] = c; r.sa[t] = sc; }
        else { r.b[t - RM] = c; r.sb[t - RM] = sc; }
    };

    v16f acc[RM][RN];
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
        for (int j = 0; j < RN; ++j) acc[i][j] = v16f{};

    // NVFP4: fragment f (A tiles, then B tiles) of step q, decoded a step ahead.
    v8h dec[2][RM + RN];
    auto decode_one = [&](const Raw<C> &r, auto QQ, auto EE, auto FF) {
        constexpr int q = decltype(QQ)::value, E = decltype(EE)::value, f = decltype(FF)::value;
        const uint4 &c = f < RM ? r.a[f < RM ? f : 0] : r.b[f < RM ? 0 : f - RM];
        const v2h s = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(f < RM ? r.sa[f < RM ? f : 0] : r.sb[f < RM ? 0 : f - RM],
                                                               1.0f, false);
        dec[E][f] = decode8(pick(c, q), v2h{s[q >> 1], s[q >> 1]});
    };
    using I0 = std::integral_constant<int, 0>;

    // prologue: scale group 0 and stages 0 .. NBUF-1 on their way, slice 0 in registers
    static_for<0, (C::GS > 1 ? C::GS : 0)>([&](auto PP) __attribute__((always_inline)) {
        static_for<0, C::SL>([&](auto I) __attribute__((always_inline)) {
            load_scale(0, decltype(PP)::value, decltype(I)::value);
        });
    });
    static_for<0, NBUF>([&](auto S) {
        constexpr int s = decltype(S)::value;
        if (s < nst) load_all(s, s, std::integral_constant<int, s & 1>{});
    });
    {
        const int behind = nst - 1;
        if (NBUF >= 4 && behind >= 3) wait_and_meet<(NBUF >= 4 ? 3 : 0) * C::LPS>();
        else if (NBUF >= 3 && behind >= 2) wait_and_meet<(NBUF >= 3 ? 2 : 0) * C::LPS>();
        else if (behind >= 1) wait_and_meet<C::LPS>();
        else wait_and_meet<0>();
    }
    Raw<C> raw[2];
    static_for<0, RM + RN>([&](auto T) { read_tile(raw[0], 0, 0, 0, T); });
    if constexpr (FMT == kNV) static_for<0, RM + RN>([&](auto F) { decode_one(raw[0], I0{}, I0{}, F); });

    // Slice u of stage s, its operands in raw[P]: reads the next slice into raw[P ^ 1]
    // and multiplies.  The last slice of a stage first meets the other waves, once
    // stage s + 1 has landed for all and all have read stage s; the loads of stage
    // s + NBUF then go out into the buffer that stage s leaves.  Reads and loads are
    // spread over the MFMAs: ahead of them, each would take its time in turn.
    int buf = 0;                                            // s % NBUF
    auto slice = [&](int s, auto UU, auto PP, auto PAR, auto STEADY) __attribute__((always_inline)) {
        constexpr int u = decltype(UU)::value, P = decltype(PP)::value;
        constexpr bool LAST = u == SUB - 1;
        using LPAR = std::integral_constant<int, (decltype(PAR)::value + NBUF) & 1>;   // of stage s + NBUF
        constexpr bool steady = decltype(STEADY)::value;    // s + NBUF < nst: no branch in the slice
        const int nbuf = buf + 1 == NBUF ? 0 : buf + 1;
        const int rs = LAST ? s + 1 : s, rbuf = LAST ? nbuf : buf, ru = LAST ? 0 : u + 1;   // the next slice's place
        if constexpr (!LAST) {
            if constexpr (!steady)
                static_for<0, RM + RN>([&](auto T) { read_tile(raw[P ^ 1], rs, ru, rbuf, T); });
        } else if constexpr (steady) {
            wait_and_meet<(NBUF - 2) * C::LPS>();
        } else if (s + 1 < nst) {
            const int behind = nst - 2 - s;                 // stages after s + 1
            if (NBUF >= 4 && behind >= 2) wait_and_meet<(NBUF >= 4 ? 2 : 0) * C::LPS>();
            else if (NBUF >= 3 && behind >= 1) wait_and_meet<(NBUF >= 3 ? 1 : 0) * C::LPS>();
            else wait_and_meet<0>();
            static_for<0, RM + RN>([&](auto T) { read_tile(raw[P ^ 1], rs, ru, rbuf, T); });
            if (s + NBUF < nst) load_all(s + NBUF, buf, LPAR{});
        } else {
            __builtin_amdgcn_s_waitcnt(0xC07F);             // raw[P], on this path too
        }
        if (steady || (int64_t)s * C::KS + 64 * (SUB * wk + u) < K) {   // else: the slice lies past K
            // parts of RN MFMAs; NVFP4's LDS reads go out with the first step's
            constexpr int STEPS = FMT == kMX ? 1 : 4, PARTS = STEPS * RM, RPARTS = RM;
            static_for<0, PARTS>([&](auto TT) {
                constexpr int part = decltype(TT)::value, q = part / RM, i = part % RM, E = q & 1;
                constexpr int r0 = part < RPARTS ? part * (RM + RN) / RPARTS : RM + RN;
                constexpr int r1 = part < RPARTS ? (part + 1) * (RM + RN) / RPARTS : RM + RN;
                constexpr int NL = LAST ? C::LPS : 0;
                constexpr int l0 = part * NL / PARTS, l1 = (part + 1) * NL / PARTS;
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (FMT == kMX) {
                    static_for<0, RN>([&](auto JJ) {
                        constexpr int j = decltype(JJ)::value;
                        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                            v8i{(int)raw[P].a[i].x, (int)raw[P].a[i].y, (int)raw[P].a[i].z, (int)raw[P].a[i].w, 0, 0, 0, 0},
                            v8i{(int)raw[P].b[j].x, (int)raw[P].b[j].y, (int)raw[P].b[j].z, (int)raw[P].b[j].w, 0, 0, 0, 0},
                            acc[i][j], 4, 4, 0, (int)raw[P].sa[i], 0, (int)raw[P].sb[j]);
                        if constexpr (steady) {
                            __builtin_amdgcn_sched_barrier(0);
                            static_for<r0 + (r1 - r0) * j / RN, r0 + (r1 - r0) * (j + 1) / RN>(
                                [&](auto T) { read_tile(raw[P ^ 1], rs, ru, rbuf, T); });
                            static_for<l0 + (l1 - l0) * j / RN, l0 + (l1 - l0) * (j + 1) / RN>(
                                [&](auto L) { load_one(s + NBUF, buf, L, LPAR{}); });
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    });
                } else {
                    if constexpr (steady) {
                        static_for<r0, r1>([&](auto T) { read_tile(raw[P ^ 1], rs, ru, rbuf, T); });
                        static_for<l0, l1>([&](auto L) { load_one(s + NBUF, buf, L, LPAR{}); });
                    }
#pragma unroll
                    for (int j = 0; j < RN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(dec[E][i], dec[E][RM + j], acc[i][j], 0, 0, 0);
                    constexpr int f0 = i * (RM + RN) / RM, f1 = (i + 1) * (RM + RN) / RM;
                    static_for<f0, f1>([&](auto F) {
                        constexpr int qn = (q + 1) & 3;
                        decode_one(q == 3 ? raw[P ^ 1] : raw[P], std::integral_constant<int, qn>{},
                                   std::integral_constant<int, (E ^ 1)>{}, F);
                    });
                    constexpr int V = (8 * (f1 - f0) + RN - 1) / RN;
                    static_for<0, RN>([&](auto) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);       // one MFMA
                        __builtin_amdgcn_sched_group_barrier(0x002, V, 0);       // its share of the decode
                    });
                    static_for<f0, f1>([&](auto F) {
                        v8h &d = dec[E ^ 1][decltype(F)::value];
                        asm volatile("" : "+v"(d));
                    });
                }
            });
            __builtin_amdgcn_sched_barrier(0);
        }
        if (LAST) buf = nbuf;
    };
    // slices of stage s; with one slice per stage the register sets alternate by stage
    auto stage = [&](int s, auto PP, auto PAR, auto STEADY) __attribute__((always_inline)) {
        constexpr int P = decltype(PP)::value;
        static_for<0, SUB>([&](auto U) {
            slice(s, U, std::integral_constant<int, (P + decltype(U)::value) & 1>{}, PAR, STEADY);
        });
    };
    using I1 = std::integral_constant<int, SUB & 1>;
    static_assert(SUB == 1 || SUB % 2 == 0, "register sets alternate over two stages");
    int s = 0;
    for (; s + 1 + NBUF < nst; s += 2) {
        stage(s, I0{}, I0{}, std::true_type{});
        stage(s + 1, I1{}, std::integral_constant<int, 1>{}, std::true_type{});
    }
    for (; s < nst; s += 2) {
        stage(s, I0{}, I0{}, std::false_type{});
        if (s + 1 < nst) stage(s + 1, I1{}, std::integral_constant<int, 1>{}, std::false_type{});
    }

    // Results, one row of MFMA tiles per wave at a time, through LDS: the WK partial
    // sums are added in the order of the waves, and rows leave in 8- or 16-byte pieces.
    // part[wave][j][register][lane]; D[m][n] of a 32 x 32 tile sits in lane
    // n + 32 ((m / 4) % 2), register 4 (m / 8) + m % 4.
    const float scale = FMT == kNV ? (*ga) * (*gb) : 1.0f;
    float *part = reinterpret_cast<float *>(smem);
#pragma unroll
    for (int i = 0; i < RM; ++i) {
        __syncthreads();                                    // the stages, or the round before, have been read
#pragma unroll
        for (int j = 0; j < RN; ++j)
#pragma unroll
            for (int k = 0; k < 16; ++k) part[((wave * RN + j) * 16 + k) * 64 + lane] = acc[i][j][k];
        __syncthreads();
        constexpr int QUADS = WM * WN * RN * 256;           // of four consecutive columns of one row
#pragma unroll
        for (int q0 = 0; q0 < QUADS; q0 += C::THREADS) {
            const int q = q0 + tid;
            if (QUADS % C::THREADS && q >= QUADS) break;
            const int l = (q & 15) * 4, k = (q >> 4) & 15, jj = q >> 8;
            v4f v = *reinterpret_cast<const v4f *>(part + q * 4);
#pragma unroll
            for (int w = 1; w < WK; ++w) v += *reinterpret_cast<const v4f *>(part + (w * QUADS + q) * 4);
            const int64_t m = m0 + 32 * (RM * (jj / RN / WN) + i) + 8 * (k >> 2) + 4 * (l >> 5) + (k & 3);
            const int64_t n = n0 + 32 * (jj % (RN * WN)) + (l & 31);
            v *= scale;
            if (m >= M || n >= N) continue;
            if (y_vec && n + 4 <= N) {
                if (y_bf16)
                    *reinterpret_cast<v4bf *>(reinterpret_cast<__bf16 *>(y) + m * ldy + n) =
                        v4bf{(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
                else
                    *reinterpret_cast<v4f *>(reinterpret_cast<float *>(y) + m * ldy + n) = v;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (n + e >= N) break;
                    if (y_bf16) reinterpret_cast<__bf16 *>(y)[m * ldy + n + e] = (__bf16)v[e];
                    else reinterpret_cast<float *>(y)[m * ldy + n + e] = v[e];
                }
            }
        }
    }
}

template <int FMT, class C, bool kPacked>
hipError_t launch_cfg(int64_t M, int64_t N, int64_t K, const uint8_t *a_codes, const uint8_t *a_scales,
                      const float *ga, const uint8_t *b_codes, const uint8_t *b_scales, const float *gb, void *y,
                      bool y_bf16, int64_t ldy, hipStream_t stream) {
    const int64_t grid = ((M + C::TM - 1) / C::TM) * ((N + C::TN - 1) / C::TN);
    const int64_t es = y_bf16 ? 2 : 4;
    const int y_vec = reinterpret_cast<uintptr_t>(y) % (4 * es) == 0 && ldy % 4 == 0;
    hipError_t e = hipFuncSetAttribute((const void *)gemm_ksplit_kernel<FMT, C, kPacked>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((gemm_ksplit_kernel<FMT, C, kPacked>), dim3((unsigned)grid), dim3(C::THREADS), C::LDS, stream, M, N, K,
                       a_codes, a_scales, ga, b_codes, b_scales, gb, y, (int)y_bf16, y_vec, ldy);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_ksplit(KsplitTile tile, Fmt fmt, int64_t M, int64_t N, int64_t K, const uint8_t *a_codes,
                              const uint8_t *a_scales, const float *ga, const uint8_t *b_codes,
                              const uint8_t *b_scales, const float *gb, void *y, bool y_bf16, int64_t ldy,
                              bool packed, hipStream_t stream) {
    // row offsets within a tile are 32-bit (128 rows of K / 2 bytes)
    if (K <= 0 || K % 128 || K > kKsplitMaxK || (packed && tile < kTile32x32)) return hipErrorInvalidValue;
    auto go = [&](auto F) {
        constexpr int f = decltype(F)::value;
        auto rows = [&](auto c) {
            return launch_cfg<f, decltype(c), false>(M, N, K, a_codes, a_scales, ga, b_codes, b_scales, gb, y, y_bf16,
                                                     ldy, stream);
        };
        auto both = [&](auto c) {
            return packed ? launch_cfg<f, decltype(c), true>(M, N, K, a_codes, a_scales, ga, b_codes, b_scales, gb, y,
                                                             y_bf16, ldy, stream)
                          : rows(c);
        };
        switch (tile) {
        case kTile32x32: return both(Cfg<f, 1, 1, 1, 1, 8, 1, 4, 32>{});
        case kTile32x128: return both(Cfg<f, 1, 2, 1, 2, 2, 2, 3, 16>{});
        case kTile64x32: return both(Cfg<f, 2, 1, 1, 1, 8, 1, 3, 32>{});
        case kTile64x64Few: return both(Cfg<f, 2, 1, 1, 2, 4, 1, 4, 16>{});
        case kTile64x64: return rows(Cfg<f, 2, 2, 1, 1, 8, 1, 4, 32>{});
        case kTile64x128: return rows(Cfg<f, 2, 2, 1, 2, 2, 2, 2, 16>{});
        case kTile128x128: return rows(Cfg<f, 2, 2, 2, 2, 1, 4, 2, 16>{});
        case kTile64x128Deep: return rows(Cfg<f, 2, 2, 1, 2, 4, 1, 4, 16>{});
        case kTile128x128Deep:
            if constexpr (f == kMX) return rows(Cfg<f, 2, 2, 2, 2, 2, 2, 3, 16>{});
        }
        return hipErrorInvalidValue;
    };
    return fmt == kMX ? go(std::integral_constant<int, kMX>{}) : go(std::integral_constant<int, kNV>{});
}

}  // namespace reqat
