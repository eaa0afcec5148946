// W4A16 product for gfx950 beyond decode sizes: Y[m][n] = sum_k x[m][k] w^[n][k],
// w^ = RN_bf16(E2M1(c) * 2^e), FP32 sums (see gemm_w4a16.hip for the decode and
// the packed image of W).
//
// A workgroup of four (eight) waves owns a TM x TN tile of Y with all of K.  Each stage of
// KS elements of K (TM rows of x, TN rows of codes and scale bytes) goes global -> LDS once,
// through a ring of NBUF buffers, and is read there by every wave that needs it; the
// kernel of gemm_w4a16.hip loads 64 rows of x for 64 rows of W and decodes W once per 64
// rows of x (512 x 27648 x 5120: 221 us, 0.65 PFLOP/s).  A wave multiplies RM x RN MFMA
// tiles of 32 x 32 (v_mfma_f32_32x32x16_bf16); where WK = 2, two sets of waves share out K
// and their partial sums meet in LDS at the end, added in a fixed order.  Weights are
// decoded in registers a step ahead of their MFMAs (four conversions per fragment, which
// apply the block's scale).  512 x 27648 x 5120: 130 us, 1.1 PFLOP/s (a large library product in
// bfloat16: 1.39); the matrix pipe busy on 0.60 of the cycles, waves waiting to issue on 0.39 of theirs
// (4.5 VALU per MFMA); 160 tiles on 256 CUs (512 x 5120 x 13824): 0.40 of the cycles.  More
// buffers, up to the whole LDS, gave at most 10% for single rounds and cost 20% elsewhere.
//
// In a 64-element slice of K, lane (r, h) takes the 32 elements of half h of row r: one MX
// block of W (16 code bytes, one E8M0 byte) and four 16-byte pieces of x; MFMA step q takes
// elements 8 q .. 8 q + 7 of them on both sides.  LDS layout: x rows of KS elements, 16-byte
// piece c at c ^ f(row), so that 32 rows read at one piece spread over the banks; codes and
// scale bytes in the order of the packed image, where 16 rows' pieces lie side by side.
#include <type_traits>

#include "fp4_device.h"
#include "g2l.h"
#include "internal.h"

namespace reqat {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef __bf16 v4bf __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

template <int RM_, int RN_, int WM_, int WN_, int WK_, int NBUF_> struct Cfg {
    static constexpr int RM = RM_, RN = RN_, WM = WM_, WN = WN_, WK = WK_, NBUF = NBUF_;
    static constexpr int WAVES = WM * WN * WK, THREADS = 64 * WAVES;
    static constexpr int TM = 32 * RM * WM, TN = 32 * RN * WN, KS = 64 * WK;
    static constexpr int XROW = 2 * KS, CH = XROW / 16, RPI = 1024 / XROW;   // bytes, pieces of a row; rows per load
    static constexpr int XB = TM * XROW, GB = 8 * KS, CB = TN / 16 * GB;     // x; codes of a row group, of the stage
    static constexpr int SB = TN * 4, STAGE = XB + CB + SB;
    static constexpr int XL = XB / 1024 / WAVES, BL = CB / 1024 / WAVES;     // loads per wave and stage
    static constexpr int SLT = SB / 256, SL = (SLT + WAVES - 1) / WAVES;     // (scales: some repeat the last one)
    static constexpr int LPS = XL + BL + SL;
    static constexpr int PART = WAVES * RN * 16 * 64 * 4;
    static constexpr int LDS = NBUF * STAGE > PART ? NBUF * STAGE : PART;
    static_assert(XB % (1024 * WAVES) == 0 && CB % (1024 * WAVES) == 0 && SB % 256 == 0, "whole loads");
    static_assert((KS == 64 || KS == 128) && NBUF >= 2 && NBUF * LPS <= 63, "stages of whole slices");
    static_assert(LDS <= 160 * 1024, "LDS");
    // repeats every 32 rows
    static __device__ __forceinline__ int f(int r) { return CH == 16 ? (r & 15) : ((r & 7) ^ ((r >> 3) & 1)); }
};

template <class C> struct Raw {
    uint4 x[C::RM][4], w[C::RN];
    uint32_t s[C::RN];
};

// Eight bfloat16 weights: codes 8 q .. 8 q + 7 times 2^e, rounded (the NaN byte 0xFF gives NaN).
__device__ __forceinline__ v8bf decode8(const uint4 &w, int q, uint32_t sb) {
    const float p2 = __builtin_bit_cast(float, sb << 23);
    const uint32_t c = q == 0 ? w.x : q == 1 ? w.y : q == 2 ? w.z : w.w;
    const v2bf d0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(c, p2, 0);
    const v2bf d1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(c, p2, 1);
    const v2bf d2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(c, p2, 2);
    const v2bf d3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(c, p2, 3);
    return v8bf{d0[0], d0[1], d1[0], d1[1], d2[0], d2[1], d3[0], d3[1]};
}

// Waits until at most n stages' loads are on their way (n <= MAX).
template <int MAX, int LPS> __device__ __forceinline__ void wait_stages(int n) {
    if constexpr (MAX > 0) {
        if (n < MAX) return wait_stages<MAX - 1, LPS>(n);
    }
    wait_and_meet<MAX * LPS>();
}

template <class C, bool kPacked>
__global__ __launch_bounds__(C::THREADS, C::LDS <= 80 * 1024 ? C::WAVES / 2 : C::WAVES / 4) void gemm_w4a16_tile_kernel(
    int64_t M, int64_t N, int64_t K, const uint8_t *__restrict__ x, int64_t ldx, const uint8_t *__restrict__ w_codes,
    const uint8_t *__restrict__ w_scales, void *__restrict__ y, int y_bf16, int y_vec, int64_t ldy) {
    constexpr int RM = C::RM, RN = C::RN, WM = C::WM, WN = C::WN, WK = C::WK, NBUF = C::NBUF;
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave / (WM * WN), wm = wave / WN % WM, wn = wave % WN;

    // Tile of this workgroup: each XCD (workgroups are dealt to the eight in turn) takes a
    // contiguous run of tiles, M fastest: neighbours share rows of W in their L2.
    const int64_t tm_n = (M + C::TM - 1) / C::TM, tn_n = (N + C::TN - 1) / C::TN, T = tm_n * tn_n;
    const int64_t xcd = blockIdx.x % 8, local = blockIdx.x / 8, per = T / 8, rem = T % 8;
    const int64_t t = xcd * per + (xcd < rem ? xcd : rem) + local;
    constexpr int GROUP_M = 1024 / C::TM;
    const int64_t width = GROUP_M * tn_n, first_m = (t / width) * GROUP_M;
    const int64_t gsz = (tm_n - first_m) < GROUP_M ? (tm_n - first_m) : GROUP_M;
    const int64_t m0 = (first_m + (t % width) % gsz) * C::TM, n0 = ((t % width) / gsz) * C::TN;

    // This wave's loads: offsets of the lane's bytes in stage 0 (rows past the edge re-read the last one)
    const int left_m = (int)(M - m0 < C::TM ? M - m0 : C::TM) - 1, left_n = (int)(N - n0 < C::TN ? N - n0 : C::TN) - 1;
    const int left_g = left_n >> 4;
    const int64_t nch = K / 128;                            // units of 16 rows x 128 elements
    const uint8_t *xb = x + m0 * ldx * 2;
    const uint8_t *wb = kPacked ? w_codes + (n0 >> 4) * nch * 1024 : w_codes + n0 * (K / 2);
    const uint8_t *sb = kPacked ? w_scales + (n0 >> 4) * nch * 64 : w_scales + n0 * (K / 32);
    uint32_t xoff[C::XL], woff[C::BL], soff[C::SL];
#pragma unroll
    for (int i = 0; i < C::XL; ++i) {
        const int row = (wave * C::XL + i) * C::RPI + lane / C::CH;
        xoff[i] = (uint32_t)(row < left_m ? row : left_m) * (uint32_t)(ldx * 2) + ((lane % C::CH) ^ C::f(row)) * 16;
    }
#pragma unroll
    for (int i = 0; i < C::BL; ++i) {
        // 16-byte piece l of the row group's (32 or 64): row l % 16, MX block l / 16 of the stage
        const int b = (wave * C::BL + i) * 1024 + lane * 16, g = b / C::GB, l = b % C::GB / 16;
        const int row = 16 * g + l % 16;
        woff[i] = kPacked ? (uint32_t)(g < left_g ? g : left_g) * (uint32_t)(nch * 1024) + l * 16
                          : (uint32_t)(row < left_n ? row : left_n) * (uint32_t)(K / 2) + l / 16 * 16;
    }
#pragma unroll
    for (int i = 0; i < C::SL; ++i) {
        const int p = wave * C::SL + i, row = (p < C::SLT ? p : C::SLT - 1) * 64 + lane, g = row / 16;
        soff[i] = kPacked ? (uint32_t)(g < left_g ? g : left_g) * (uint32_t)(nch * 64) + row % 16 * 4
                          : (uint32_t)(row < left_n ? row : left_n) * (uint32_t)(K / 32);
    }
    // Load L of this wave's share of stage s
    auto load_one = [&](int s, int buf, auto LL) {
        constexpr int L = decltype(LL)::value;
        uint8_t *st = smem + buf * C::STAGE;
        if constexpr (L < C::XL) {
            g2l16(xb + (int64_t)s * C::XROW, xoff[L], st + (wave * C::XL + L) * 1024);
        } else if constexpr (L < C::XL + C::BL) {
            constexpr int i = L - C::XL;
            const int64_t at = kPacked ? (int64_t)s * C::GB : (int64_t)s * (C::KS / 2);
            g2l16(wb + at, woff[i], st + C::XB + (wave * C::BL + i) * 1024);
        } else {
            constexpr int i = L - C::XL - C::BL;
            const int p = wave * C::SL + i, u = s * C::KS / 128;
            g2l4(sb + (int64_t)u * (kPacked ? 64 : 4), soff[i],
                 st + C::XB + C::CB + (p < C::SLT ? p : C::SLT - 1) * 256);
        }
    };

    // Reads of the wave's 64 elements of stage s, in the order of use: W, then x by MFMA step
    const int lr = lane & 31, h = lane >> 5;
    constexpr int READS = RN + 4 * RM;
    auto read_one = [&](Raw<C> &r, int s, int buf, auto TT) {
        constexpr int t = decltype(TT)::value;
        const uint8_t *st = smem + buf * C::STAGE;
        if constexpr (t < RN) {
            const int row = (wn * RN + t) * 32 + lr, blk = 2 * wk + h;          // MX block of the stage
            r.w[t] = *reinterpret_cast<const uint4 *>(st + C::XB + (row >> 4) * C::GB + 256 * blk + 16 * (row & 15));
            r.s[t] = st[C::XB + C::CB + row * 4 + ((C::KS == 64 ? 2 * (s & 1) : 0) + blk)];
        } else {
            constexpr int q = (t - RN) / RM, i = (t - RN) % RM;
            const int row = (wm * RM + i) * 32 + lr;
            r.x[i][q] = *reinterpret_cast<const uint4 *>(st + row * C::XROW + (((8 * wk + 4 * h + q) ^ C::f(lr)) << 4));
        }
    };

    v16f acc[RM][RN];
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
        for (int j = 0; j < RN; ++j) acc[i][j] = v16f{};

    const int nst = (int)(K / C::KS);                       // K % 128 == 0
    static_for<0, NBUF>([&](auto S) {
        constexpr int s = decltype(S)::value;
        if (s < nst) static_for<0, C::LPS>([&](auto L) { load_one(s, s, L); });
    });
    wait_stages<NBUF - 1, C::LPS>(nst - 1);
    Raw<C> raw[2];
    static_for<0, READS>([&](auto T) { read_one(raw[0], 0, 0, T); });

    // Stage s, its operands in raw[P]: the waves meet once stage s + 1 has landed for all and all have
    // read stage s; then its reads into raw[P ^ 1], the loads of stage s + NBUF into the buffer that
    // stage s leaves, and the decode of the next step go out between the MFMAs.
    int buf = 0;                                            // s % NBUF
    v8bf dec[2][RN];
    static_for<0, RN>([&](auto J) {
        constexpr int j = decltype(J)::value;
        dec[0][j] = decode8(raw[0].w[j], 0, raw[0].s[j]);
    });
    auto stage = [&](int s, auto PP, auto STEADY) __attribute__((always_inline)) {
        constexpr int P = decltype(PP)::value;
        constexpr bool steady = decltype(STEADY)::value;    // s + NBUF < nst
        const int nbuf = buf + 1 == NBUF ? 0 : buf + 1;
        if constexpr (steady) {
            wait_and_meet<(NBUF - 2) * C::LPS>();
        } else if (s + 1 < nst) {
            wait_stages<NBUF - 2, C::LPS>(nst - 2 - s);     // the stages after s + 1
            static_for<0, READS>([&](auto T) { read_one(raw[P ^ 1], s + 1, nbuf, T); });
            if (s + NBUF < nst) static_for<0, C::LPS>([&](auto L) { load_one(s + NBUF, buf, L); });
        } else {
            __builtin_amdgcn_s_waitcnt(0xC07F);
        }
        // parts of RN MFMAs; the reads go out with the first three steps (the fourth decodes from them)
        constexpr int PARTS = 4 * RM, RPARTS = 3 * RM;
        static_for<0, PARTS>([&](auto TT) {
            constexpr int part = decltype(TT)::value, q = part / RM, i = part % RM, E = q & 1;
            constexpr int r0 = part < RPARTS ? part * READS / RPARTS : READS;
            constexpr int r1 = part < RPARTS ? (part + 1) * READS / RPARTS : READS;
            constexpr int l0 = part * C::LPS / PARTS, l1 = (part + 1) * C::LPS / PARTS;
            constexpr int f0 = i * RN / RM, f1 = (i + 1) * RN / RM;     // next step's W fragments
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (steady) {
                static_for<r0, r1>([&](auto T) { read_one(raw[P ^ 1], s + 1, nbuf, T); });
                static_for<l0, l1>([&](auto L) { load_one(s + NBUF, buf, L); });
            }
#pragma unroll
            for (int j = 0; j < RN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, raw[P].x[i][q]), dec[E][j],
                                                                    acc[i][j], 0, 0, 0);
            static_for<f0, f1>([&](auto F) {
                constexpr int j = decltype(F)::value;
                dec[E ^ 1][j] = q == 3 ? decode8(raw[P ^ 1].w[j], 0, raw[P ^ 1].s[j])
                                       : decode8(raw[P].w[j], (q + 1) & 3, raw[P].s[j]);
            });
            static_for<0, RN>([&](auto) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                        // one MFMA
                __builtin_amdgcn_sched_group_barrier(0x002, (6 * (f1 - f0) + RN - 1) / RN, 0);   // its share of the decode
            });
        });
        __builtin_amdgcn_sched_barrier(0);
        buf = nbuf;
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    int s = 0;
    for (; s + 1 + NBUF < nst; s += 2) {
        stage(s, I0{}, std::true_type{});
        stage(s + 1, I1{}, std::true_type{});
    }
    for (; s < nst; s += 2) {
        stage(s, I0{}, std::false_type{});
        if (s + 1 < nst) stage(s + 1, I1{}, std::false_type{});
    }

    // Results, one row of MFMA tiles per wave at a time, through LDS: partial sums are added in
    // the order of the waves and rows leave in 8- or 16-byte pieces.  part[wave][j][register][lane];
    // D[m][n] of a 32 x 32 tile sits in lane n + 32 ((m / 4) % 2), register 4 (m / 8) + m % 4.
    float *part = reinterpret_cast<float *>(smem);
#pragma unroll
    for (int i = 0; i < RM; ++i) {
        __syncthreads();
#pragma unroll
        for (int j = 0; j < RN; ++j)
#pragma unroll
            for (int k = 0; k < 16; ++k) part[((wave * RN + j) * 16 + k) * 64 + lane] = acc[i][j][k];
        __syncthreads();
        constexpr int QUADS = WM * WN * RN * 256;           // of four consecutive columns of one row
        static_assert(QUADS % C::THREADS == 0, "whole rounds");
#pragma unroll
        for (int q0 = 0; q0 < QUADS; q0 += C::THREADS) {
            const int q = q0 + tid;
            const int l = (q & 15) * 4, k = (q >> 4) & 15, jj = q >> 8;
            v4f v = *reinterpret_cast<const v4f *>(part + q * 4);
#pragma unroll
            for (int w = 1; w < WK; ++w) v += *reinterpret_cast<const v4f *>(part + (w * QUADS + q) * 4);
            const int64_t m = m0 + 32 * (RM * (jj / RN / WN) + i) + 8 * (k >> 2) + 4 * (l >> 5) + (k & 3);
            const int64_t n = n0 + 32 * (jj % (RN * WN)) + (l & 31);
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

template <class C>
hipError_t launch_cfg(int64_t M, int64_t N, int64_t K, const uint16_t *x, int64_t ldx, const uint8_t *w_codes,
                      const uint8_t *w_scales, bool packed, void *y, bool y_bf16, int64_t ldy, hipStream_t stream) {
    const int64_t grid = ((M + C::TM - 1) / C::TM) * ((N + C::TN - 1) / C::TN);
    const int64_t es = y_bf16 ? 2 : 4;
    const int y_vec = reinterpret_cast<uintptr_t>(y) % (4 * es) == 0 && ldy % 4 == 0;
    auto go = [&](auto kernel) {
        hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(C::THREADS), C::LDS, stream, M, N, K,
                           reinterpret_cast<const uint8_t *>(x), ldx, w_codes, w_scales, y, (int)y_bf16, y_vec, ldy);
        return hipGetLastError();
    };
    return packed ? go(gemm_w4a16_tile_kernel<C, true>) : go(gemm_w4a16_tile_kernel<C, false>);
}

}  // namespace

hipError_t launch_gemm_w4a16_tile(W16Tile tile, int64_t M, int64_t N, int64_t K, const uint16_t *x, int64_t ldx,
                                  const uint8_t *w_codes, const uint8_t *w_scales, bool packed, void *y, bool y_bf16,
                                  int64_t ldy, hipStream_t stream) {
    auto cfg = [&](auto c) {
        return launch_cfg<decltype(c)>(M, N, K, x, ldx, w_codes, w_scales, packed, y, y_bf16, ldy, stream);
    };
    // row offsets within a tile are 32-bit (128 rows of 2 ldx bytes)
    if (M <= 0 || N <= 0 || K <= 0 || K % 128 || K > kW16TileMaxLd || ldx > kW16TileMaxLd) return hipErrorInvalidValue;
    switch (tile) {
    case kW16Tile64x64: return cfg(Cfg<1, 2, 2, 1, 2, 3>{});
    case kW16Tile64x128: return cfg(Cfg<2, 2, 1, 2, 2, 3>{});
    case kW16Tile128x128: return cfg(Cfg<2, 2, 2, 2, 1, 3>{});
    default: return cfg(Cfg<2, 2, 2, 2, 2, 3>{});
    }
}

}  // namespace reqat
