// omc_dequant_gemm / omc_dequant_gemm_dx on codes of any width B (2 .. 16 bits; S1E4M3 with bias 7 has a kernel of its own).
//
// C[M x N] = A[M x K] * (s W + b), W packed as [K x N] (forward) or [N x K] (TRANS).  Steps of 64 k, two LDS stages.  A goes from
// global memory straight into LDS as rows of 128 bytes (16-byte pieces XOR-swizzled by half the row: 64 banks hold two rows).  W passes through
// registers: a thread takes 32 consecutive codes = B whole dwords, so that every shift is a compile-time constant,
// decodes them in the bit domain and stores 32 bfloat16 values: forward as a part of a k row [k][BN] that the transposing
// 16-bit read turns into fragments, TRANS as half of a column's 64 k, laid out like A.  Each code is decoded once per
// workgroup, during the products of the step before; its dwords were asked for two steps before.
//
// Forward W rows: the 64 bytes of a unit go to group g ^ f(k) of the row, f = (k & 3) + 4 * (bit 3 of k) as far as the row has
// groups, and its four pieces are rotated by g / 2: the eight k rows of a transposing read and the eight lanes of a store then
// lie on different banks.  (No conflict is counted forward; TRANS 2.1 - 4.2 million cycles over all compute units in a launch of 84 - 91 us.)
//
// What bounds it: the decode, about five vector instructions per code, beside 64 KB through LDS per 16 k of a 256 x 256 tile.  Measured on 11-bit codes against the kernels before (256 x 128 or 128 x 128 tile,
// A staged through registers, a patch of 4 x 4 codes per thread with run-time shifts; 256 x 128 by 16 waves for long contractions):
// forward 8192 x 4096 x 1024 104 -> 82 us, 2048 x 2048 x 512 18.6 -> 11.4, input gradient 2048 x 512 x 2048 53.6 -> 13.
#pragma once
#include <algorithm>

#include "omc_mma.h"

#pragma clang fp contract(off)

namespace omc {

struct BitsArgs {
    const uint16_t *A;
    const uint32_t *codes;
    const float *sb;
    float *C;
    uint32_t N, K, tiles_m, tiles_n;
    FmtParams fp;
};

// U consecutive codes (U = 32 or 16) as dwords.  Sixteen codes of an odd width start in the middle of a dword every other time;
// their dwords never reach past those of the 32 codes they belong to.
template <int B, int U>
struct Unit {
    static constexpr int kDwords = (U * B + 31) / 32;
    static constexpr bool kShifted = (U * B) % 32 != 0;
    uint32_t w[kDwords];
};
template <int B, int U>
__device__ __forceinline__ void load_unit(const uint32_t *__restrict__ from, Unit<B, U> &u) {
    typedef uint32_t x4 __attribute__((ext_vector_type(4), aligned(4)));
    typedef uint32_t x2 __attribute__((ext_vector_type(2), aligned(4)));
    constexpr int n = Unit<B, U>::kDwords;
    int i = 0;
#pragma unroll
    for (; i + 4 <= n; i += 4) {
        const x4 t = *reinterpret_cast<const x4 *>(from + i);
        u.w[i] = t[0]; u.w[i + 1] = t[1]; u.w[i + 2] = t[2]; u.w[i + 3] = t[3];
    }
    if constexpr ((n & 2) != 0) {
        const x2 t = *reinterpret_cast<const x2 *>(from + (n & ~3));
        u.w[n & ~3] = t[0];
        u.w[(n & ~3) + 1] = t[1];
    }
    if constexpr ((n & 1) != 0) u.w[n - 1] = from[n - 1];
}
// moves the codes of a unit that starts `shift` bits into its first dword to bit 0
template <int B, int U>
__device__ __forceinline__ void align_unit(Unit<B, U> &u, uint32_t shift) {
    if constexpr (Unit<B, U>::kShifted) {
#pragma unroll
        for (int i = 0; i < Unit<B, U>::kDwords; ++i)
            u.w[i] = __builtin_amdgcn_alignbit(i + 1 < Unit<B, U>::kDwords ? u.w[i + 1] : 0u, u.w[i], shift);
    }
}
// code i with its sign bit at bit 31 (what lies below is masked by the decoder)
template <int B, int U>
__device__ __forceinline__ uint32_t unit_code(const Unit<B, U> &u, int i) {
    const int p = i * B, idx = p >> 5, off = p & 31;
    if (off + B <= 32) return u.w[idx] << (32 - B - off);
    return __builtin_amdgcn_alignbit(u.w[idx + 1], u.w[idx], off + B - 32);
}
// codes 8 i .. 8 i + 7 of a unit as bfloat16 (their fp32 images have nothing in the low 16 bits)
template <int B, int U>
__device__ __forceinline__ u32x4 decode_piece(const Unit<B, U> &u, int i, const FmtParams &fp) {
    u32x4 o;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const uint32_t lo = __float_as_uint(decode_top(unit_code<B, U>(u, 8 * i + 2 * p), fp));
        const uint32_t hi = __float_as_uint(decode_top(unit_code<B, U>(u, 8 * i + 2 * p + 1), fp));
        o[p] = __builtin_amdgcn_perm(hi, lo, 0x07060302u);
    }
    return o;
}

// WM x WN waves of TM x TN matrix tiles (32 x 32) each, TEAMS times: team t multiplies the steps t, t + TEAMS, ... of the
// contraction in LDS stages of its own, and team 0 adds up the teams' tiles in order.  A team's sums are CHAINS chains (which of
// them, the quarter of the step decides).  OCC waves per SIMD.
template <int B, int U, int WM, int WN, int TM, int TN, int TEAMS, int CHAINS, int OCC, bool TRANS>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * WM * WN * TEAMS, 64 * WM * WN * TEAMS))) __attribute__((amdgpu_waves_per_eu(OCC, OCC)))
void gemm_bits_kernel(BitsArgs ga) {
    constexpr int NW = WM * WN, NT = 64 * NW, BM = 32 * TM * WM, BN = 32 * TN * WN;
    constexpr int kALoads = BM / 8 / NW, kUnits = 64 * BN / U, kGroups = BN / 32, kRowUnits = BN / U;
    constexpr uint32_t kABytes = BM * 128, kStage = kABytes + BN * 128;
    static_assert(WM == 2 && (WN == 2 || WN == 4), "how the quarters are dealt below");
    static_assert(BM % (8 * NW) == 0 && kUnits == NT, "whole loads, one unit per thread");
    __shared__ __attribute__((aligned(1024))) uint8_t lds_all[TEAMS * 2 * kStage];
    const uint32_t team = TEAMS == 1 ? 0u : __builtin_amdgcn_readfirstlane(threadIdx.x / NT);
    uint8_t *lds = lds_all + team * (2 * kStage);
    const uint32_t lds0 = lds_offset(lds);
    const uint32_t tid = TEAMS == 1 ? threadIdx.x : threadIdx.x % NT, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave / WN, wn = wave % WN;
    const uint32_t N = ga.N, K = ga.K;
    const FmtParams fp = ga.fp;
    uint32_t m0, n0;
    tile_of_block(BM == 256 ? 4 : 8, ga.tiles_m, ga.tiles_n, m0, n0);
    m0 *= BM;
    n0 *= BN;

    // ---- global -> LDS / registers.  The last step may be half empty (K % 64 == 32): the upper half is then the lower one again
    // instead of a read past the row, and nobody multiplies it
    const uint32_t full_k = K / 64, steps_k = (K + 63) / 64;
    const uint32_t full = (full_k + TEAMS - 1 - team) / TEAMS, steps = (steps_k + TEAMS - 1 - team) / TEAMS;   // this team's
    const uint8_t *a_base = reinterpret_cast<const uint8_t *>(ga.A) + static_cast<uint64_t>(m0) * K * 2;
    const uint32_t a_row = lane >> 3, a_piece = (lane & 7u) ^ ((a_row >> 1) + 4 * (wave & 1u));
    auto load_a = [&](uint32_t at, uint32_t i) {
        const uint32_t j = team + TEAMS * i;
        const uint32_t a_off = a_row * K * 2 + (j == full_k ? a_piece & 3u : a_piece) * 16;
#pragma unroll
        for (int q = 0; q < kALoads; ++q) {
            const uint32_t c = wave + NW * q;                 // rows 8 c ..
            load_to_lds(a_base + static_cast<uint64_t>(j) * 128 + static_cast<uint64_t>(c) * 16 * K, a_off, lds0 + at + c * 1024);
        }
    };
    // this thread's unit: TRANS column u_row, part u_part of its 64 k; forward k row u_row, part u_part of its BN columns
    constexpr uint32_t kParts = TRANS ? 64 / U : kRowUnits, kPieces = U / 8;
    const uint32_t u_row = tid / kParts, u_part = tid % kParts;
    const uint32_t u_shift = Unit<B, U>::kShifted ? 16u * (u_part & 1u) : 0u;
    auto load_w = [&](uint32_t i, Unit<B, U> &u) {
        const uint32_t j = team + TEAMS * i;
        const bool half = j == full_k;
        const uint64_t e = TRANS ? (static_cast<uint64_t>(n0 + u_row) * K + static_cast<uint64_t>(j) * 64 + U * (half ? u_part % (32 / U) : u_part))
                                 : ((static_cast<uint64_t>(j) * 64 + (half ? u_row & 31u : u_row)) * N + n0 + U * u_part);
        load_unit<B, U>(ga.codes + (e * B >> 5), u);
    };
    auto swizzle_f = [](uint32_t k) { return ((k & 3u) | ((k >> 1) & 4u)) & (kGroups - 1); };
    uint32_t u_at[kPieces];
#pragma unroll
    for (uint32_t i = 0; i < kPieces; ++i) {
        const uint32_t piece = u_part * kPieces + i, group = piece / 4;
        u_at[i] = kABytes + (TRANS ? u_row * 128 + ((piece ^ ((u_row >> 1) & 7u)) << 4)
                                   : u_row * (2 * BN) + ((group ^ swizzle_f(u_row)) * 4 + ((piece & 3u) ^ ((group >> 1) & 3u))) * 16);
    }
    auto store_piece = [&](uint32_t at, const Unit<B, U> &u, int i) {
        *reinterpret_cast<u32x4 *>(lds + at + u_at[i]) = decode_piece<B, U>(u, i, fp);
    };

    // ---- LDS -> fragments
    const uint32_t f_row = lane & 31u, f_half = lane >> 5;
    auto a_place = [&](uint32_t ks) {
        const uint32_t row = 32 * TM * wm + f_row;
        return row * 128 + (((2 * ks + f_half) ^ ((row >> 1) & 7u)) << 4);
    };
    const uint32_t block = lane >> 4, in = lane & 15u;          // forward: 16 lanes point at 4 k rows x 16 columns
    uint32_t w_base[TN];                                        // forward: quarter 0's place per column block
#pragma unroll
    for (uint32_t ni = 0; ni < TN; ++ni) {
        const uint32_t g = TN * wn + ni, k = 8 * (block >> 1) + (in >> 2), piece = 2 * (block & 1u) + ((in >> 1) & 1u);
        w_base[ni] = kABytes + k * (2 * BN) + ((g ^ swizzle_f(k)) * 4 + (piece ^ ((g >> 1) & 3u))) * 16 + 8 * (in & 1u);
    }
    auto w_place = [&](uint32_t ks) {                           // TRANS: place of column block 0; forward: step to quarter ks
        if (!TRANS) return ks * 16 * (2 * BN);
        const uint32_t col = 32 * TN * wn + f_row;
        return kABytes + col * 128 + (((2 * ks + f_half) ^ ((col >> 1) & 7u)) << 4);
    };
    uint32_t a_at[4], w_at[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const uint32_t ks = (p + wn + 2 * wm) & 3u;
        a_at[p] = a_place(ks);
        w_at[p] = w_place(ks);
    }
    struct Frags {
        bf16x8 a[TM], w[TN];
    };
    auto read_frags = [&](uint32_t at, uint32_t a_off, uint32_t w_off, Frags &f) {
#pragma unroll
        for (int mi = 0; mi < TM; ++mi) f.a[mi] = *reinterpret_cast<const bf16x8 *>(lds + at + a_off + 32 * 128 * mi);
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) {
            if (TRANS) {
                f.w[ni] = *reinterpret_cast<const bf16x8 *>(lds + at + w_off + 32 * 128 * ni);
            } else {
                typedef short s16x8 __attribute__((ext_vector_type(8)));
                uint8_t *q = lds + (at + w_off + w_base[ni]);
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((OMC_LDS s16x4 *)(q));
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((OMC_LDS s16x4 *)(q + 4 * 2 * BN));
                const s16x8 both = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                f.w[ni] = __builtin_bit_cast(bf16x8, both);
            }
        }
    };

    f32x16 acc[CHAINS][TM][TN];
    RowSums<WN, TM, CHAINS> rsum;
    auto multiply = [&](const Frags &f, auto quarter, bool sum) {
        constexpr int Q = decltype(quarter)::value, chain = Q % CHAINS;
#pragma unroll
        for (int ni = 0; ni < TN; ++ni)
#pragma unroll
            for (int mi = 0; mi < TM; ++mi)
                acc[chain][mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[mi], f.w[ni], acc[chain][mi][ni], 0, 0, 0);
        if (sum) rsum.template add<Q>(f.a);
    };

    // step i: A and W of the step are in stage `cur`; the dwords of step i + 1 are in `next` (asked for during step i - 1)
    Frags f0, f1;
    uint32_t cur = 0;
    Unit<B, U> now, next;
#pragma unroll
    for (int i = 0; i < Unit<B, U>::kDwords; ++i) next.w[i] = 0;
    auto clear = [&]() {
        clear_chains(acc);
        rsum.clear();
    };
    if (CHAINS == 1) clear();
    if (steps > 0) {
        load_a(0, 0);
        load_w(0, next);
    }
    if (CHAINS > 1) clear();                                  // (while they are on their way)
    if (steps > 0) {
        now = next;
        if (steps > 1) load_w(1, next);
        align_unit<B, U>(now, u_shift);
#pragma unroll
        for (int i = 0; i < static_cast<int>(kPieces); ++i) store_piece(0, now, i);
    }
    auto step = [&](uint32_t i, bool first, bool more1, bool more2) {
        wait_loads_and_sync<0>();
#pragma unroll
        for (int q = 0; q < Unit<B, U>::kDwords; ++q) pin(next.w[q]);   // they have arrived: their uses need no wait of their own
        now = next;
        const uint32_t other = kStage - cur;
        read_frags(cur, a_at[0], w_at[0], f0);
        if (more1) load_a(other, i + 1);
        if (more2) load_w(i + 2, next);
        if (more1) align_unit<B, U>(now, u_shift);
        if (!first) multiply(f1, UintTag<3>{}, false);
        read_frags(cur, a_at[1], w_at[1], f1);
        if (more1) store_piece(other, now, 0);
        multiply(f0, UintTag<0>{}, true);
        read_frags(cur, a_at[2], w_at[2], f0);
        if (more1) store_piece(other, now, 1);
        multiply(f1, UintTag<1>{}, false);
        read_frags(cur, a_at[3], w_at[3], f1);
        if (more1 && kPieces > 2) store_piece(other, now, 2);
        multiply(f0, UintTag<2>{}, WN == 2);
        if (more1 && kPieces > 2) store_piece(other, now, 3);
        cur = other;
    };
    if (full > 0) {
        step(0, true, steps > 1, steps > 2);
        uint32_t i = 1;
        for (; i + 2 < steps; ++i) step(i, false, true, true);
        for (; i < full; ++i) step(i, false, i + 1 < steps, i + 2 < steps);
        multiply(f1, UintTag<3>{}, false);
    }
    if (full < steps) {                                       // 32 k more: two quarters
        wait_loads_and_sync<0>();
        auto quarter = [&](auto ks) {
            read_frags(cur, a_place(ks.value), w_place(ks.value), f0);
            multiply(f0, ks, false);
            if (ks.value % WN == wn) rsum.template add<0>(f0.a);
        };
        quarter(UintTag<0>{});
        quarter(UintTag<1>{});
    }
    for (uint32_t i = steps; i < (steps_k + TEAMS - 1) / TEAMS; ++i) wait_loads_and_sync<0>();   // teams wait for each other
    wait_loads_and_sync<0>();                                 // nobody reads a stage any more
    const float s = ga.sb ? ga.sb[0] : 1.0f, b = ga.sb ? ga.sb[1] : 0.0f;
    float *rowsum = reinterpret_cast<float *>(lds_all);       // [TEAMS * WN][BM]
    join_chains(acc);
    publish_row_sums<WN, BM, TM>(rowsum, rsum.total(), ga.sb != nullptr, team, 32 * TM * wm, wn, lane);
    if (!add_teams<TEAMS, NW, TM, TN>(rowsum + TEAMS * WN * BM, acc[0], team, wave, lane)) return;
    store_tile<TEAMS * WN, BM, TM, TN>(ga.C + static_cast<uint64_t>(m0) * N + n0 + 32 * TN * wn, N, acc[0], rowsum, 32 * TM * wm, lane, s, b);
}

// 256 x 128 by four waves, one to a SIMD, each of 128 x 64, decodes a code for 256 rows and reads its fragments from LDS half as often as 128 x 256 by eight
// (9216 x 896 x 1120, input gradient, 13 bits, 28 us; 36 with 128 x 128; 8192 x 1024 x 2048 45, 50 with 128 x 256); the latter is faster forward where
// every unit has one tile and a result has few columns (15360 x 512 x 1120, 11 bits: 27 us, 32 with 256 x 128).  128 x 64 by four waves, three
// workgroups on a unit, fills the chip with half the decoding of 64 x 64 (2304 x 3712 x 192 12.6 us, 14.5 with 128 x 128; 1536 x 2944 x 704 16.4, 18.4), which
// wins on short contractions (8192 x 128 x 320, 11 bits: 5.5 us, 5.8 with 128 x 64).  8192 x 4096 x 1024: 82 us with 256 x 256, 107 with 128 x 128; 2048 x
// 512 x 2048: 50 with 256 x 256, 27 with 128 x 128, 14 / 13 with 64 x 64 and 2 / 4 teams.
// Fitted to 1532 sizes in 6, 8, 11 and 13 bits.  On 1180 others the chosen tile takes 0.6 % longer than the best one on average, more than 7 % longer on 33 of
// them, at worst 29 % (13056 x 256 x 3744, 11 bits, input gradient: 72 us with 128 x 128, 56 with 128 x 64); in 4 and 16 bits, which are not in the fit, 0.8 and 0.9 %, at
// worst 15 and 27 % (120 sizes each); on 90 with K = 32 - 96, smaller than any in the fit, 1.4 %, at worst 9 %.
static constexpr GemmTile kBitsTiles[] = {
    {256, 256, 1, 1, 1, 2.271, 1.395, 1.354, 11.2, 0.065}, {256, 128, 1, 1, 1, 2.589, 0.728, 1.008, 5.458, 0.082},
    {128, 256, 1, 1, 1, 2.2, 0.561, 1.087, 4.948, 0.057}, {128, 128, 1, 2, 2, 3.136, 0.679, 0.572, 1.55, 0.051},
    {128, 64, 1, 1, 3, 3.229, 0.578, 0.346, 0.638, 0.075}, {64, 64, 1, 2, 4, 2.533, 0.549, 0.281, 0.235, 0.099},
    {64, 64, 2, 2, 2, 2.397, 0.715, 0.462, 0.732, 0.088}, {64, 64, 4, 1, 1, 3.275, 0.993, 0.881, 0.934, 0.088},
};
static constexpr double kBitsUneven = 1.0;

// Chains of fp32 sums that a contraction is dealt into, by the result's 64 x 64 tiles and the steps: at least as many as it was dealt into when the
// choice fell on two or four teams for more of the small products (11 bits, 5888 x 256 x 192: 2.7e-8 off 64 bits in two chains, 3.1e-8 in one).  The
// second chain of 128 x 128 does not fit 128 registers: that kernel has a compute unit to itself, which costs nothing, as results that
// want two chains have at most 192 of these tiles.
inline uint32_t bits_chains(uint32_t M, uint32_t N, uint32_t K) {
    const uint64_t small_tiles = static_cast<uint64_t>(M / 64) * (N / 64), steps = (static_cast<uint64_t>(K) + 63) / 64;
    if (steps >= 3 && small_tiles <= std::min<uint64_t>(256, 16 + 9 * steps)) return 4;
    return small_tiles <= (steps > 40 ? 768 : steps <= 3 ? 400 : std::min<uint64_t>(512, 428 + 6 * steps)) ? 2 : 1;
}
inline int gemm_bits_tile(uint32_t M, uint32_t N, uint32_t K) { return pick_tile(kBitsTiles, kBitsUneven, M, N, K, bits_chains(M, N, K)); }
inline uint32_t gemm_bits_sums(uint32_t M, uint32_t N, uint32_t K) {
    const int which = gemm_bits_tile(M, N, K);
    return which < 0 ? 0 : kBitsTiles[which].teams * chains_per_team(kBitsTiles[which], bits_chains(M, N, K));
}

template <int B, int WN, int U, int TM, int TN, int TEAMS, int CHAINS, int OCC, bool TRANS>
inline void launch_bits_one(const BitsArgs &ga, hipStream_t st) {
    gemm_bits_kernel<B, U, 2, WN, TM, TN, TEAMS, CHAINS, OCC, TRANS><<<dim3(ga.tiles_m * ga.tiles_n), dim3(128 * WN * TEAMS), 0, st>>>(ga);
}
template <int B, bool TRANS>
inline int launch_bits_tile(int which, uint32_t chains, const BitsArgs &ga, hipStream_t st) {
    switch (which) {
        case 0: launch_bits_one<B, 4, 32, 4, 2, 1, 1, 2, TRANS>(ga, st); break;
        case 1: launch_bits_one<B, 2, 32, 4, 2, 1, 1, 1, TRANS>(ga, st); break;
        case 2: launch_bits_one<B, 4, 32, 2, 2, 1, 1, 2, TRANS>(ga, st); break;
        case 3:
            if (chains == 2) launch_bits_one<B, 4, 16, 2, 1, 1, 2, 2, TRANS>(ga, st);
            else launch_bits_one<B, 4, 16, 2, 1, 1, 1, 4, TRANS>(ga, st);
            break;
        case 4: launch_bits_one<B, 2, 16, 2, 1, 1, 1, 3, TRANS>(ga, st); break;
        case 5:
            if (chains == 2) launch_bits_one<B, 2, 16, 1, 1, 1, 2, 4, TRANS>(ga, st);
            else launch_bits_one<B, 2, 16, 1, 1, 1, 1, 4, TRANS>(ga, st);
            break;
        case 6:
            if (chains == 2) launch_bits_one<B, 2, 16, 1, 1, 2, 2, 4, TRANS>(ga, st);
            else launch_bits_one<B, 2, 16, 1, 1, 2, 1, 4, TRANS>(ga, st);
            break;
        case 7: launch_bits_one<B, 2, 16, 1, 1, 4, 1, 4, TRANS>(ga, st); break;
        default: return static_cast<int>(hipErrorInvalidValue);
    }
    return static_cast<int>(hipGetLastError());
}
template <int B>
inline int launch_bits(const BitsArgs &args, uint32_t M, int trans, hipStream_t st) {
    const int which = gemm_bits_tile(M, args.N, args.K);
    if (which < 0) return static_cast<int>(hipErrorInvalidValue);
    BitsArgs ga = args;
    ga.tiles_m = M / kBitsTiles[which].bm;
    ga.tiles_n = args.N / kBitsTiles[which].bn;
    const uint32_t chains = chains_per_team(kBitsTiles[which], bits_chains(M, args.N, args.K));
    return trans ? launch_bits_tile<B, true>(which, chains, ga, st) : launch_bits_tile<B, false>(which, chains, ga, st);
}

// one translation unit per range of widths
int launch_gemm_bits_2_5(const BitsArgs &ga, uint32_t M, int trans, hipStream_t st);
int launch_gemm_bits_6_8(const BitsArgs &ga, uint32_t M, int trans, hipStream_t st);
int launch_gemm_bits_9_11(const BitsArgs &ga, uint32_t M, int trans, hipStream_t st);
int launch_gemm_bits_12_14(const BitsArgs &ga, uint32_t M, int trans, hipStream_t st);
int launch_gemm_bits_15_16(const BitsArgs &ga, uint32_t M, int trans, hipStream_t st);

}  // namespace omc
