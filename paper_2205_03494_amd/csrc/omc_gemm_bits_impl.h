// omc_dequant_gemm / omc_dequant_gemm_dx on codes of any width B (2 .. 16 bits; S1E4M3 with bias 7 has a kernel of its own).
//
// C[M x N] = A[M x K] * (s W + b), W packed as [K x N] (forward) or [N x K] (TRANS).  Steps of 64 k, two LDS stages.  A goes from
// global memory straight into LDS as rows of 128 bytes (16-byte pieces XOR-swizzled by half the row: 64 banks hold two rows).  W passes through
// registers: a thread takes 32 consecutive codes = B whole dwords, so that every shift is a compile-time constant,
// decodes them in the bit domain and stores 32 bfloat16 values: forward as a part of a k row [k][BN] that the transposing
// 16-bit read turns into fragments, TRANS as half of a column's 64 k, laid out like A.  Each code is decoded once per
// workgroup, during the products of the step before; its dwords were asked for two steps before.
//
// Forward W rows: a row's 64-byte groups are exchanged by the lowest bits of k, so that four rows of one group lie on different banks, and the 16-byte pieces in a group by bit 3 of k, so that
// the eight rows that a transposing read takes at a time do, and by the group, so that the eight lanes of a store do.
//
// The order of the instructions is written down, a column of matrix tiles at a time, as in the FP8 kernel; vector and scalar arithmetic may move, and the decoding of a step's codes is spread evenly over its
// columns.  11 bits, us, 32 x 32 x 16 instructions and the compiler's order -> this: 2048 x 2048 x 512 10.9 -> 10.2, 2304 x 3712 x 192 12.5 -> 11.3, 4096 x 1024 x 1056 17.2 -> 16.6, 512 x 512 x 512 5.73 -> 5.49.  The tiles of 256
// rows are faster the old way and have a kernel of their own (omc_gemm_bits_large.h).
//
// What bounds it: the decode, about five vector instructions per code, which hold up the matrix cores by some 3 clocks each (64 x 128 x 32 by 32 matrix instructions, 64 vector instructions beside
// them: 512 -> 703 clocks).  Measured on 11-bit codes against the first kernels (256 x 128 or 128 x 128 tile,
// A staged through registers, a patch of 4 x 4 codes per thread with run-time shifts; 256 x 128 by 16 waves for long contractions):
// forward 8192 x 4096 x 1024 104 -> 80 us, 2048 x 2048 x 512 18.6 -> 10.2, input gradient 2048 x 512 x 2048 53.6 -> 13.
#pragma once
#include <algorithm>

#include "omc_gemm_bits_codes.h"
#include "omc_gemm_bits_large.h"

#pragma clang fp contract(off)

namespace omc {

// WM x WN waves of TM x TN matrix tiles (16 x 16) each, TEAMS times: team t multiplies the steps t, t + TEAMS, ... of the
// contraction in LDS stages of its own, and team 0 adds up the teams' tiles in order.  A team's sums are CHAINS chains (which of
// them, the half of the step decides).  OCC waves per SIMD.
template <int B, int U, int WM, int WN, int TM, int TN, int TEAMS, int CHAINS, int OCC, bool TRANS, bool HW>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * WM * WN * TEAMS, 64 * WM * WN * TEAMS))) __attribute__((amdgpu_waves_per_eu(OCC, OCC)))
void gemm_bits_kernel(BitsArgs ga) {
    constexpr int NW = WM * WN, NT = 64 * NW, BM = 16 * TM * WM, BN = 16 * TN * WN;
    constexpr int kALoads = BM / 8 / NW, kUnits = 64 * BN / U, kGroups = BN / 32, kRowUnits = BN / U;
    constexpr uint32_t kABytes = BM * 128, kStage = kABytes + BN * 128;
    static_assert(WM == 2 && (WN == 2 || WN == 4), "how the row sums are dealt below");
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
    tile_of_block(8, ga.tiles_m, ga.tiles_n, m0, n0);
    m0 *= BM;
    n0 *= BN;

    // ---- global -> LDS / registers.  The last step may be half empty (K % 64 == 32): the upper half is then the lower one again
    // instead of a read past the row, and nobody multiplies it
    const uint32_t full_k = K / 64, steps_k = (K + 63) / 64;
    const uint32_t full = (full_k + TEAMS - 1 - team) / TEAMS, steps = (steps_k + TEAMS - 1 - team) / TEAMS;   // this team's
    const uint8_t *a_base = reinterpret_cast<const uint8_t *>(ga.A) + static_cast<uint64_t>(m0) * K * 2;
    const uint32_t a_row = lane >> 3, a_piece = (lane & 7u) ^ ((a_row >> 1) + 4 * (wave & 1u));
    const uint8_t *a_from = a_base + static_cast<uint64_t>(8 * wave) * 2 * K + 128 * team;   // of the step that is asked for next
    const uint64_t a_stride = 16ull * NW * K;                 // between a wave's kilobytes
    auto load_a = [&](uint32_t at, uint32_t i) {
        const uint32_t a_off = a_row * K * 2 + (team + TEAMS * i == full_k ? a_piece & 3u : a_piece) * 16;
#pragma unroll
        for (int q = 0; q < kALoads; ++q) load_to_lds(a_from + q * a_stride, a_off, lds0 + at + (wave + NW * q) * 1024);
        a_from += 128 * TEAMS;
    };
    // this thread's unit: TRANS column u_row, part u_part of its 64 k; forward k row u_row, part u_part of its BN columns
    constexpr uint32_t kUnitParts = TRANS ? 64 / U : kRowUnits, kPieces = U / 8;
    const uint32_t u_row = tid / kUnitParts, u_part = tid % kUnitParts;
    const uint32_t u_shift = Unit<B, U>::kShifted ? 16u * (u_part & 1u) : 0u;
    const uint64_t first_code = TRANS ? static_cast<uint64_t>(n0 + u_row) * K + 64 * team + U * u_part : (64ull * team + u_row) * N + n0 + U * u_part;
    const uint32_t *w_from = ga.codes + (first_code * B >> 5);   // of the step that is asked for next
    const uint64_t w_step = TRANS ? 2ull * B * TEAMS : 2ull * B * TEAMS * N;   // (64 codes or rows of them are whole dwords)
    auto load_w = [&](uint32_t i, Unit<B, U> &u) {
        const bool back = team + TEAMS * i == full_k && (TRANS ? u_part >= 32 / U : u_row >= 32);
        load_unit<B, U>(back ? w_from - (TRANS ? B : static_cast<uint64_t>(B) * N) : w_from, u);
        w_from += w_step;
    };
    // forward: where piece `piece` (16 bytes, of the whole row) of k row `k` lies
    auto w_row_place = [](uint32_t k, uint32_t piece) {
        const uint32_t group = piece / 4, other_group = kGroups >= 4 ? k & 3u : (k >> 1) & 1u;
        return kABytes + k * (2 * BN) + ((group ^ other_group) * 4 + ((piece & 3u) ^ ((k >> 2) & 2u) ^ (group & 1u) ^ ((group >> 1) & 2u))) * 16;
    };
    // where its first piece goes; the others lie beside it, before the swizzle
    const uint32_t u_at = TRANS ? kABytes + u_row * 128 + (((u_part * kPieces) ^ ((u_row >> 1) & 7u)) << 4) : w_row_place(u_row, u_part * kPieces);
    auto store_piece = [&](uint32_t at, uint32_t i, u32x4 piece) { *reinterpret_cast<u32x4 *>(lds + at + (u_at ^ (16u * i))) = piece; };

    // ---- LDS -> fragments of 32 k
    const uint32_t f_row = lane & 15u, f_k = lane >> 4;
    typedef RowOrder<WN, TM> Order;
    const Order order(wn);
    auto a_place = [&](uint32_t half) {
        const uint32_t row = 16 * TM * wm + f_row;            // (of the wave's first row tile, which need not be the one it multiplies first)
        return row * 128 + (((4 * half + f_k) ^ ((row >> 1) & 7u)) << 4);
    };
    // A step's products in parts, two to a half: its first and its last TM / 2 row tiles, column by column of the tiles.  A's fragments of a part are read
    // beside the products of the part before, those of the first part behind the step's barrier, and W's of a half each as soon as its predecessor has been multiplied
    // for the last time.
    constexpr int kRows = TM / 2, kParts = 2;
    static_assert(Order::kSlots % kRows == 0, "the rows of a part follow each other");
    uint32_t a_part[kParts];                                    // where the parts' rows begin
#pragma unroll
    for (uint32_t q = 0; q < kParts; ++q) a_part[q] = 128 * order.row(q * kRows);
    uint32_t w_first[TN / 2];                                   // forward: the first half's place per two column tiles; 16 lanes point at 4 k rows x 16 columns
#pragma unroll
    for (uint32_t n2 = 0; n2 < TN / 2; ++n2) w_first[n2] = w_row_place(8 * f_k + (f_row >> 2), 2 * (TN * wn + 2 * n2) + ((f_row >> 1) & 1u)) + 8 * (f_row & 1u);
    auto w_place = [&](uint32_t half) {                         // TRANS: place of column tile 0; forward: step to the half
        if (!TRANS) return half * 32 * (2 * BN);
        const uint32_t col = 16 * TN * wn + f_row;
        return kABytes + col * 128 + (((4 * half + f_k) ^ ((col >> 1) & 7u)) << 4);
    };
    uint32_t a_at[2], w_at[2];                                  // of the half that is multiplied first, and the other one
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        a_at[p] = a_place((p + wn) & 1u);
        w_at[p] = w_place((p + wn) & 1u);
    }
    bf16x8 fa[2][kRows], fw[TN];
    uint32_t cur = 0;
    auto read_a = [&](uint32_t a_off, auto part, auto index) {
        constexpr int P = decltype(part)::value, I = decltype(index)::value;
        fa[P % 2][I] = *reinterpret_cast<const bf16x8 *>(lds + cur + a_off + a_part[P % kParts] + 16 * 128 * I);
    };
    auto read_w = [&](uint32_t w_off, auto index) {
        constexpr int ni = decltype(index)::value;
        if (TRANS) {
            fw[ni] = *reinterpret_cast<const bf16x8 *>(lds + cur + w_off + 16 * 128 * ni);
        } else {
            typedef short s16x8 __attribute__((ext_vector_type(8)));
            uint8_t *q = lds + (cur + w_off + (w_first[ni / 2] ^ (32u * (ni & 1))));   // (the second of two: two pieces on, before the swizzle)
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((OMC_LDS s16x4 *)(q));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((OMC_LDS s16x4 *)(q + 4 * 2 * BN));
            const s16x8 both = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            fw[ni] = __builtin_bit_cast(bf16x8, both);
        }
    };

    Sums<CHAINS, TM, TN> acc;
    RowSums<WN, TM, true> rsum;
    Unit<B, U> next;
    Pairs<B, U, HW> now;
    // NEXT: the part whose fragments are read meanwhile, or kAll; PAIRS: of the unit's pairs of codes those from FIRST on are decoded meanwhile, and whole pieces stored in the other stage
    constexpr int kAll = 2 * kParts, kPairs = U / 2;
    u32x4 piece = {0, 0, 0, 0};
    auto multiply = [&](auto part, auto odd, auto next_part, auto first_pair, auto pairs) {
        constexpr int P = decltype(part)::value, NEXT = decltype(next_part)::value, HALF = P / kParts, chain = HALF % CHAINS;
        constexpr int FIRST = decltype(first_pair)::value, PAIRS = decltype(pairs)::value, R = (P % kParts) * kRows;
        for_constants<TN>([&](auto group) {
            constexpr int G = decltype(group)::value, R0 = G * kRows / TN, R1 = (G + 1) * kRows / TN, D0 = FIRST + G * PAIRS / TN, D1 = FIRST + (G + 1) * PAIRS / TN;
            if constexpr (NEXT < kAll) for_constants<R1 - R0>([&](auto i) { read_a(a_at[NEXT / kParts], next_part, UintTag<R0 + decltype(i)::value>{}); });
#pragma unroll
            for (int mi = 0; mi < kRows; ++mi)
                acc[chain][R + mi][G] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[P % 2][mi], fw[G], acc[chain][R + mi][G], 0, 0, 0);
            for_constants<R1 - R0>([&](auto i) { rsum.template add<R + R0 + decltype(i)::value, HALF, decltype(odd)::value>(fa[P % 2][R0 + decltype(i)::value]); });
            if constexpr (NEXT < kAll && NEXT % kParts == 0) read_w(w_at[NEXT / kParts], group);
            for_constants<D1 - D0>([&](auto i) {
                constexpr int pair = D0 + decltype(i)::value;
                piece[pair % 4] = now.pair(pair, fp);
                if constexpr (pair % 4 == 3) store_piece(kStage - cur, pair / 4, piece);
            });
            __builtin_amdgcn_sched_barrier(0x6);              // the columns keep their order, but for vector and scalar arithmetic
        });
    };

    // step i: A and W of the step are in stage `cur`, the dwords of step i + 1 in `next` (asked for during step i - 1)
    auto clear = [&]() {
        clear_chains<CHAINS, TM, TN>(acc);
        rsum.clear();
    };
#pragma unroll
    for (int i = 0; i < Unit<B, U>::kDwords; ++i) next.w[i] = 0;
    if (CHAINS == 1) clear();
    if (steps > 0) {
        load_a(0, 0);
        load_w(0, next);
    }
    if (CHAINS > 1) clear();                                  // (while they are on their way)
    if (steps > 0) {
        now.take(next, u_shift);
        if (steps > 1) load_w(1, next);
#pragma unroll
        for (int i = 0; i < static_cast<int>(kPieces); ++i) {
#pragma unroll
            for (int p = 0; p < 4; ++p) piece[p] = now.pair(4 * i + p, fp);
            store_piece(0, i, piece);
        }
    }
    const UintTag<0> p0;
    const UintTag<kAll - 1> last;
    const UintTag<kAll> nothing;
    // the step's decoding is spread evenly over its parts, of which the one before its own first comes first
    auto pairs_before = [](int place) { return place * kPairs / kAll; };
    // `odd`: the step's number, or what passes for it at the ends
    auto step = [&](uint32_t i, auto first, auto more1, bool more2, auto odd) {
        constexpr bool FIRST = decltype(first)::value, MORE = decltype(more1)::value;
        wait_loads_and_sync<0>();
#pragma unroll
        for (int q = 0; q < Unit<B, U>::kDwords; ++q) pin(next.w[q]);   // they have arrived: their uses need no wait of their own
        if constexpr (MORE) now.take(next, u_shift);
        if constexpr (MORE) load_a(kStage - cur, i + 1);
        if (more2) load_w(i + 2, next);
        constexpr int kBegin = FIRST ? 0 : pairs_before(1);   // (the first step has no part before its own)
        if constexpr (FIRST) {
            for_constants<TN>([&](auto n) { read_w(w_at[0], n); });
            for_constants<kRows>([&](auto n) { read_a(a_at[0], p0, n); });
        } else {
            multiply(last, BoolTag<!decltype(odd)::value>{}, p0, p0, UintTag<MORE ? kBegin : 0>{});
        }
        for_constants<kAll - 1>([&](auto part) {
            constexpr int P = decltype(part)::value, D0 = P == 0 ? kBegin : pairs_before(P + 1), D1 = pairs_before(P + 2);
            multiply(part, odd, UintTag<P + 1>{}, UintTag<D0>{}, UintTag<MORE ? D1 - D0 : 0>{});
        });
        cur = kStage - cur;
    };
    const BoolTag<true> yes;
    const BoolTag<false> no;
    if (full > 0) {
        if (steps > 1) step(0, yes, yes, steps > 2, no);
        else step(0, yes, no, false, no);
        uint32_t i = 1;
        for (; i + 3 < steps; i += 2) {
            step(i, no, yes, true, yes);
            step(i + 1, no, yes, true, no);
        }
        if (i + 2 < steps) step(i++, no, yes, true, yes);
        if (i + 1 < steps && i < full) step(i++, no, yes, false, no);   // (of whole steps only the last has none behind it)
        if (i < full) step(i, no, no, false, yes);
        multiply(last, no, nothing, p0, p0);
    }
    if (full < steps) {                                       // 32 k more, the same ones first in all waves
        wait_loads_and_sync<0>();
        a_at[0] = a_place(0);
        const uint32_t w_off = w_place(0);
        const auto before = rsum;                             // (where two waves share the rows, one's are enough)
        for_constants<TN>([&](auto n) { read_w(w_off, n); });
        for_constants<kRows>([&](auto n) { read_a(a_at[0], p0, n); });
        for_constants<kParts - 1>([&](auto part) {
            constexpr int P = decltype(part)::value;
            multiply(part, no, UintTag<P + 1>{}, p0, p0);
        });
        multiply(UintTag<kParts - 1>{}, no, nothing, p0, p0);
        if (Order::kByHalf && (wn & 1u)) rsum = before;
    }
    for (uint32_t i = steps; i < (steps_k + TEAMS - 1) / TEAMS; ++i) wait_loads_and_sync<0>();   // teams wait for each other
    wait_loads_and_sync<0>();                                 // nobody reads a stage any more
    const float s = ga.sb ? ga.sb[0] : 1.0f, b = ga.sb ? ga.sb[1] : 0.0f;
    float *rowsum = reinterpret_cast<float *>(lds_all);       // [TEAMS * kParts][BM]
    join_chains<CHAINS, TM, TN>(acc);
    publish_row_sums<WN, BM, TM>(rowsum, rsum, ga.sb != nullptr, team, 16 * TM * wm, wn, lane);
    if (!add_teams<TEAMS, NW, TM, TN>(rowsum + TEAMS * Order::kParts * BM, acc[0], team, wave, lane)) return;
    store_tile<TEAMS * Order::kParts, BM, TM, TN>(ga.C + static_cast<uint64_t>(m0) * N + n0 + 16 * TN * wn, N, acc[0], rowsum, 16 * TM * wm, order, lane, s, b);
}

// 256 x 128 by four waves, one to a SIMD, each of 128 x 64, decodes a code for 256 rows and reads its fragments from LDS half as often as 128 x 256 by eight
// (9216 x 896 x 1120, input gradient, 13 bits, 28 us; 36 with 128 x 128; 8192 x 1024 x 2048 45, 50 with 128 x 256); the latter is faster forward where
// every unit has one tile and a result has few columns (15360 x 512 x 1120, 11 bits: 27 us, 32 with 256 x 128).  128 x 64 by four waves, three
// workgroups on a unit, fills the chip with half the decoding of 64 x 64 (2304 x 3712 x 192 12.6 us, 14.5 with 128 x 128; 1536 x 2944 x 704 16.4, 18.4), which
// wins on short contractions (8192 x 128 x 320, 11 bits: 5.5 us, 5.8 with 128 x 64).  8192 x 4096 x 1024: 82 us with 256 x 256, 107 with 128 x 128; 2048 x
// 512 x 2048: 50 with 256 x 256, 27 with 128 x 128, 14 / 13 with 64 x 64 and 2 / 4 teams.
// (These times and the fit were taken with matrix instructions of 32 x 32 x 16 and the bit-domain decode throughout; with the present ones the tiles of 64 and 128 rows are 2 - 10 % faster.)
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

template <int B, int WN, int U, int TM, int TN, int TEAMS, int CHAINS, int OCC, bool TRANS, bool HW>
inline void launch_bits_one(const BitsArgs &ga, hipStream_t st) {
    gemm_bits_kernel<B, U, 2, WN, TM, TN, TEAMS, CHAINS, OCC, TRANS, HW><<<dim3(ga.tiles_m * ga.tiles_n), dim3(128 * WN * TEAMS), 0, st>>>(ga);
}
template <int B, bool TRANS, bool HW>
inline int launch_bits_tile(int which, uint32_t chains, const BitsArgs &ga, hipStream_t st) {
    switch (which) {
        case 0: gemm_bits_large_kernel<B, 4, TRANS, HW><<<dim3(ga.tiles_m * ga.tiles_n), dim3(512), 0, st>>>(ga); break;
        case 1: gemm_bits_large_kernel<B, 2, TRANS, HW><<<dim3(ga.tiles_m * ga.tiles_n), dim3(256), 0, st>>>(ga); break;
        case 2: launch_bits_one<B, 4, 32, 4, 4, 1, 1, 2, TRANS, HW>(ga, st); break;
        case 3:
            if (chains == 2) launch_bits_one<B, 4, 16, 4, 2, 1, 2, 2, TRANS, HW>(ga, st);
            else launch_bits_one<B, 4, 16, 4, 2, 1, 1, 4, TRANS, HW>(ga, st);
            break;
        case 4: launch_bits_one<B, 2, 16, 4, 2, 1, 1, 3, TRANS, HW>(ga, st); break;
        case 5:
            if (chains == 2) launch_bits_one<B, 2, 16, 2, 2, 1, 2, 4, TRANS, HW>(ga, st);
            else launch_bits_one<B, 2, 16, 2, 2, 1, 1, 4, TRANS, HW>(ga, st);
            break;
        case 6:
            if (chains == 2) launch_bits_one<B, 2, 16, 2, 2, 2, 2, 4, TRANS, HW>(ga, st);
            else launch_bits_one<B, 2, 16, 2, 2, 2, 1, 4, TRANS, HW>(ga, st);
            break;
        case 7: launch_bits_one<B, 2, 16, 2, 2, 4, 1, 4, TRANS, HW>(ga, st); break;
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
    if constexpr (B == 6 || B == 8) {
        if (hardware_converts(ga.fp)) return trans ? launch_bits_tile<B, true, true>(which, chains, ga, st) : launch_bits_tile<B, false, true>(which, chains, ga, st);
    }
    return trans ? launch_bits_tile<B, true, false>(which, chains, ga, st) : launch_bits_tile<B, false, false>(which, chains, ga, st);
}

// one translation unit per range of widths
int launch_gemm_bits_2_5(const BitsArgs &ga, uint32_t M, int trans, hipStream_t st);
int launch_gemm_bits_6_8(const BitsArgs &ga, uint32_t M, int trans, hipStream_t st);
int launch_gemm_bits_9_11(const BitsArgs &ga, uint32_t M, int trans, hipStream_t st);
int launch_gemm_bits_12_14(const BitsArgs &ga, uint32_t M, int trans, hipStream_t st);
int launch_gemm_bits_15_16(const BitsArgs &ga, uint32_t M, int trans, hipStream_t st);

}  // namespace omc
