// omc_dequant_gemm / omc_dequant_gemm_dx on S1E4M3 codes with bias 7 (OCP FP8 E4M3 but for the value of the top code).
//
// C[M x N] = A[M x K] * (s W + b), W packed as [K x N] (forward) or [N x K] (TRANS, the input gradient).  Both operands go
// from global memory straight into a ring of S LDS stages of 64 k each, as they are: A as rows of 128 bytes, W as bytes.  A
// wave takes A fragments with 16-byte reads and W fragments as eight codes per lane -- forward with the transposing 8-bit read
// (ds_read_b64_tr_b8: of 16 lanes that point at eight k rows x two 8-byte chunks, lane c receives column c's eight k), TRANS
// with a plain read of eight consecutive codes -- and converts them to bfloat16 in registers, four instructions for eight
// codes.  Staging costs no vector instruction and W passes through LDS at one byte per weight.
//
// 16-byte pieces are XOR-swizzled on their way in (the lane picks the piece, its LDS place is fixed): A pieces by half the row,
// forward W pieces by the k row as far as a row has pieces, TRANS W pieces by a quarter of the column, so that the 16 pieces of A that one read takes at
// a time, or the 16 k rows of one piece of W, lie on different ones of the 64 banks.  No bank conflict is counted in either direction.
//
// The order of the instructions is written down, a column of matrix tiles at a time: its products, and beside them a share of the reads of the next part's fragments, the conversion of
// the next column, and a share of the loads of a later stage.  Left to itself the compiler puts the reads right before their use, and the address arithmetic of the loads in one run of 100
// scalar instructions; addresses now advance from stage to stage.  The last part of a step is multiplied after the
// barrier of the next step, under that step's first reads.  The column waves start with different halves of a step.
//
// The top code reads as NaN in the hardware conversion, without its sign.  No pass over the codes looks for it beforehand, and no
// instruction in the loop: it makes every row of its column NaN, so a wave looks at one row of its sums, and a workgroup that finds
// one computes its tile again with a conversion that is right for it (as it does, to the same result, where A itself is not finite).
// The large tiles also look once after an eighth of a long contraction, and stop there: where top codes are all over the matrix, the
// second pass is then nearly all it costs.  8192 x 4096 x 1024 / 8192 x 1024 x 4096, us: one code in 1000 a top code 90 / 89 (154 / 150 where
// the second pass decoded in the bit domain and the first one always ran to its end; 95 / 109 with a pass over the codes first and a
// kernel of other formats behind it); a top code in one column of 64, in the last row of k, 134 / 135 (156 / 154; 95 / 108); none 65 / 58
// either way.  Looking more often costs up to 9 % where there is none, and so does looking in small tiles (up to 4 %).
//
// Measured (us, 8192 x 4096 x 1024 / 8192 x 1024 x 4096, fp32 output, new operands each time): 65 / 59 with matrix instructions of 32 x 32 x 16, row sums by dot products and the
// compiler's order, 62 / 57 now.  What bounds it: power.  With two waves a SIMD and 8192 x 4096 x 4096 it ran at 1.77 GHz, the matrix cores busy in 80 % of the cycles (of two tiles a compute unit); now it is 1.88 GHz, and 1.83 / 1.80 GHz at the first shape (forward / input gradient), of 2.4.  Instructions
// taken out of the loop make the clock fall again, by and large: without the reads of fragments it is 2.38 GHz, without the loads 2.23.  At a contraction of 1024 also the C stores: a workgroup's take 5 us, in which
// the other one of the unit has the matrix cores to itself and uses them half as well as two.
#include <algorithm>

#include "omc_mma.h"

#pragma clang fp contract(off)

namespace omc {

// Eight codes as bfloat16.  EXACT: right for the top code too.  It is converted as the code below it, 448 = 0x43e0 in bfloat16, and
// gets the bit that is missing to 480 = 0x43f0 afterwards: 24 instructions for eight codes instead of four (the bit-domain
// decode of the other formats takes 44).
template <bool EXACT>
__device__ __forceinline__ bf16x8 fp8x8_to_bf16(u32x2 c) {
    u32x4 o;
#pragma unroll
    for (int d = 0; d < 2; ++d) {
        uint32_t codes = c[d], top = 0;
        if (EXACT) {
            top = ((codes & 0x7f7f7f7fu) + 0x01010101u) & 0x80808080u;   // bit 7 of the bytes that hold it
            codes -= top >> 7;
            top >>= 3;
        }
        o[2 * d] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(codes, 1.0f, false));
        o[2 * d + 1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(codes, 1.0f, true));
        if (EXACT) {
            o[2 * d] |= __builtin_amdgcn_perm(0u, top, 0x0c010c00u);
            o[2 * d + 1] |= __builtin_amdgcn_perm(0u, top, 0x0c030c02u);
        }
    }
    return __builtin_bit_cast(bf16x8, o);
}

struct Fp8Args {
    const uint16_t *A;
    const uint8_t *codes;
    const float *sb;
    float *C;
    uint32_t N, K, tiles_m, tiles_n;
};

// WM x WN waves of TM x TN matrix tiles (16 x 16) each, TEAMS times: team t multiplies the steps t, t + TEAMS, ... of the
// contraction in LDS stages of its own, and team 0 adds up the teams' tiles in order.  A team's sums are CHAINS chains (which
// of them, the half of the step decides, of four also whether the step is odd).  S stages, OCC waves per SIMD.
template <int WM, int WN, int TM, int TN, int TEAMS, int CHAINS, int S, int OCC, bool TRANS>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * WM * WN * TEAMS, 64 * WM * WN * TEAMS))) __attribute__((amdgpu_waves_per_eu(OCC, OCC)))
void gemm_fp8_kernel(Fp8Args ga) {
    constexpr int NW = WM * WN, BM = 16 * TM * WM, BN = 16 * TN * WN;
    constexpr int kALoads = BM / 8 / NW, kWLoads = BN / 16 / NW, kLoads = kALoads + kWLoads;   // 1 KB loads per wave and stage
    constexpr int kPieces = BN / 16;                        // 16-byte pieces in a k row of the forward W tile
    constexpr uint32_t kABytes = BM * 128, kStage = kABytes + BN * 64;
    constexpr bool kLookEarly = BM * BN >= 128 * 256;
    static_assert(WM == 2 && (WN == 2 || WN == 4), "how the row sums are dealt below; with an even number of waves a wave's loads bring one half of 16 rows");
    static_assert(BM % (8 * NW) == 0 && BN % (16 * NW) == 0 && (64 / kPieces) * NW % 16 == 0, "whole loads, one swizzle per wave");
    __shared__ __attribute__((aligned(1024))) uint8_t lds_all[TEAMS * S * kStage];
    __shared__ uint32_t top_met;
    const uint32_t team = TEAMS == 1 ? 0u : __builtin_amdgcn_readfirstlane(threadIdx.x / (64 * NW));
    uint8_t *lds = lds_all + team * (S * kStage);
    const uint32_t lds0 = lds_offset(lds);
    const uint32_t tid = TEAMS == 1 ? threadIdx.x : threadIdx.x % (64 * NW), lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave / WN, wn = wave % WN;
    const uint32_t N = ga.N, K = ga.K;
    uint32_t m0, n0;
    tile_of_block(BM == 256 ? 4 : 8, ga.tiles_m, ga.tiles_n, m0, n0);
    m0 *= BM;
    n0 *= BN;

    // ---- global -> LDS: stage j holds k in [64 j, 64 j + 64); the last one may be half empty (K % 64 == 32), its lanes then
    // bring the lower half twice instead of reading past the row, and nobody multiplies the upper half
    const uint32_t full_k = K / 64, stages_k = (K + 63) / 64;
    const uint32_t full = (full_k + TEAMS - 1 - team) / TEAMS, stages = (stages_k + TEAMS - 1 - team) / TEAMS;   // this team's
    const uint32_t a_row = lane >> 3, a_piece = (lane & 7u) ^ ((a_row >> 1) + 4 * (wave & 1u));
    const uint32_t w_row = TRANS ? lane >> 2 : lane / kPieces;
    auto w_swizzle = [](uint32_t k_row) { return k_row * kPieces / 16 & (kPieces - 1u); };
    const uint32_t w_piece = TRANS ? (lane & 3u) ^ (lane >> 4) : (lane % kPieces) ^ w_swizzle(wave * (64 / kPieces) + w_row);
    const uint8_t *a_from, *w_from;                           // of the stage that is asked for next: this wave's first kilobyte
    uint32_t a_off, w_off;                                    // this lane's piece of a kilobyte
    auto first_stage = [&]() {
        a_from = reinterpret_cast<const uint8_t *>(ga.A) + static_cast<uint64_t>(m0 + 8 * wave) * K * 2 + 128 * team;
        w_from = TRANS ? ga.codes + static_cast<uint64_t>(n0 + 16 * wave) * K + 64 * team
                       : ga.codes + static_cast<uint64_t>(64 * team + 64 / kPieces * wave) * N + n0;
        a_off = a_row * K * 2 + a_piece * 16;
        w_off = TRANS ? w_row * K + w_piece * 16 : w_row * N + w_piece * 16;
    };
    auto next_stage = [&]() {
        a_from += 128 * TEAMS;
        w_from += TRANS ? 64 * TEAMS : 64ull * TEAMS * N;
    };
    const uint64_t a_stride = 16ull * NW * K, w_stride = TRANS ? 16ull * NW * K : 64ull / kPieces * NW * N;   // between a wave's kilobytes
    auto load_one = [&](uint32_t at, auto index, bool half) {
        constexpr uint32_t I = decltype(index)::value;
        if constexpr (I < kALoads) {
            load_to_lds(a_from + I * a_stride, half ? a_off - (a_piece & 4u) * 16 : a_off, lds0 + at + (wave + NW * I) * 1024);
        } else {
            constexpr uint32_t i = I - kALoads;
            if (TRANS) {
                load_to_lds(w_from + i * w_stride, half ? w_off - (w_piece & 2u) * 16 : w_off, lds0 + at + kABytes + (wave + NW * i) * 1024);
            } else {                                          // k rows from 32 on: 32 rows back (these are whole kilobytes)
                const bool back = half && (wave + NW * i) * (64 / kPieces) >= 32;
                load_to_lds(back ? w_from + i * w_stride - 32ull * N : w_from + i * w_stride, w_off, lds0 + at + kABytes + (wave + NW * i) * 1024);
            }
        }
    };
    auto is_half = [&](uint32_t step) { return team + TEAMS * step == full_k; };
    auto load_stage = [&](uint32_t at, uint32_t step) {
        const bool half = is_half(step);
        for_constants<kLoads>([&](auto i) { load_one(at, i, half); });
        next_stage();
    };

    // ---- LDS -> fragments of 32 k
    const uint32_t f_row = lane & 15u, f_k = lane >> 4;
    auto a_place = [&](uint32_t half) {
        const uint32_t row = 16 * TM * wm + f_row;            // (of the wave's first row tile, which need not be the one it multiplies first)
        return row * 128 + (((4 * half + f_k) ^ ((row >> 1) & 7u)) << 4);
    };
    auto w_place = [&](uint32_t half) {
        if (TRANS) {
            const uint32_t col = 16 * TN * wn + f_row;
            return kABytes + col * 64 + (((2 * half + (f_k >> 1)) ^ ((col >> 2) & 3u)) << 4) + 8 * (f_k & 1u);
        }
        const uint32_t row = 32 * half + 8 * f_k + (f_row >> 1);   // 16 lanes: 16 columns x 8 k
        return kABytes + row * BN + (((TN * wn) ^ w_swizzle(row)) << 4) + 8 * (f_row & 1u);
    };
    uint32_t a_at[2], w_at[2];                                // of the half that is multiplied first, and the other one
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        a_at[p] = a_place((p + wn) & 1u);
        w_at[p] = w_place((p + wn) & 1u);
    }
    typedef RowOrder<WN, TM> Order;
    const Order order(wn);
    constexpr int kRun = Order::kSlots < TM / 2 ? Order::kSlots : TM / 2;   // so many of its row tiles follow each other
    uint32_t a_run[TM / kRun];                                // where the runs begin
#pragma unroll
    for (uint32_t r = 0; r < TM / kRun; ++r) a_run[r] = 128 * order.row(r * kRun);
    typedef StepFrags<TM, TN, bf16x8, u32x2> Frags;
    Frags f;
    // read `index` of phase P's, in the order they are needed
    auto read_one = [&](uint32_t at, uint32_t a_off, uint32_t w_off, auto phase, auto index) {
        constexpr int P = decltype(phase)::value, I = decltype(index)::value;
        constexpr bool kReadsB = Frags::reads_b(P);
        constexpr int mi = Frags::reads_a(P) ? I - (kReadsB ? 1 : 0) : -1;
        if constexpr (mi >= 0 && mi < Frags::kRows) {
            constexpr int tile = Frags::first_row(P) + mi;
            f.a[Frags::a_slot(P)][mi] = *reinterpret_cast<const bf16x8 *>(lds + at + a_off + a_run[tile / kRun] + 16 * 128 * (tile % kRun));
        } else {
            constexpr int i = I == 0 ? 0 : I - (Frags::reads_a(P) ? Frags::kRows : 0), ni = Frags::first_col(P) + i;
            if (TRANS) {
                // volatile: of two columns' reads the compiler makes one instruction that takes 16 bytes a lane, lanes of the same half of a 16-byte piece together, on half of the banks
                // (512 x 3584 x 1920 13.3 us, 12.3 apart; 3072 x 640 x 4096 24.2, 23.0)
                f.b[Frags::b_slot(P)][i] = *(const volatile OMC_LDS u32x2 *)(lds + at + w_off + 16 * 64 * ni);
            } else {                                          // 16 columns on: a piece on, before the swizzle
                const i32x2 t = __builtin_amdgcn_ds_read_tr8_b64_v2i32((OMC_LDS i32x2 *)(lds + at + (w_off ^ (16u * ni))));
                f.b[Frags::b_slot(P)][i] = u32x2{static_cast<uint32_t>(t[0]), static_cast<uint32_t>(t[1])};
            }
        }
    };
    auto read_frags = [&](uint32_t at, uint32_t a_off, uint32_t w_off, auto phase) {
        for_constants<Frags::reads(decltype(phase)::value)>([&](auto i) { read_one(at, a_off, w_off, phase, i); });
    };

    Sums<CHAINS, TM, TN> acc;
    uint32_t cur = 0, far = 0;
    // (3072 x 640 x 4096 by 64 x 128 in one chain: forward 22.5 us by parity, 24.6 otherwise, input gradient 24.8, 24.2; two chains, 1536 x 768 x 4096, 23.4, 21.5 and 23.2, 22.0)
    constexpr bool kByParity = TM * TN < 32 && (WN == 2 || (TM == 2 && CHAINS == 1 && !TRANS));
    RowSums<WN, TM, kByParity> rsum;
    auto holds_nan = [&]() {                                  // one row of every column tells
        bool bad = false;
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) bad = bad || acc[0][0][ni][0] != acc[0][0][ni][0];
        return __any(bad);
    };
    // Without EXACT it may stop on the way, in all waves of the workgroup alike, with a NaN in some wave's sums.
    auto compute = [&](auto exact_tag) {
        constexpr bool EXACT = decltype(exact_tag)::value;
        constexpr int kLast = Frags::kPhases - 1, kGroups = Frags::kCols;
        // Over so many columns of a step its loads are spread: over all of them, or where the next step waits for them over half (8192 x 4096 x 1024 by two stages 62.0 us, 65.7 over
        // all; 2048 x 2048 x 512 by three 8.40 over all, 8.56 over half).
        constexpr int kLoadColumns = kGroups * Frags::kPhases / (S == 2 ? 2 : 1);
        bf16x8 w;                                             // the column of fragments that is multiplied next
        auto convert = [&](auto phase, auto col) { w = fp8x8_to_bf16<EXACT>(f.b[Frags::b_slot(decltype(phase)::value)][decltype(col)::value]); };
        // The products of a phase, column by column of its tiles.  Beside each column: a share of the reads of phase NEXT from the stage at `at`, the conversion of the column after
        // it, and a share of the stage's loads (the step begins with its last phase's share).
        auto multiply = [&](auto phase, auto odd, auto next, uint32_t at, auto load, bool half) {
            constexpr int P = decltype(phase)::value, NEXT = decltype(next)::value, chain = (Frags::half(P) + 2 * static_cast<int>(decltype(odd)::value)) % CHAINS;
            constexpr int A = Frags::a_slot(P), R = Frags::first_row(P), C = Frags::first_col(P);
            for_constants<kGroups>([&](auto group) {
                constexpr int G = decltype(group)::value;
                const bf16x8 now = w;
                if constexpr (NEXT <= kLast) {
                    constexpr int N0 = G * Frags::reads(NEXT) / kGroups, N1 = (G + 1) * Frags::reads(NEXT) / kGroups;
                    for_constants<N1 - N0>([&](auto i) { read_one(at, a_at[Frags::half(NEXT)], w_at[Frags::half(NEXT)], next, UintTag<N0 + decltype(i)::value>{}); });
                }
                if constexpr (decltype(load)::value) {
                    constexpr int place = ((P + 1) % Frags::kPhases) * kGroups + G, here = place < kLoadColumns ? place : kLoadColumns;
                    constexpr int L0 = here * kLoads / kLoadColumns, L1 = here < kLoadColumns ? (here + 1) * kLoads / kLoadColumns : L0;
                    for_constants<L1 - L0>([&](auto i) { load_one(far, UintTag<L0 + decltype(i)::value>{}, half); });
                }
#pragma unroll
                for (int mi = 0; mi < Frags::kRows; ++mi)
                    acc[chain][R + mi][C + G] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a[A][mi], now, acc[chain][R + mi][C + G], 0, 0, 0);
                if constexpr (G + 1 < kGroups) convert(phase, UintTag<G + 1>{});
                else if constexpr (NEXT <= kLast) convert(next, UintTag<0>{});
                if constexpr (Frags::reads_a(P)) {
                    constexpr int S0 = G * Frags::kRows / kGroups, S1 = (G + 1) * Frags::kRows / kGroups;
                    for_constants<S1 - S0>([&](auto i) { rsum.template add<R + S0 + decltype(i)::value, Frags::half(P), decltype(odd)::value>(f.a[A][S0 + decltype(i)::value]); });
                }
                if constexpr (Frags::kParts == 2) __builtin_amdgcn_sched_barrier(0);   // (in waves of 32 x 32 the compiler's order is as good or better)
            });
        };
        auto clear = [&]() {
            clear_chains<CHAINS, TM, TN>(acc);
            rsum.clear();
        };
        if (CHAINS == 1) clear();
        const uint32_t shortest = stages_k / TEAMS;
        uint32_t steady_end = stages > S - 1 ? stages - (S - 1) : 0, full_end = full, slots = (stages_k + TEAMS - 1) / TEAMS;
        bool half = full < stages;
        cur = 0;
        far = (S - 1) * kStage;
        const BoolTag<false> no;
        const UintTag<kLast + 1> nothing;
        auto rest_of_step = [&](auto odd, auto load, bool half_stage) {   // everything but the first part's reads and the last one's products
            for_constants<kLast>([&](auto phase) { multiply(phase, odd, UintTag<decltype(phase)::value + 1>{}, cur, load, half_stage); });
            cur = cur == (S - 1) * kStage ? 0 : cur + kStage;
            far = far == (S - 1) * kStage ? 0 : far + kStage;
        };
        // `what` for an even or an odd step, where its chains depend on that
        auto by_parity = [&](uint32_t j, auto what) {
            if (CHAINS == 4 && (j & 1u) != 0) what(BoolTag<true>{}, BoolTag<false>{});
            else what(BoolTag<false>{}, BoolTag<true>{});
        };
        if (!EXACT && kLookEarly && threadIdx.x == 0) top_met = 0;
        first_stage();
#pragma unroll
        for (uint32_t i = 0; i < S - 1; ++i)
            if (i < stages) load_stage(i * kStage, i);
        if (CHAINS > 1) clear();                              // (while the first stages are on their way)
        if (full > 0) {
            wait_stage<S, kLoads>(0, stages);
            read_frags(cur, a_at[0], w_at[0], UintTag<0>{});
            if (stages > S - 1) load_stage(far, S - 1);
            convert(UintTag<0>{}, UintTag<0>{});
            rest_of_step(no, no, false);
            uint32_t j = 1;
            auto steady = [&](uint32_t i, auto odd, auto even) {
                wait_loads_and_sync<(S - 2) * kLoads>();
                const bool half_stage = is_half(i + S - 1);
                multiply(UintTag<kLast>{}, even, UintTag<0>{}, cur, BoolTag<true>{}, half_stage);
                rest_of_step(odd, BoolTag<true>{}, half_stage);
                next_stage();
            };
            auto steps_before = [&](uint32_t end) {
                if constexpr (kByParity) {                    // (without a branch in every step: four chains of 256 x 384 x 704 5.99 -> 5.49 us)
                    for (; j + 1 < end; j += 2) {
                        steady(j, BoolTag<true>{}, BoolTag<false>{});
                        steady(j + 1, BoolTag<false>{}, BoolTag<true>{});
                    }
                    if (j < end) {
                        by_parity(j, [&](auto odd, auto even) { steady(j, odd, even); });
                        ++j;
                    }
                } else {
                    while (j < end) {
                        const uint32_t chain_end = std::min(end, j / kChainSteps * kChainSteps + kChainSteps);
                        for (; j < chain_end; ++j) steady(j, BoolTag<false>{}, BoolTag<false>{});
                        if (j < end) rsum.end_chains(lane);
                    }
                }
            };
            if (!EXACT && kLookEarly && shortest >= 16) {     // (every team gets this far)
                steps_before(shortest / 8);
                if (holds_nan() && lane == 0) top_met = 1;
                sync_lds();
                if (__builtin_amdgcn_readfirstlane(top_met) != 0) {
                    steady_end = full_end = slots = 0;        // the same in all waves: nothing more is multiplied in this pass
                    half = false;
                }
            }
            steps_before(steady_end);
            for (; j < full_end; ++j) {
                wait_stage<S, kLoads>(j, stages);
                by_parity(j, [&](auto odd, auto even) {
                    multiply(UintTag<kLast>{}, even, UintTag<0>{}, cur, no, false);
                    rest_of_step(odd, no, false);
                });
            }
            by_parity(j, [&](auto, auto even) { multiply(UintTag<kLast>{}, even, nothing, 0, no, false); });
        }
        if (half) {                                           // 32 k more, the same ones first in all waves
            wait_loads_and_sync<0>();
            if (wn & 1u) {
                a_at[0] = a_place(0);
                w_at[0] = w_place(0);
            }
            const auto before = rsum;                         // (where two waves share the rows, one's are enough)
            read_frags(cur, a_at[0], w_at[0], UintTag<0>{});
            convert(UintTag<0>{}, UintTag<0>{});
            if constexpr (kLast == 3) {
                multiply(UintTag<0>{}, no, UintTag<1>{}, cur, no, false);
                multiply(UintTag<1>{}, no, nothing, cur, no, false);
            } else {
                multiply(UintTag<0>{}, no, nothing, cur, no, false);
            }
            if (Order::kByHalf && (wn & 1u)) rsum = before;
            if (wn & 1u) {
                a_at[0] = a_place(1);
                w_at[0] = w_place(1);
            }
        }
        for (uint32_t i = stages; i < slots; ++i) wait_loads_and_sync<0>();   // teams wait for each other
        wait_loads_and_sync<0>();                             // nobody reads a stage any more
        join_chains<CHAINS, TM, TN>(acc);
    };

    float *rowsum = reinterpret_cast<float *>(lds_all);       // [TEAMS * kParts][BM], then a flag per wave, then the other teams' tiles
    uint32_t *tops = reinterpret_cast<uint32_t *>(rowsum + TEAMS * Order::kParts * BM);
    float *parts = reinterpret_cast<float *>(tops + 64);
    static_assert(4 * (TEAMS * Order::kParts * BM + 64 + (TEAMS - 1) * BM * BN) <= TEAMS * S * static_cast<int>(kStage), "fits the stages");
    compute(BoolTag<false>{});
    const bool mine = holds_nan();
    if (lane == 0) tops[team * NW + wave] = mine ? 1u : 0u;
    __syncthreads();
    uint32_t any_top = 0;
#pragma unroll
    for (int w = 0; w < NW * TEAMS; ++w) any_top |= tops[w];
    __syncthreads();                                          // the flags are read before anything overwrites them
    if (__builtin_amdgcn_readfirstlane(any_top) != 0) compute(BoolTag<true>{});
    const float s = ga.sb ? ga.sb[0] : 1.0f, b = ga.sb ? ga.sb[1] : 0.0f;
    publish_row_sums<WN, BM, TM>(rowsum, rsum, ga.sb != nullptr, team, 16 * TM * wm, wn, lane);
    if (!add_teams<TEAMS, NW, TM, TN>(parts, acc[0], team, wave, lane)) return;
    store_tile<TEAMS * Order::kParts, BM, TM, TN>(ga.C + static_cast<uint64_t>(m0) * N + n0 + 16 * TN * wn, N, acc[0], rowsum, 16 * TM * wm, order, lane, s, b);
}

// 128 x 256 by four waves has two workgroups on a compute unit, so that one's C stores pass under the other's products: it
// wins wherever a unit gets several tiles of a contraction that is not very long (8192 x 4096 x 1024, new operands each time: 66 us; 70
// with 256 x 256, one workgroup of eight waves per unit, whose loop is the fastest but whose stores nothing covers: 213 to 224 us at
// K = 4096).  The third one is the same tile by eight waves with a third stage, better when every unit has one tile
// (8192 x 1024 x 4096: 60 to 62 us).  The small tiles win where they spread a short product over more units, and several teams where
// even those leave most of them idle (2048 x 512 x 2048: 25 us with 128 x 256, 19 with 128 x 128, 12 with 64 x 128, 11.6 / 9.2 / 10.5
// with 64 x 64 and 1 / 2 / 4 teams).
// (These times, the fit below and those of top codes above were taken with matrix instructions of 32 x 32 x 16; with the present ones every tile is 2 - 9 % faster.)
// Fitted to 1308 sizes.  On 918 others the chosen tile takes 0.5 % longer than the best one on average, more than 7 % longer on 15 of them, at worst
// 17 % (5888 x 384 x 992, input gradient: 13.2 us with 64 x 128, 11.3 with 128 x 128); on 90 with K = 32 - 96, smaller than any in the fit, 0.3 % and 9 %.
static constexpr GemmTile kFp8Tiles[] = {
    {256, 256, 1, 1, 1, 2.628, 1.024, 1.283, 11.45, 0.078}, {128, 256, 1, 1, 2, 2.2, 0.948, 0.658, 4.66, 0.112},
    {128, 256, 1, 1, 1, 2.2, 0.595, 0.788, 6.411, 0.037}, {128, 128, 1, 1, 2, 2.915, 0.462, 0.456, 1.795, 0.057},
    {64, 128, 1, 2, 2, 2.682, 0.238, 0.287, 1.055, 0.067}, {64, 64, 1, 4, 4, 2.646, 0.238, 0.192, 0.249, 0.08},
    {64, 64, 2, 2, 2, 3.007, 0.375, 0.363, 0.551, 0.055}, {64, 64, 4, 1, 1, 3.396, 0.722, 0.895, 0.293, 0.072},
};
static constexpr double kFp8Uneven = 0.5;

// Chains of fp32 sums that a contraction is dealt into, by the result's 64 x 64 tiles and the steps: at least as many as when the choice fell
// on four or two teams of waves for nearly every small product.  Those are slower than one team or two on most of them, but an error against 64 bits grows
// with a chain's length: 512 x 512 x 512 3.4e-8 in four chains, 4.0e-8 in one, 512 x 512 x 4096 6.0e-8 in four, 7.2e-8 in two, 5120 x 256 x 1472 5.2e-8 in
// two, 6.5e-8 in one.  So one team keeps the chains of four: 64 more registers (two waves a SIMD are enough, as results that want four chains have at most one of these tiles a compute unit) and 48 additions at the end, 4.33 -> 4.45 us for 256 x 384 x 416
// (5.29 with four teams), 9.27 -> 9.7 for 2048 x 512 x 2048 with two teams of two chains (9.8 - 10.0 with four).
static uint32_t fp8_chains(uint32_t M, uint32_t N, uint32_t K) {
    const uint64_t small_tiles = static_cast<uint64_t>(M / 64) * (N / 64), steps = (static_cast<uint64_t>(K) + 63) / 64;
    if (small_tiles <= (steps <= 2 ? 120 : std::min<uint64_t>(256, 156 + 4 * steps))) return 4;
    return steps >= 4 && small_tiles <= std::min<uint64_t>(432, 248 + 8 * steps) ? 2 : 1;
}

template <int WM, int WN, int TM, int TN, int TEAMS, int CHAINS, int S, int OCC, bool TRANS>
static void launch_one(const Fp8Args &ga, hipStream_t st) {
    gemm_fp8_kernel<WM, WN, TM, TN, TEAMS, CHAINS, S, OCC, TRANS><<<dim3(ga.tiles_m * ga.tiles_n), dim3(64 * WM * WN * TEAMS), 0, st>>>(ga);
}
// `chains`: of each team
template <bool TRANS>
static int launch_tile(int which, uint32_t chains, const Fp8Args &ga, hipStream_t st) {
    switch (which) {
        case 0: launch_one<2, 4, 8, 4, 1, 1, 3, 2, TRANS>(ga, st); break;
        case 1: launch_one<2, 2, 4, 8, 1, 1, 2, 2, TRANS>(ga, st); break;
        case 2: launch_one<2, 4, 4, 4, 1, 1, 3, 2, TRANS>(ga, st); break;
        case 3: launch_one<2, 2, 4, 4, 1, 1, 3, 2, TRANS>(ga, st); break;
        case 4:
            if (chains == 2) launch_one<2, 4, 2, 2, 1, 2, 3, 4, TRANS>(ga, st);
            else launch_one<2, 4, 2, 2, 1, 1, 3, 4, TRANS>(ga, st);
            break;
        case 5:
            if (chains == 4) launch_one<2, 2, 2, 2, 1, 4, 3, 2, TRANS>(ga, st);
            else if (chains == 2) launch_one<2, 2, 2, 2, 1, 2, 3, 4, TRANS>(ga, st);
            else launch_one<2, 2, 2, 2, 1, 1, 3, 4, TRANS>(ga, st);
            break;
        case 6:
            if (chains == 2) launch_one<2, 2, 2, 2, 2, 2, 3, 4, TRANS>(ga, st);
            else launch_one<2, 2, 2, 2, 2, 1, 3, 4, TRANS>(ga, st);
            break;
        case 7: launch_one<2, 2, 2, 2, 4, 1, 3, 4, TRANS>(ga, st); break;
        default: return static_cast<int>(hipErrorInvalidValue);
    }
    return static_cast<int>(hipGetLastError());
}

int gemm_fp8_tile(uint32_t M, uint32_t N, uint32_t K) { return pick_tile(kFp8Tiles, kFp8Uneven, M, N, K, fp8_chains(M, N, K)); }
uint32_t gemm_fp8_sums(uint32_t M, uint32_t N, uint32_t K) {
    const int which = gemm_fp8_tile(M, N, K);
    return which < 0 ? 0 : kFp8Tiles[which].teams * chains_per_team(kFp8Tiles[which], fp8_chains(M, N, K));
}

int launch_gemm_fp8(const uint16_t *A, const void *codes, const float *sb, float *C, uint32_t M, uint32_t N, uint32_t K, int trans, hipStream_t st) {
    const int which = gemm_fp8_tile(M, N, K);
    if (which < 0) return static_cast<int>(hipErrorInvalidValue);
    const GemmTile &t = kFp8Tiles[which];
    const Fp8Args ga{A, static_cast<const uint8_t *>(codes), sb, C, N, K, M / t.bm, N / t.bn};
    const uint32_t chains = chains_per_team(t, fp8_chains(M, N, K));
    return trans ? launch_tile<true>(which, chains, ga, st) : launch_tile<false>(which, chains, ga, st);
}

}  // namespace omc
