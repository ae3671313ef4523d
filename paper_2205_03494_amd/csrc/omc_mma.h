// Building blocks of the matrix-core kernels whose operands travel from global memory straight into LDS.
#pragma once
#include "omc_stream.h"

namespace omc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
#define OMC_LDS __attribute__((address_space(3)))

template <bool B>
struct BoolTag {
    static constexpr bool value = B;
};

template <uint32_t V>
struct UintTag {
    static constexpr uint32_t value = V;
};

// f(UintTag<0>) .. f(UintTag<COUNT - 1>)
template <int COUNT, int FROM = 0, typename F>
__device__ __forceinline__ void for_constants(F &&f) {
    if constexpr (FROM < COUNT) {
        f(UintTag<FROM>{});
        for_constants<COUNT, FROM + 1>(f);
    }
}

// LDS byte offset of a __shared__ object, as the direct-to-LDS loads take it.
__device__ __forceinline__ uint32_t lds_offset(const void *p) {
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const OMC_LDS uint8_t *)(p)));
}

// One wave copies 64 pieces of 16 bytes from global memory into 1 KB of LDS at `dst` (the same in every lane), lane l's
// piece to dst + 16 l, from base + off (off per lane).  No register is written, so nothing can be overwritten under
// a load in flight.  Written as asm because the compiler makes every LDS read it cannot tell apart from the target wait for
// all such loads; the kernels wait for them by count instead (wait_loads_and_sync), which is sound because
// these are the only vector-memory operations of their loops and return in order.
__device__ __forceinline__ void load_to_lds(const uint8_t *base, uint32_t off, uint32_t dst) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(off), "s"(base) : "memory", "m0");
}

// Waits until at most LATER of this wave's vector-memory operations are in flight and its LDS accesses are done, then for
// the whole workgroup: what the older loads of all waves brought is in LDS, and what was read before may be overwritten.
template <int LATER>
__device__ __forceinline__ void wait_loads_and_sync() {
    static_assert(LATER >= 0 && LATER <= 63, "the counter has six bits");
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(LATER) : "memory");
}

// A barrier that waits for this wave's LDS accesses and leaves its loads in flight.
__device__ __forceinline__ void sync_lds() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// The ring of S stages: waits for stage j of `total` when up to S - 1 of them have been asked for; PER = loads per stage.
template <int S, int PER>
__device__ __forceinline__ void wait_stage(uint32_t j, uint32_t total) {
    static_assert(S >= 2 && S <= 5, "cases below");
    const uint32_t later = total - 1 - j;
    if (later >= S - 2) wait_loads_and_sync<(S - 2) * PER>();
    else if (S > 4 && later == 2) wait_loads_and_sync<(S > 4 ? 2 : 0) * PER>();
    else if (S > 3 && later == 1) wait_loads_and_sync<(S > 3 ? 1 : 0) * PER>();
    else wait_loads_and_sync<0>();
}

// Host: which of a kernel's tile sizes to launch for an M x N result over K, by an estimate of its time.  In us: `base` is a launch; `step` a step of
// 64 k (of TEAMS times as many with several teams) of workgroups that nothing else slows down, `resident` of them on a compute unit; `loaded` what a step
// costs per workgroup of a unit where all units are busy (matrix cores, LDS and memory together); `stores` the C stores of 256 tiles; `fresh` a megabyte
// of A and W on its way from memory, W at a byte a code.  A launch ends with the unit that has the most workgroups, and while others have run out of
// theirs it is faster: `uneven` is the share of its surplus over the average that counts (9728 x 128 x 3680, input gradient: 304 tiles
// of 64 x 64, two on some units, 37 us by two teams; 152 of 64 x 128, one on a unit, 34).
// Each row is fitted to its tile's own times, and all rows were then moved by at most 12 % towards the choices that cost least.  A row gives the times of its tile
// within 6 - 9 % (standard deviation, sizes where it is within 1.5 of the best).  How good the choice is was measured on other sizes, see the tables.
struct GemmTile {
    uint32_t bm, bn, teams, chains, resident;                 // chains: the most that one team can keep
    double base, step, loaded, stores, fresh;
};
inline uint32_t chains_per_team(const GemmTile &t, uint32_t chains) { return (chains + t.teams - 1) / t.teams; }
// `chains`: into how many chains of fp32 sums the contraction is to be dealt at least
template <int COUNT>
inline int pick_tile(const GemmTile (&tiles)[COUNT], double uneven, uint32_t M, uint32_t N, uint32_t K, uint32_t chains) {
    const double megabytes = (2.0 * M + N) * K / 1e6;
    int best = -1;
    double best_cost = 0.0;
    for (int i = 0; i < COUNT; ++i) {
        const GemmTile &t = tiles[i];
        if (M % t.bm != 0 || N % t.bn != 0 || chains_per_team(t, chains) > t.chains) continue;
        const uint64_t count = static_cast<uint64_t>(M / t.bm) * (N / t.bn);
        if (count > 0x7fffffffull) continue;
        const double per_unit = static_cast<double>(count) / 256.0;
        const double alone = t.step * static_cast<double>((count + 256ull * t.resident - 1) / (256ull * t.resident));
        const double busy = t.loaded * (per_unit + uneven * (static_cast<double>((count + 255) / 256) - per_unit));
        const uint64_t steps = (static_cast<uint64_t>(K) + 64ull * t.teams - 1) / (64ull * t.teams);
        const double cost = t.base + t.stores * per_unit + t.fresh * megabytes + static_cast<double>(steps) * (alone > busy ? alone : busy);
        if (best < 0 || cost < best_cost) {
            best = i;
            best_cost = cost;
        }
    }
    return best;
}

// Tile of this workgroup in a grid of tiles_m x tiles_n (one-dimensional launch).  Workgroups go to the 8 dies in turn and
// each die has an L2 of its own, so every die gets a contiguous run of the tile order, in which groups of `group_rows` tile rows
// share their columns.  The tiles of a die at one time should need as many bytes of the one operand as of the other: eight rows for
// tiles whose two sides weigh the same, fewer for 256-row tiles (256 x 256 of bf16 by bytes, 8192 x 4096 x 1024: 70 us with 4 rows, 79
// with 8, 82 with 16; 11-bit codes 82, 89, 93; weight gradient in 256 x 128, 8192 rows, 4096 x 1024: 71 with 2, 72 with 4, 75 with 8).
__device__ __forceinline__ void tile_of_block(uint32_t group_rows, uint32_t tiles_m, uint32_t tiles_n, uint32_t &tm, uint32_t &tn) {
    const uint32_t total = tiles_m * tiles_n, q = total / 8, r = total % 8, die = blockIdx.x % 8;
    const uint32_t id = die * q + (die < r ? die : r) + blockIdx.x / 8;
    const uint32_t rows = tiles_m < group_rows ? tiles_m : group_rows;
    const uint32_t group = id / (rows * tiles_n), first = group * rows;
    const uint32_t height = tiles_m - first < rows ? tiles_m - first : rows;
    const uint32_t in = id - group * rows * tiles_n;
    tm = first + in % height;
    tn = in / height;
}

// The products are matrix instructions of 16 x 16 results over 32 k, not of 32 x 32 over 16.  Both multiply 512 pairs per clock and SIMD, but large
// products run at the card's power limit (8192 x 4096 x 1024 on S1E4M3 codes, call after call: 1.83 GHz of 2.4), and the smaller ones take less power: registers full of normal values, nothing but matrix instructions, 1750 TFLOP/s
// at 1.71 GHz with 32 x 32 x 16, 1935 at 1.95 GHz with 16 x 16 x 32.  Either adds up its k in the same order (results bit for bit the same over K = 64 - 8192).
// A: lane l holds row l % 16, k 8 (l / 16) ..; B likewise its column; the result's value v of lane l is row 4 (l / 16) + v, column l % 16.
template <int CHAINS, int TM, int TN>
using Sums = f32x4[CHAINS][TM][TN];

// How the row sums of A are dealt out over the WN column waves that multiply the same rows, and where the rows of a wave's tiles lie.  Each wave sums the rows of its first
// tiles, over either half of the steps; where it has few tiles (kByHalf), of four waves two share the rows and each takes the half that it multiplies first.  So that
// those are other rows in each wave, their order differs: tile mi lies at row 16 * (mi ^ flip).
template <int WN, int TM>
struct RowOrder {
    static constexpr bool kByHalf = WN == 4 && TM < 8;
    static constexpr int kSlots = kByHalf ? TM / 2 : TM / WN, kParts = kByHalf ? 2 : 1;   // kParts: waves that share a row
    uint32_t flip;
    __device__ __forceinline__ explicit RowOrder(uint32_t wn) : flip((kByHalf ? wn >> 1 : wn) * kSlots) {}
    __device__ __forceinline__ uint32_t row(uint32_t mi) const { return 16 * (mi ^ flip); }
};
// A wave's share of them: products with ones.  One costs a 16 x 32 fragment 16 clocks of the matrix cores; the four two-element dot products of a lane that
// do the same hold them up for 40, as they cannot run beside them (64 matrix instructions and 16 of the former a step of 256 x 256: 205000 clocks for 8192 x 4096 x 4096, 160000 without any).
// Each half of a step has a chain of its own (of waves that share rows, each its half), and with that alone they are too long: 8192 x 8192 x 8192, A of one sign 11.4e-8 off 64 bits, mean zero 6.1e-8, where
// dot products dealt out over lanes and waves were 4.3e-8 and 5.1e-8.  BY_PARITY: odd steps have chains of their own, which costs no instruction in a loop of two steps (4.4e-8 - 5.1e-8 and 5.1e-8 - 5.3e-8 over 8192).
// Otherwise the chains end every kChainSteps steps, and a sum of 64 bits takes what they hold (2.2e-8 - 3.1e-8 and 2.8e-8 - 4.0e-8).  Which one is measured, by kernel: waves of 128 x 64 and 64 x 128 have no registers for the
// former (they spill 20 - 50), and ending chains makes the compiler move the loads of the other codes' kernels (11 bits, 1536 x 1536 x 4096, input gradient: 48.1 us, 51.9 so, 47.4 by parity).
constexpr uint32_t kChainSteps = 8;
template <int WN, int TM, bool BY_PARITY>
struct RowSums {
    typedef RowOrder<WN, TM> Order;
    static constexpr int kHalves = Order::kByHalf ? 1 : 2, kChains = BY_PARITY ? 2 * kHalves : kHalves;
    u32x4 ones;
    f32x4 sum[Order::kSlots][kChains];
    double ended[Order::kSlots];                              // of row 4 (lane / 16) + lane % 4: every column of the products with ones holds the sums
    __device__ __forceinline__ void clear() {
        ones = u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
        asm volatile("" : "+v"(ones));                        // they stay in registers
#pragma unroll
        for (int mi = 0; mi < Order::kSlots; ++mi) {
            ended[mi] = 0.0;
#pragma unroll
            for (int c = 0; c < kChains; ++c) sum[mi][c] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
    }
    __device__ __forceinline__ f32x4 joined(int mi) const {   // (BY_PARITY) of rows 4 (lane / 16) ..
        f32x4 t;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            t[v] = sum[mi][0][v] + sum[mi][kHalves][v];
            if constexpr (kHalves == 2) t[v] += sum[mi][1][v] + sum[mi][3][v];
        }
        return t;
    }
    __device__ __forceinline__ void end_chains(uint32_t lane) {
#pragma unroll
        for (int mi = 0; mi < Order::kSlots; ++mi)
#pragma unroll
            for (int c = 0; c < kChains; ++c) {
                const f32x4 x = sum[mi][c];
                const float lower = (lane & 1u) ? x[1] : x[0], upper = (lane & 1u) ? x[3] : x[2];
                ended[mi] += static_cast<double>((lane & 2u) ? upper : lower);
                sum[mi][c] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            }
    }
    template <int MI, int HALF, bool ODD>
    __device__ __forceinline__ void add(bf16x8 a) {
        constexpr int chain = HALF + (BY_PARITY && ODD ? kHalves : 0);
        if constexpr (MI < Order::kSlots && HALF < kHalves) sum[MI][chain] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, ones), sum[MI][chain], 0, 0, 0);
    }
};

template <int CHAINS, int TM, int TN>
__device__ __forceinline__ void clear_chains(Sums<CHAINS, TM, TN> &acc) {
#pragma unroll
    for (int c = 0; c < CHAINS; ++c)
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
#pragma unroll
            for (int ni = 0; ni < TN; ++ni) acc[c][mi][ni] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
}
// The chains' sums, added in order, in the first one.
template <int CHAINS, int TM, int TN>
__device__ __forceinline__ void join_chains(Sums<CHAINS, TM, TN> &acc) {
#pragma unroll
    for (int c = 1; c < CHAINS; ++c)
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
#pragma unroll
            for (int ni = 0; ni < TN; ++ni)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[0][mi][ni][v] += acc[c][mi][ni][v];
}

// The fragments of a step of 64 k in the order they are multiplied: two halves of 32 k, of which each is dealt into parts of rows or columns, whichever the wave has
// more of, while the other operand's fragments stay.  Those of a part are read while the part before is multiplied; the last part is
// multiplied after the barrier of the next step, under that step's first reads.  A wave of 64 x 128 has 48 registers of them (operands of the FP8 kernel), with whole halves
// it would be 64.
template <int TM, int TN, typename FragA, typename FragB>
struct StepFrags {
    static constexpr bool kSplitN = TN >= 4 && TN > TM, kSplitM = !kSplitN && TM >= 4;
    static constexpr int kParts = kSplitN || kSplitM ? 2 : 1, kPhases = 2 * kParts;     // of a step
    static constexpr int kRows = kSplitM ? TM / 2 : TM, kCols = kSplitN ? TN / 2 : TN;  // tiles in a part
    FragA a[2][kRows];
    FragB b[2][kCols];
    static constexpr int half(int phase) { return phase / kParts; }
    static constexpr int part(int phase) { return phase % kParts; }
    static constexpr int a_slot(int phase) { return kSplitM ? part(phase) : half(phase); }
    static constexpr int b_slot(int phase) { return kSplitN ? part(phase) : half(phase); }
    static constexpr int first_row(int phase) { return kSplitM ? part(phase) * kRows : 0; }
    static constexpr int first_col(int phase) { return kSplitN ? part(phase) * kCols : 0; }
    static constexpr bool reads_a(int phase) { return kSplitM || part(phase) == 0; }
    static constexpr bool reads_b(int phase) { return kSplitN || part(phase) == 0; }
    static constexpr int reads(int phase) { return (reads_a(phase) ? kRows : 0) + (reads_b(phase) ? kCols : 0); }
};

// A wave's share of the row sums of A to LDS, [team * kParts + part][BM]; without an offset they must not enter the result,
// whatever they are.
template <int WN, int BM, int TM, bool BY_PARITY>
__device__ __forceinline__ void publish_row_sums(float *rowsum, RowSums<WN, TM, BY_PARITY> &rsum, bool wanted, uint32_t team, uint32_t row0,
                                                 uint32_t wn, uint32_t lane) {
    typedef RowOrder<WN, TM> Order;
    const Order order(wn);
    float *to = rowsum + (team * Order::kParts + (Order::kByHalf ? wn & 1u : 0u)) * BM + row0 + 4 * (lane >> 4);
    if constexpr (BY_PARITY) {
#pragma unroll
        for (int mi = 0; mi < Order::kSlots; ++mi) {
            f32x4 t = rsum.joined(mi);
            if (!wanted) t = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            if ((lane & 15u) == 0) *reinterpret_cast<f32x4 *>(to + order.row(mi)) = t;
        }
    } else {
        rsum.end_chains(lane);
#pragma unroll
        for (int mi = 0; mi < Order::kSlots; ++mi)
            if ((lane & 15u) < 4) to[order.row(mi) + (lane & 3u)] = wanted ? static_cast<float>(rsum.ended[mi]) : 0.0f;
    }
}

// Team 0's waves add the other teams' tiles to theirs, in order; true for team 0.  `parts`: LDS for (TEAMS - 1) tiles.
// The barrier also makes the row sums visible.
template <int TEAMS, int NW, int TM, int TN>
__device__ __forceinline__ bool add_teams(float *parts, f32x4 (&acc)[TM][TN], uint32_t team, uint32_t wave, uint32_t lane) {
    constexpr uint32_t kWaveQuads = TM * TN * 64;
    f32x4 *quads = reinterpret_cast<f32x4 *>(parts);
    if (TEAMS > 1 && team > 0) {
        f32x4 *to = quads + ((team - 1) * NW + wave) * kWaveQuads + lane;
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
#pragma unroll
            for (int ni = 0; ni < TN; ++ni) to[(mi * TN + ni) * 64] = acc[mi][ni];
    }
    __syncthreads();
    if (TEAMS > 1 && team > 0) return false;
#pragma unroll
    for (int t = 1; t < TEAMS; ++t) {
        const f32x4 *from = quads + ((t - 1) * NW + wave) * kWaveQuads + lane;
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
#pragma unroll
            for (int ni = 0; ni < TN; ++ni) {
                const f32x4 q = from[(mi * TN + ni) * 64];
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[mi][ni][v] += q[v];
            }
    }
    return true;
}

// Value v of two tiles that lie side by side, exchanged between lanes so that an access takes two rows of 32 neighbouring values: `x` becomes row 8 (lane / 32) + v of
// them, `y` the row four below, both column lane % 32.
__device__ __forceinline__ void side_by_side(float &x, float &y) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    x = __uint_as_float(r[0]);
    y = __uint_as_float(r[1]);
}

// C tile = s * acc + b * row sums.  PARTS waves have each summed a part of the
// contraction: `rowsum` in LDS, [PARTS][BM].  A store instruction of a wave writes two rows of 128 contiguous bytes.  The result is
// read by another kernel at the earliest: with ordinary stores it displaces the operands, 71.2 instead of 66.4 us and 84 instead
// of 80 (8192 x 1024 x 4096 and 8192 x 4096 x 1024, new operands each time).
template <int PARTS, int BM, int TM, int TN, typename Order>
__device__ __forceinline__ void store_tile(float *__restrict__ C, uint32_t ldc, const f32x4 (&acc)[TM][TN], const float *rowsum,
                                           uint32_t row0, const Order &order, uint32_t lane, float s, float b) {
    static_assert(TN % 2 == 0, "pairs of tiles");
    const uint32_t col = lane & 31u, row8 = 8 * (lane >> 5);
#pragma unroll
    for (int mi = 0; mi < TM; ++mi) {
        const uint32_t row = row0 + order.row(mi) + row8;
        f32x4 add[2];                                         // rows row .. row + 3, row + 4 ..
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            add[r] = *reinterpret_cast<const f32x4 *>(rowsum + row + 4 * r);
#pragma unroll
            for (int q = 1; q < PARTS; ++q) {
                const f32x4 t = *reinterpret_cast<const f32x4 *>(rowsum + q * BM + row + 4 * r);
#pragma unroll
                for (int v = 0; v < 4; ++v) add[r][v] += t[v];
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) add[r][v] = b * add[r][v];
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float *to = C + static_cast<uint64_t>(row + v) * ldc + col;
#pragma unroll
            for (int ni = 0; ni < TN; ni += 2) {
                float x = acc[mi][ni][v], y = acc[mi][ni + 1][v];
                side_by_side(x, y);
                __builtin_nontemporal_store(s * x + add[0][v], to + 16 * ni);
                __builtin_nontemporal_store(s * y + add[1][v], to + 4 * static_cast<uint64_t>(ldc) + 16 * ni);
            }
        }
    }
}

}  // namespace omc
