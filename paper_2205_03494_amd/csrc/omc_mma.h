// Building blocks of the matrix-core kernels whose operands travel from global memory straight into LDS.
#pragma once
#include "omc_stream.h"

namespace omc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
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

// acc[0] .. acc[PARTS - 1] += the 8 bfloat16 values of a fragment, two at a time, dealt out in turn
template <int PARTS>
__device__ __forceinline__ void add_fragment(bf16x8 f, float *acc) {
    const bf16x2 ones = {static_cast<__bf16>(1.0f), static_cast<__bf16>(1.0f)};
    const u32x4 x = __builtin_bit_cast(u32x4, f);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t w = x[i];
        acc[i % PARTS] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), ones, acc[i % PARTS], false);
    }
}

// A wave's share of the row sums of A.  With two column waves it sums two quarters of each step (the first and third that it
// multiplies), with four one, and where the products are summed in several chains so are these.
template <int WN, int TM, int CHAINS>
struct RowSums {
    static constexpr int kChains = WN == 2 ? CHAINS : 1, kPerFragment = kChains == 4 ? 2 : 1;
    float sum[TM][kChains];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
#pragma unroll
            for (int c = 0; c < kChains; ++c) sum[mi][c] = 0.0f;
    }
    template <int QUARTER>
    __device__ __forceinline__ void add(const bf16x8 (&a)[TM]) {
#pragma unroll
        for (int mi = 0; mi < TM; ++mi) add_fragment<kPerFragment>(a[mi], sum[mi] + (QUARTER == 2 ? kChains / 2 : 0));
    }
    struct Total {
        float row[TM];
    };
    __device__ __forceinline__ Total total() const {
        Total t;
#pragma unroll
        for (int mi = 0; mi < TM; ++mi) {
            t.row[mi] = sum[mi][0];
#pragma unroll
            for (int c = 1; c < kChains; ++c) t.row[mi] += sum[mi][c];
        }
        return t;
    }
};

template <int CHAINS, int TM, int TN>
__device__ __forceinline__ void clear_chains(f32x16 (&acc)[CHAINS][TM][TN]) {
#pragma unroll
    for (int c = 0; c < CHAINS; ++c)
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
#pragma unroll
            for (int ni = 0; ni < TN; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[c][mi][ni][v] = 0.0f;
}
// The chains' sums, added in order, in the first one.
template <int CHAINS, int TM, int TN>
__device__ __forceinline__ void join_chains(f32x16 (&acc)[CHAINS][TM][TN]) {
#pragma unroll
    for (int c = 1; c < CHAINS; ++c)
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
#pragma unroll
            for (int ni = 0; ni < TN; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[0][mi][ni][v] += acc[c][mi][ni][v];
}

// A wave's share of the row sums of A to LDS, [team * WN + column wave][BM]; without an offset they must not enter the result,
// whatever they are.
template <int WN, int BM, int TM, typename Total>
__device__ __forceinline__ void publish_row_sums(float *rowsum, const Total &rsum, bool wanted, uint32_t team, uint32_t row0,
                                                 uint32_t wn, uint32_t lane) {
#pragma unroll
    for (int mi = 0; mi < TM; ++mi) {
        const float t = rsum.row[mi] + __shfl_xor(rsum.row[mi], 32);
        if (lane < 32) rowsum[(team * WN + wn) * BM + row0 + 32 * mi + lane] = wanted ? t : 0.0f;
    }
}

// Team 0's waves add the other teams' tiles to theirs, in order; true for team 0.  `parts`: LDS for (TEAMS - 1) tiles.
// The barrier also makes the row sums visible.
template <int TEAMS, int NW, int TM, int TN>
__device__ __forceinline__ bool add_teams(float *parts, f32x16 (&acc)[TM][TN], uint32_t team, uint32_t wave, uint32_t lane) {
    constexpr uint32_t kWaveFloats = TM * TN * 16 * 64;
    if (TEAMS > 1 && team > 0) {
        float *to = parts + ((team - 1) * NW + wave) * kWaveFloats + lane;
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
#pragma unroll
            for (int ni = 0; ni < TN; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) to[((mi * TN + ni) * 16 + v) * 64] = acc[mi][ni][v];
    }
    __syncthreads();
    if (TEAMS > 1 && team > 0) return false;
#pragma unroll
    for (int t = 1; t < TEAMS; ++t) {
        const float *from = parts + ((t - 1) * NW + wave) * kWaveFloats + lane;
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
#pragma unroll
            for (int ni = 0; ni < TN; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[mi][ni][v] += from[((mi * TN + ni) * 16 + v) * 64];
    }
    return true;
}

// C tile = s * acc + b * row sums.  Several waves (PARTS) have each summed a part of the
// contraction: `rowsum` in LDS, [PARTS][BM].  A lane's accumulators are one column of each 32-column block, so a store instruction of a wave writes two rows
// of 128 contiguous bytes.  The result is
// read by another kernel at the earliest: with ordinary stores it displaces the operands, 71.2 instead of 66.4 us and 84 instead
// of 80 (8192 x 1024 x 4096 and 8192 x 4096 x 1024, new operands each time).
template <int PARTS, int BM, int TM, int TN>
__device__ __forceinline__ void store_tile(float *__restrict__ C, uint32_t ldc, const f32x16 (&acc)[TM][TN], const float *rowsum,
                                           uint32_t row0, uint32_t lane, float s, float b) {
    const uint32_t f_row = lane & 31u, f_half = lane >> 5;
#pragma unroll
    for (int mi = 0; mi < TM; ++mi) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const uint32_t row = row0 + 32 * mi + 8 * (v >> 2) + 4 * f_half + (v & 3);
            float sum = rowsum[row];
#pragma unroll
            for (int q = 1; q < PARTS; ++q) sum += rowsum[q * BM + row];
            const float add = b * sum;
            float *to = C + static_cast<uint64_t>(row) * ldc + f_row;
#pragma unroll
            for (int ni = 0; ni < TN; ++ni) __builtin_nontemporal_store(s * acc[mi][ni][v] + add, to + 32 * ni);
        }
    }
}

}  // namespace omc
