// Step kernel over the quantized variables of one code width; included once per optimizer.
#pragma once
#include "omc_stream.h"

namespace omc {

#ifndef OMC_TUNE_WAVES_FP6
#define OMC_TUNE_WAVES_FP6 2
#endif
#ifndef OMC_TUNE_OCP_MAXMODE
#define OMC_TUNE_OCP_MAXMODE 2      // kStepSgd: the hardware FP8 variant serves plain SGD only
#endif
#ifndef OMC_TUNE_SGD8_MAX_WAVES
#define OMC_TUNE_SGD8_MAX_WAVES 2      // waves per SIMD of the 8-bit SGD kernel with hardware conversion (0: no cap)
#endif
#ifndef OMC_TUNE_FP6_MAXMODE
#define OMC_TUNE_FP6_MAXMODE 2      // kStepSgd: the hardware 6-bit variant serves plain SGD only
#endif

struct StepArgs {
    uint8_t *arena;
    const uint8_t *plan;      // device copy of the plan blob
    uint64_t var_off, item_off;
    uint32_t first_item, nitems;
    uint32_t fp32_first, fp32_nitems;   // work items of fp32 variables appended to this launch's grid
    uint32_t tail_first, tail_nitems;   // ragged tails, the first workgroups of this launch's grid
    float *sb_table;
    const float *grads;
    float *st0, *st1;
    Partial *ws;
    OptConst oc;
    uint32_t fp32_keep_items;           // the first so many fp32 work items keep their values cached from step to step
    uint32_t fp32_item_by_item;         // parts of the fp32 items on this launch's grid: an item's one after the other, or the first ones of all items first
};

// Variables kept in fp32 (paper Sec. 2.4, 2.5): the update alone, 16-byte pieces, coalesced.
// Every stream is touched once per step, so all loads and stores are non-temporal; all pieces of a lane
// are loaded before any of them is updated (memory-level parallelism is all that is needed).
#ifndef OMC_TUNE_FP32_NT
#define OMC_TUNE_FP32_NT 1
#endif
#ifndef OMC_TUNE_FP32_PARTS
#define OMC_TUNE_FP32_PARTS 8
#endif
// An fp32 item goes to eight waves, each with all its loads in flight at once: a wave that goes on to a second batch waits for the stores
// of the first, as stores and loads share a counter.  Half of 115 M elements in fp32, 2 waves of two batches of four pieces / 4 of
// one / 8 of one batch of two, us: Adam 569 / 556 / 538, momentum 366 / 356 / 352, SGD 195 / 190 / 184 (one wave, four batches: 591, 374, 201).
constexpr uint32_t kFp32Parts = OMC_TUNE_FP32_PARTS;
constexpr int kFp32PartElems = kChunkElems / static_cast<int>(kFp32Parts);
template <int MODE, bool KEEPW>
__device__ __forceinline__ void fp32_item_body(const StepArgs &sa, uint32_t item, uint32_t part) {
    constexpr bool NT = OMC_TUNE_FP32_NT != 0;
    constexpr bool NTW = NT && !KEEPW;                   // the values themselves: read and rewritten by every step
    const PlanItem *items = reinterpret_cast<const PlanItem *>(sa.plan + sa.item_off);
    const PlanVar *vars = reinterpret_cast<const PlanVar *>(sa.plan + sa.var_off);
    const PlanItem it = to_scalar_regs(items[item]);
    const PlanVar pv = to_scalar_regs(vars[it.var]);
    const uint32_t lane = threadIdx.x & 63u;
    float *__restrict__ w = reinterpret_cast<float *>(sa.arena + pv.data_offset);
    const float *__restrict__ g = sa.grads + pv.aux_offset;
    float *__restrict__ m = sa.st0 ? sa.st0 + pv.aux_offset : nullptr;
    float *__restrict__ v = sa.st1 ? sa.st1 + pv.aux_offset : nullptr;
    const uint64_t n = pv.n;
    const uint64_t begin = static_cast<uint64_t>(it.chunk) * kChunkElems + part * kFp32PartElems;
    constexpr int kPieces = kFp32PartElems / 256;            // per lane
    auto ld = [&](const float *p, bool nt = NT) {
        const f32x4 *q = reinterpret_cast<const f32x4 *>(p);
        return nt ? __builtin_nontemporal_load(q) : *q;
    };
    auto st = [&](float *p, const f32x4 &x, bool nt = NT) {
        f32x4 *q = reinterpret_cast<f32x4 *>(p);
        if (nt) __builtin_nontemporal_store(x, q); else *q = x;
    };
    const uint64_t e0 = begin + static_cast<uint64_t>(lane) * 4;
    f32x4 xw[kPieces], xg[kPieces], xm[kPieces], xv[kPieces];
    auto update = [&](int u) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float tm = xm[u][c], tv = xv[u][c];
            xw[u][c] = apply_update<MODE>(xw[u][c], xg[u][c], tm, tv, sa.oc);
            xm[u][c] = tm;
            xv[u][c] = tv;
        }
    };
    if (begin + kFp32PartElems <= n) {                       // the whole part is inside: wave-uniform
#pragma unroll
        for (int u = 0; u < kPieces; ++u) {
            const uint64_t e = e0 + static_cast<uint64_t>(u) * 256;
            xw[u] = ld(w + e, NTW);
            xg[u] = ld(g + e);
            xm[u] = (MODE >= kStepMomentum) ? ld(m + e) : f32x4{0, 0, 0, 0};
            xv[u] = (MODE == kStepAdam) ? ld(v + e) : f32x4{0, 0, 0, 0};
        }
#pragma unroll
        for (int u = 0; u < kPieces; ++u) {
            const uint64_t e = e0 + static_cast<uint64_t>(u) * 256;
            update(u);
            st(w + e, xw[u], NTW);
            if (MODE >= kStepMomentum) st(m + e, xm[u]);
            if (MODE == kStepAdam) st(v + e, xv[u]);
        }
        return;
    }
    if (begin >= n) return;
    // the variable ends in this part: whole pieces where there are any, all loads in flight together
    uint32_t live[kPieces];                                  // this lane's elements of a piece
    auto ld_live = [&](const float *p, uint32_t count) {
        f32x4 x = {0, 0, 0, 0};
        if (count == 4) x = ld(p);
        else
            for (uint32_t c = 0; c < 3; ++c)
                if (c < count) x[c] = p[c];
        return x;
    };
    auto st_live = [&](float *p, const f32x4 &x, uint32_t count) {
        if (count == 4) st(p, x);
        else
            for (uint32_t c = 0; c < 3; ++c)
                if (c < count) p[c] = x[c];
    };
#pragma unroll
    for (int u = 0; u < kPieces; ++u) {
        const uint64_t e = e0 + static_cast<uint64_t>(u) * 256;
        live[u] = e >= n ? 0u : n - e < 4 ? static_cast<uint32_t>(n - e) : 4u;
        xw[u] = ld_live(w + e, live[u]);
        xg[u] = ld_live(g + e, live[u]);
        xm[u] = (MODE >= kStepMomentum) ? ld_live(m + e, live[u]) : f32x4{0, 0, 0, 0};
        xv[u] = (MODE == kStepAdam) ? ld_live(v + e, live[u]) : f32x4{0, 0, 0, 0};
    }
#pragma unroll
    for (int u = 0; u < kPieces; ++u) {
        const uint64_t e = e0 + static_cast<uint64_t>(u) * 256;
        update(u);
        st_live(w + e, xw[u], live[u]);
        if (MODE >= kStepMomentum) st_live(m + e, xm[u], live[u]);
        if (MODE == kStepAdam) st_live(v + e, xv[u], live[u]);
    }
}

template <int MODE>
__device__ __forceinline__ void do_fp32_item(const StepArgs &sa, uint32_t item, uint32_t part) {
    if (item - sa.fp32_first < sa.fp32_keep_items) fp32_item_body<MODE, true>(sa, item, part);
    else fp32_item_body<MODE, false>(sa, item, part);
}

// What the kernels need of one quantized variable.
__device__ __forceinline__ void step_tile_args(const StepArgs &sa, const PlanVar &pv, TileArgs &a) {
    a.codes = reinterpret_cast<uint32_t *>(sa.arena + pv.data_offset);
    a.total_dwords = pv.total_dwords;
    a.grad = sa.grads + pv.aux_offset;
    a.st0 = sa.st0 ? sa.st0 + pv.aux_offset : nullptr;
    a.st1 = sa.st1 ? sa.st1 + pv.aux_offset : nullptr;
    a.n = pv.n;
    a.s = to_scalar_regs(sa.sb_table[2 * static_cast<uint64_t>(pv.sb_index)]);
    a.b = to_scalar_regs(sa.sb_table[2 * static_cast<uint64_t>(pv.sb_index) + 1]);
}

// A ragged tail as one workgroup (code width read from the plan); `lds`: kLdsDwords dwords.
template <int MODE>
__device__ __forceinline__ void step_tail(const StepArgs &sa, uint32_t index, uint32_t *lds) {
    const PlanItem *items = reinterpret_cast<const PlanItem *>(sa.plan + sa.item_off);
    const PlanVar *vars = reinterpret_cast<const PlanVar *>(sa.plan + sa.var_off);
    const uint32_t item = sa.tail_first + index;
    const PlanItem it = to_scalar_regs(items[item]);
    const PlanVar pv = to_scalar_regs(vars[it.var]);
    TileArgs a{};
    step_tile_args(sa, pv, a);
    const FmtParams fp = pv.fp;
    do_tail<MODE>(a, fp, sa.oc, lds, sa.ws + item);
}

// KEEP: the launch's work items keep their packed codes cached from step to step; without it the code
// loads and stores carry the non-temporal hint.
// Occupancy: the register budget follows Tuning<>::waves (waves per SIMD the compiler must make room for).  The
// 8-bit SGD kernel with hardware conversion needs few registers and would run four waves per SIMD; it is held
// at two (8 workgroups per compute unit), because fewer streams open at once suit the memory system better when
// the traffic really comes from HBM (codes streamed, caches flushed between steps: 120 -> 113 us; caps of 10
// workgroups measure like 8, 6 and 4 are slower).  The kernels with more arithmetic per element lose 7-10 %
// under the same cap and are left alone.
template <int B, int MODE, int VARIANT>
struct StepOccupancy {
    static constexpr int min_waves = (VARIANT == 3) ? OMC_TUNE_WAVES_FP6 : Tuning<MODE, B>::waves;
    static constexpr bool capped = (VARIANT == 2 && MODE == kStepSgd && OMC_TUNE_SGD8_MAX_WAVES > 0);
    static constexpr int lo = capped ? (min_waves < OMC_TUNE_SGD8_MAX_WAVES ? min_waves : OMC_TUNE_SGD8_MAX_WAVES) : min_waves;
    static constexpr int hi = capped ? OMC_TUNE_SGD8_MAX_WAVES : 8;
};
template <int B, int MODE, int VARIANT, bool KEEP>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * Tuning<MODE, B>::item_waves, 64 * Tuning<MODE, B>::item_waves)))
__attribute__((amdgpu_waves_per_eu(StepOccupancy<B, MODE, VARIANT>::lo, StepOccupancy<B, MODE, VARIANT>::hi)))
void step_kernel(StepArgs sa) {
    constexpr int NW = Tuning<MODE, B>::item_waves;
    __shared__ __attribute__((aligned(16))) uint32_t lds[NW * kLdsDwords];
    if (blockIdx.x < sa.tail_nitems) {
        if (NW == 1 || threadIdx.x < 64) step_tail<MODE>(sa, blockIdx.x, lds);
        return;
    }
    const uint32_t block = blockIdx.x - sa.tail_nitems;
    if (block >= sa.nitems) {                            // the workgroups past the end serve fp32 variables, a wave a part of an item
        const uint32_t part = (block - sa.nitems) * NW + (NW == 1 ? 0u : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
        const bool whole = sa.fp32_item_by_item != 0;
        do_fp32_item<MODE>(sa, sa.fp32_first + (whole ? part / kFp32Parts : part % sa.fp32_nitems), whole ? part % kFp32Parts : part / sa.fp32_nitems);
        return;
    }
    const PlanItem *items = reinterpret_cast<const PlanItem *>(sa.plan + sa.item_off);
    const PlanVar *vars = reinterpret_cast<const PlanVar *>(sa.plan + sa.var_off);
    const uint32_t item = sa.first_item + block;
    const PlanItem it = to_scalar_regs(items[item]);
    const PlanVar pv = to_scalar_regs(vars[it.var]);
    TileArgs a{};
    step_tile_args(sa, pv, a);
    const FmtParams fp = pv.fp;
    do_chunk<B, MODE, VARIANT, KEEP, NW>(a, fp, sa.oc, it.chunk, lds, sa.ws + item);
}

// Tails, the quantized variables' items and the parts of the fp32 ones.
template <int BITS, int MODE>
inline dim3 step_grid(const StepArgs &sa) {
    constexpr uint32_t kPartsPerBlock = Tuning<MODE, BITS>::item_waves;
    static_assert(kFp32Parts % kPartsPerBlock == 0, "an fp32 item is whole workgroups");
    return dim3(sa.tail_nitems + sa.nitems + sa.fp32_nitems * (kFp32Parts / kPartsPerBlock));
}

// Variants 0 / 1 and, for code widths that can hold 16 mantissa bits, 4 / 5 (error-carrying sums).
template <int BITS, int MODE, bool KEEP>
inline void launch_step_generic_variant(uint32_t variant, const StepArgs &sa, hipStream_t st) {
    const dim3 grid = step_grid<BITS, MODE>(sa), block(64 * Tuning<MODE, BITS>::item_waves);
    if constexpr (BITS >= 18) {
        if (variant == 4) { step_kernel<BITS, MODE, 4, KEEP><<<grid, block, 0, st>>>(sa); return; }
        if (variant == 5) { step_kernel<BITS, MODE, 5, KEEP><<<grid, block, 0, st>>>(sa); return; }
    }
    if (variant == 1) step_kernel<BITS, MODE, 1, KEEP><<<grid, block, 0, st>>>(sa);
    else step_kernel<BITS, MODE, 0, KEEP><<<grid, block, 0, st>>>(sa);
}

template <int MODE, bool KEEP>
inline int launch_step_group_keep(uint32_t bits, uint32_t variant, const StepArgs &sa, hipStream_t st) {
    // the hardware-conversion variant pays off where the vector ALU is the limit: plain SGD
    if (bits == 8 && variant == 2 && MODE <= OMC_TUNE_OCP_MAXMODE) {
        step_kernel<8, MODE, 2, KEEP><<<step_grid<8, MODE>(sa), dim3(64 * Tuning<MODE, 8>::item_waves), 0, st>>>(sa);
        return static_cast<int>(hipGetLastError());
    }
    if (bits == 6 && variant == 3 && MODE <= OMC_TUNE_FP6_MAXMODE) {
        step_kernel<6, MODE, 3, KEEP><<<step_grid<6, MODE>(sa), dim3(64 * Tuning<MODE, 6>::item_waves), 0, st>>>(sa);
        return static_cast<int>(hipGetLastError());
    }
    switch (bits) {
#define X(BITS)                                                              \
    case BITS:                                                               \
        launch_step_generic_variant<BITS, MODE, KEEP>(variant, sa, st);      \
        break;
        OMC_FOR_EACH_BITS(X)
#undef X
        default:
            return static_cast<int>(hipErrorInvalidValue);
    }
    return static_cast<int>(hipGetLastError());
}

template <int MODE>
inline int launch_step_group_mode(uint32_t bits, uint32_t variant, const StepArgs &sa, bool keep, hipStream_t st) {
    return keep ? launch_step_group_keep<MODE, true>(bits, variant, sa, st)
                : launch_step_group_keep<MODE, false>(bits, variant, sa, st);
}

int launch_step_group_sgd(uint32_t bits, uint32_t variant, const StepArgs &sa, bool keep, hipStream_t st);
int launch_step_group_momentum(uint32_t bits, uint32_t variant, const StepArgs &sa, bool keep, hipStream_t st);
int launch_step_group_adam(uint32_t bits, uint32_t variant, const StepArgs &sa, bool keep, hipStream_t st);

}  // namespace omc
