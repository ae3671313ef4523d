// Kernels shared by the single-variable calls (omc_compress, omc_decompress) and the variable-set
// calls (omc_compress_set, omc_decompress_set): the same full-tile / tail device code, fed either
// from one variable described in the kernel arguments or from a plan's work items.
#pragma once
#include "omc_stream.h"

namespace omc {

struct CodecArgs {
    uint8_t *arena;              // base of the data offsets (single variable: its packed buffer)
    const uint8_t *plan;         // device plan blob, or nullptr: one variable, described by `single`
    uint64_t var_off, item_off;
    uint32_t first_item, nitems;
    uint32_t fp32_first, fp32_nitems;   // set calls: copies of fp32 variables appended to the grid
    uint32_t tail_first, tail_nitems;   // ragged tails, the first workgroups of the grid (set calls: a run of the plan's
                                        // work items; single variable: 0 or 1, its partial sums go to slot tail_first)
    PlanVar single;
    uint32_t single_tiles;       // single variable: full tiles per work item
    const float *sb_in;          // decompress: (s, b) table / pair, nullptr = (1, 0)
    const float *vin;            // compress: fp32 values, indexed by aux_offset
    float *vout;                 // decompress: fp32 output, indexed by aux_offset
    Partial *ws;
};

// What rides along with a set's first full-tile launch (the tail groups follow each other in the item list).
struct SetGroups {
    uint32_t fp32_first, fp32_nitems, tail_first, tail_nitems;
};
inline SetGroups set_groups(const PlanGroup *groups, uint32_t ngroups) {
    SetGroups sg{};
    for (uint32_t gi = 0; gi < ngroups; ++gi) {
        if (groups[gi].nitems == 0) continue;
        if (groups[gi].kind == kGroupFp32) {
            sg.fp32_first = groups[gi].first_item;
            sg.fp32_nitems = groups[gi].nitems;
        } else if (groups[gi].kind == kGroupTail) {
            if (sg.tail_nitems == 0) sg.tail_first = groups[gi].first_item;
            sg.tail_nitems += groups[gi].nitems;
        }
    }
    return sg;
}

#ifndef OMC_TUNE_COPY_PARTS
#define OMC_TUNE_COPY_PARTS 4
#endif
// Four waves to an item, each with all its loads in flight at once and no load behind its own stores: conversions of 115 M elements 199 -> 195
// us, a change of a tenth of the 11-bit variables and the message 150 -> 143; eight waves 195 and 147.
constexpr uint32_t kCopyParts = OMC_TUNE_COPY_PARTS;
constexpr int kCopyPartElems = kChunkElems / static_cast<int>(kCopyParts);
// fp32 variable of a set: plain copy between the aux-indexed array and the arena (16-byte pieces)
template <int MODE>
__device__ __forceinline__ void copy_fp32_item(const CodecArgs &ca, uint32_t item, uint32_t part) {
    const PlanItem *items = reinterpret_cast<const PlanItem *>(ca.plan + ca.item_off);
    const PlanVar *vars = reinterpret_cast<const PlanVar *>(ca.plan + ca.var_off);
    const PlanItem it = to_scalar_regs(items[item]);
    const PlanVar pv = to_scalar_regs(vars[it.var]);
    const uint32_t lane = threadIdx.x & 63u;
    float *in_arena = reinterpret_cast<float *>(ca.arena + pv.data_offset);
    const float *src = (MODE == kCompress) ? ca.vin + pv.aux_offset : in_arena;
    float *dst = (MODE == kCompress) ? in_arena : ca.vout + pv.aux_offset;
    const uint64_t begin = static_cast<uint64_t>(it.chunk) * kChunkElems + part * kCopyPartElems;
    // Pieces per lane in flight; both streams are touched once.  (A part is one batch; written without the loop, small
    // re-selections take 1 % longer, 24.3 -> 24.5 us.)
    constexpr int kBatch = kCopyPartElems / 256 < 8 ? kCopyPartElems / 256 : 8;
    for (int j0 = 0; j0 < kCopyPartElems / 256; j0 += kBatch) {
        const uint64_t e0 = begin + (static_cast<uint64_t>(j0) * 64 + lane) * 4;
        if (begin + static_cast<uint64_t>(j0 + kBatch) * 256 <= pv.n) {   // the whole batch is inside: wave-uniform
            f32x4 x[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
                x[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(src + e0 + static_cast<uint64_t>(u) * 256));
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
                __builtin_nontemporal_store(x[u], reinterpret_cast<f32x4 *>(dst + e0 + static_cast<uint64_t>(u) * 256));
            continue;
        }
        if (begin + static_cast<uint64_t>(j0) * 256 >= pv.n) return;
        f32x4 x[kBatch];                                     // the variable ends in this batch: whole pieces where there are any
        uint32_t live[kBatch];                               // this lane's elements of a piece
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const uint64_t e = e0 + static_cast<uint64_t>(u) * 256;
            live[u] = e >= pv.n ? 0u : pv.n - e < 4 ? static_cast<uint32_t>(pv.n - e) : 4u;
            x[u] = f32x4{0, 0, 0, 0};
            if (live[u] == 4) x[u] = *reinterpret_cast<const f32x4 *>(src + e);
            else
                for (uint32_t c = 0; c < 3; ++c)
                    if (c < live[u]) x[u][c] = src[e + c];
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const uint64_t e = e0 + static_cast<uint64_t>(u) * 256;
            if (live[u] == 4) *reinterpret_cast<f32x4 *>(dst + e) = x[u];
            else
                for (uint32_t c = 0; c < 3; ++c)
                    if (c < live[u]) dst[e + c] = x[u][c];
        }
    }
}

template <int MODE>
__device__ __forceinline__ void codec_tile_args(const CodecArgs &ca, const PlanVar &pv, uint32_t var, TileArgs &a) {
    a.codes = reinterpret_cast<uint32_t *>(ca.arena + pv.data_offset);
    a.total_dwords = pv.total_dwords;
    a.n = pv.n;
    a.s = 1.0f;
    a.b = 0.0f;
    if (MODE == kCompress) {
        a.vin = ca.vin + pv.aux_offset;
    } else {
        a.vout = ca.vout + pv.aux_offset;
        if (ca.sb_in) {
            a.s = to_scalar_regs(ca.sb_in[2 * static_cast<uint64_t>(var)]);
            a.b = to_scalar_regs(ca.sb_in[2 * static_cast<uint64_t>(var) + 1]);
        }
    }
}

// A ragged tail as one workgroup; `lds`: kLdsDwords dwords.
template <int MODE>
__device__ __forceinline__ void codec_tail(const CodecArgs &ca, uint32_t index, uint32_t *lds) {
    const uint32_t item = ca.tail_first + index;
    uint32_t var = 0;
    PlanVar pv = ca.single;
    if (ca.plan) {
        const PlanItem *items = reinterpret_cast<const PlanItem *>(ca.plan + ca.item_off);
        const PlanVar *vars = reinterpret_cast<const PlanVar *>(ca.plan + ca.var_off);
        const PlanItem it = to_scalar_regs(items[item]);
        pv = to_scalar_regs(vars[it.var]);
        var = pv.sb_index;
    }
    TileArgs a{};
    codec_tile_args<MODE>(ca, pv, var, a);
    OptConst oc{};
    do_tail<MODE>(a, pv.fp, oc, lds, ca.ws + item);
}

// Grid: ragged tails, then full-tile work items, then copies of fp32 variables: more than FEW_COPIES copy by copy, neighbouring addresses at the same time, fewer by
// the first parts of all of them first, the parts that are empty last.
template <int B, int MODE, int VARIANT, uint32_t FEW_COPIES = 0>
__device__ __forceinline__ void codec_block(const CodecArgs &ca, uint32_t index, uint32_t *lds) {
    if (index < ca.tail_nitems) {
        codec_tail<MODE>(ca, index, lds);
        return;
    }
    const uint32_t block = index - ca.tail_nitems;
    if (block >= ca.nitems) {
        const uint32_t part = block - ca.nitems;
        const bool whole = ca.fp32_nitems > FEW_COPIES;
        copy_fp32_item<MODE>(ca, ca.fp32_first + (whole ? part / kCopyParts : part % ca.fp32_nitems), whole ? part % kCopyParts : part / ca.fp32_nitems);
        return;
    }
    uint32_t item = block, var = 0, chunk = block;
    PlanVar pv = ca.single;
    uint32_t tiles = ca.single_tiles;
    if (ca.plan) {
        const PlanItem *items = reinterpret_cast<const PlanItem *>(ca.plan + ca.item_off);
        const PlanVar *vars = reinterpret_cast<const PlanVar *>(ca.plan + ca.var_off);
        item = ca.first_item + block;
        const PlanItem it = to_scalar_regs(items[item]);
        chunk = it.chunk;
        pv = to_scalar_regs(vars[it.var]);
        var = pv.sb_index;
        tiles = tiles_per_chunk(B);
    }
    TileArgs a{};
    codec_tile_args<MODE>(ca, pv, var, a);
    OptConst oc{};
    do_chunk<B, MODE, VARIANT>(a, pv.fp, oc, chunk, lds, ca.ws + item, tiles);
}

template <int B, int MODE, int VARIANT>
__global__ __launch_bounds__(64, (Tuning<MODE, B>::waves)) void codec_kernel(CodecArgs ca) {
    __shared__ __attribute__((aligned(16))) uint32_t lds[kLdsDwords];
    codec_block<B, MODE, VARIANT>(ca, blockIdx.x, lds);
}

// Tails, the quantized variables' items and the parts of the copies.
inline uint32_t codec_blocks(const CodecArgs &ca) { return ca.tail_nitems + ca.nitems + ca.fp32_nitems * kCopyParts; }
template <int B, int MODE, int VARIANT>
inline void launch_codec(const CodecArgs &ca, hipStream_t st) {
    static_assert(Tuning<MODE, B>::item_waves == 1, "one wave per workgroup");
    codec_kernel<B, MODE, VARIANT><<<dim3(codec_blocks(ca)), dim3(64), 0, st>>>(ca);
}

// Moves what is left of a set's copies, at most one launch's share, to this launch.
inline void take_copies(SetGroups &rest, CodecArgs &ca) {
    ca.fp32_first = rest.fp32_first;
    ca.fp32_nitems = rest.fp32_nitems < kMostSharingBlocks / kCopyParts ? rest.fp32_nitems : kMostSharingBlocks / kCopyParts;
    rest.fp32_first += ca.fp32_nitems;
    rest.fp32_nitems -= ca.fp32_nitems;
}
inline void take_tails(SetGroups &rest, CodecArgs &ca) {
    ca.tail_first = rest.tail_first;
    ca.tail_nitems = rest.tail_nitems;
    rest.tail_nitems = 0;
}

// Tails of a set that has no full tile at all.
template <int MODE>
__global__ __launch_bounds__(64) void codec_tail_kernel(CodecArgs ca) {
    __shared__ uint32_t lds[kLdsDwords];
    codec_tail<MODE>(ca, blockIdx.x, lds);
}

}  // namespace omc
