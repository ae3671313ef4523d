// omc_aggregate_mean: the server's side of a federated round (paper Sec. 1: the clients' trained
// models come back and are aggregated; Sec. 2.5: every client quantizes its own subset of the
// variables).  out[i] = (v_0[i] + v_1[i] + ... + v_{R-1}[i]) / R over the clients' decompressed
// values, summed in client order in fp32, every operation rounded once.  One pass: each client's
// copy is read once in the form it arrived in (packed codes or fp32), the mean is written once.
#include <algorithm>

#include "omc_stream.h"

#ifndef OMC_TUNE_AGG_NT
#define OMC_TUNE_AGG_NT 1      // the clients' codes are read once per round: non-temporal
#endif

namespace omc {

// Loads of a batch of clients are in flight together.  Byte codes: eight clients at three waves per SIMD 291 us, four at four 301, two at
// six 304 (115 M elements, 8 clients; one at eight 311).  A batch takes 16 registers a client, as a client may be in fp32, and at three waves 12 registers
// are spilled: 16 bytes a lane out and back per slab of 1024 elements, of which hardly any leaves the caches (1 % of the bytes written to memory).  The other
// widths hold a client in 32 registers, and more waves are worth more than more clients: 10 layers of 397 x 1191 in 11 bits, 4 clients, one client at four waves 66 us, two at three 71, four at two 80.
constexpr uint32_t kByteBatch = 8, kByteWaves = 3, kTileWaves = 4, kFlatBatch = 8, kTailBatchClients = 4;
constexpr uint32_t kTailPart = 256;       // elements of a ragged tail that one workgroup takes: four per lane
constexpr uint32_t kTailParts = kTileElems / kTailPart;
constexpr uint32_t kFlatParts = 4;        // workgroups that share an all-fp32 item
// A work item is shared by several workgroups until there are this many: about what the chip holds at a time (same sets: 4096 74 us,
// 8192 and more 71).
constexpr uint32_t kEnoughBlocks = 8192;

struct AggArgs {
    const uint8_t *plan;                 // device copy of the aggregation plan blob
    uint64_t var_off, src_off, item_off;
    uint32_t first_item;
    uint32_t tail_first, tail_blocks;    // ragged tails: kTailParts workgroups an item, the first ones of the launch
    uint32_t full_blocks, parts;         // full tiles: `parts` workgroups an item
    uint32_t flat_first;                 // items of all-fp32 variables: kFlatParts workgroups an item, the last ones of the launch
    uint32_t nreplicas;
    float count;                         // R as a float
    AggPointers p;
    float *out;
};

// The variable of a work item and where its copies lie: lane r holds client r's.  All clients' descriptors take three dependent
// loads together; fetched one client after the other, where they were needed, they were two for each.
struct AggView {
    AggVar av;
    uint32_t chunk;
    uint32_t addr_lo, addr_hi, quantized;
    float s, b;
    __device__ __forceinline__ const uint8_t *copy(uint32_t r) const {
        return reinterpret_cast<const uint8_t *>((static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(addr_hi, r))) << 32) |
                                                 static_cast<uint32_t>(__builtin_amdgcn_readlane(addr_lo, r)));
    }
    __device__ __forceinline__ bool is_quantized(uint32_t r) const { return __builtin_amdgcn_readlane(quantized, r) != 0; }
    __device__ __forceinline__ float scale(uint32_t r) const { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(s), r)); }
    __device__ __forceinline__ float offset(uint32_t r) const { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(b), r)); }
};
__device__ __forceinline__ AggView load_view(const AggArgs &aa, uint32_t item) {
    AggView v{};
    const PlanItem it = to_scalar_regs(reinterpret_cast<const PlanItem *>(aa.plan + aa.item_off)[item]);
    v.chunk = it.chunk;
    const uint32_t r = threadIdx.x;
    if (r < aa.nreplicas) {
        const AggSrc src = (reinterpret_cast<const AggSrc *>(aa.plan + aa.src_off) + static_cast<uint64_t>(it.var) * aa.nreplicas)[r];
        const uint64_t addr = reinterpret_cast<uint64_t>(aa.p.arena[r]) + src.data_offset;
        v.addr_lo = static_cast<uint32_t>(addr);
        v.addr_hi = static_cast<uint32_t>(addr >> 32);
        v.quantized = src.quantized;
        const float *sb = aa.p.sb[r] + 2 * static_cast<uint64_t>(it.var);
        v.s = sb[0];
        v.b = sb[1];
    }
    v.av = to_scalar_regs(reinterpret_cast<const AggVar *>(aa.plan + aa.var_off)[it.var]);
    return v;
}

// Variables that are fp32 at every client: 16-byte pieces, coalesced, bounds-checked at the end.
__device__ __forceinline__ void aggregate_flat_part(const AggArgs &aa, uint32_t block) {
    const AggView v = load_view(aa, aa.flat_first + block / kFlatParts);
    const uint32_t lane = threadIdx.x;
    float *dst = aa.out + v.av.aux_offset;
    const uint64_t begin = static_cast<uint64_t>(v.chunk) * kChunkElems;
    for (uint32_t j = block % kFlatParts; j < kChunkElems / 256; j += kFlatParts) {
        const uint64_t e = begin + (static_cast<uint64_t>(j) * 64 + lane) * 4;
        if (begin + static_cast<uint64_t>(j) * 256 >= v.av.n) break;
        const uint32_t left = e >= v.av.n ? 0u : v.av.n - e < 4 ? static_cast<uint32_t>(v.av.n - e) : 4u;   // this lane's elements
        f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
        for (uint32_t r0 = 0; r0 < aa.nreplicas; r0 += kFlatBatch) {
            f32x4 x[kFlatBatch];
#pragma unroll
            for (uint32_t g = 0; g < kFlatBatch; ++g) {
                x[g] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                if (r0 + g >= aa.nreplicas) continue;
                const float *from = reinterpret_cast<const float *>(v.copy(r0 + g));
                if (left == 4) x[g] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(from + e));
                else
                    for (uint32_t c = 0; c < 3; ++c)
                        if (c < left) x[g][c] = from[e + c];
            }
#pragma unroll
            for (uint32_t g = 0; g < kFlatBatch; ++g)
                if (r0 + g < aa.nreplicas)
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[c] = (r0 + g == 0) ? x[g][c] : acc[c] + x[g][c];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] = acc[c] / aa.count;
        if (left == 4) __builtin_nontemporal_store(acc, reinterpret_cast<f32x4 *>(dst + e));
        else
            for (uint32_t c = 0; c < 3; ++c)
                if (c < left) dst[e + c] = acc[c];
    }
}

// Ragged tails of variables that at least one client quantized: run-time code width, every access checked.  A workgroup takes 256
// elements, a lane every 64th of them, and asks for those of four clients at a time.  What bounds it is latency: with 32 consecutive
// elements per lane, one client's after the other's, and a launch behind the full tiles, sets of odd sizes took, 8 clients of 4 blocks of
// 134 x 273 (41 MB) 128 us, now 12; 6 clients of 15 blocks of 100 x 305 in 16 bits (70 MB) 138, now 22.
__device__ __forceinline__ void aggregate_tail_part(const AggArgs &aa, uint32_t block) {
    const AggView v = load_view(aa, aa.tail_first + block / kTailParts);
    const FmtParams fp = v.av.fp;
    const uint32_t B = fp.bits, lane = threadIdx.x;
    const uint32_t cmask = (B == 32) ? 0xffffffffu : ((1u << B) - 1u);
    const uint64_t e0 = (v.av.n / kTileElems) * kTileElems;
    const uint32_t count = static_cast<uint32_t>(v.av.n - e0), begin = block % kTailParts * kTailPart;
    if (begin >= count) return;
    const uint64_t dw0 = (e0 >> 5) * B;                      // the tail's first dword
    const uint32_t dwords = static_cast<uint32_t>(v.av.total_dwords - dw0);
    constexpr uint32_t kEach = kTailPart / 64, G = kTailBatchClients;
    float acc[kEach] = {};
    for (uint32_t r0 = 0; r0 < aa.nreplicas; r0 += G) {
        uint32_t lo[G][kEach], hi[G][kEach];
#pragma unroll
        for (uint32_t g = 0; g < G; ++g) {
#pragma unroll
            for (uint32_t u = 0; u < kEach; ++u) lo[g][u] = hi[g][u] = 0u;
            if (r0 + g >= aa.nreplicas) continue;
            const uint8_t *copy = v.copy(r0 + g);
            if (v.is_quantized(r0 + g)) {
                const uint32_t *codes = reinterpret_cast<const uint32_t *>(copy) + dw0;
#pragma unroll
                for (uint32_t u = 0; u < kEach; ++u) {
                    const uint32_t i = begin + lane + 64u * u, d = (i * B) >> 5;
                    if (i < count) lo[g][u] = codes[d];
                    if (i < count && d + 1 < dwords) hi[g][u] = codes[d + 1];
                }
            } else {
                const uint32_t *values = reinterpret_cast<const uint32_t *>(copy) + e0;
#pragma unroll
                for (uint32_t u = 0; u < kEach; ++u) {
                    const uint32_t i = begin + lane + 64u * u;
                    if (i < count) lo[g][u] = values[i];
                }
            }
        }
#pragma unroll
        for (uint32_t g = 0; g < G; ++g) {
            if (r0 + g >= aa.nreplicas) continue;
            const bool quantized = v.is_quantized(r0 + g);
            const float s = v.scale(r0 + g), b = v.offset(r0 + g);
#pragma unroll
            for (uint32_t u = 0; u < kEach; ++u) {
                float x = __uint_as_float(lo[g][u]);
                if (quantized) {
                    const uint32_t i = begin + lane + 64u * u;
                    const uint64_t both = (static_cast<uint64_t>(hi[g][u]) << 32) | lo[g][u];
                    const uint32_t code = static_cast<uint32_t>(both >> ((i * B) & 31u)) & cmask;
                    const float vt = decode_top(code << (32u - B), fp);
                    const float sv = s * vt;
                    x = sv + b;
                }
                acc[u] = (r0 + g == 0) ? x : acc[u] + x;
            }
        }
    }
#pragma unroll
    for (uint32_t u = 0; u < kEach; ++u) {
        const uint32_t i = begin + lane + 64u * u;
        if (i < count) aa.out[v.av.aux_offset + e0 + i] = acc[u] / aa.count;
    }
}

// The workgroups of a launch that take tails (the first ones) and all-fp32 items (the last ones); true if this is one of them.
__device__ __forceinline__ bool aggregate_rest(const AggArgs &aa) {
    if (blockIdx.x < aa.tail_blocks) {
        aggregate_tail_part(aa, blockIdx.x);
        return true;
    }
    if (blockIdx.x >= aa.tail_blocks + aa.full_blocks) {
        aggregate_flat_part(aa, blockIdx.x - aa.tail_blocks - aa.full_blocks);
        return true;
    }
    return false;
}

// Full tiles of a variable that at least one client quantized (code width B).  A lane owns 32
// consecutive elements; a client's tile reaches that layout through LDS from coalesced 16-byte
// pieces, whether it holds codes or fp32 values.
template <int B>
__global__ __launch_bounds__(64, kTileWaves) void aggregate_kernel(AggArgs aa) {
    __shared__ __attribute__((aligned(16))) uint32_t lds[kLdsDwords];
    if (aggregate_rest(aa)) return;
    const uint32_t lane = threadIdx.x, block = blockIdx.x - aa.tail_blocks;
    const AggView v = load_view(aa, aa.first_item + block / aa.parts);
    const FmtParams fp = v.av.fp;
    const uint64_t first_tile = static_cast<uint64_t>(v.chunk) * tiles_per_chunk(B);
    const uint64_t full_tiles = v.av.n / kTileElems;
    const uint32_t ntiles = static_cast<uint32_t>(
        (full_tiles - first_tile < tiles_per_chunk(B)) ? full_tiles - first_tile : tiles_per_chunk(B));
    for (uint32_t t = block % aa.parts; t < ntiles; t += aa.parts) {
        const uint64_t e0 = (first_tile + t) * kTileElems;
        float acc[32];
        for (uint32_t r = 0; r < aa.nreplicas; ++r) {
            const uint8_t *copy = v.copy(r);
            float val[32];
            if (v.is_quantized(r)) {
                const float sc = v.scale(r), of = v.offset(r);
                u32x4 cq[CodePieces<B>::rounds];
                load_code_pieces<B, OMC_TUNE_AGG_NT != 0>(reinterpret_cast<const uint32_t *>(copy) + (e0 >> 5) * B, lane, cq);
                uint32_t w[B];
                code_pieces_to_lanes<B>(cq, w, lds, lane);
#pragma unroll
                for (int i = 0; i < 32; ++i) {
                    const float vt = decode_top(code_at_top<B>(w, i), fp);
                    const float sv = sc * vt;
                    val[i] = sv + of;
                }
            } else {
                f32x4 g[8];
                load_f32_pieces<true>(reinterpret_cast<const float *>(copy) + e0, lane, g);
                pieces_to_lanes(g, val, lds, lane);
            }
#pragma unroll
            for (int i = 0; i < 32; ++i) acc[i] = (r == 0) ? val[i] : acc[i] + val[i];
        }
#pragma unroll
        for (int i = 0; i < 32; ++i) acc[i] = acc[i] / aa.count;
        f32x4 o[8];
        lanes_to_pieces(acc, o, lds, lane);
        store_f32_pieces<true>(aa.out + v.av.aux_offset + e0, lane, o);
    }
}

// Byte codes need no transposition: a lane takes dwords of four codes at the same element offsets as
// its 16-byte pieces of the fp32 copies and of the output (slab of 1024 elements: piece j of lane l =
// elements 256 j + 4 l ..).  Everything stays coalesced and LDS is not used.  S1E4M3 / bias 7 is
// decoded by the hardware's FP8 conversion; its one deviating code (the top code reads as NaN) leaves a
// NaN in the sums, and such a slab is redone with the generic decode.
template <bool HW>
__device__ __forceinline__ void aggregate_byte_slab(const AggArgs &aa, const AggView &v, const FmtParams &fp, uint64_t e0,
                                                    uint32_t lane, f32x4 (&acc)[4]) {
    for (uint32_t r0 = 0; r0 < aa.nreplicas; r0 += kByteBatch) {
        f32x4 in[kByteBatch][4];                              // four codes (in the first element) or values
#pragma unroll
        for (uint32_t g = 0; g < kByteBatch; ++g) {
            if (r0 + g >= aa.nreplicas) continue;
            const uint8_t *copy = v.copy(r0 + g);
            if (v.is_quantized(r0 + g)) {
                const uint32_t *c = reinterpret_cast<const uint32_t *>(copy) + (e0 >> 2);
#pragma unroll
                for (int j = 0; j < 4; ++j) in[g][j][0] = __uint_as_float(OMC_TUNE_AGG_NT ? __builtin_nontemporal_load(c + (64 * j + lane)) : c[64 * j + lane]);
            } else {
                const f32x4 *x = reinterpret_cast<const f32x4 *>(reinterpret_cast<const float *>(copy) + e0);
#pragma unroll
                for (int j = 0; j < 4; ++j) in[g][j] = __builtin_nontemporal_load(x + (64 * j + lane));
            }
        }
#pragma unroll
        for (uint32_t g = 0; g < kByteBatch; ++g) {
            if (r0 + g >= aa.nreplicas) continue;
            const bool quantized = v.is_quantized(r0 + g);
            const float sc = v.scale(r0 + g), of = v.offset(r0 + g);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f32x4 val = in[g][j];
                if (quantized) {
                    const uint32_t w = __float_as_uint(in[g][j][0]);
                    float vt[4];
                    if (HW) {
                        const f32x2 lo = __builtin_amdgcn_cvt_pk_f32_fp8(static_cast<int>(w), false);
                        const f32x2 hi = __builtin_amdgcn_cvt_pk_f32_fp8(static_cast<int>(w), true);
                        vt[0] = lo[0]; vt[1] = lo[1]; vt[2] = hi[0]; vt[3] = hi[1];
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i) vt[i] = decode_top(w << (24 - 8 * i), fp);
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float sv = sc * vt[i];
                        val[i] = sv + of;
                    }
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[j][i] = (r0 + g == 0) ? val[i] : acc[j][i] + val[i];
            }
        }
    }
}

__global__ __launch_bounds__(64, kByteWaves) void aggregate_byte_kernel(AggArgs aa) {
    if (aggregate_rest(aa)) return;
    const uint32_t lane = threadIdx.x, block = blockIdx.x - aa.tail_blocks;
    const AggView v = load_view(aa, aa.first_item + block / aa.parts);
    const FmtParams fp = v.av.fp;
    const uint64_t first_tile = static_cast<uint64_t>(v.chunk) * tiles_per_chunk(8);
    const uint64_t full_tiles = v.av.n / kTileElems;
    const uint32_t ntiles = static_cast<uint32_t>(
        (full_tiles - first_tile < tiles_per_chunk(8)) ? full_tiles - first_tile : tiles_per_chunk(8));
    const bool hw = fp.variant == 2;
    for (uint32_t sl = block % aa.parts; sl < 2 * ntiles; sl += aa.parts) {
        const uint64_t e0 = first_tile * kTileElems + static_cast<uint64_t>(sl) * 1024;
        f32x4 acc[4];
        bool done = false;
        if (hw) {
            aggregate_byte_slab<true>(aa, v, fp, e0, lane, acc);
            bool bad = false;
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i) bad = bad || (acc[j][i] != acc[j][i]);
            done = !__any(bad);
        }
        if (!done) aggregate_byte_slab<false>(aa, v, fp, e0, lane, acc);
        f32x4 *dst = reinterpret_cast<f32x4 *>(aa.out + v.av.aux_offset + e0);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            f32x4 o;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = acc[j][i] / aa.count;
            __builtin_nontemporal_store(o, dst + (64 * j + lane));
        }
    }
}

// tails and all-fp32 items alone (no full-tile launch to ride on)
__global__ __launch_bounds__(64) void aggregate_rest_kernel(AggArgs aa) { aggregate_rest(aa); }

// Workgroups that share a work item: its slabs of byte codes or its tiles, where the items alone are too few to fill the chip.
static uint32_t parts_of(uint32_t bits, uint32_t nitems) {
    const uint32_t most = bits == 8 ? 2 * tiles_per_chunk(8) : tiles_per_chunk(bits);
    uint32_t parts = 1;
    while (parts < most && nitems * static_cast<uint64_t>(parts) < kEnoughBlocks) parts *= 2;
    return parts;
}

int launch_aggregate_mean(const AggHeader *ah, const void *agg_dev, const AggPointers &ptrs, float *out,
                          void *stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    const PlanGroup *groups = reinterpret_cast<const PlanGroup *>(reinterpret_cast<const uint8_t *>(ah) + ah->group_off);
    AggArgs aa{};
    aa.plan = static_cast<const uint8_t *>(agg_dev);
    aa.var_off = ah->var_off;
    aa.src_off = ah->src_off;
    aa.item_off = ah->item_off;
    aa.nreplicas = ah->nreplicas;
    aa.count = static_cast<float>(ah->nreplicas);
    aa.p = ptrs;
    aa.out = out;
    // the tails and the all-fp32 items ride on the first full-tile launch
    const PlanGroup *flat = nullptr, *tail = nullptr;
    for (uint32_t gi = 0; gi < ah->ngroups; ++gi) {
        if (groups[gi].kind == kGroupFp32 && groups[gi].nitems > 0) flat = &groups[gi];
        if (groups[gi].kind == kGroupTail && groups[gi].nitems > 0) tail = &groups[gi];
    }
    uint32_t tails = 0, tails_left = tail ? tail->nitems : 0, flats = 0, flats_left = flat ? flat->nitems : 0;
    auto take_rest = [&]() -> uint64_t {                     // at most one launch's share of what is left: its workgroups
        aa.tail_first = tail ? tail->first_item + tails : 0;
        aa.flat_first = flat ? flat->first_item + flats : 0;
        const uint32_t nt = std::min(tails_left, kMostSharingBlocks / kTailParts), nf = std::min(flats_left, kMostSharingBlocks / kFlatParts);
        tails += nt;
        tails_left -= nt;
        flats += nf;
        flats_left -= nf;
        aa.tail_blocks = nt * kTailParts;
        return static_cast<uint64_t>(aa.tail_blocks) + nf * kFlatParts;
    };
    for (uint32_t gi = 0; gi < ah->ngroups; ++gi) {
        const PlanGroup &g = groups[gi];
        if (g.nitems == 0 || g.kind != kGroupFull) continue;
        aa.first_item = g.first_item;
        aa.parts = parts_of(g.bits, g.nitems);
        const uint64_t blocks = static_cast<uint64_t>(g.nitems) * aa.parts + take_rest();
        if (blocks > 0x7fffffffull) return static_cast<int>(hipErrorInvalidValue);
        aa.full_blocks = g.nitems * aa.parts;
        const dim3 grid(static_cast<uint32_t>(blocks));
        if (g.bits == 8) {
            aggregate_byte_kernel<<<grid, dim3(64), 0, st>>>(aa);
        } else {
            switch (g.bits) {
#define X(BITS) case BITS: aggregate_kernel<BITS><<<grid, dim3(64), 0, st>>>(aa); break;
                OMC_FOR_EACH_BITS(X)
#undef X
                default: return static_cast<int>(hipErrorInvalidValue);
            }
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return static_cast<int>(e);
    }
    while (tails_left > 0 || flats_left > 0) {               // what no full tile's launch took
        const uint64_t blocks = take_rest();
        aa.full_blocks = 0;
        aggregate_rest_kernel<<<dim3(static_cast<uint32_t>(blocks)), dim3(64), 0, st>>>(aa);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return static_cast<int>(e);
    }
    return 0;
}

}  // namespace omc
