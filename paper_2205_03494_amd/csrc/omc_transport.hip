// Device side of omc_transport_pack (paper Sec. 1: parameters are kept and transported in compressed
// form).  Pure data movement: no arithmetic of the method happens here.
#include "omc_stream.h"

namespace omc {

constexpr int kMetaThreads = 1024;   // at most: one wave for every 64 variables up to there

// What the message says of variable i: its record and its (s, b).  Returns the record's share of the checksum.
__device__ __forceinline__ uint64_t write_record(const PlanVar &pv, uint32_t i, uint64_t payload_offset, const float *__restrict__ sb_table, uint8_t *__restrict__ msg,
                                                 const TransportHeader &th) {
    TransportVar tv;
    tv.payload_offset = payload_offset;
    tv.aux_offset = pv.aux_offset;
    tv.n = pv.n;
    const bool q = (pv.flags & OMC_VAR_QUANTIZED) != 0;
    tv.exp_bits = q ? static_cast<uint8_t>(pv.fp.exp_bits) : 8;
    tv.man_bits = q ? static_cast<uint8_t>(pv.fp.man_bits) : 23;
    tv.exp_bias = q ? static_cast<int16_t>(pv.fp.bias) : 127;
    tv.flags = pv.flags;
    reinterpret_cast<TransportVar *>(msg + sizeof(TransportHeader))[i] = tv;
    float *sb_out = reinterpret_cast<float *>(msg + th.sb_off) + 2 * static_cast<uint64_t>(i);
    sb_out[0] = q ? sb_table[2 * static_cast<uint64_t>(pv.sb_index)] : 1.0f;
    sb_out[1] = q ? sb_table[2 * static_cast<uint64_t>(pv.sb_index) + 1] : 0.0f;
    return transport_var_hash(i, tv);
}

// The header with the checksum, once the workgroup's records are written; `wave_sum`: a word a wave.
__device__ __forceinline__ void write_header(uint64_t hash_sum, uint64_t *wave_sum, uint8_t *__restrict__ msg, TransportHeader &th) {
    for (int off = 32; off >= 1; off >>= 1) hash_sum += __shfl_xor(hash_sum, off);
    __syncthreads();
    if ((threadIdx.x & 63u) == 0) wave_sum[threadIdx.x >> 6] = hash_sum;
    __syncthreads();
    if (threadIdx.x != 0) return;
    hash_sum = 0;
    for (uint32_t w = 0; w < blockDim.x / 64; ++w) hash_sum += wave_sum[w];
    th.checksum = transport_header_hash(th, hash_sum);
    *reinterpret_cast<TransportHeader *>(msg) = th;
}

// One workgroup: walks the plan's variable table in order, gives every variable its 16-byte aligned place
// in the payload (a running sum of the sizes), writes the message's variable table and (s, b) table, and
// finally the header with the checksum over both.
__global__ __launch_bounds__(kMetaThreads) void transport_meta_kernel(const uint8_t *__restrict__ plan, uint64_t var_off,
                                                                       const float *__restrict__ sb_table,
                                                                       uint8_t *__restrict__ msg, TransportHeader th) {
    __shared__ uint64_t wave_sum[kMetaThreads / 64];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, threads = blockDim.x, waves = threads / 64;
    const PlanVar *vars = reinterpret_cast<const PlanVar *>(plan + var_off);
    uint64_t carry = 0;                                         // the same in every thread
    uint64_t hash_sum = 0;
    for (uint32_t base = 0; base < th.nvars; base += threads) {
        const uint32_t i = base + tid;
        uint64_t bytes = 0;
        PlanVar pv{};
        if (i < th.nvars) {
            pv = vars[i];
            bytes = (pv.flags & OMC_VAR_QUANTIZED) ? pv.total_dwords * 4 : (4 * pv.n + 15) / 16 * 16;
        }
        uint64_t upto = bytes;                                   // inclusive scan of the sizes: within the wave ...
        for (int off = 1; off < 64; off <<= 1) {
            const uint64_t add = __shfl_up(upto, off);
            if (lane >= static_cast<uint32_t>(off)) upto += add;
        }
        __syncthreads();                                         // (the sums of the round before are read)
        if (lane == 63) wave_sum[wave] = upto;
        __syncthreads();
        uint64_t total = 0;                                      // ... and over the waves before it
        for (uint32_t w = 0; w < waves; ++w) {
            if (w == wave) upto += carry + total;
            total += wave_sum[w];
        }
        carry += total;
        if (i < th.nvars) hash_sum += write_record(pv, i, upto - bytes, sb_table, msg, th);
    }
    write_header(hash_sum, wave_sum, msg, th);
}

// The payload in runs of 32 KB (of less, down to 2 KB, where that would be fewer than 1024), one workgroup each: up to eight 16-byte pieces
// per thread, all in flight together.  Most arenas are laid out like a payload: in table order, without gaps but for the padding to 16 bytes.  Such a DENSE set's runs are found in the plan, the
// places being the arena's own, and the table, (s, b) and header are written beside the copies, by the first workgroup of the only launch: a round's change and its message, 599 variables in 11 bits 135.8 -> 131.5 us;
// 4 blocks of 170 x 511 in three formats 32.5 -> 27.0.  Of any other set a run is found in the message's own table, which the meta kernel has written before.  Of a set of up to 256
// variables every thread takes one entry to LDS; of a larger one the threads look at one entry in every `stride`, then at the entries
// between, two dependent loads.  A run that lies in one variable is copied by all threads; in the others each wave takes one variable
// after the other.  Large messages are bound by memory (both streams are touched once and carry the hint): 190.7 MB of 599 variables 60 us; with
// 64 workgroups per variable, whatever its size, and four pieces per thread 71 us.  Small ones are bound by dependent loads, above all
// by the variables that a wave takes one after the other: 100 variables of 1000 11-bit codes 5.8 us, 11.2 with runs of 32 KB and a table
// made by 1024 threads; 3000 variables of 300 codes 18 us, 33 so.
constexpr uint32_t kPackThreads = 256, kPackBatch = 8;
constexpr uint64_t kPackLongest = 16ull * kPackThreads * kPackBatch, kPackShortest = 2048, kPackRuns = 1024;
inline uint64_t pack_run(uint64_t payload_bytes) {
    const uint64_t even = (payload_bytes / kPackRuns + kPackShortest - 1) / kPackShortest * kPackShortest;
    return even < kPackShortest ? kPackShortest : even > kPackLongest ? kPackLongest : even;
}

// pieces [p0, p1) of a variable by THREADS threads, `t` being this one; `bytes` is the variable's size in the arena
template <uint32_t THREADS>
__device__ __forceinline__ void pack_pieces(const uint8_t *src8, uint8_t *dst8, uint64_t bytes, uint64_t p0, uint64_t p1, uint32_t t) {
    const u32x4 *src = reinterpret_cast<const u32x4 *>(src8);
    u32x4 *dst = reinterpret_cast<u32x4 *>(dst8);
    const uint64_t full = bytes / 16, end = p1 < full ? p1 : full;
    for (uint64_t p = p0 + t; p < end; p += THREADS * kPackBatch) {
        u32x4 x[kPackBatch];
#pragma unroll
        for (uint32_t u = 0; u < kPackBatch; ++u)
            if (p + u * THREADS < end) x[u] = __builtin_nontemporal_load(src + p + u * THREADS);
#pragma unroll
        for (uint32_t u = 0; u < kPackBatch; ++u)
            if (p + u * THREADS < end) __builtin_nontemporal_store(x[u], dst + p + u * THREADS);
    }
    if (t == 0 && p0 <= full && full < p1 && bytes % 16) {        // an fp32 variable whose size is no multiple of four
        const uint32_t *s = reinterpret_cast<const uint32_t *>(src + full);
        uint32_t *d = reinterpret_cast<uint32_t *>(dst + full);
        const uint32_t left = static_cast<uint32_t>(bytes % 16) / 4;
        for (uint32_t k = 0; k < 4; ++k) d[k] = k < left ? s[k] : 0u;
    }
}

template <bool DENSE>
__global__ __launch_bounds__(kPackThreads) void transport_pack_kernel(const uint8_t *__restrict__ plan, uint64_t var_off,
                                                                      const uint8_t *__restrict__ arena, const float *__restrict__ sb_table,
                                                                      uint8_t *__restrict__ msg, TransportHeader th, uint64_t run) {
    const PlanVar *vars = reinterpret_cast<const PlanVar *>(plan + var_off);
    const TransportVar *tvs = reinterpret_cast<const TransportVar *>(msg + sizeof(TransportHeader));
    const uint32_t tid = threadIdx.x, nvars = th.nvars;
    const uint64_t arena_first = DENSE ? vars[0].data_offset : 0;
    auto place = [&](uint32_t i) { return DENSE ? vars[i].data_offset - arena_first : tvs[i].payload_offset; };   // in the payload
    if (DENSE && blockIdx.x == 0) {
        __shared__ uint64_t wave_sum[kPackThreads / 64];
        uint64_t hash_sum = 0;
        for (uint32_t i = tid; i < nvars; i += kPackThreads) hash_sum += write_record(vars[i], i, place(i), sb_table, msg, th);
        write_header(hash_sum, wave_sum, msg, th);
        return;
    }
    const uint64_t payload_off = th.payload_off, payload_bytes = th.payload_bytes;
    const uint64_t lo = static_cast<uint64_t>(blockIdx.x - (DENSE ? 1 : 0)) * run, hi = lo + run < payload_bytes ? lo + run : payload_bytes;
    struct Entry {
        uint64_t to, from, bytes;                             // place in the payload, place in the arena, size there
    };
    auto look_up = [&](uint32_t i) {
        const PlanVar &pv = vars[i];
        return Entry{place(i), pv.data_offset, (pv.flags & OMC_VAR_QUANTIZED) ? pv.total_dwords * 4 : 4 * pv.n};
    };
    __shared__ Entry table[kPackThreads];                     // of a set that it holds: one round trip for all of it
    const bool in_table = nvars > 1 && nvars <= kPackThreads;
    auto entry = [&](uint32_t i) { return in_table ? table[i] : look_up(i); };
    // the last variable that starts at or before lo (variable 0 starts at 0)
    uint32_t first = 0;
    if (in_table) {
        Entry mine{};
        if (tid < nvars) table[tid] = mine = look_up(tid);
        first = static_cast<uint32_t>(__syncthreads_count(tid < nvars && mine.to <= lo)) - 1;   // offsets ascend
    }
    for (uint32_t span = in_table ? 1 : nvars; span > 1;) {
        const uint32_t stride = (span + kPackThreads - 1) / kPackThreads, at = first + tid * stride;
        const bool below = tid * stride < span && place(at) <= lo;
        const uint32_t steps = static_cast<uint32_t>(__syncthreads_count(below)) - 1;   // entry `first` is below
        const uint32_t rest = span - steps * stride;
        first += steps * stride;
        span = rest < stride ? rest : stride;
    }
    const Entry e = to_scalar_regs(entry(first));
    uint8_t *payload = msg + payload_off;
    if (e.to + (e.bytes + 15) / 16 * 16 >= hi) {
        pack_pieces<kPackThreads>(arena + e.from, payload + e.to, e.bytes, (lo - e.to) / 16, (hi - e.to) / 16, tid);
        return;
    }
    for (uint32_t i = first + (tid >> 6); i < nvars; i += kPackThreads / 64) {
        const Entry w = to_scalar_regs(entry(i));
        if (w.to >= hi) return;
        const uint64_t end = w.to + (w.bytes + 15) / 16 * 16;
        pack_pieces<64>(arena + w.from, payload + w.to, w.bytes, lo > w.to ? (lo - w.to) / 16 : 0, ((end < hi ? end : hi) - w.to) / 16, tid & 63u);
    }
}

int launch_transport_pack(const PlanHeader *ph, const void *plan_dev, const void *arena, bool dense, const float *sb_table,
                          void *msg_dev, const TransportHeader &th, void *stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    const uint8_t *plan = static_cast<const uint8_t *>(plan_dev), *from = static_cast<const uint8_t *>(arena);
    uint8_t *msg = static_cast<uint8_t *>(msg_dev);
    const uint64_t run = pack_run(th.payload_bytes), runs = (th.payload_bytes + run - 1) / run;
    if (runs > 0x7ffffffeull) return static_cast<int>(hipErrorInvalidValue);
    if (dense) {
        transport_pack_kernel<true><<<dim3(static_cast<uint32_t>(runs) + 1), dim3(kPackThreads), 0, st>>>(plan, ph->var_off, from, sb_table, msg, th, run);
        return static_cast<int>(hipGetLastError());
    }
    transport_meta_kernel<<<dim3(1), dim3(ph->nvars < kMetaThreads ? (ph->nvars + 63) / 64 * 64 : kMetaThreads), 0, st>>>(plan, ph->var_off, sb_table, msg, th);
    const int rc = static_cast<int>(hipGetLastError());
    if (rc != 0) return rc;
    transport_pack_kernel<false><<<dim3(static_cast<uint32_t>(runs)), dim3(kPackThreads), 0, st>>>(plan, ph->var_off, from, sb_table, msg, th, run);
    return static_cast<int>(hipGetLastError());
}

}  // namespace omc
