// The tiles of 256 rows of the products on codes of any width: WN column waves, two row waves, each of 4 x 2 matrix tiles of 32 x 32: 256 x 256 by eight waves, 256 x 128 by four.
//
// Built like gemm_bits_kernel, but on matrix instructions of 32 x 32 x 16.  A wave decodes 32 codes a step beside its products, 3 vector instructions in every 16 clocks, and with the
// smaller matrix instructions there is then an instruction to issue in every slot.  256 x 256, 11 bits, 8192 x 4096 x 1024 / 8192 x 4096 x 4096: 80 / 243 us this way, 86 / 258 with 16 x 16 x 32 (other orders of
// the fragments, two or four row tiles at a time, decoding in place or a step ahead: 85 - 88 / 256 - 270), though those take less power; no part of a step stands out there either: without the decoding
// 80 / 231, without the loads of A 81 / 229, without reading its fragments 81 / 238.  256 x 128, 13 bits, 5632 x 1280 x 2560 50.3 / 53.2 us, 2816 x 2432 x 3136 58.8 / 60.7, 7936 x 1024 x 1472 34.0 / 33.0.
#pragma once
#include "omc_gemm_bits_codes.h"

#pragma clang fp contract(off)

namespace omc {

typedef float f32x16 __attribute__((ext_vector_type(16)));

template <int B, int WN, bool TRANS, bool HW>
__global__ __attribute__((amdgpu_flat_work_group_size(128 * WN, 128 * WN))) __attribute__((amdgpu_waves_per_eu(WN / 2, WN / 2)))
void gemm_bits_large_kernel(BitsArgs ga) {
    constexpr int U = 32, WM = 2, TM = 4, TN = 2, NW = WM * WN, BM = 32 * TM * WM, BN = 32 * TN * WN;
    constexpr int kALoads = BM / 8 / NW, kGroups = BN / 32, kRowUnits = BN / U;
    constexpr uint32_t kABytes = BM * 128, kStage = kABytes + BN * 128;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[2 * kStage];
    const uint32_t lds0 = lds_offset(lds);
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave / WN, wn = wave % WN;
    const uint32_t N = ga.N, K = ga.K;
    const FmtParams fp = ga.fp;
    uint32_t m0, n0;
    tile_of_block(4, ga.tiles_m, ga.tiles_n, m0, n0);
    m0 *= BM;
    n0 *= BN;

    // ---- global -> LDS / registers.  The last step may be half empty (K % 64 == 32): the upper half is then the lower one again
    // instead of a read past the row, and nobody multiplies it
    const uint32_t full = K / 64, steps = (K + 63) / 64;
    const uint8_t *a_base = reinterpret_cast<const uint8_t *>(ga.A) + static_cast<uint64_t>(m0) * K * 2;
    const uint32_t a_row = lane >> 3, a_piece = (lane & 7u) ^ ((a_row >> 1) + 4 * (wave & 1u));
    auto load_a = [&](uint32_t at, uint32_t j) {
        const uint32_t a_off = a_row * K * 2 + (j == full ? a_piece & 3u : a_piece) * 16;
#pragma unroll
        for (int q = 0; q < kALoads; ++q) {
            const uint32_t c = wave + NW * q;                 // rows 8 c ..
            load_to_lds(a_base + static_cast<uint64_t>(j) * 128 + static_cast<uint64_t>(c) * 16 * K, a_off, lds0 + at + c * 1024);
        }
    };
    // this thread's unit: TRANS column u_row, part u_part of its 64 k; forward k row u_row, part u_part of its BN columns
    constexpr uint32_t kParts = TRANS ? 64 / U : kRowUnits, kPieces = U / 8;
    const uint32_t u_row = tid / kParts, u_part = tid % kParts;
    auto load_w = [&](uint32_t j, Unit<B, U> &u) {
        const bool half = j == full;
        const uint64_t e = TRANS ? (static_cast<uint64_t>(n0 + u_row) * K + static_cast<uint64_t>(j) * 64 + U * (half ? 0 : u_part))
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
    auto store_piece = [&](uint32_t at, const Pairs<B, U, HW> &u, int i) {
        u32x4 piece;
#pragma unroll
        for (int p = 0; p < 4; ++p) piece[p] = u.pair(4 * i + p, fp);
        *reinterpret_cast<u32x4 *>(lds + at + u_at[i]) = piece;
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

    f32x16 acc[TM][TN];
    float rsum[TM];                                             // its share of the row sums of A: of the quarter of a step that it multiplies first, with two column waves also the third
    auto add_row_sums = [&](const Frags &f) {
#pragma unroll
        for (int mi = 0; mi < TM; ++mi) {
            const bf16x2 ones = {static_cast<__bf16>(1.0f), static_cast<__bf16>(1.0f)};
            const u32x4 x = __builtin_bit_cast(u32x4, f.a[mi]);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t two = x[i];
                rsum[mi] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, two), ones, rsum[mi], false);
            }
        }
    };
    auto multiply = [&](const Frags &f) {
#pragma unroll
        for (int ni = 0; ni < TN; ++ni)
#pragma unroll
            for (int mi = 0; mi < TM; ++mi)
                acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[mi], f.w[ni], acc[mi][ni], 0, 0, 0);
    };

    // step i: A and W of the step are in stage `cur`; the dwords of step i + 1 are in `next` (asked for during step i - 1)
    Frags f0, f1;
    uint32_t cur = 0;
    Unit<B, U> next;
    Pairs<B, U, HW> now;
#pragma unroll
    for (int i = 0; i < Unit<B, U>::kDwords; ++i) next.w[i] = 0;
#pragma unroll
    for (int mi = 0; mi < TM; ++mi) {
        rsum[mi] = 0.0f;
#pragma unroll
        for (int ni = 0; ni < TN; ++ni)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.0f;
    }
    load_a(0, 0);
    load_w(0, next);
    now.take(next, 0);
    if (steps > 1) load_w(1, next);
#pragma unroll
    for (int i = 0; i < static_cast<int>(kPieces); ++i) store_piece(0, now, i);
    auto step = [&](uint32_t i, bool first, bool more1, bool more2) {
        wait_loads_and_sync<0>();
#pragma unroll
        for (int q = 0; q < Unit<B, U>::kDwords; ++q) pin(next.w[q]);   // they have arrived: their uses need no wait of their own
        now.take(next, 0);
        const uint32_t other = kStage - cur;
        read_frags(cur, a_at[0], w_at[0], f0);
        if (more1) load_a(other, i + 1);
        if (more2) load_w(i + 2, next);
        if (!first) multiply(f1);
        read_frags(cur, a_at[1], w_at[1], f1);
        if (more1) store_piece(other, now, 0);
        multiply(f0);
        add_row_sums(f0);
        read_frags(cur, a_at[2], w_at[2], f0);
        if (more1) store_piece(other, now, 1);
        multiply(f1);
        read_frags(cur, a_at[3], w_at[3], f1);
        if (more1) store_piece(other, now, 2);
        multiply(f0);
        if (WN == 2) add_row_sums(f0);
        if (more1) store_piece(other, now, 3);
        cur = other;
    };
    if (full > 0) {
        step(0, true, steps > 1, steps > 2);
        uint32_t i = 1;
        for (; i + 2 < steps; ++i) step(i, false, true, true);
        for (; i < full; ++i) step(i, false, i + 1 < steps, i + 2 < steps);
        multiply(f1);
    }
    if (full < steps) {                                       // 32 k more: two quarters
        wait_loads_and_sync<0>();
        auto quarter = [&](auto ks) {
            read_frags(cur, a_place(ks.value), w_place(ks.value), f0);
            multiply(f0);
            if (ks.value % WN == wn) add_row_sums(f0);
        };
        quarter(UintTag<0>{});
        quarter(UintTag<1>{});
    }
    wait_loads_and_sync<0>();                                 // nobody reads a stage any more
    const float s = ga.sb ? ga.sb[0] : 1.0f, b = ga.sb ? ga.sb[1] : 0.0f;
    float *rowsum = reinterpret_cast<float *>(lds);            // [WN][BM]
    const uint32_t row0 = 32 * TM * wm;
#pragma unroll
    for (int mi = 0; mi < TM; ++mi) {
        const float t = rsum[mi] + __shfl_xor(rsum[mi], 32);
        if (lane < 32) rowsum[wn * BM + row0 + 32 * mi + lane] = ga.sb ? t : 0.0f;   // without an offset they must not enter the result, whatever they are
    }
    __syncthreads();
    float *C = ga.C + static_cast<uint64_t>(m0) * N + n0 + 32 * TN * wn + f_row;
#pragma unroll
    for (int mi = 0; mi < TM; ++mi) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {                         // two rows of 128 bytes a store, non-temporal as in the other kernels
            const uint32_t row = row0 + 32 * mi + 8 * (v >> 2) + 4 * f_half + (v & 3);
            float sum = rowsum[row];
#pragma unroll
            for (int q = 1; q < WN; ++q) sum += rowsum[q * BM + row];
            const float add = b * sum;
#pragma unroll
            for (int ni = 0; ni < TN; ++ni) __builtin_nontemporal_store(s * acc[mi][ni][v] + add, C + static_cast<uint64_t>(row) * N + 32 * ni);
        }
    }
}

}  // namespace omc
