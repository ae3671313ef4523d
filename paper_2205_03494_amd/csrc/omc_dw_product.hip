// The weight gradient dW[K x N] = X^T dY of omc_dw_update_recompress (paper Sec. 2.1, backward propagation: decompress the layer's
// parameters, apply the gradients, compress, discard), either as `nsplit` partial sums over runs of the M rows, row-major in the
// workspace, which the update kernels add in order; or, for 8-bit codes, consumed in the epilogue: the tile of the gradient
// goes to LDS, a thread takes four consecutive weights of a row at a time, one dword of codes, decodes and transforms them
// (Sec. 2.2, 2.3), updates, rounds, stores them back and takes the sums of the fit, and the fp32 gradient is nowhere in memory
// (unless the caller asks for a copy).
//
// Both operands lie along the contraction, X as [M x K] and dY as [M x N], and go from global memory straight into a ring of S LDS
// stages of 32 rows, as they are.  The transposing 16-bit read (ds_read_b64_tr_b16) makes matrix fragments of them: of 16 lanes
// that point at four rows x 16 columns, lane c receives column c's four rows.  Staging costs no vector instruction.  On the way in
// (the lane picks the piece, its LDS place is fixed) the 64-byte groups of a row are exchanged by the lowest bits of the row and the 16-byte pieces in them by its bit 3: the eight rows of
// one read then lie on different banks.
//
// A weight matrix gives few tiles (4 M weights = 128 of 256 x 128) and the contraction is long, so it is shared out twice: between
// TEAMS of waves of a workgroup, which add up their tiles through LDS, and between workgroups (nsplit).
//
// Matrix instructions of 16 x 16 x 32 and the order of reads and products written down, a column of tiles at a time: 8192 rows, 4096 x 1024 weights, 8 bits, momentum, with the update: 3 of 77 us less than 32 x 32 x 16 and the compiler's order.
//
// A stage is asked for behind the products that hide the step's first reads, not before them: 8448 rows, 4864 x 1024 weights 111 -> 104 us (105 with 32 x 32 x 16), 4096 rows, 4096 x 2048 76.5 -> 72.3.
//
// What bounds it: power (2.0 GHz of 2.4, that size) and the loads (at the matrix cores' rate 64 bytes per clock and compute unit with 128 x 128 tiles, 48 with 256 x 128), not the LDS reads: plain or 16-byte reads in their place change nothing.
#include "omc_dw_args.h"
#include "omc_mma.h"

namespace omc {

struct ProductArgs {
    const uint16_t *X, *dY;
    float *partials;                     // [nsplit][K][N]
    uint32_t N, K, steps, nsplit;        // steps of 32 rows in all
    uint32_t tiles_k, tiles_n, group_rows;
};

// Epilogue of the one-kernel route on a tile [ROWS][COLS] of the gradient in LDS, by all THREADS of the workgroup.
template <int ROWS, int COLS, int THREADS, int MODE, bool WIDE>
__device__ __forceinline__ void update_tile(const DwArgs &a, const float *grad, uint32_t k0, uint32_t n0, FitAcc &fit) {
    constexpr int kPieces = ROWS * COLS / 4 / THREADS, kMost = MODE == kStepAdam ? 2 : 4, kBatch = kPieces < kMost ? kPieces : kMost;
    static_assert(kPieces * 4 * THREADS == ROWS * COLS && kPieces % kBatch == 0, "whole batches of whole pieces");
    const float s = to_scalar_regs(a.sb[0]), b = to_scalar_regs(a.sb[1]);
    const FmtParams fp = a.fp;
    for (int i = 0; i < kPieces; i += kBatch) {
        uint32_t cw[kBatch];
        f32x4 g4[kBatch], m4[kBatch], v4[kBatch];
        uint64_t e[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const uint32_t q = (i + u) * THREADS + threadIdx.x;
            e[u] = static_cast<uint64_t>(k0 + q / (COLS / 4)) * a.N + n0 + 4 * (q % (COLS / 4));
            cw[u] = a.codes[e[u] >> 2];
            if (MODE >= kStepMomentum) m4[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(a.st0 + e[u]));
            if (MODE == kStepAdam) v4[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(a.st1 + e[u]));
            g4[u] = reinterpret_cast<const f32x4 *>(grad)[q];
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            pin(cw[u]);
            uint32_t out = 0;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float vt = decode_top(cw[u] << (24 - 8 * c), fp);
                const float sv = s * vt;
                float x = sv + b;
                float mm = MODE >= kStepMomentum ? m4[u][c] : 0.0f, vv = MODE == kStepAdam ? v4[u][c] : 0.0f;
                x = apply_update<MODE>(x, g4[u][c], mm, vv, a.oc);
                if (MODE >= kStepMomentum) m4[u][c] = mm;
                if (MODE == kStepAdam) v4[u][c] = vv;
                uint32_t code;
                float tq;
                encode<WIDE>(x, fp, code, tq);
                fit.seed(tq);
                fit.add(x, tq);
                out |= code << (8 * c);
            }
            // keep the pieces in program order: the arithmetic must not pile up above the serial fp64 accumulation
            fit.pin_sums();
            pin(out);
            a.codes[e[u] >> 2] = out;
            if (MODE >= kStepMomentum) __builtin_nontemporal_store(m4[u], reinterpret_cast<f32x4 *>(a.st0 + e[u]));
            if (MODE == kStepAdam) __builtin_nontemporal_store(v4[u], reinterpret_cast<f32x4 *>(a.st1 + e[u]));
            if (a.dW_out) __builtin_nontemporal_store(g4[u], reinterpret_cast<f32x4 *>(a.dW_out + e[u]));
        }
    }
}

// WM x WN waves of TM x TN matrix tiles (16 x 16) each, TEAMS times; S stages, OCC waves per SIMD.  MODE: kPark for partial sums, else
// the optimizer of the one-kernel route.
constexpr int kPark = -1;
template <int WM, int WN, int TM, int TN, int TEAMS, int S, int OCC, int MODE>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * WM * WN * TEAMS, 64 * WM * WN * TEAMS))) __attribute__((amdgpu_waves_per_eu(OCC, OCC)))
void dw_product_kernel(ProductArgs pa, DwArgs a) {
    constexpr int NW = WM * WN, BK = 16 * TM * WM, BN = 16 * TN * WN;
    constexpr int kXLoads = BK / 16 / NW, kYLoads = BN / 16 / NW, kLoads = kXLoads + kYLoads;   // 1 KB loads per wave and stage
    constexpr uint32_t kXBytes = BK * 64, kStage = kXBytes + BN * 64;
    static_assert(BK % (16 * NW) == 0 && BN % (16 * NW) == 0, "whole loads");
    // (the one-kernel route's sums lie behind its tile)
    constexpr int kExtra = MODE != kPark && BK * BN * 4 + 16 * static_cast<int>(sizeof(Partial)) > TEAMS * S * static_cast<int>(kStage) ? 16 * static_cast<int>(sizeof(Partial)) : 0;
    __shared__ __attribute__((aligned(1024))) uint8_t lds_all[TEAMS * S * kStage + kExtra];
    const uint32_t team = TEAMS == 1 ? 0u : __builtin_amdgcn_readfirstlane(threadIdx.x / (64 * NW));
    uint8_t *lds = lds_all + team * (S * kStage);
    const uint32_t lds0 = lds_offset(lds);
    const uint32_t tid = TEAMS == 1 ? threadIdx.x : threadIdx.x % (64 * NW), lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave / WN, wn = wave % WN;
    const uint32_t N = pa.N, K = pa.K;
    uint32_t k0, n0;
    tile_of_block(pa.group_rows, pa.tiles_k, pa.tiles_n, k0, n0);
    k0 *= BK;
    n0 *= BN;
    // this workgroup's steps, and its teams' shares of them: team t takes t, t + TEAMS, ...
    const uint32_t split = blockIdx.y;
    const uint32_t begin = static_cast<uint32_t>(static_cast<uint64_t>(pa.steps) * split / pa.nsplit);
    const uint32_t end = static_cast<uint32_t>(static_cast<uint64_t>(pa.steps) * (split + 1) / pa.nsplit);
    const uint32_t mine = (end - begin + TEAMS - 1 - team) / TEAMS, most = (end - begin + TEAMS - 1) / TEAMS;

    // ---- global -> LDS: stage i holds the rows of this team's step i
    auto swizzle_group = [](uint32_t row, uint32_t groups) { return groups >= 4 ? row & 3u : (row >> 1) & 1u; };
    auto swizzle_piece = [](uint32_t row) { return (row >> 2) & 2u; };
    const uint64_t first_row = 32ull * (begin + team);
    const uint8_t *x_from = reinterpret_cast<const uint8_t *>(pa.X + first_row * K + k0), *y_from = reinterpret_cast<const uint8_t *>(pa.dY + first_row * N + n0);
    auto load_operand = [&](auto width, const uint8_t *from, uint32_t ld, uint32_t at) {
        constexpr uint32_t W = decltype(width)::value, kRows = 512 / W, kSlots = W / 8;
#pragma unroll
        for (uint32_t i = 0; i < W / 16 / NW; ++i) {
            const uint32_t c = wave + NW * i, in = lane / kSlots, row = c * kRows + in, slot = lane % kSlots;
            const uint32_t piece = (((slot >> 2) ^ swizzle_group(row, W / 32)) << 2) | ((slot & 3u) ^ swizzle_piece(row));
            load_to_lds(from + static_cast<uint64_t>(c) * kRows * ld * 2, in * ld * 2 + piece * 16, lds0 + at + c * 1024);
        }
    };
    auto load_stage = [&](uint32_t at) {
        load_operand(UintTag<BK>{}, x_from, K, at);
        load_operand(UintTag<BN>{}, y_from, N, at + kXBytes);
        x_from += 64ull * TEAMS * K;
        y_from += 64ull * TEAMS * N;
    };

    // ---- LDS -> fragments of 32 rows: 16 lanes take 8 of them
    const uint32_t row = 8 * (lane >> 4) + ((lane & 15u) >> 2), byte = 8 * (lane & 1u);
    auto place = [&](uint32_t tile, uint32_t width) {
        const uint32_t piece = 2 * (tile & 1u) + ((lane >> 1) & 1u);
        return row * (2 * width) + (((tile >> 1) ^ swizzle_group(row, width / 32)) * 4 + (piece ^ swizzle_piece(row))) * 16 + byte;
    };
    uint32_t x_at[TM], y_at[TN];
#pragma unroll
    for (uint32_t mi = 0; mi < TM; ++mi) x_at[mi] = place(TM * wm + mi, BK);
#pragma unroll
    for (uint32_t ni = 0; ni < TN; ++ni) y_at[ni] = kXBytes + place(TN * wn + ni, BN);
    uint32_t cur = 0, far = (S - 1) * kStage;
    auto read_one = [&](uint32_t at, uint32_t four_rows) {
        typedef short s16x8 __attribute__((ext_vector_type(8)));
        uint8_t *q = lds + at;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((OMC_LDS s16x4 *)(q));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((OMC_LDS s16x4 *)(q + four_rows));
        const s16x8 both = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        return __builtin_bit_cast(bf16x8, both);
    };
    // A step's products in two parts, the first and the last TM / 2 tiles of X by all of dY, column by column of the tiles.  X's fragments of a part are read beside the products of the part
    // before, those of the first part behind the step's barrier, and dY's of a step each as soon as its predecessor has been multiplied for the last time.
    constexpr int kRows = TM / 2;
    bf16x8 x[2][kRows], y[TN];
    f32x4 acc[TM][TN];
#pragma unroll
    for (int mi = 0; mi < TM; ++mi)
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) acc[mi][ni] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    auto read_x = [&](auto part, auto index) {
        constexpr int P = decltype(part)::value, I = decltype(index)::value;
        x[P][I] = read_one(cur + x_at[P * kRows + I], 4 * 2 * BK);
    };
    auto read_y = [&](auto index) { y[decltype(index)::value] = read_one(cur + y_at[decltype(index)::value], 4 * 2 * BN); };
    // `more`: with the reads for the part behind it
    auto multiply = [&](auto part, auto more) {
        constexpr int P = decltype(part)::value;
        for_constants<TN>([&](auto group) {
            constexpr int G = decltype(group)::value, R0 = G * kRows / TN, R1 = (G + 1) * kRows / TN;
            if constexpr (decltype(more)::value) for_constants<R1 - R0>([&](auto i) { read_x(UintTag<1 - P>{}, UintTag<R0 + decltype(i)::value>{}); });
#pragma unroll
            for (int mi = 0; mi < kRows; ++mi)
                acc[P * kRows + mi][G] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[P][mi], y[G], acc[P * kRows + mi][G], 0, 0, 0);
            if constexpr (P == 1 && decltype(more)::value) read_y(group);
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    const BoolTag<true> yes;
    auto first_part = [&]() {
        multiply(UintTag<0>{}, yes);
        cur = cur == (S - 1) * kStage ? 0 : cur + kStage;
        far = far == (S - 1) * kStage ? 0 : far + kStage;
    };
#pragma unroll
    for (uint32_t i = 0; i < S - 1; ++i)
        if (i < mine) load_stage(i * kStage);
    if (mine > 0) {
        wait_stage<S, kLoads>(0, mine);
        for_constants<TN>([&](auto i) { read_y(i); });
        for_constants<kRows>([&](auto i) { read_x(UintTag<0>{}, i); });
        if (mine > S - 1) load_stage(far);
        first_part();
        uint32_t i = 1;
        for (; i + (S - 1) < mine; ++i) {
            wait_loads_and_sync<(S - 2) * kLoads>();
            multiply(UintTag<1>{}, yes);
            load_stage(far);
            first_part();
        }
        for (; i < mine; ++i) {
            wait_stage<S, kLoads>(i, mine);
            multiply(UintTag<1>{}, yes);
            first_part();
        }
        multiply(UintTag<1>{}, BoolTag<false>{});
    }
    for (uint32_t i = mine; i < most; ++i) wait_loads_and_sync<0>();   // teams wait for each other
    wait_loads_and_sync<0>();                                 // nobody reads a stage any more
    static_assert((TEAMS - 1) * BK * BN * 4 <= TEAMS * S * static_cast<int>(kStage), "the other teams' tiles fit the stages");
    const bool lead = add_teams<TEAMS, NW, TM, TN>(reinterpret_cast<float *>(lds_all), acc, team, wave, lane);
    if constexpr (MODE == kPark) {
        if (!lead) return;
        float *to = pa.partials + static_cast<uint64_t>(split) * K * N + static_cast<uint64_t>(k0 + 16 * TM * wm + 8 * (lane >> 5)) * N +
                    n0 + 16 * TN * wn + (lane & 31u);
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int ni = 0; ni < TN; ni += 2) {
                    float p = acc[mi][ni][v], q = acc[mi][ni + 1][v];
                    side_by_side(p, q);
                    to[static_cast<uint64_t>(16 * mi + v) * N + 16 * ni] = p;
                    to[static_cast<uint64_t>(16 * mi + v + 4) * N + 16 * ni] = q;
                }
    } else {
        static_assert(BK * BN * 4 + 16 * static_cast<int>(sizeof(Partial)) <= TEAMS * S * static_cast<int>(kStage) + kExtra, "the tile fits the stages");
        float *tile = reinterpret_cast<float *>(lds_all);
        Partial *sums = reinterpret_cast<Partial *>(lds_all + BK * BN * 4);
        if (TEAMS > 1) __syncthreads();                       // the other teams' tiles are read
        if (lead) {
            float *to = tile + (16 * TM * wm + 8 * (lane >> 5)) * BN + 16 * TN * wn + (lane & 31u);
#pragma unroll
            for (int mi = 0; mi < TM; ++mi)
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int ni = 0; ni < TN; ni += 2) {
                        float p = acc[mi][ni][v], q = acc[mi][ni + 1][v];
                        side_by_side(p, q);
                        to[(16 * mi + v) * BN + 16 * ni] = p;
                        to[(16 * mi + v + 4) * BN + 16 * ni] = q;
                    }
        }
        __syncthreads();
        FitAcc fit;
        fit.clear();
        if (a.fp.wide) update_tile<BK, BN, 64 * NW * TEAMS, MODE, true>(a, tile, k0, n0, fit);
        else update_tile<BK, BN, 64 * NW * TEAMS, MODE, false>(a, tile, k0, n0, fit);
        fit.reduce_and_store<false>(sums + team * NW + wave);  // (8-bit formats: plain fp64 sums within a wave)
        __syncthreads();
        if (threadIdx.x < 64) {                               // one partial per tile: the waves' sums, each addition's error kept
            constexpr uint32_t kWaves = NW * TEAMS;
            static_assert(kWaves <= 16 && (kWaves & (kWaves - 1)) == 0, "one lane of the first wave per wave and sum");
            const Partial *from = sums + (lane & (kWaves - 1));
            DD one{(&from->sV)[lane >> 4], 0.0};              // 16 lanes a sum: V, Vt, V Vt, Vt^2
            float tmin = from->tmin, tmax = from->tmax;
            if constexpr (kWaves > 8) one = dd_add(one, dd_xor_in_row<8>(one));
            if constexpr (kWaves > 4) one = dd_add(one, dd_xor_in_row<4>(one));
            if constexpr (kWaves > 2) one = dd_add(one, dd_xor_in_row<2>(one));
            if constexpr (kWaves > 1) one = dd_add(one, dd_xor_in_row<1>(one));
#pragma unroll
            for (int off = kWaves / 2; off >= 1; off >>= 1) {
                tmin = fminf(tmin, __shfl_xor(tmin, off));
                tmax = fmaxf(tmax, __shfl_xor(tmax, off));
            }
            Partial *out = a.ws + blockIdx.x;
            if ((lane & 15u) == 0) {
                (&out->sV)[lane >> 4] = one.hi;
                (&out->lV)[lane >> 4] = one.lo;
            }
            if (lane == 0) {
                out->tmin = tmin;
                out->tmax = tmax;
            }
        }
    }
}

// Tiles (fitted with matrix instructions of 32 x 32 x 16): their figures are for steps of 32 rows (of TEAMS times as many with several teams), see GemmTile
// (`fresh` is not counted here).
static constexpr GemmTile kProductTiles[] = {
    {256, 128, 2, 1, 1, 6.2, 0.64, 0.88, 0.0, 0.0}, {128, 128, 1, 1, 2, 3.5, 0.30, 0.28, 0.0, 0.0}, {128, 128, 2, 1, 1, 4.7, 0.355, 0.57, 0.0, 0.0},
    {64, 64, 1, 1, 4, 3.2, 0.13, 0.126, 0.0, 0.0},  {64, 64, 2, 1, 2, 1.0, 0.20, 0.215, 3.0, 0.0},  {64, 64, 4, 1, 1, 1.0, 0.40, 0.46, 3.0, 0.0},
};

// What the one-kernel route's epilogue takes, in us per workgroup of a compute unit, under momentum (under SGD 0.6 of it, under
// Adam 2: the sizes alone decide, so that the gradient's bits depend on them alone).
static constexpr double kEpilogue[] = {13.7, 6.9, 9.3, 2.0, 1.5, 4.0};

// The tile, number of splits and estimated time (us) of a product, by the estimate that pick_tile makes, over any number of splits up
// to what the workspace has room for, or none.  The contraction is cut into at least `room` parts, by splits and teams together:
// so that no fp32 sum runs over more products than M / room, which keeps its error where a workspace of that size puts it (2e-7 for 4096
// products, 3e-7 for 8192).  A split costs its partial sums, written here and read by the update (4 bytes each way at 5 TB/s, half of the
// writing covered).  8192 rows, 4096 x 1024 weights: two splits of 256 x 128 by two teams 71, one of 128 x 128 by two teams 78, one
// of 128 x 128 81, four of 256 x 128 80, 64 x 64 124 - 133.  2048 rows, 512 x 2048 weights: 10 with 64 x 64, 12 - 19 with the others.
// On matrices of more than one 256 x 128 tile per compute unit that leave no room for partial sums, the epilogue, codes and state, is no
// small part of the call and is counted.  Where a unit has one workgroup at a time nothing runs beside it; where it has several, half of
// the shorter of epilogue and product passes under the longer one.  8-bit codes, 128 rows on 8192 x 8192 weights, SGD / momentum / Adam:
// 96 / 142 / 250 with 128 x 128, 119 / 155 / 278 with 256 x 128 by two teams, which the products alone would choose, 125 / 162 / 271 with
// 64 x 64.  (Smaller ones: over 100 random sizes the chosen tile is 3 % off the best one with and without it.)
static bool fills_several_times(uint32_t N, uint32_t K) { return static_cast<uint64_t>(K) * N > 256ull * 256 * 128; }
struct ProductChoice {
    int tile;
    uint32_t splits;
    double us;
};
static ProductChoice choose_product(uint32_t M, uint32_t N, uint32_t K, uint32_t room, bool parked) {
    const uint32_t most_splits = parked ? room : 1;
    ProductChoice best{-1, 1, 0.0};
    const uint32_t all_steps = M / 32;
    for (int i = 0; i < static_cast<int>(sizeof(kProductTiles) / sizeof(kProductTiles[0])); ++i) {
        const GemmTile &t = kProductTiles[i];
        if (K % t.bm != 0 || N % t.bn != 0) continue;
        const uint64_t tiles = static_cast<uint64_t>(K / t.bm) * (N / t.bn);
        if (tiles > 0x7fffffffull) continue;
        for (uint32_t splits = 1; splits <= most_splits && splits <= all_steps; ++splits) {
            if (splits * t.teams < room) continue;
            const uint64_t count = tiles * splits;
            const double per_unit = static_cast<double>(count) / 256.0;
            const double alone = t.step * static_cast<double>((count + 256ull * t.resident - 1) / (256ull * t.resident));
            const double busy = t.loaded * per_unit;
            const uint32_t steps = ((all_steps + splits - 1) / splits + t.teams - 1) / t.teams;
            const double product = steps * (alone > busy ? alone : busy);
            double us = t.base + t.stores * per_unit;
            if (room > 0 || !fills_several_times(N, K)) {
                us += product;
                if (parked) us += splits * 6.0 * K * N / 5e6;
            } else {
                const double epilogue = kEpilogue[i] * (t.resident > 1 ? per_unit : static_cast<double>((count + 255) / 256));
                const double longer = product > epilogue ? product : epilogue, shorter = product > epilogue ? epilogue : product;
                us += longer + (t.resident > 1 ? 0.5 : 1.0) * shorter;
            }
            if (best.tile < 0 || us < best.us) best = ProductChoice{i, splits, us};
        }
    }
    return best;
}

// Tile rows in a group of the tile order.  For the operands' sake eight, or two of the 256-row tiles.  The epilogue also moves codes and state
// of the tiles that are under way at one time, and with eight tile rows of a matrix whose rows are a multiple of 8 KB long these lie in
// a part of every such stretch only, as if in a part of the memory's channels: 32 rows on 4096 x 4096 weights, momentum 48 us, Adam 65 - 99
// depending on where the buffers lie.  Where the product is short enough not to miss the shared operands, the tiles under way on a die
// therefore cover whole rows of the weights: 38 and 65 us; 1024 rows 73 -> 65 and 97 - 121 -> 93.  (Smaller matrices have all their tiles under
// way at once; rows of 5120 weights take 108 us under Adam as it is, 115 so.)
static uint32_t tile_group(const GemmTile &t, uint32_t tiles_n, uint32_t M, uint32_t N, uint32_t K, bool moves_state) {
    const uint32_t usual = t.bm == 256 ? 2 : 8;
    if (!moves_state || t.bn < 128 || M > 1024 || N % 2048 != 0 || !fills_several_times(N, K)) return usual;
    const uint32_t whole = 32 * t.resident / tiles_n;         // 32 compute units on a die
    if (whole < 2) return M <= 256 ? 1 : usual;
    return whole < usual ? whole : usual;
}

template <int MODE>
static int launch_product(int tile, ProductArgs pa, const DwArgs &a, hipStream_t st) {
    if (tile < 0) return static_cast<int>(hipErrorInvalidValue);
    pa.tiles_k = pa.K / kProductTiles[tile].bm;
    pa.tiles_n = pa.N / kProductTiles[tile].bn;
    pa.group_rows = tile_group(kProductTiles[tile], pa.tiles_n, 32 * pa.steps, pa.N, pa.K, MODE >= kStepMomentum);
    const dim3 grid(pa.tiles_k * pa.tiles_n, pa.nsplit);
    switch (tile) {
        case 0: dw_product_kernel<2, 2, 8, 4, 2, 3, 2, MODE><<<grid, dim3(512), 0, st>>>(pa, a); break;
        case 1: dw_product_kernel<2, 2, 4, 4, 1, 4, 2, MODE><<<grid, dim3(256), 0, st>>>(pa, a); break;
        case 2: dw_product_kernel<2, 2, 4, 4, 2, 4, 2, MODE><<<grid, dim3(512), 0, st>>>(pa, a); break;
        case 3: dw_product_kernel<2, 2, 2, 2, 1, 4, 4, MODE><<<grid, dim3(256), 0, st>>>(pa, a); break;
        case 4: dw_product_kernel<2, 2, 2, 2, 2, 4, 4, MODE><<<grid, dim3(512), 0, st>>>(pa, a); break;
        default: dw_product_kernel<2, 2, 2, 2, 4, 4, 4, MODE><<<grid, dim3(1024), 0, st>>>(pa, a); break;
    }
    return static_cast<int>(hipGetLastError());
}

int launch_dw_product(const DwArgs &a, float *partials, uint32_t room, uint32_t *nsplit, hipStream_t st) {
    const ProductChoice c = choose_product(a.M, a.N, a.K, room, true);
    *nsplit = c.splits;
    return launch_product<kPark>(c.tile, ProductArgs{a.X, a.dY, partials, a.N, a.K, a.M / 32, c.splits, 0, 0, 0}, a, st);
}

// What the update kernel costs besides reading the partial sums: its launch, and codes and state, which the one-kernel route's
// epilogue moves mostly under other workgroups' products (8192 rows, 4096 x 1024 weights, 8 bits, momentum: one kernel 79 us,
// product and update 71 + 17).
bool dw_one_kernel_is_faster(uint32_t M, uint32_t N, uint32_t K, uint32_t room) {
    const ProductChoice one = choose_product(M, N, K, room, false), two = choose_product(M, N, K, room, true);
    return one.tile >= 0 && (two.tile < 0 || one.us <= two.us + 3.0 + 6.0 * K * N / 5e6);
}

uint32_t dw_tile_and_splits(uint32_t M, uint32_t N, uint32_t K, uint32_t room, bool parked) {
    const ProductChoice c = choose_product(M, N, K, room, parked);
    return static_cast<uint32_t>(c.tile) * 100 + c.splits;
}

int launch_dw_one_kernel(const DwArgs &a, uint32_t room, int opt_kind, uint32_t *nparts, hipStream_t st) {
    const ProductChoice c = choose_product(a.M, a.N, a.K, room, false);
    if (c.tile >= 0) *nparts = (a.K / kProductTiles[c.tile].bm) * (a.N / kProductTiles[c.tile].bn);
    const ProductArgs pa{a.X, a.dY, nullptr, a.N, a.K, a.M / 32, 1, 0, 0, 0};
    if (opt_kind == OMC_SGD) return launch_product<kStepSgd>(c.tile, pa, a, st);
    if (opt_kind == OMC_MOMENTUM) return launch_product<kStepMomentum>(c.tile, pa, a, st);
    return launch_product<kStepAdam>(c.tile, pa, a, st);
}

}  // namespace omc
