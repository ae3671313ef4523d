// omc_reselect (paper Sec. 2.5: the quantized subset changes from round to round): variables that become quantized are compressed and
// unchanged ones copied by one derived plan, variables that become fp32 are decompressed by another.
#include "omc_codec_impl.h"

namespace omc {

// Both plans' work of one code width in one launch: the workgroups of the compression, then those of the decompression.  They read
// the old arena and write different variables of the new one.  A launch that only drains and fills again costs 3 - 5 us: change of the
// subset and message of 599 variables in 11 bits 141.5 -> 135 us, of 4 blocks of 170 x 511 in three formats 39 -> 30 (with the two launches for
// (s, b) in one, and in the latter figure the shorter copies).
// A few copies beside the conversions, codes and vectors of all sizes: their first parts first (encoder of 9 blocks, 229 wide, 19 bits, with the message
// 30.7 us, 31.3 copy by copy; 16 blocks, 495 wide, three formats 158.2, 160.9).  The conversions of a whole set prefer copy by copy however few they are (1019 copies
// 24.0 us, 25.2 the other way; 393 54.0, 54.5).
constexpr uint32_t kFewCopies = 1024;
template <int B, int VARIANT>
__global__ __launch_bounds__(64, (Tuning<kCompress, B>::waves)) void reselect_kernel(CodecArgs to_codes, uint32_t first, CodecArgs to_fp32) {
    __shared__ __attribute__((aligned(16))) uint32_t lds[kLdsDwords];
    if (blockIdx.x < first) codec_block<B, kCompress, VARIANT, kFewCopies>(to_codes, blockIdx.x, lds);
    else codec_block<B, kDecompress, 0, kFewCopies>(to_fp32, blockIdx.x - first, lds);
}

template <int B, int VARIANT>
static void launch_one(const CodecArgs &c, const CodecArgs &d, hipStream_t st) {
    const uint32_t first = codec_blocks(c);
    reselect_kernel<B, VARIANT><<<dim3(first + codec_blocks(d)), dim3(64), 0, st>>>(c, first, d);
}

template <int BITS>
static void launch_variant(uint32_t variant, const CodecArgs &c, const CodecArgs &d, hipStream_t st) {
    if constexpr (BITS >= 18) {
        if (variant == 4) { launch_one<BITS, 4>(c, d, st); return; }
        if (variant == 5) { launch_one<BITS, 5>(c, d, st); return; }
    }
    if constexpr (BITS == 8) {
        if (variant == 2) { launch_one<BITS, 2>(c, d, st); return; }
    }
    if constexpr (BITS == 6) {
        if (variant == 3) { launch_one<BITS, 3>(c, d, st); return; }
    }
    if (variant == 1) launch_one<BITS, 1>(c, d, st);
    else launch_one<BITS, 0>(c, d, st);
}

static int launch_width(uint32_t bits, uint32_t variant, const CodecArgs &c, const CodecArgs &d, hipStream_t st) {
    switch (bits) {
#define X(BITS)                                          \
    case BITS:                                           \
        launch_variant<BITS>(variant, c, d, st);         \
        break;
        OMC_FOR_EACH_BITS(X)
#undef X
        default:
            return static_cast<int>(hipErrorInvalidValue);
    }
    return static_cast<int>(hipGetLastError());
}

// (s, b) of a new subset.  The first workgroups, one per variable of the derived plan, fit the newly quantized variables; the
// others copy (s, b) of the variables that stay quantized and write (1, 0) for those that are fp32 afterwards.  One launch for both:
// each takes 4 - 5 us, whatever the set.
__global__ __launch_bounds__(64 * kFinalizeWaves) void reselect_sb_kernel(const uint8_t *__restrict__ plan, uint64_t var_off, uint32_t fits,
                                                                          const Partial *__restrict__ ws,
                                                                          const uint32_t *__restrict__ actions, uint32_t nvars,
                                                                          const float *__restrict__ sb_old, float *__restrict__ sb_new) {
    __shared__ double red[kFinalizeWaves * 10];
    if (blockIdx.x < fits) {
        const PlanVar pv = to_scalar_regs(reinterpret_cast<const PlanVar *>(plan + var_off)[blockIdx.x]);
        if (pv.flags & OMC_VAR_QUANTIZED) finalize_plan_variable<kFinalizeWaves>(pv, ws, sb_new, red);
        return;
    }
    const uint32_t i = (blockIdx.x - fits) * (64 * kFinalizeWaves) + threadIdx.x;
    if (i >= nvars) return;
    const uint32_t a = actions[i];
    if (a == kRsCopyQuantized) {
        sb_new[2 * static_cast<uint64_t>(i)] = sb_old[2 * static_cast<uint64_t>(i)];
        sb_new[2 * static_cast<uint64_t>(i) + 1] = sb_old[2 * static_cast<uint64_t>(i) + 1];
    } else if (a != kRsToQuantized) {
        sb_new[2 * static_cast<uint64_t>(i)] = 1.0f;
        sb_new[2 * static_cast<uint64_t>(i) + 1] = 0.0f;
    }
}

// A plan's full-tile groups; tails and copies ride on whichever launch is first (of more copies than one launch takes, the others on the next ones).
struct Side {
    CodecArgs args;
    const PlanGroup *groups;
    uint32_t ngroups;
    SetGroups rest;
    Side(const PlanPair &plan) : args{}, groups(nullptr), ngroups(0), rest{} {
        if (!plan.host) return;
        args.plan = plan.dev;
        args.var_off = plan.host->var_off;
        args.item_off = plan.host->item_off;
        groups = reinterpret_cast<const PlanGroup *>(reinterpret_cast<const uint8_t *>(plan.host) + plan.host->group_off);
        ngroups = plan.host->ngroups;
        rest = set_groups(groups, ngroups);
    }
    // arguments for this group (nullptr: none of its width), with what is left of the tails and copies
    CodecArgs take(const PlanGroup *g) {
        CodecArgs ca = args;
        if (g) {
            ca.first_item = g->first_item;
            ca.nitems = g->nitems;
        }
        take_copies(rest, ca);
        take_tails(rest, ca);
        return ca;
    }
    const PlanGroup *full(uint32_t i) const { return groups[i].kind == kGroupFull && groups[i].nitems > 0 ? &groups[i] : nullptr; }
    bool left() const { return rest.tail_nitems > 0 || rest.fp32_nitems > 0; }
};

int launch_reselect(const void *arena_old, const float *sb_old, void *arena_new, float *sb_new, const PlanPair &to_codes,
                    const PlanPair &to_fp32, const uint32_t *actions_dev, uint32_t nvars, Partial *ws, void *stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    Side c(to_codes), d(to_fp32);
    c.args.arena = static_cast<uint8_t *>(arena_new);
    c.args.vin = static_cast<const float *>(arena_old);
    c.args.ws = ws;
    d.args.arena = static_cast<uint8_t *>(const_cast<void *>(arena_old));    // never written in this mode
    d.args.sb_in = sb_old;
    d.args.vout = static_cast<float *>(arena_new);
    auto same = [](const Side &side, const PlanGroup *g) -> const PlanGroup * {     // the other side's group of this width and rounding
        for (uint32_t k = 0; k < side.ngroups; ++k)
            if (side.full(k) && side.full(k)->bits == g->bits && side.full(k)->wide == g->wide) return side.full(k);
        return nullptr;
    };
    for (uint32_t i = 0; i < c.ngroups; ++i) {
        const PlanGroup *g = c.full(i);
        if (!g) continue;
        const PlanGroup *other = same(d, g);
        const int rc = launch_width(g->bits, g->wide, c.take(g), other || d.left() ? d.take(other) : CodecArgs{}, st);
        if (rc != 0) return rc;
    }
    for (uint32_t i = 0; i < d.ngroups; ++i) {
        const PlanGroup *g = d.full(i);
        if (!g || same(c, g)) continue;
        const int rc = launch_width(g->bits, 0, c.left() ? c.take(nullptr) : CodecArgs{}, d.take(g), st);
        if (rc != 0) return rc;
    }
    while (c.left() || d.left()) {                           // what no full tile's launch took: any width serves
        const int rc = launch_width(8, 0, c.left() ? c.take(nullptr) : CodecArgs{}, d.left() ? d.take(nullptr) : CodecArgs{}, st);
        if (rc != 0) return rc;
    }
    const PlanHeader *ph = to_codes.host;
    const uint32_t fits = ph && ph->nquant > 0 ? ph->nvars : 0, copies = (nvars - 1) / (64 * kFinalizeWaves) + 1;
    reselect_sb_kernel<<<dim3(fits + copies), dim3(64 * kFinalizeWaves), 0, st>>>(to_codes.dev, ph ? ph->var_off : 0, fits, ws, actions_dev, nvars, sb_old, sb_new);
    return static_cast<int>(hipGetLastError());
}

}  // namespace omc
