// omc_step_update_recompress: orchestration over the plan's groups, the fp32-variable kernels
// and the per-variable finalize.
#include <algorithm>

#include "omc_step_impl.h"

#ifndef OMC_TUNE_KEEP_BUDGET_MIB
#define OMC_TUNE_KEEP_BUDGET_MIB 224     // packed codes that stay cached when the set's codes do not fit as a whole
#endif
#ifndef OMC_TUNE_KEEP_FP32
#define OMC_TUNE_KEEP_FP32 1             // bit k: optimizer kind k keeps fp32 values cached (measured: pays for SGD only)
#endif
#ifndef OMC_TUNE_KEEP_ALL_MIB
#define OMC_TUNE_KEEP_ALL_MIB 264        // up to this size all codes stay cached
#endif

namespace omc {

template <int MODE>
__global__ __launch_bounds__(64) void step_fp32_kernel(StepArgs sa) {
    do_fp32_item<MODE>(sa, sa.first_item + blockIdx.x / kFp32Parts, blockIdx.x % kFp32Parts);
}

// Ragged tails of a set that has no full tile at all, one wave each.
template <int MODE>
__global__ __launch_bounds__(64) void step_tail_kernel(StepArgs sa) {
    __shared__ uint32_t lds[kLdsDwords];
    step_tail<MODE>(sa, blockIdx.x, lds);
}

int launch_step(void *arena, const PlanHeader *ph, const void *plan_dev, float *sb_table, const float *grads,
                float *state0, float *state1, const omc_opt &opt, Partial *ws, void *stream,
                void *const *events) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    uint32_t launch = 0;
    auto mark = [&](uint32_t which) -> int {   // optional caller-owned events around each launch
        if (!events) return 0;
        return static_cast<int>(hipEventRecord(static_cast<hipEvent_t>(events[2 * launch + which]), st));
    };
    const uint8_t *ph_bytes = reinterpret_cast<const uint8_t *>(ph);
    const PlanGroup *groups = reinterpret_cast<const PlanGroup *>(ph_bytes + ph->group_off);
    StepArgs sa{};
    sa.arena = static_cast<uint8_t *>(arena);
    sa.plan = static_cast<const uint8_t *>(plan_dev);
    sa.var_off = ph->var_off;
    sa.item_off = ph->item_off;
    sa.sb_table = sb_table;
    sa.grads = grads;
    sa.st0 = opt.kind >= OMC_MOMENTUM ? state0 : nullptr;
    sa.st1 = opt.kind == OMC_ADAM ? state1 : nullptr;
    sa.ws = ws;
    sa.oc = OptConst{opt.lr, opt.momentum, opt.beta1, opt.beta2, opt.eps, opt.one_minus_beta1,
                     opt.one_minus_beta2, opt.bias_corr1, opt.bias_corr2};
    // the fp32 variables and the ragged tails ride along with the first full-tile launch as extra workgroups
    const PlanGroup *fp32_group = nullptr;
    uint32_t tail_first = 0, tail_nitems = 0;              // the tail groups follow each other in the item list
    bool fuse = false;
    for (uint32_t gi = 0; gi < ph->ngroups; ++gi) {
        if (groups[gi].nitems == 0) continue;
        if (groups[gi].kind == kGroupFp32) fp32_group = &groups[gi];
        if (groups[gi].kind == kGroupFull) fuse = true;
        if (groups[gi].kind == kGroupTail) {
            if (tail_nitems == 0) tail_first = groups[gi].first_item;
            tail_nitems += groups[gi].nitems;
        }
    }
    bool fused_done = false;
    // Packed codes are read and rewritten by every step.  In a training loop a forward and a backward pass lie
    // between two steps and nothing survives in the caches, so by default every code access carries the
    // non-temporal hint.  A caller that runs steps back to back asks for OMC_OPT_KEEP_CODES: the codes then
    // come back from the memory-side cache at the next step if they still sit there.  Work items get to keep
    // their codes cached, in launch order, up to a budget below that cache's 256 MB; the codes of all other
    // items carry the non-temporal hint and pass it by.  A group whose items fall on both sides of the limit
    // is launched in two parts.
    uint64_t keep_budget = 0;                              // bytes of packed codes that stay cached
    uint32_t fp32_keep_items = 0;                          // fp32 work items whose values stay cached
    if (opt.flags & OMC_OPT_KEEP_CODES) {                  // (default: other work runs between two steps, nothing would survive)
        const uint64_t cache = static_cast<uint64_t>(OMC_TUNE_KEEP_BUDGET_MIB) << 20;
        uint64_t all_codes = 0;
        for (uint32_t gi = 0; gi < ph->ngroups; ++gi)
            if (groups[gi].kind == kGroupFull) all_codes += static_cast<uint64_t>(groups[gi].nitems) * tiles_per_chunk(groups[gi].bits) * kTileElems * groups[gi].bits / 8;
        // a set that exceeds the cache by little still gets most of its hits and is not worth a second, small launch
        keep_budget = all_codes <= (static_cast<uint64_t>(OMC_TUNE_KEEP_ALL_MIB) << 20) ? all_codes : cache;
        // what the codes leave goes to the values of the fp32 variables, which are read and rewritten in place as well
        // (optimizer state is not worth keeping: measured slower)
        const uint64_t left = cache > all_codes ? cache - all_codes : 0;
        if (fp32_group && ((OMC_TUNE_KEEP_FP32 >> opt.kind) & 1)) fp32_keep_items = static_cast<uint32_t>(std::min<uint64_t>(fp32_group->nitems, left / (4ull * kChunkElems)));
    }
    // fp32 items from this one of the group on, in launches of their own (see kMostSharingBlocks)
    constexpr uint32_t kFp32Run = kMostSharingBlocks / kFp32Parts;
    auto launch_fp32 = [&](uint32_t from) -> int {
        for (; from < fp32_group->nitems; from += kFp32Run) {
            sa.first_item = sa.fp32_first = fp32_group->first_item + from;
            sa.fp32_keep_items = fp32_keep_items > from ? fp32_keep_items - from : 0;
            const dim3 grid(std::min(fp32_group->nitems - from, kFp32Run) * kFp32Parts);
            if (opt.kind == OMC_SGD) step_fp32_kernel<kStepSgd><<<grid, dim3(64), 0, st>>>(sa);
            else if (opt.kind == OMC_MOMENTUM) step_fp32_kernel<kStepMomentum><<<grid, dim3(64), 0, st>>>(sa);
            else step_fp32_kernel<kStepAdam><<<grid, dim3(64), 0, st>>>(sa);
            const int rc = static_cast<int>(hipGetLastError());
            if (rc != 0) return rc;
        }
        return 0;
    };
    // The order of the parts of fp32 items: an item's one after the other, neighbouring addresses at the same time; of few items that are largely
    // vectors the first parts of all items first and the empty parts last, which counts most where a compute unit holds few waves (Adam of 13 bits and
    // more).  Small encoders, us, one after the other against first parts first; items, and how many they would be if every one were full: momentum
    // 1698, 1569 38 : 42; 1019, 886 25.2 : 26.8, Adam 35.7 : 37.7; Adam in 16 bits 721, 648 37.6 : 38.3; but Adam in 19 bits 782, 455 41 : 33; 982, 682 146 : 141, in 13
    // bits 534, 360 30.1 : 28.5; and up to 512 items whatever they hold, momentum 332, 242 14.1 : 13.6; 374, 306 18.6 : 18.3.
    auto item_by_item = [&]() -> bool {
        const uint32_t nitems = fp32_group->nitems;
        if (nitems <= 512 || nitems > 1024) return nitems > 1024;
        const PlanVar *vars = reinterpret_cast<const PlanVar *>(ph_bytes + ph->var_off);
        uint64_t elements = 0;
        for (uint32_t i = 0; i < ph->nvars; ++i)
            if (!(vars[i].flags & OMC_VAR_QUANTIZED)) elements += vars[i].n;
        return 4 * elements >= 3ull * nitems * kChunkElems;
    };
    auto take = [&](uint32_t nitems, uint64_t item_bytes) -> uint32_t {   // how many of nitems the budget still covers
        const uint64_t k = std::min<uint64_t>(nitems, keep_budget / item_bytes);
        keep_budget -= k * item_bytes;
        return static_cast<uint32_t>(k);
    };
    for (uint32_t gi = 0; gi < ph->ngroups; ++gi) {
        const PlanGroup &g = groups[gi];
        if (g.nitems == 0) continue;
        if (fuse && g.kind != kGroupFull) continue;
        if (g.kind == kGroupTail && g.first_item != tail_first) continue;   // both tail groups are one launch
        sa.first_item = g.first_item;
        sa.nitems = g.nitems;
        sa.fp32_first = 0;
        sa.fp32_nitems = 0;
        auto ride_along = [&]() {                                          // with the first full-tile launch of the step
            sa.fp32_nitems = 0;
            sa.tail_nitems = 0;
            if (fused_done) return;
            sa.tail_first = tail_first;
            sa.tail_nitems = tail_nitems;
            if (fp32_group) {
                sa.fp32_first = fp32_group->first_item;
                sa.fp32_nitems = std::min(fp32_group->nitems, kFp32Run);
                sa.fp32_keep_items = fp32_keep_items;
                sa.fp32_item_by_item = item_by_item() ? 1u : 0u;
            }
            fused_done = true;
        };
        int rc = mark(0);
        if (rc != 0) return rc;
        if (g.kind == kGroupTail) {
            sa.tail_first = tail_first;
            if (opt.kind == OMC_SGD) step_tail_kernel<kStepSgd><<<dim3(tail_nitems), dim3(64), 0, st>>>(sa);
            else if (opt.kind == OMC_MOMENTUM) step_tail_kernel<kStepMomentum><<<dim3(tail_nitems), dim3(64), 0, st>>>(sa);
            else step_tail_kernel<kStepAdam><<<dim3(tail_nitems), dim3(64), 0, st>>>(sa);
            rc = static_cast<int>(hipGetLastError());
        } else if (g.kind == kGroupFp32) {
            rc = launch_fp32(0);
        } else {
            const uint32_t kept = take(g.nitems, static_cast<uint64_t>(tiles_per_chunk(g.bits)) * kTileElems * g.bits / 8);
            for (int part = 0; part < 2 && rc == 0; ++part) {              // the cached items, then the streaming ones
                sa.first_item = g.first_item + (part == 0 ? 0 : kept);
                sa.nitems = part == 0 ? kept : g.nitems - kept;
                if (sa.nitems == 0) continue;
                const bool first = !fused_done;
                ride_along();
                if (opt.kind == OMC_SGD) rc = launch_step_group_sgd(g.bits, g.wide, sa, part == 0, st);
                else if (opt.kind == OMC_MOMENTUM) rc = launch_step_group_momentum(g.bits, g.wide, sa, part == 0, st);
                else rc = launch_step_group_adam(g.bits, g.wide, sa, part == 0, st);
                if (rc == 0 && first && fp32_group) rc = launch_fp32(kFp32Run);
            }
        }
        if (rc != 0) return rc;
        rc = mark(1);
        if (rc != 0) return rc;
        ++launch;
    }
    if (ph->nquant > 0) {
        int rc = mark(0);
        if (rc != 0) return rc;
        finalize_plan_kernel<kFinalizeWaves><<<dim3(ph->nvars), dim3(64 * kFinalizeWaves), 0, st>>>(sa.plan, ph->var_off, ws, sb_table);
        rc = static_cast<int>(hipGetLastError());
        if (rc != 0) return rc;
        return mark(1);
    }
    return 0;
}

}  // namespace omc
