// Update kernel of the fused weight-gradient step, any code width (included once per optimizer).  The gradient lies in the
// workspace as partial sums over runs of the rows, row-major like the variable: one wave takes a tile of 2048 consecutive
// elements, adds the partial sums in order and runs the cycle of the streaming step kernels on it.  Bound by memory (a 4 M-element
// 8-bit variable under momentum with two partial sums: 75 MB in 16 us).
#pragma once
#include "omc_dw_args.h"

namespace omc {

template <int B, int MODE, int VARIANT>
__global__ __launch_bounds__(64, (Tuning<MODE, B>::waves)) void dw_reduce_update_kernel(DwArgs a) {
    __shared__ __attribute__((aligned(16))) uint32_t lds[kLdsDwords];
    const uint32_t lane = threadIdx.x;
    const uint64_t n = static_cast<uint64_t>(a.K) * a.N, e0 = static_cast<uint64_t>(blockIdx.x) * kTileElems;
    TileArgs ta{};
    ta.codes = a.codes;
    ta.total_dwords = n / 32 * B;
    ta.grad = a.partials;
    ta.st0 = a.st0;
    ta.st1 = a.st1;
    ta.n = n;
    ta.s = to_scalar_regs(a.sb[0]);
    ta.b = to_scalar_regs(a.sb[1]);
    Stage<B, MODE> st;
    issue_loads<B, MODE, true>(ta, e0, lane, st);            // the next forward pass reads the codes: they stay cached
    for (uint32_t sp = 1; sp < a.nsplit; ++sp) {
        f32x4 more[8];
        load_f32_pieces<true>(a.partials + sp * n + e0, lane, more);
#pragma unroll
        for (int j = 0; j < 8; ++j) st.gq[j] = st.gq[j] + more[j];
    }
    if (a.dW_out) store_f32_pieces<true>(a.dW_out + e0, lane, st.gq);   // the gradient as consumed
    FitAcc fit;
    fit.clear();
    finish_tile<B, MODE, VARIANT, false, true>(ta, a.fp, a.oc, e0, lane, lds, st, fit);
    fit.template reduce_and_store<variant_exact(VARIANT)>(a.ws + blockIdx.x);
}

// FmtParams::variant: 0 / 1 rounding by add-subtract / ldexp (7 exponent bits, so 8 bits in all, are the fewest that reach the
// binades of the latter); 4 / 5 the same with error-carrying sums, which only code widths of 18 bits and more can ask for; the
// hardware conversions (2 / 3) serve plain SGD.
template <int BITS, int MODE>
inline void launch_dw_update_width(dim3 grid, const DwArgs &a, hipStream_t st) {
    const uint32_t variant = a.fp.variant;
    if constexpr (BITS >= 18) {
        if (variant == 4) { dw_reduce_update_kernel<BITS, MODE, 4><<<grid, dim3(64), 0, st>>>(a); return; }
        if (variant == 5) { dw_reduce_update_kernel<BITS, MODE, 5><<<grid, dim3(64), 0, st>>>(a); return; }
    }
    if constexpr (BITS == 8 && MODE == kStepSgd) {
        if (variant == 2) { dw_reduce_update_kernel<8, MODE, 2><<<grid, dim3(64), 0, st>>>(a); return; }
    }
    if constexpr (BITS == 6 && MODE == kStepSgd) {
        if (variant == 3) { dw_reduce_update_kernel<6, MODE, 3><<<grid, dim3(64), 0, st>>>(a); return; }
    }
    if constexpr (BITS >= 8) {
        if (variant == 1) { dw_reduce_update_kernel<BITS, MODE, 1><<<grid, dim3(64), 0, st>>>(a); return; }
    }
    dw_reduce_update_kernel<BITS, MODE, 0><<<grid, dim3(64), 0, st>>>(a);
}

template <int MODE>
inline int launch_dw_update_mode(const DwArgs &a, hipStream_t st) {
    const dim3 grid(static_cast<uint32_t>(static_cast<uint64_t>(a.K) * a.N / kTileElems));
    switch (a.fp.bits) {
#define X(BITS)                                            \
    case BITS:                                             \
        launch_dw_update_width<BITS, MODE>(grid, a, st);   \
        break;
        OMC_FOR_EACH_BITS(X)
#undef X
        default:
            return static_cast<int>(hipErrorInvalidValue);
    }
    return static_cast<int>(hipGetLastError());
}

}  // namespace omc
