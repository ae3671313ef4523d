// Shared by the kernels of omc_dw_update_recompress.
#pragma once
#include "omc_stream.h"

namespace omc {

struct DwArgs {
    const uint16_t *X, *dY;
    uint32_t *codes;
    const float *sb;
    float *st0, *st1;
    float *dW_out;
    Partial *ws;
    const float *partials;   // two-kernel route: [nsplit][K * N] partial sums of the gradient
    uint32_t nsplit;
    FmtParams fp;
    OptConst oc;
    uint32_t M, N, K;
};

// First kernel of the two-kernel route: the gradient as *nsplit <= room partial sums.
int launch_dw_product(const DwArgs &a, float *partials, uint32_t room, uint32_t *nsplit, hipStream_t st);
// The one-kernel route (8-bit codes); *nparts: how many partial sums of the fit it leaves.  `room`: how many copies of the
// gradient the workspace holds, 0 or more; none is written.
int launch_dw_one_kernel(const DwArgs &a, uint32_t room, int opt_kind, uint32_t *nparts, hipStream_t st);
bool dw_one_kernel_is_faster(uint32_t M, uint32_t N, uint32_t K, uint32_t room);
// 100 * tile + splits of a route.
uint32_t dw_tile_and_splits(uint32_t M, uint32_t N, uint32_t K, uint32_t room, bool parked);

// Second kernel: adds them up and runs the cycle; one launcher per optimizer.
int launch_dw_update_sgd(const DwArgs &a, hipStream_t st);
int launch_dw_update_momentum(const DwArgs &a, hipStream_t st);
int launch_dw_update_adam(const DwArgs &a, hipStream_t st);

}  // namespace omc
