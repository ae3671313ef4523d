// Shared by the kernels of omc_dw_update_recompress.
#pragma once
#include "omc_stream.h"

namespace omc {

constexpr int kDwCols = 128, kDwStep = 32;

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

// First kernel of the two-kernel route: the gradient as *nsplit <= most_splits partial sums.
int launch_dw_product(const uint16_t *X, const uint16_t *dY, float *partials, uint32_t M, uint32_t N, uint32_t K, uint32_t most_splits,
                      uint32_t *nsplit, hipStream_t st);

// Second kernel: adds them up and runs the cycle; one launcher per optimizer.
int launch_dw_update_sgd(const DwArgs &a, hipStream_t st);
int launch_dw_update_momentum(const DwArgs &a, hipStream_t st);
int launch_dw_update_adam(const DwArgs &a, hipStream_t st);

}  // namespace omc
