// omc_dw_update_recompress: the backward pass of a linear layer on a compressed weight matrix
// (paper Sec. 2.1, backward propagation: decompress the layer's parameters, apply the gradients,
// compress, discard).  The weight gradient dW = X^T dY is formed on the matrix cores and consumed at once: in that kernel's
// epilogue, or by a second kernel that reads it as partial sums from the workspace; then the per-variable finalize.
#include "omc_dw_args.h"

namespace omc {

template <int NW>
__global__ __launch_bounds__(64 * NW) void dw_finalize_kernel(const Partial *__restrict__ ws, uint32_t nparts, uint64_t n,
                                                              int use_pvt, int exact, float *__restrict__ sb) {
    __shared__ double red[NW * 10];
    finalize_variable<NW>(ws, nparts, nullptr, n, use_pvt != 0, exact != 0, sb, red);
}

// one Partial per 2048 elements (the finest grain any of the update kernels uses)
static size_t dw_fit_bytes(uint32_t N, uint32_t K) {
    return (static_cast<size_t>(K) * N / kTileElems * sizeof(Partial) + 255) / 256 * 256;
}

// How many fp32 copies of the gradient the workspace holds.  This is part of what callers size their workspace by, whether the route taken
// writes them or not: as many as keep 256 compute units busy with 256 x 128 tiles on runs of at least 2048 rows, where that gives at
// least 128 workgroups (one copy also for 8-bit codes, which the one-kernel route leaves unused); else as many as give 512
// workgroups, with those tiles or half of them, on runs of at least 512 rows, at most 8, and none for 8-bit codes where one would do.
static uint32_t gradient_room(uint32_t bits, uint32_t M, uint32_t N, uint32_t K) {
    const uint64_t tiles = static_cast<uint64_t>(K / 256) * (N / 128);
    auto splits_for = [&](uint64_t count, uint64_t enough, uint32_t rows) {
        uint32_t sp = 1;
        while (count * sp < enough && sp < 8 && M % (2 * sp * 32) == 0 && M / (2 * sp) >= rows) sp *= 2;
        return sp;
    };
    if (tiles <= 256) {
        const uint32_t sp = splits_for(tiles, 129, 2048);     // doubled while the doubled count is at most 256
        if (M / sp >= 2048 && tiles * sp >= 128) return sp;
    }
    uint32_t sp = splits_for(tiles, 512, 512);
    if (tiles * sp < 512) sp = splits_for(2 * tiles, 512, 512);
    return bits == 8 && sp == 1 ? 0u : sp;
}

// Host only, not part of the interface: which kernels a call of these sizes takes, 10000 for the one-kernel route + 100 * tile + splits.
extern "C" uint32_t omc_internal_dw_route(uint32_t bits, uint32_t M, uint32_t N, uint32_t K) {
    const uint32_t room = gradient_room(bits, M, N, K);
    const bool one_kernel = bits == 8 && dw_one_kernel_is_faster(M, N, K, room);
    return (one_kernel ? 10000u : 0u) + dw_tile_and_splits(M, N, K, room, !one_kernel);
}

int launch_dw_update(const uint16_t *X, const uint16_t *dY, void *codes, const FmtParams &fp, float *sb, int use_pvt,
                     float *state0, float *state1, const omc_opt &opt, float *dW_out, uint32_t M, uint32_t N,
                     uint32_t K, void *ws, void *stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    const uint32_t room = gradient_room(fp.bits, M, N, K);
    // workspace: the fit's partials | the gradient's partial sums
    uint8_t *w8 = static_cast<uint8_t *>(ws);
    float *sums = reinterpret_cast<float *>(w8 + dw_fit_bytes(N, K));
    DwArgs a{};
    a.X = X;
    a.dY = dY;
    a.codes = static_cast<uint32_t *>(codes);
    a.sb = sb;
    a.st0 = opt.kind >= OMC_MOMENTUM ? state0 : nullptr;
    a.st1 = opt.kind == OMC_ADAM ? state1 : nullptr;
    a.dW_out = dW_out;
    a.ws = reinterpret_cast<Partial *>(w8);
    a.partials = sums;
    a.fp = fp;
    a.oc = OptConst{opt.lr, opt.momentum, opt.beta1, opt.beta2, opt.eps, opt.one_minus_beta1,
                    opt.one_minus_beta2, opt.bias_corr1, opt.bias_corr2};
    a.M = M;
    a.N = N;
    a.K = K;
    uint32_t nparts = 0;
    int rc;
    const bool one_kernel = fp.bits == 8 && dw_one_kernel_is_faster(M, N, K, room);
    if (one_kernel) {
        rc = launch_dw_one_kernel(a, room, opt.kind, &nparts, st);
    } else {
        nparts = static_cast<uint32_t>(static_cast<uint64_t>(K) * N / kTileElems);
        rc = launch_dw_product(a, sums, room, &a.nsplit, st);
        if (rc != 0) return rc;
        if (opt.kind == OMC_SGD) rc = launch_dw_update_sgd(a, st);
        else if (opt.kind == OMC_MOMENTUM) rc = launch_dw_update_momentum(a, st);
        else rc = launch_dw_update_adam(a, st);
    }
    if (rc != 0) return rc;
    const uint64_t n = static_cast<uint64_t>(K) * N;
    // the width of the reduction depends on the sizes alone, so results do not depend on the run
    const int exact = one_kernel || variant_exact(fp.variant) ? 1 : 0;   // the partials carry error words
    if (nparts <= 256) dw_finalize_kernel<1><<<dim3(1), dim3(64), 0, st>>>(a.ws, nparts, n, use_pvt, exact, sb);
    else if (nparts <= 2048) dw_finalize_kernel<4><<<dim3(1), dim3(256), 0, st>>>(a.ws, nparts, n, use_pvt, exact, sb);
    else dw_finalize_kernel<16><<<dim3(1), dim3(1024), 0, st>>>(a.ws, nparts, n, use_pvt, exact, sb);
    return static_cast<int>(hipGetLastError());
}

size_t dw_workspace_bytes(uint32_t bits, uint32_t M, uint32_t N, uint32_t K) {
    return dw_fit_bytes(N, K) + static_cast<size_t>(gradient_room(bits, M, N, K)) * K * N * sizeof(float);
}

}  // namespace omc
