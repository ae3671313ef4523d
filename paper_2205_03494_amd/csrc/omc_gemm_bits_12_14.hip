// Products on packed weights, codes of 12 to 14 bits.
#include "omc_gemm_bits_impl.h"

namespace omc {
int launch_gemm_bits_12_14(const BitsArgs &ga, uint32_t M, int trans, hipStream_t st) {
    switch (ga.fp.bits) {
        case 12: return launch_bits<12>(ga, M, trans, st);
        case 13: return launch_bits<13>(ga, M, trans, st);
        case 14: return launch_bits<14>(ga, M, trans, st);
        default: return static_cast<int>(hipErrorInvalidValue);
    }
}
}  // namespace omc
