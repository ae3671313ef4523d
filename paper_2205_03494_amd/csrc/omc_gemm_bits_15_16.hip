// Products on packed weights, codes of 15 to 16 bits.
#include "omc_gemm_bits_impl.h"

namespace omc {
int launch_gemm_bits_15_16(const BitsArgs &ga, uint32_t M, int trans, hipStream_t st) {
    switch (ga.fp.bits) {
        case 15: return launch_bits<15>(ga, M, trans, st);
        case 16: return launch_bits<16>(ga, M, trans, st);
        default: return static_cast<int>(hipErrorInvalidValue);
    }
}
}  // namespace omc
