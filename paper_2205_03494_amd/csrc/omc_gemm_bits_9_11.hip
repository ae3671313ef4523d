// Products on packed weights, codes of 9 to 11 bits.
#include "omc_gemm_bits_impl.h"

namespace omc {
int launch_gemm_bits_9_11(const BitsArgs &ga, uint32_t M, int trans, hipStream_t st) {
    switch (ga.fp.bits) {
        case 9: return launch_bits<9>(ga, M, trans, st);
        case 10: return launch_bits<10>(ga, M, trans, st);
        case 11: return launch_bits<11>(ga, M, trans, st);
        default: return static_cast<int>(hipErrorInvalidValue);
    }
}
}  // namespace omc
