// Products on packed weights, codes of 6 to 8 bits.
#include "omc_gemm_bits_impl.h"

namespace omc {
int launch_gemm_bits_6_8(const BitsArgs &ga, uint32_t M, int trans, hipStream_t st) {
    switch (ga.fp.bits) {
        case 6: return launch_bits<6>(ga, M, trans, st);
        case 7: return launch_bits<7>(ga, M, trans, st);
        case 8: return launch_bits<8>(ga, M, trans, st);
        default: return static_cast<int>(hipErrorInvalidValue);
    }
}
}  // namespace omc
