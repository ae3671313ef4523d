// Products on packed weights, codes of 2 to 5 bits.
#include "omc_gemm_bits_impl.h"

namespace omc {
int launch_gemm_bits_2_5(const BitsArgs &ga, uint32_t M, int trans, hipStream_t st) {
    switch (ga.fp.bits) {
        case 2: return launch_bits<2>(ga, M, trans, st);
        case 3: return launch_bits<3>(ga, M, trans, st);
        case 4: return launch_bits<4>(ga, M, trans, st);
        case 5: return launch_bits<5>(ga, M, trans, st);
        default: return static_cast<int>(hipErrorInvalidValue);
    }
}
}  // namespace omc
