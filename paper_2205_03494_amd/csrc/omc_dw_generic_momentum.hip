// Update kernels of the fused weight-gradient step for every code width, momentum optimizer.
#include "omc_dw_generic_impl.h"

namespace omc {
int launch_dw_update_momentum(const DwArgs &a, hipStream_t st) { return launch_dw_update_mode<kStepMomentum>(a, st); }
}  // namespace omc
