// Update kernels of the fused weight-gradient step for every code width, adam optimizer.
#include "omc_dw_generic_impl.h"

namespace omc {
int launch_dw_update_adam(const DwArgs &a, hipStream_t st) { return launch_dw_update_mode<kStepAdam>(a, st); }
}  // namespace omc
