// Update kernels of the fused weight-gradient step for every code width, sgd optimizer.
#include "omc_dw_generic_impl.h"

namespace omc {
int launch_dw_update_sgd(const DwArgs &a, hipStream_t st) { return launch_dw_update_mode<kStepSgd>(a, st); }
}  // namespace omc
