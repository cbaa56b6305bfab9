// The step kernel of small ensembles (four lanes per planet, wh_wide.h) in
// Jacobi coordinates, on the default schedule (build.py).
#include "wh_wide_kernel.h"

namespace wh {

template __global__ void k_step_wide<false, WH_DKD, 0, 0, true>(StepParams);
template __global__ void k_step_wide<true, WH_DKD, 0, 0, true>(StepParams);
template __global__ void k_step_wide<false, WH_KDK, 0, 0, true>(StepParams);
template __global__ void k_step_wide<true, WH_KDK, 0, 0, true>(StepParams);
template __global__ void k_step_wide<false, SCHEME_SABA, 0, 0, true>(StepParams);
template __global__ void k_step_wide<true, SCHEME_SABA, 0, 0, true>(StepParams);

}  // namespace wh
