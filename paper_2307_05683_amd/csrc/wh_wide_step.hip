// The step kernel of small ensembles (four lanes per planet, wh_wide.h), DHC: a
// translation unit of its own, as the pair layout's, for its schedule (build.py).
#include "wh_wide_kernel.h"

namespace wh {

#define WH_WIDE(STORAGE)                                                     \
  template __global__ void k_step_wide<false, WH_DKD, 0, STORAGE>(StepParams); \
  template __global__ void k_step_wide<true, WH_DKD, 0, STORAGE>(StepParams);  \
  template __global__ void k_step_wide<false, WH_KDK, 0, STORAGE>(StepParams); \
  template __global__ void k_step_wide<true, WH_KDK, 0, STORAGE>(StepParams);  \
  template __global__ void k_step_wide<false, WH_DKD, 1, STORAGE>(StepParams); \
  template __global__ void k_step_wide<true, WH_DKD, 1, STORAGE>(StepParams);  \
  template __global__ void k_step_wide<false, WH_KDK, 1, STORAGE>(StepParams); \
  template __global__ void k_step_wide<true, WH_KDK, 1, STORAGE>(StepParams);  \
  template __global__ void k_step_wide<false, SCHEME_SABA, 0, STORAGE>(StepParams)
WH_WIDE(0);
WH_WIDE(1);
#undef WH_WIDE

}  // namespace wh
