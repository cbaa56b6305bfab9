// Definition of k_step_wide (declared in wh_wide.h), for the translation units
// that instantiate it.
#pragma once
#include "wh_wide.h"

namespace wh {

template <bool GR, int SCHEME, int KC, int STORAGE, bool JAC>
__global__ __launch_bounds__(256) void k_step_wide(StepParams p) {
  __shared__ double lds[4 * WIDE_LDS];
  const int lane = threadIdx.x & 63, wb = threadIdx.x >> 6;
  double* block = lds + wb * WIDE_LDS;
  // 4 wavefronts per wave of 64 slots, 2 per wave of the split packing
  const int w = (int)(blockIdx.x * (blockDim.x >> 6)) + wb;
  if constexpr (STORAGE == 1) {
    if (w < 2 * p.w8) wide_group<8, GR, SCHEME, KC, 1, false>(p, w, block, lane);
    return;
  }
  if (w >= 4 * p.w8) return;
  if (w < 4 * p.w1) wide_group<1, GR, SCHEME, KC, 0, JAC>(p, w, block, lane);
  else if (w < 4 * p.w2) wide_group<2, GR, SCHEME, KC, 0, JAC>(p, w, block, lane);
  else if (w < 4 * p.w4) wide_group<4, GR, SCHEME, KC, 0, JAC>(p, w, block, lane);
  else wide_group<8, GR, SCHEME, KC, 0, JAC>(p, w, block, lane);
}

}  // namespace wh
