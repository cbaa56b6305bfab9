// The reverse-mode kernel of small ensembles (four lanes per planet,
// wh_wide_adjoint.h), a translation unit of its own for its schedule: with one
// wavefront per SIMD it is scheduled for latency (max-ilp).
#include "wh_wide_adjoint.h"

namespace wh {

template <bool GR, bool SPLIT, int SCH, bool FIN> __global__ __launch_bounds__(64) void k_adj_wide(AdjParams q) {
  __shared__ double lds[WIDE_ADJ_LDS];
  const StepParams& p = q.sp;
  const int lane = threadIdx.x, ww = q.wide_waves;
  int w = (int)blockIdx.x;
  const bool sweep = !FIN && w < q.sweep_waves;
  if (!sweep) w -= q.sweep_waves;
  if (w >= ww) return;
  if (sweep) {
    const bool first = q.first_synced != 0;
    if (SPLIT) wide_sweep<8, GR, SCH, 1>(p, q.grad, q.tape, ww, q.n_seg, first, w, lds, lane);
    else if (w < 4 * p.w1) wide_sweep<1, GR, SCH, 0>(p, q.grad, q.tape, ww, q.n_seg, first, w, lds, lane);
    else if (w < 4 * p.w2) wide_sweep<2, GR, SCH, 0>(p, q.grad, q.tape, ww, q.n_seg, first, w, lds, lane);
    else if (w < 4 * p.w4) wide_sweep<4, GR, SCH, 0>(p, q.grad, q.tape, ww, q.n_seg, first, w, lds, lane);
    else wide_sweep<8, GR, SCH, 0>(p, q.grad, q.tape, ww, q.n_seg, first, w, lds, lane);
  } else {
    const bool first = q.rec_first_synced != 0;
    if (SPLIT) wide_record<8, GR, SCH, 1, FIN>(p, q.ck_rec, q.tape_rec, ww, q.n_rec, first, w, lds, lane);
    else if (w < 4 * p.w1) wide_record<1, GR, SCH, 0, FIN>(p, q.ck_rec, q.tape_rec, ww, q.n_rec, first, w, lds, lane);
    else if (w < 4 * p.w2) wide_record<2, GR, SCH, 0, FIN>(p, q.ck_rec, q.tape_rec, ww, q.n_rec, first, w, lds, lane);
    else if (w < 4 * p.w4) wide_record<4, GR, SCH, 0, FIN>(p, q.ck_rec, q.tape_rec, ww, q.n_rec, first, w, lds, lane);
    else wide_record<8, GR, SCH, 0, FIN>(p, q.ck_rec, q.tape_rec, ww, q.n_rec, first, w, lds, lane);
  }
}

#define WH_ADJ_WIDE(SPLIT, FIN)                                                  \
  template __global__ void k_adj_wide<false, SPLIT, WH_DKD, FIN>(AdjParams);     \
  template __global__ void k_adj_wide<true, SPLIT, WH_DKD, FIN>(AdjParams);      \
  template __global__ void k_adj_wide<false, SPLIT, WH_KDK, FIN>(AdjParams);     \
  template __global__ void k_adj_wide<true, SPLIT, WH_KDK, FIN>(AdjParams);      \
  template __global__ void k_adj_wide<false, SPLIT, SCHEME_SABA, FIN>(AdjParams)
WH_ADJ_WIDE(false, false);
WH_ADJ_WIDE(false, true);
WH_ADJ_WIDE(true, false);
WH_ADJ_WIDE(true, true);
#undef WH_ADJ_WIDE

}  // namespace wh
