// The form that one call of n_steps takes outside balanced launches, by the
// library's own rules (wh_host.h), for tests that compare two forms: launches
// in even shares, 1 for a single one.  Exported for ctypes.
#include "wh_host.h"

extern "C" int step_form_launches(int S, const int32_t* n_planets, int packing, int scheme, int gr, int simds,
                                  int n_steps) {
  using namespace wh_host;
  wh_config cfg;
  config_defaults(&cfg, S);
  cfg.scheme = scheme;
  cfg.gr_c = gr ? 100.0 : 0.0;
  Packing P;
  std::string why;
  if (!make_packing(S, n_planets, packing, P, &why)) return -1;
  EvenShare e{};
  return choose_even(P, cfg, simds, n_steps, e) ? e.slices : 1;
}
