// The launches that choose_even and a balanced plan cut into even shares
// (wh_host.h), by the library's own rules, costs and slice caps: in no slice
// may both parts of a cut wave have steps (two wavefronts of one launch would
// then step the same systems), the lower bin's part comes first, and every
// wave runs all its steps.  Long launches are where the roundings of a bin's
// ends count most.
#include "wh_host.h"

#include <cstdio>
#include <random>

using namespace wh_host;

static int used = 0;

// The steps of every wave, counted slice by slice.
static bool whole(EvenShare e) {
  const int W = e.first[5];
  std::vector<int> done(W, 0), slice_of(W, -1);
  for (e.slice = 0; e.slice < e.slices; ++e.slice)
    for (int b = 0; b < e.bins; ++b) {
      int w = 0, s = 0;
      for (int i = 0; even_piece(e, b, i, w, s); ++i) {
        if (i >= EVEN_PIECES) return std::printf("too many pieces\n"), false;
        if (s == 0) continue;
        if (s < 0 || w < 0 || w >= W) return std::printf("out of range\n"), false;
        if (slice_of[w] == e.slice) return std::printf("wave %d twice in slice %d of %d\n", w, e.slice, e.slices), false;
        slice_of[w] = e.slice;
        done[w] += s;
      }
    }
  for (int w = 0; w < W; ++w)
    if (done[w] != e.steps) return std::printf("wave %d: %d of %d steps\n", w, done[w], e.steps), false;
  return true;
}

// The cut waves alone: bin b's first piece (the wave cut at its end) and bin
// b + 1's last.
static bool cuts(EvenShare e) {
  std::vector<int> last(e.bins, -1);   // the last slice of the lower part
  for (e.slice = 0; e.slice < e.slices; ++e.slice)
    for (int b = 0; b < e.bins; ++b) {
      int w = 0, s = 0;
      if (even_piece(e, b, 0, w, s) && s > 0) last[b] = e.slice;
    }
  for (e.slice = 0; e.slice < e.slices; ++e.slice)
    for (int b = 1; b < e.bins; ++b) {
      int lower = 0, w = -1, s = 0, steps = 0, i = 0, wi;
      even_piece(e, b - 1, 0, lower, s);
      // pieces are wave-ordered: the tail, if there is one, is the last
      while (even_piece(e, b, i, wi, s)) w = wi, steps = s, ++i;
      if (w == lower && steps > 0 && e.slice <= last[b - 1])
        return std::printf("wave %d in bins %d and %d of slice %d of %d\n", w, b - 1, b, e.slice, e.slices), false;
    }
  return true;
}

static bool check(const Packing& P, const wh_config& cfg, int steps, bool all) {
  EvenShare e{};
  bool ok = true;
  if (choose_even(P, cfg, 1024, steps, e)) ++used, ok = all ? whole(e) : cuts(e);
  for (int k = 1; ok && k <= 4 && all; ++k)   // a balanced plan's bins
    if (P.nwaves > k * 1024 && even_form(P, cfg, k * 1024, steps, e = EvenShare{})) ++used, ok = whole(e);
  if (!ok) std::printf("%d waves, %d steps, scheme %d, gr %d\n", P.nwaves, steps, cfg.scheme, cfg.gr_c > 0);
  return ok;
}

static Packing eights(int waves) {
  Packing P;
  P.nwaves = P.wm = P.w8 = waves;
  P.ns = 64 * waves;
  return P;
}

int main() {
  wh_config cfg;
  config_defaults(&cfg, 1);
  for (double gr : {0.0, 100.0}) {
    cfg.gr_c = gr;
    for (int W = 1025; W <= 4096; ++W) {
      if (!check(eights(W), cfg, 4096, false)) return 1;
      for (int steps : {1000, 8192, 50000, 1000000})
        if (W % 16 == steps % 7 && !check(eights(W), cfg, steps, false)) return 1;
    }
    for (int W : {1079, 2129, 2158, 2171, 2197, 2343, 2121})
      for (int steps : {128, 1000, 4096, 50000})
        if (!check(eights(W), cfg, steps, true)) return 1;
  }
  std::mt19937 r(2);
  for (int t = 0; t < 60; ++t) {
    const int S = 8000 + r() % 34000, hi = 2 + r() % 7, lo = 1 + r() % hi;
    std::vector<int32_t> n(S);
    for (int& x : n) x = lo + r() % (hi - lo + 1);
    cfg.gr_c = t % 2 ? 100.0 : 0.0;
    cfg.packing = t % 3 == 0 ? WH_PACK_MIXED : WH_PACK_POW2;
    cfg.scheme = t % 5 == 0 && cfg.packing == WH_PACK_POW2 && !cfg.gr_c ? WH_SABA4 : WH_DKD;
    Packing P;
    std::string why;
    if (!make_packing(S, n.data(), cfg.packing, P, &why)) return std::printf("%s\n", why.c_str()), 1;
    const int steps[] = {256, 1000, 4096, 8192, 100000};
    if (!check(P, cfg, steps[r() % 5], true)) return 1;
  }
  if (used < 4000) return std::printf("only %d shares\n", used), 1;
  std::printf("even share cuts ok (%d)\n", used);
  return 0;
}
