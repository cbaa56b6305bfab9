// Even shares of a launch (EvenShare, wh_host.h): every wave runs all its
// steps, none appears twice in a slice (the two parts of a cut wave lie in
// different ones, the first part first), and the bins' slices weigh the same.
#include "wh_host.h"

#include <cstdio>
#include <random>

using namespace wh_host;

int main() {
  std::mt19937 r(1);
  const int costs[2][5] = {{316, 331, 378, 478, 543}, {330, 367, 416, 526, 598}}, bins[] = {1024, 2048, 7, 64};
  const int steps[] = {64, 100, 300, 1000, 4096, 1000000};
  int used = 0, by_slices[7] = {0};
  for (int t = 0; t < 1500; ++t) {
    EvenShare e{};
    const int c = r() % 2;
    e.bins = bins[r() % 4];
    e.steps = steps[r() % 6];
    for (int g = 0; g < 5; ++g) {
      e.cost[g] = costs[c][g];
      e.first[g + 1] = e.first[g] + (r() % 3 == 0 ? 0 : (int)(r() % (5 * e.bins / 4)));
    }
    const int W = e.first[5];
    if (W == 0 || (e.slices = even_slices(e, 6)) == 0) continue;
    ++used;
    ++by_slices[e.slices];
    std::vector<int> done(W, 0);
    const double share = even_total(e) / e.bins * e.steps / e.slices;
    for (e.slice = 0; e.slice < e.slices; ++e.slice) {
      std::vector<char> seen(W, 0);
      for (int b = 0; b < e.bins; ++b) {
        double weight = 0.0;
        int w = 0, s = 0;
        for (int i = 0; even_piece(e, b, i, w, s); ++i) {
          if (i >= EVEN_PIECES) return std::printf("too many pieces\n"), 1;
          if (s == 0) continue;
          if (s < 0 || w < 0 || w >= W) return std::printf("out of range\n"), 1;
          if (seen[w]) return std::printf("wave %d twice in slice %d of %d\n", w, e.slice, e.slices), 1;
          seen[w] = 1;
          done[w] += s;
          weight += (double)s * e.cost[w < e.first[1] ? 0 : w < e.first[2] ? 1 : w < e.first[3] ? 2 : w < e.first[4] ? 3 : 4];
        }
        // a bin's ends are rounded to whole units of a step's cost, its cuts
        // to whole steps
        if (weight > share + e.steps + 4 * 598) return std::printf("slice %g of %g\n", weight, share), 1;
      }
    }
    for (int w = 0; w < W; ++w)
      if (done[w] != e.steps) return std::printf("wave %d: %d of %d steps\n", w, done[w], e.steps), 1;
  }
  if (used < 200 || !by_slices[2] || !by_slices[3] || !by_slices[6]) return std::printf("only %d used\n", used), 1;
  std::printf("even shares ok\n");
  return 0;
}
