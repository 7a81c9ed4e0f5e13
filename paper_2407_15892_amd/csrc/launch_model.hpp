// Host side: estimates, in microseconds, of launches of large tiles (one workgroup per compute unit) on a whole chip.
// They only have to rank the ways of cutting a problem.
//
// Fitted to launches of the 8B-shaped configurations at S = 200 to 32768.  A 256 x 256 tile takes 1.375 per K step with all
// compute units busy (the chip is power limited then), 1.25 otherwise, plus what its ends take; a dW tile's ends: 12 plus
// 0.1 per K step up to 20, and 10 more where it is read.  A launch takes whole rounds of kNumCu tiles at the faster rate,
// all its tiles at the slower one, or its bytes at 4.6 TB/s, whichever is longest, plus 2.  Two kinds of tiles in one
// launch: those of the first kind first, those of the second as compute units come free; bound by bytes it takes a third
// longer than the bytes alone (200 rows, V = 128256: dH's loads wait behind dW's stores, 930 for the 3.3 GB that take 740
// in two launches).
#pragma once
#include <stdint.h>

#include <algorithm>

namespace mst {

constexpr int kNumCu = 256;          // MI355X compute units
constexpr double kBusyStepUs = 1.375, kStepUs = 1.25, kHbmBytesPerUs = 4.6e6;
struct TileCost {
  double ksteps, ends;
  double step = kStepUs, busy_step = kBusyStepUs;
  double busy() const { return busy_step * ksteps + ends; }
  double alone() const { return step * ksteps + ends; }
};
inline TileCost tile_cost(int64_t k, double ends) { return {(double)((k + 63) / 64), ends}; }
inline TileCost dw_cost(int64_t rows, bool add) {
  TileCost c = tile_cost(rows, 0.0);
  c.ends = 12.0 + (c.ksteps < 80.0 ? 0.1 * c.ksteps : 8.0) + (add ? 10.0 : 0.0);
  return c;
}
inline double launch_us(int64_t tiles, TileCost c, double bytes) {
  const double rounds = (double)((tiles + kNumCu - 1) / kNumCu) * c.alone(), busy = (double)tiles / kNumCu * c.busy();
  return 2.0 + std::max(std::max(rounds, busy), bytes / kHbmBytesPerUs);
}
// The time until n1 pieces of work of t1, then n2 of t2, handed out in this order to `units`, are done: n1 % units of them are
// late for the second kind by one piece of the first, and the others take pieces of it meanwhile.  The end is that of the
// n2-th piece: a multiple of t2 after the moment `a` when the others are free, or after the late ones are.
inline double span_us(int64_t n1, double t1, int64_t n2, double t2, int64_t units) {
  const double a = (double)(n1 / units) * t1;
  const int64_t late = n1 % units, others = units - late;
  const int64_t f = late ? (int64_t)(t1 / t2) : 0, c = late ? f + 1 : 0;    // whole pieces before the late ones' first, + 1
  auto up = [](int64_t n, int64_t by) { return n > 0 ? (n + by - 1) / by : 0; };
  const int64_t j = up(n2, others);
  const double with_others = (double)(j <= c ? j : up(n2 + late * c, units)) * t2;
  const double with_late = t1 + (double)up(n2 - others * f, units) * t2;
  return a + (late ? std::max(t1, std::min(with_others, with_late)) : with_others);
}
// n1 tiles of c1, then n2 of c2
inline double launch_us(int64_t n1, TileCost c1, int64_t n2, TileCost c2, double bytes) {
  const double span = span_us(n1, c1.alone(), n2, c2.alone(), kNumCu);
  const double busy = ((double)n1 * c1.busy() + (double)n2 * c2.busy()) / kNumCu;
  return 2.0 + std::max(std::max(span, busy), 1.3 * bytes / kHbmBytesPerUs);
}

}  // namespace mst
