// gmg_plan.hpp -- launch shapes found by a search on the host (no device
// code, no HIP: a host compiler alone builds it).
#pragma once

#include <algorithm>

namespace gmg {

// z-chunk of a column-marching launch with `cols` blocks per chunk column
// and `resident` blocks running at once: the chunk (at least min_kc planes, a
// multiple of step) that minimises the rounds of blocks times the planes a
// block marches (its chunk plus `extra`), the smallest chunk for each chunk
// count, among chunks that give at least min_rounds rounds when any does; and
// that product.  (A round with few blocks leaves most CUs idle: at level 1 of
// the 512^3 grid, 11-plane chunks made 1032 blocks of one per CU, 4.03 rounds
// on 256 CUs; 24-plane chunks, 473 blocks in 2 rounds, took 110.5 us per sweep
// against 137.8.  An even chunk is chosen as such: rounding the best chunk
// down instead made 2 rounds of 1, 285 us against 166 for the fused residual
// sweep at 320^3.)
//
// The search goes from one chunk count to the next, about 2 sqrt(nz) of them:
// sweeps ask once per launch.  (A look at every chunk length took 1.2 us at
// nz = 256, 2.7 at 512 and 140 at 32768, as long as a kernel on such a grid;
// this takes 0.3, 0.5 and 4.)
struct Rounds {
  int kc;
  double planes;
};
inline Rounds rounds_of(int nz, long long cols, long long resident, int min_kc, int extra, int min_rounds = 1,
                        int step = 1) {
  auto up = [step](int kc) { return (kc + step - 1) / step * step; };
  const int first = std::max(step, up(std::min(nz, min_kc)));
  Rounds best{first, 1e300}, any{first, 1e300};
  for (int kc = first;;) {
    const int gz = (nz + kc - 1) / kc;
    const long long rounds = (cols * gz + resident - 1) / resident;
    const double cost = (double)rounds * (kc + extra);
    if (cost < any.planes) any = {kc, cost};
    if (rounds >= min_rounds && cost < best.planes) best = {kc, cost};
    if (gz == 1) break;
    kc = up((nz + gz - 2) / (gz - 1));  // the smallest chunk of fewer than gz chunks
  }
  return best.planes < 1e300 ? best : any;
}
inline int rounds_kc(int nz, long long cols, long long resident, int min_kc, int extra, int min_rounds = 1) {
  return std::min(nz, rounds_of(nz, cols, resident, min_kc, extra, min_rounds).kc);
}

}  // namespace gmg
