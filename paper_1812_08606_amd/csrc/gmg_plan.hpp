// gmg_plan.hpp -- launch shapes found by a search on the host (no device
// code, no HIP: a host compiler alone builds it).
#pragma once

#include <algorithm>
#include <array>
#include <vector>

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

// Pairs of the box and its halo: at most PPT per thread, as many as the
// registers hold (15 weights and right sides a pair).  LDS elements of one
// colour: the pairs, a frame of one row and plane, and one before and after.
template <typename T>
struct LegShape {
  static constexpr int threads = sizeof(T) == 4 ? 1024 : 512;
  static constexpr int max_pairs = sizeof(T) == 4 ? 4096 : 2560;
  static constexpr int lds = sizeof(T) == 4 ? 7168 : 4608;
  static constexpr int own = 2048;
};

// One launch of a leg.
struct LegPlan {
  int sweeps;          // symmetric sweeps
  int tx, ty, tz;      // owned box: pairs, rows, planes
  int hx, hy;          // halo: pairs; rows and planes
};

// Time of one launch of a leg (clocks, a model fitted to the bottom kernel's
// and the leg's measured phases): launch and first loads, then per pair of
// the box with its halo the loads and each half-sweep, times the rounds of
// blocks (one per CU).
template <typename T>
double leg_cost(long long blocks, int pairs, int nh, int cus) {
  const double load = sizeof(T) == 4 ? 1.6 : 3.2, half = sizeof(T) == 4 ? 0.55 : 0.75;
  return 9000.0 + (double)((blocks + cus - 1) / cus) * (4000.0 + pairs * (load + half * nh));
}

// Launches of the legs of one level: the boxes and the splits that cost least.
template <typename T>
class LegSearch {
 public:
  LegSearch(int nx, int ny, int nz, int cus) : nx_(nx), ny_(ny), nz_(nz), cus_(cus) {}

  // A leg of nu sweeps (from x = 0 when zero, the residual after it when
  // resid) as launches of one to three sweeps; their cost, 1e300 when there is
  // none.  The cheapest way to run the last n sweeps, which start from an
  // iterate, is found for n = 1, 2, ...  (a leg splits in 81 ways at 8 sweeps:
  // trying each took 0.6 ms of the set-up per level, this 0.02).
  double split(int nu, bool zero, bool resid, std::vector<LegPlan>& out) {
    std::vector<double> cost(nu + 1, 1e300);
    std::vector<int> first(nu + 1, 0);
    cost[0] = 0.0;
    for (int n = 1; n <= nu; ++n)
      for (int f = 1; f <= std::min(n, 3); ++f) {
        const Box& b = box(f, zero && n == nu, resid && f == n);
        if (b.cost < 1e300 && b.cost + cost[n - f] < cost[n]) {
          cost[n] = b.cost + cost[n - f];
          first[n] = f;
        }
      }
    out.clear();
    if (cost[nu] < 1e300)
      for (int n = nu; n > 0; n -= first[n]) out.push_back(box(first[n], zero && n == nu, resid && first[n] == n).plan);
    return cost[nu];
  }

 private:
  struct Box {
    bool known = false;
    double cost = 1e300;
    LegPlan plan{};
  };

  // The cheapest box for `sweeps` symmetric sweeps: halo of 2 sweeps cells (one
  // more with the residual, one less from x = 0).
  const Box& box(int sweeps, bool zero, bool resid) {
    Box& best = boxes_[(sweeps - 1) * 4 + zero * 2 + resid];
    if (best.known) return best;
    best.known = true;
    const int nh = 2 * sweeps, R = nh + (resid ? 1 : 0) - (zero ? 1 : 0), H = nx_ / 2;
    for (int tx = H;; tx = (tx + 1) / 2) {
      const int hx = tx == H ? 0 : (R + 1) / 2;
      for (int ty = 2; ty <= 16; ty += 2)
        for (int tz = 2; tz <= 16; tz += 2) {
          const long long rx = tx + 2 * hx, ry = ty + 2 * R, rz = tz + 2 * R;
          if (rx * ry * rz > LegShape<T>::max_pairs || rx * (ry + 2) * (rz + 2) + 2 > LegShape<T>::lds ||
              tx * ty * tz > LegShape<T>::own)
            continue;
          const long long blocks =
              (long long)((H + tx - 1) / tx) * ((ny_ + ty - 1) / ty) * ((nz_ + tz - 1) / tz);
          const double c = leg_cost<T>(blocks, (int)(rx * ry * rz), nh, cus_);
          if (c < best.cost) {
            best.cost = c;
            best.plan = {sweeps, tx, ty, tz, hx, R};
          }
        }
      if (tx <= 8) break;
    }
    return best;
  }

  int nx_, ny_, nz_, cus_;
  std::array<Box, 12> boxes_;
};

}  // namespace gmg
