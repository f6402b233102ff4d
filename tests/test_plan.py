"""The host searches for launch shapes (gmg_plan.hpp) against plain searches
over everything, and what they cost, on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

ROUNDS = r"""
#include <chrono>
#include <cstdio>
#include <random>
#include "gmg_plan.hpp"
using namespace gmg;

// every chunk length of the range, the smallest of each chunk count
Rounds all(int nz, long long cols, long long resident, int min_kc, int extra, int min_rounds, int step) {
  const int first = std::max(step, (std::min(nz, min_kc) + step - 1) / step * step);
  Rounds best{first, 1e300}, any{first, 1e300};
  for (int kc = first; kc < nz + step; kc += step) {
    const long long gz = (nz + kc - 1) / kc;
    if (kc > first && (nz + kc - step - 1) / (kc - step) == gz) continue;
    const long long rounds = (cols * gz + resident - 1) / resident;
    const double cost = (double)rounds * (kc + extra);
    if (cost < any.planes) any = {kc, cost};
    if (rounds >= min_rounds && cost < best.planes) best = {kc, cost};
  }
  return best.planes < 1e300 ? best : any;
}

int main() {
  std::mt19937 r(1);
  auto pick = [&](int lo, int hi) { return (int)(lo + r() % (unsigned)(hi - lo + 1)); };
  for (int t = 0; t < 200000; ++t) {
    const int step = pick(1, 2), nz = pick(1, 8) == 1 ? pick(1, 20) * step : pick(1, 700) * step;
    const int min_kc = pick(1, 40), extra = pick(0, 3), min_rounds = pick(1, 4);
    const long long cols = pick(1, 4000), resident = 256LL * pick(1, 8);
    const Rounds a = all(nz, cols, resident, min_kc, extra, min_rounds, step);
    const Rounds b = rounds_of(nz, cols, resident, min_kc, extra, min_rounds, step);
    if (a.kc != b.kc || a.planes != b.planes) {
      std::printf("nz %d cols %lld resident %lld min_kc %d extra %d min_rounds %d step %d: %d, expected %d\n", nz, cols,
                  resident, min_kc, extra, min_rounds, step, b.kc, a.kc);
      return 1;
    }
  }
  volatile int sink = 0;
  auto us = [&](auto f) {
    const auto t0 = std::chrono::steady_clock::now();
    for (int i = 0; i < 50; ++i) sink = f(65536 + i).kc;
    return std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count() / 50;
  };
  const double plain = us([](int nz) { return all(nz, 16, 1024, 1, 2, 1, 1); });
  const double found = us([](int nz) { return rounds_of(nz, 16, 1024, 1, 2, 1, 1); });
  std::printf("65536 planes: %.2f us, over every chunk %.2f us\n", found, plain);
  return found < 0.1 * plain ? 0 : 2;
}
"""

LEGS = r"""
#include <chrono>
#include <cstdio>
#include <random>
#include "gmg_plan.hpp"
using namespace gmg;

struct Shape { int nx, ny, nz; };

// every box, every split
template <typename T>
bool box(const Shape& s, int sweeps, bool zero, bool resid, int cus, LegPlan& best, double& cost) {
  const int nh = 2 * sweeps, R = nh + (resid ? 1 : 0) - (zero ? 1 : 0), H = s.nx / 2;
  cost = 1e300;
  for (int tx = H;; tx = (tx + 1) / 2) {
    const int hx = tx == H ? 0 : (R + 1) / 2;
    for (int ty = 2; ty <= 16; ty += 2)
      for (int tz = 2; tz <= 16; tz += 2) {
        const int rx = tx + 2 * hx, ry = ty + 2 * R, rz = tz + 2 * R, pairs = rx * ry * rz;
        if (pairs > LegShape<T>::max_pairs || rx * (ry + 2) * (rz + 2) + 2 > LegShape<T>::lds ||
            tx * ty * tz > LegShape<T>::own)
          continue;
        const long long blocks = (long long)((H + tx - 1) / tx) * ((s.ny + ty - 1) / ty) * ((s.nz + tz - 1) / tz);
        const double c = leg_cost<T>(blocks, pairs, nh, cus);
        if (c < cost) {
          cost = c;
          best = {sweeps, tx, ty, tz, hx, R};
        }
      }
    if (tx <= 8) break;
  }
  return cost < 1e300;
}
template <typename T>
double split(const Shape& s, int nu, bool zero, bool resid, int cus, std::vector<LegPlan>& out) {
  double best = 1e300;
  for (int first = 1; first <= std::min(nu, 3); ++first) {
    LegPlan p{};
    double c;
    if (!box<T>(s, first, zero, resid && first == nu, cus, p, c)) continue;
    std::vector<LegPlan> rest;
    if (first < nu) c += split<T>(s, nu - first, false, resid, cus, rest);
    if (c < best) {
      best = c;
      out.assign(1, p);
      out.insert(out.end(), rest.begin(), rest.end());
    }
  }
  return best;
}

template <typename T>
int compare(const Shape& s, int nu) {
  LegSearch<T> search(s.nx, s.ny, s.nz, 256);
  for (int which = 0; which < 3; ++which) {
    const bool zero = which == 0, resid = which != 2;
    std::vector<LegPlan> a, b;
    const double ca = split<T>(s, nu, zero, resid, 256, a), cb = search.split(nu, zero, resid, b);
    bool same = ca == cb && a.size() == b.size();
    for (size_t i = 0; same && i < a.size(); ++i)
      same = a[i].sweeps == b[i].sweeps && a[i].tx == b[i].tx && a[i].ty == b[i].ty && a[i].tz == b[i].tz &&
             a[i].hx == b[i].hx && a[i].hy == b[i].hy;
    if (!same) {
      std::printf("%d x %d x %d, %d sweeps, leg %d, %d bytes: %g, expected %g\n", s.nx, s.ny, s.nz, nu, which,
                  (int)sizeof(T), cb, ca);
      return 1;
    }
  }
  return 0;
}

int main() {
  std::mt19937 r(2);
  auto even = [&](int hi) { return 2 * (1 + (int)(r() % (unsigned)(hi / 2))); };
  for (int t = 0; t < 150; ++t) {
    const Shape s{t % 10 ? even(160) : even(6000), even(160), even(160)};
    for (int nu = 1; nu <= 6; ++nu)
      if (compare<float>(s, nu) || compare<double>(s, nu)) return 1;
  }
  const Shape s{64, 64, 64};
  if (compare<float>(s, 8) || compare<double>(s, 8)) return 1;
  auto us = [&](auto f) {
    const auto t0 = std::chrono::steady_clock::now();
    for (int i = 0; i < 5; ++i) f();
    return std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count() / 5;
  };
  std::vector<LegPlan> out;
  const double plain = us([&] { split<float>(s, 8, false, true, 256, out); });
  const double found = us([&] { LegSearch<float>(s.nx, s.ny, s.nz, 256).split(8, false, true, out); });
  std::printf("8 sweeps: %.1f us, over every split %.1f us\n", found, plain);
  return found < 0.25 * plain ? 0 : 2;
}
"""


def _run(tmp_path, source):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(source)
    subprocess.run([cxx, "-O2", "-std=c++17", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_1812_08606_amd", "csrc"), "-o", str(exe), str(src)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert done.returncode == 0, done.stdout + done.stderr
    return done.stdout


def test_rounds_search(tmp_path):
    """The same chunk and product as a search over every chunk length, in well
    under a tenth of its time on 65536 planes (about 512 chunk counts)."""
    print(_run(tmp_path, ROUNDS))


def test_leg_search(tmp_path):
    """The same boxes and splits as trying every split of a leg, without its
    growth with the number of sweeps (176 boxes per leg of 8 sweeps)."""
    print(_run(tmp_path, LEGS))
