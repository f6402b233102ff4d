// gmg_bottom.hpp -- the bottom of the multigrid cycle (levels of at most 4096
// cells down to the coarsest) in one workgroup.
#pragma once

#include "gmg_kernels.hpp"
#include "gmg_sym.hpp"

namespace gmg {

// One launch runs every level from the first bottom level (at most 4096
// cells) to the coarsest: smoothing, residual and restriction, the direct
// coarsest solve, prolongation and post-smoothing, with LDS barriers between
// the phases instead of kernel launches.  Its time is the chain of its 30 to
// 90 short phases, so a phase is made as short as it can be: every x-pair of
// every smoothed level has one owner thread, which computes the pair's face
// weights, reciprocal diagonals and right sides once, at the start, and keeps
// them in registers; a half-sweep is then six LDS reads, six multiply-adds
// and one LDS write.  The iterates lie in LDS, one array per colour (a
// half-sweep then reads and writes consecutive words: at 16^3 its time is LDS
// throughput), with a plane of zeros below and above each level: through a
// plate the mirrored ghost doubles the face coefficient and its neighbour
// value is the zero plane's, so plates need no case of their own, and a
// missing side face has weight 0.  (Recomputing
// index, weights and diagonal from face coefficients in LDS in each phase
// took 1.3 us per phase: 39.7 us per V-cycle and 72 us per full multigrid
// cycle of 16^3 and below, V(2,2), float32, against 16 and 32 now; float64 45
// and 73, now 19 and 32.  Of the V-cycle's 38000 clocks 10000 are the
// launch's first loads and set-up, 1100 each half-sweep at 16^3, 350-700 each
// phase on the levels below, which wait for LDS and the barrier.)
constexpr int BOTTOM_MAX_LEVELS = 4;  // 4096, 512, 64 and 8 cells: every halved dimension is at least 2
// Threads of the workgroup and x-pairs of the first level each owns (2048
// pairs at most): 1024 threads leave 128 registers, enough for two float32
// pairs; 512 leave 256, enough for four float64 ones.  Coarsest inverses up to
// inv_lds rows are read into LDS with the weights, as many as fit beside the
// rest (on the way to a solve of 80 rows the read of its inverse was most of
// the solve).
template <typename T>
struct BottomShape {
  static constexpr int threads = sizeof(T) == 4 ? 1024 : 512;
  static constexpr int pairs = 2048 / threads;
  static constexpr int inv_lds = sizeof(T) == 4 ? 128 : 96;
};
// LDS elements of one colour: 2048 + 256 + 32 pairs on the smoothed levels,
// and two planes of pairs per level (a smoothed level's dimensions are at
// least 4: a plane has at most 512, 64 and 8 pairs).
constexpr int BOTTOM_LDS_X = 2048 + 256 + 32 + 2 * (512 + 64 + 8);

template <typename T>
struct BottomArgs {
  FaceCoef<T> co[BOTTOM_MAX_LEVELS];
  Geom g[BOTTOM_MAX_LEVELS];
  T* x0;
  const T* b0;
  const T* Ainv;
  int nlev;  // levels handled, the last one the coarsest
  int nu_pre, nu_post;
  int xoff[BOTTOM_MAX_LEVELS];  // offset of each smoothed level's first pair in the LDS iterates
};

__device__ __forceinline__ int geom_cells(const Geom& g) { return g.nx * g.ny * g.nz; }

// a / d for 0 <= a < 8192 and 1 <= d <= 1024 with rd = 1 / d to 1 ulp: the
// float product lies within 2e-3 of the quotient plus 1/(2d), away from an
// integer by at least 1/(2d), so truncation gives the exact quotient (checked
// for every such a and d).
__device__ __forceinline__ int small_div(int a, float rd) { return (int)(((float)a + 0.5f) * rd); }

// Coordinates of item p of rows of n items on planes of ny rows.
struct BottomAt {
  int m, j, k;
  __device__ __forceinline__ BottomAt(int p, int n, int ny) {
    // (opaque: recomputed in each phase rather than kept in registers the
    // weights need)
    asm volatile("" : "+v"(p));
    const int row = small_div(p, 1.0f / (float)n);
    m = p - row * n;
    k = small_div(row, 1.0f / (float)ny);
    j = row - k * ny;
  }
};

// Where a pair's interpolation reads the next level: the natural index of its
// parent row's cell m (9 bits, at most 512 cells), the steps to the nearer
// coarse row and plane (-1, 0, 1; 0 outside the grid), whether the coarse
// cells m - 1 and m + 1 exist, and the colour of cell m.  (Found once: the
// coordinates and clamps took most of the interpolation's instructions.)
__device__ __forceinline__ int bottom_parent(const Geom& g, int p) {
  const int NX = g.nx >> 1, NY = g.ny >> 1, NZ = g.nz >> 1;
  const BottomAt at(p, NX, g.ny);
  const int J = at.j >> 1, K = at.k >> 1;
  const int dJ = at.j & 1 ? (J < NY - 1 ? 1 : 0) : (J > 0 ? -1 : 0);
  const int dK = at.k & 1 ? (K < NZ - 1 ? 1 : 0) : (K > 0 ? -1 : 0);
  return ((K * NY + J) * NX + at.m) | (dJ + 1) << 9 | (dK + 1) << 11 | (at.m > 0) << 13 | (at.m < NX - 1) << 14 |
         ((at.m + J + K) & 1) << 15;
}

// One x-pair (cells 2m, 2m + 1 of row j, plane k) of a smoothed level: colour
// c's cell is [c], cell 2m + e_c with e_c = (c + j + k) % 2.
template <typename T>
struct BottomPair {
  int at;                 // its index in the LDS array of either colour
  int dx;                 // colour 0's outer x-neighbour, in colour 1's array, is at + dx; colour 1's at - dx
  int pk;                 // bottom_parent
  T wi;                   // face between the two cells
  T wo[2], ws[2], wn[2];  // outer x-face and y-faces (0 where there is none)
  T wb[2], wt[2];         // z-faces (doubled on the plates)
  T rd[2];                // reciprocal diagonal
  T b[2];                 // right side
};

// Weights and diagonals of the pair (m, j, k) of a level with stored faces.
template <typename T>
__device__ __forceinline__ void pair_weights(BottomPair<T>& q, const FaceCoef<T>& co, const Geom& g, int m, int j,
                                             int k) {
  const int H = g.nx >> 1;
  const size_t c = cidx(g, 2 * m, j, k), sy = (size_t)g.nx, sz = (size_t)g.nx * g.ny;
  const T ix = (T)g.ihx2, iy = (T)g.ihy2, iz = (T)g.ihz2;
  const bool top = k == g.nz - 1, he = m < H - 1, hn = j < g.ny - 1;
  const T* wtp = top ? co.tp + (size_t)j * g.nx + 2 * m : co.wz + c + sz;
  const size_t cn = hn ? c + sy : c;
  T xw[3] = {co.wx[c], co.wx[c + 1], co.wx[he ? c + 2 : c + 1]};
  T ys[2] = {co.wy[c], co.wy[c + 1]}, yn[2] = {co.wy[cn], co.wy[cn + 1]};
  T zb[2] = {co.wz[c], co.wz[c + 1]}, zt[2] = {wtp[0], wtp[1]};
  const int par = (j + k) & 1;  // e_0
  q.dx = par ? 1 : -1;
  q.wi = xw[1] * ix;
  const T fb = k == 0 ? T(2) : T(1), ft = top ? T(2) : T(1);
#pragma unroll
  for (int cc = 0; cc < 2; ++cc) {
    const bool e = par != cc;  // cell 2m + 1
    q.wo[cc] = e ? (he ? xw[2] * ix : T(0)) : (m > 0 ? xw[0] * ix : T(0));
    q.ws[cc] = j > 0 ? (e ? ys[1] : ys[0]) * iy : T(0);
    q.wn[cc] = hn ? (e ? yn[1] : yn[0]) * iy : T(0);
    q.wb[cc] = fb * ((e ? zb[1] : zb[0]) * iz);
    q.wt[cc] = ft * ((e ? zt[1] : zt[0]) * iz);
    q.rd[cc] = recip(q.wi + q.wo[cc] + q.ws[cc] + q.wn[cc] + q.wb[cc] + q.wt[cc]);
  }
}

template <typename T>
__device__ __forceinline__ void bottom_setup(BottomPair<T>& q, const FaceCoef<T>& co, const Geom& g, int xoff, int p) {
  const BottomAt at(p, g.nx >> 1, g.ny);
  pair_weights(q, co, g, at.m, at.j, at.k);
  q.at = xoff + p;
  q.pk = bottom_parent(g, p);
  q.b[0] = q.b[1] = T(0);
}

// Neighbour values of the pair's colour-C cell (i: the pair's other cell, o:
// the one outside the pair).
template <typename T>
struct BottomNbrs {
  T i, o, s, n, b, t;
};

template <int C, typename T, int N>
__device__ __forceinline__ BottomNbrs<T> bottom_nbrs(const BottomPair<T>& q, const T (&lx)[2][N], int sy, int sz) {
  // (opaque: the neighbours' addresses are recomputed in each phase rather
  // than kept in registers)
  int at = q.at;
  asm volatile("" : "+v"(at));
  const T* p = lx[1 - C] + at;
  return BottomNbrs<T>{p[0], p[C ? -q.dx : q.dx], p[-sy], p[sy], p[-sz], p[sz]};
}

template <int C, typename T, int N>
__device__ __forceinline__ void bottom_update(const BottomPair<T>& q, const BottomNbrs<T>& v, T (&lx)[2][N]) {
  const T off = q.wi * v.i + q.wo[C] * v.o + q.ws[C] * v.s + q.wn[C] * v.n + q.wb[C] * v.b + q.wt[C] * v.t;
  lx[C][q.at] = (q.b[C] + off) * q.rd[C];
}

template <int C, typename T>
__device__ __forceinline__ T bottom_residual(const BottomPair<T>& q, const BottomNbrs<T>& v, T x) {
  return q.b[C] - (q.wi * (x - v.i) + q.wo[C] * (x - v.o) + q.ws[C] * (x - v.s) + q.wn[C] * (x - v.n) +
                   q.wb[C] * (x - v.b) + q.wt[C] * (x - v.t));
}

// Interpolated coarse value (cell-centred trilinear; mirrored ghosts on the
// sides, negated ones through the plates) at cell 2m + e of the pair whose
// parent is pk; at(natural index, colour): the coarse value.
template <typename T, typename F>
__device__ __forceinline__ T bottom_interp(F&& at, int pk, const Geom& gc, bool e) {
  asm volatile("" : "+v"(pk));  // (opaque: unpacked in each call, not kept unpacked)
  const int nat = pk & 511, dJ = ((pk >> 9) & 3) - 1, dK = ((pk >> 11) & 3) - 1, col = (pk >> 15) & 1;
  const int dI = e ? (pk >> 14) & 1 : -((pk >> 13) & 1);
  const int sJ = dJ * gc.nx, sK = dK * (gc.nx * gc.ny);
  T c[4], s[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int i = nat + (u & 1 ? sJ : 0) + (u & 2 ? sK : 0);
    const int cu = col ^ (u & 1 ? dJ & 1 : 0) ^ (u & 2 ? dK & 1 : 0);
    c[u] = at(i, cu);
    s[u] = at(i + dI, cu ^ (dI & 1));
  }
  const T q3 = T(0.75), q1 = T(0.25), sk = dK == 0 ? T(-1) : T(1);
  const T p0 = q3 * (q3 * c[0] + q1 * s[0]) + q1 * (q3 * c[1] + q1 * s[1]);
  const T p1 = q3 * (q3 * c[2] + q1 * s[2]) + q1 * (q3 * c[3] + q1 * s[3]);
  return q3 * p0 + q1 * sk * p1;
}

// FMG false: one V-cycle from zero for the right side b0.  FMG true: the
// full multigrid cycle over these levels: b0 restricted (mean of 8) to every
// level, the coarsest solved, then on each finer level one V-cycle from the
// interpolated coarser solution.  The result of the first bottom level goes
// to x0.  (Two instantiations, so that each inlines the V-cycle once.)
template <typename T, bool FMG>
__global__ __launch_bounds__(BottomShape<T>::threads) void k_vcycle_bottom(const BottomArgs<T> A) {
  constexpr int NT = BottomShape<T>::threads, NP0 = BottomShape<T>::pairs;
  __shared__ T lx[2][BOTTOM_LDS_X];
  __shared__ T part[2048];  // a pair's sum of residuals (or right sides) of the level being restricted
  __shared__ T lbc[512], lxc[512];  // right side and solution of the coarsest level
  __shared__ T linv[BottomShape<T>::inv_lds * BottomShape<T>::inv_lds];
  const int t = threadIdx.x, L = A.nlev - 1;
  const int nu_pre = A.nu_pre, nu_post = A.nu_post;
  const Geom gL = A.g[L];
  const int nc = geom_cells(gL);
  // owners: the first level's pairs t, t + NT, ...; one pair of the second or
  // third level
  const Geom g0 = A.g[0];
  const int np0 = geom_cells(g0) >> 1;
  const int np1 = L > 1 ? geom_cells(A.g[1]) >> 1 : 0, np2 = L > 2 ? geom_cells(A.g[2]) >> 1 : 0;
  const int lev = t < np1 ? 1 : (t < np1 + np2 ? 2 : -1);
  const int p1 = lev == 2 ? t - np1 : t;
  BottomPair<T> q0[NP0], q1;
#pragma unroll
  for (int u = 0; u < NP0; ++u) {
    const int p = t + u * NT;
    bottom_setup(q0[u], A.co[0], g0, A.xoff[0], p < np0 ? p : 0);
    if (p < np0) {
      const T b0 = A.b0[2 * p], b1 = A.b0[2 * p + 1];
      q0[u].b[0] = q0[u].dx > 0 ? b1 : b0;
      q0[u].b[1] = q0[u].dx > 0 ? b0 : b1;
    }
    if (u & 1) __builtin_amdgcn_sched_barrier(0);  // the loads of two pairs at a time: registers
  }
  if (lev > 0) bottom_setup(q1, A.co[lev], A.g[lev], A.xoff[lev], p1);
  for (int c = t; c < BOTTOM_LDS_X; c += NT) lx[0][c] = lx[1][c] = T(0);
  if (nc <= BottomShape<T>::inv_lds)
    for (int c = t; c < nc * nc; c += NT) linv[c] = A.Ainv[c];
  __syncthreads();

  // fn(pair, pair number) over this thread's pairs of level l
  auto each = [&](int l, auto&& fn) {
    if (l == 0) {
#pragma unroll
      for (int u = 0; u < NP0; ++u) {
        if (t + u * NT < np0) fn(q0[u], t + u * NT);
        __builtin_amdgcn_sched_barrier(0);  // one pair at a time: registers
      }
    } else if (lev == l) {
      fn(q1, p1);
    }
  };
  // half-sweep of colour C: every pair's neighbour values are read before the
  // first is stored
  auto half = [&](int l, auto cc) {
    constexpr int C = decltype(cc)::value;
    const int sy = A.g[l].nx >> 1, sz = sy * A.g[l].ny;
    if (l == 0) {
      BottomNbrs<T> v[NP0];
#pragma unroll
      for (int u = 0; u < NP0; ++u)
        if (t + u * NT < np0) v[u] = bottom_nbrs<C>(q0[u], lx, sy, sz);
#pragma unroll
      for (int u = 0; u < NP0; ++u)
        if (t + u * NT < np0) bottom_update<C>(q0[u], v[u], lx);
    } else if (lev == l) {
      bottom_update<C>(q1, bottom_nbrs<C>(q1, lx, sy, sz), lx);
    }
    lds_barrier();
  };
  constexpr std::integral_constant<int, 0> RED{};
  constexpr std::integral_constant<int, 1> BLACK{};
  // part of level l's pairs -> right side of level l + 1 (mean of 8)
  auto gather = [&](int l) {
    const Geom g = A.g[l + 1];
    const int fy = A.g[l].ny;
    auto mean = [&](int I, int J, int K) {
      const T* r = part + ((2 * K) * fy + 2 * J) * g.nx + I;
      return (r[0] + r[g.nx] + (r[fy * g.nx] + r[(fy + 1) * g.nx])) * T(0.125);
    };
    if (l + 1 == L) {
      if (t < nc) {
        const BottomAt c(t, gL.nx, gL.ny);
        lbc[t] = mean(c.m, c.j, c.k);
      }
    } else if (lev == l + 1) {
      const BottomAt c(p1, g.nx >> 1, g.ny);
      const T b0 = mean(2 * c.m, c.j, c.k), b1 = mean(2 * c.m + 1, c.j, c.k);
      q1.b[0] = q1.dx > 0 ? b1 : b0;
      q1.b[1] = q1.dx > 0 ? b0 : b1;
    }
    lds_barrier();
  };
  auto coarsest = [&]() {
    T* x = lxc;
    if (nc <= BottomShape<T>::inv_lds) {
      // four lanes per row, each every fourth column
      const int r = t >> 2;
      if (r < nc) {
        T acc = T(0);
        for (int c = t & 3; c < nc; c += 4) acc += linv[c * nc + r] * lbc[c];
        acc += __shfl_xor(acc, 1, 64);
        acc += __shfl_xor(acc, 2, 64);
        if (!(t & 3)) x[r] = acc;
      }
    } else {
      // eight rows of the inverse per wave at a time, the lanes across the row
      const int lane = t & 63, wave = t >> 6;
      for (int r0 = 8 * wave; r0 < nc; r0 += 8 * (NT / 64)) {
        T acc[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc[u] = T(0);
        for (int c = lane; c < nc; c += 64) {
          const T bv = lbc[c];
#pragma unroll
          for (int u = 0; u < 8; ++u) acc[u] += A.Ainv[(size_t)min(r0 + u, nc - 1) * nc + c] * bv;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
#pragma unroll
          for (int off = 32; off > 0; off >>= 1) acc[u] += __shfl_down(acc[u], off, 64);
          if (lane == 0 && r0 + u < nc) x[r0 + u] = acc[u];
        }
      }
    }
    lds_barrier();
  };
  // x += P x_{l+1}, or x = P x_{l+1} when set; of the colours in cmask (1
  // red, 2 black): the colour that the next half-sweep overwrites without
  // reading it is left out
  auto prolong = [&](int l, bool set, int cmask) {
    const Geom gc = A.g[l + 1];
    const int xoff = l + 1 < L ? A.xoff[l + 1] : 0;
    each(l, [&](BottomPair<T>& q, int) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        if (!((cmask >> c) & 1)) continue;
        const bool e = (q.dx > 0) != (c == 1);
        const T v = l + 1 == L ? bottom_interp<T>([&](int i, int) { return lxc[i]; }, q.pk, gc, e)
                               : bottom_interp<T>([&](int i, int col) { return lx[col][xoff + (i >> 1)]; }, q.pk, gc, e);
        lx[c][q.at] = set ? v : lx[c][q.at] + v;
      }
    });
    lds_barrier();
  };
  // V-cycle on the levels l0 .. L; from x = 0, or from the guess in x of
  // level l0 when from_x (the coarser levels start from 0 either way)
  auto cycle = [&](int l0, bool from_x) {
    for (int l = l0; l < L; ++l) {
      const bool guess = from_x && l == l0;
      if (!guess) {
        each(l, [&](BottomPair<T>& q, int) {
          // red from x = 0 (black stays 0)
          lx[0][q.at] = nu_pre > 0 ? q.b[0] * q.rd[0] : T(0);
          lx[1][q.at] = T(0);
        });
        lds_barrier();
      }
      for (int it = 0; it < nu_pre; ++it) {
        if (it > 0 || guess) half(l, RED);
        half(l, BLACK);
      }
      const int sy = A.g[l].nx >> 1, sz = sy * A.g[l].ny;
      each(l, [&](BottomPair<T>& q, int p) {
        const BottomNbrs<T> v0 = bottom_nbrs<0>(q, lx, sy, sz), v1 = bottom_nbrs<1>(q, lx, sy, sz);
        part[p] = bottom_residual<0>(q, v0, v1.i) + bottom_residual<1>(q, v1, v0.i);
      });
      lds_barrier();
      gather(l);
    }
    coarsest();
    for (int l = L - 1; l >= l0; --l) {
      prolong(l, false, nu_post > 0 ? 1 : 3);
      for (int it = 0; it < nu_post; ++it) {
        half(l, BLACK);
        half(l, RED);
      }
    }
  };

  if (!FMG) {
    cycle(0, false);
  } else {
    for (int l = 0; l < L; ++l) {  // right sides of every level
      each(l, [&](BottomPair<T>& q, int p) { part[p] = q.b[0] + q.b[1]; });
      lds_barrier();
      gather(l);
    }
    coarsest();
    for (int l = L - 1; l >= 0; --l) {
      prolong(l, true, nu_pre > 0 ? 2 : 3);
      cycle(l, true);
    }
  }
#pragma unroll
  for (int u = 0; u < NP0; ++u) {
    const int p = t + u * NT;
    if (p < np0) {
      const T v0 = lx[0][q0[u].at], v1 = lx[1][q0[u].at];
      A.x0[2 * p] = q0[u].dx > 0 ? v1 : v0;
      A.x0[2 * p + 1] = q0[u].dx > 0 ? v0 : v1;
    }
  }
}

}  // namespace gmg
