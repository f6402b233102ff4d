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
// every smoothed level has one owner thread, which loads the pair's face
// weights and reciprocal diagonals (packed at each renewal) and right sides
// once, at the start, and keeps them in registers; a half-sweep is then six
// LDS reads, six multiply-adds and one LDS write.  The iterates lie in LDS, one
// array per colour (a half-sweep then reads and writes consecutive words: at
// 16^3 its time is LDS throughput), with a plane of zeros below and above each
// level: through a plate the mirrored ghost doubles the face coefficient and
// its neighbour value is the zero plane's, so plates need no case of their own,
// and a missing side face has weight 0.  (Recomputing index, weights and
// diagonal from face coefficients in LDS in each phase took 1.3 us per phase:
// 39.7 us per V-cycle and 72 us per full multigrid cycle of 16^3 and below,
// V(2,2), float32, against 12.3 and 19.8 now; float64 V-cycle 45, now 17.  Of the V-cycle's 27000 clocks 7000 are the
// launch's first loads and set-up, 1100 each half-sweep at 16^3, 3000 its
// interpolation, 350-700 each phase on the level below, which waits for LDS
// and the barrier.)
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

// A 4 x 4 x 4 level (over a coarsest 2 x 2 x 2) is not smoothed either: its
// V-cycle from zero and its full multigrid cycle are linear maps of its 64
// right-side values, found at each renewal by running them on the unit vectors
// (64 workgroups), and one matrix-vector product then takes the place of the
// 12 shortest phases, three times in a full multigrid cycle.  MAP_LD elements
// from column to column: the 64 (float64: 32) lanes that read 8 columns of a
// few rows fall on different LDS banks.  (Float32, 16^3 and below: V-cycle 15.6
// -> 14.0 us, full multigrid 28.3 -> 22.0; finding the maps takes 16 us of a
// renewal.)
constexpr int MAP_CELLS = 64;
template <typename T>
constexpr int MAP_LD = sizeof(T) == 4 ? 72 : 68;

template <typename T>
struct BottomArgs {
  Geom g[BOTTOM_MAX_LEVELS];
  const T* w;                    // packed pairs of every smoothed level
  int npairs;                    // their number
  int poff[BOTTOM_MAX_LEVELS];   // first pair of each level
  T* x0;
  const T* b0;        // null: the workgroups take the unit vectors, the c-th result c * MAP_LD beyond x0
  const T* Ainv;      // solves the last level: element (r, c) at c * ld + r
  const T* Afirst;    // full multigrid: the last level's first solution (Ainv unless that is a whole cycle's map)
  int ld;
  int nlev;  // levels handled, the last one solved by Ainv
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
// coarse row and plane (-1, 0, 1; 0 outside the grid), and whether the coarse
// cells m - 1 and m + 1 exist.  (Found once: the coordinates and clamps took
// most of the interpolation's instructions.)
__device__ __forceinline__ int bottom_parent(const Geom& g, int p) {
  const int NX = g.nx >> 1, NY = g.ny >> 1, NZ = g.nz >> 1;
  const BottomAt at(p, NX, g.ny);
  const int J = at.j >> 1, K = at.k >> 1;
  const int dJ = at.j & 1 ? (J < NY - 1 ? 1 : 0) : (J > 0 ? -1 : 0);
  const int dK = at.k & 1 ? (K < NZ - 1 ? 1 : 0) : (K > 0 ? -1 : 0);
  return ((K * NY + J) * NX + at.m) | (dJ + 1) << 9 | (dK + 1) << 11 | (at.m > 0) << 13 | (at.m < NX - 1) << 14;
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

// Stored faces of the pair (m, j, k) of a level.
template <typename T>
struct PairFaces {
  T xw[3], ys[2], yn[2], zb[2], zt[2];
};

template <typename T>
__device__ __forceinline__ PairFaces<T> pair_faces(const FaceCoef<T>& co, const Geom& g, int m, int j, int k) {
  const size_t c = cidx(g, 2 * m, j, k), sy = (size_t)g.nx, sz = (size_t)g.nx * g.ny;
  const T* wtp = k == g.nz - 1 ? co.tp + (size_t)j * g.nx + 2 * m : co.wz + c + sz;
  const size_t cn = j < g.ny - 1 ? c + sy : c;
  return PairFaces<T>{{co.wx[c], co.wx[c + 1], co.wx[m < (g.nx >> 1) - 1 ? c + 2 : c + 1]},
                      {co.wy[c], co.wy[c + 1]},
                      {co.wy[cn], co.wy[cn + 1]},
                      {co.wz[c], co.wz[c + 1]},
                      {wtp[0], wtp[1]}};
}

// Weights and diagonals of the pair (m, j, k) from its stored faces.
template <typename T>
__device__ __forceinline__ void pair_weights(BottomPair<T>& q, const PairFaces<T>& f, const Geom& g, int m, int j,
                                             int k) {
  const T ix = (T)g.ihx2, iy = (T)g.ihy2, iz = (T)g.ihz2;
  const bool top = k == g.nz - 1, he = m < (g.nx >> 1) - 1, hn = j < g.ny - 1;
  const int par = (j + k) & 1;  // e_0
  q.dx = par ? 1 : -1;
  q.wi = f.xw[1] * ix;
  const T fb = k == 0 ? T(2) : T(1), ft = top ? T(2) : T(1);
#pragma unroll
  for (int cc = 0; cc < 2; ++cc) {
    const bool e = par != cc;  // cell 2m + 1
    q.wo[cc] = e ? (he ? f.xw[2] * ix : T(0)) : (m > 0 ? f.xw[0] * ix : T(0));
    q.ws[cc] = j > 0 ? (e ? f.ys[1] : f.ys[0]) * iy : T(0);
    q.wn[cc] = hn ? (e ? f.yn[1] : f.yn[0]) * iy : T(0);
    q.wb[cc] = fb * ((e ? f.zb[1] : f.zb[0]) * iz);
    q.wt[cc] = ft * ((e ? f.zt[1] : f.zt[0]) * iz);
    q.rd[cc] = recip(q.wi + q.wo[cc] + q.ws[cc] + q.wn[cc] + q.wb[cc] + q.wt[cc]);
  }
}

// The pairs of the smoothed bottom levels as the launches read them: weights,
// reciprocal diagonals and position (bottom_parent, and bit 16: dx > 0) in
// chunks of 16 bytes, chunk i of pair p at (i * npairs + p) * 16.  (Faces to
// weights and positions in every launch: V-cycle of 16^3 and below 14.0 us in
// float32, now 12.3; of 3840 cells and below in float64 17.0, now 14.4; packing
// takes 3 us of a renewal.)
template <typename T>
struct PackedPair {
  static constexpr int per = 16 / sizeof(T);
  static constexpr int chunks = (14 + per - 1) / per;  // 4 in float32, 7 in float64
  typedef T Chunk __attribute__((ext_vector_type(per)));
  Chunk c[chunks];
  __device__ __forceinline__ T get(int i) const { return c[i / per][i % per]; }
  __device__ __forceinline__ void set(int i, T v) { c[i / per][i % per] = v; }
  __device__ __forceinline__ void load(const T* w, int npairs, int p) {
#pragma unroll
    for (int i = 0; i < chunks; ++i) c[i] = reinterpret_cast<const Chunk*>(w)[i * npairs + p];
  }
};

template <typename T>
struct PackArgs {
  FaceCoef<T> co[BOTTOM_MAX_LEVELS];
  Geom g[BOTTOM_MAX_LEVELS];
  int poff[BOTTOM_MAX_LEVELS];
  int nlev, npairs;
  T* w;
};

// One thread per pair of the smoothed bottom levels.
template <typename T>
__global__ __launch_bounds__(256) void k_bottom_pack(const PackArgs<T> A) {
  const int p = blockIdx.x * 256 + threadIdx.x;
  if (p >= A.npairs) return;
  int l = 0;
  while (l + 1 < A.nlev && p >= A.poff[l + 1]) ++l;
  const Geom g = A.g[l];
  const int q = p - A.poff[l];
  const BottomAt at(q, g.nx >> 1, g.ny);
  BottomPair<T> b;
  pair_weights(b, pair_faces(A.co[l], g, at.m, at.j, at.k), g, at.m, at.j, at.k);
  PackedPair<T> r{};
  r.set(0, b.wi);
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    r.set(1 + c, b.wo[c]);
    r.set(3 + c, b.ws[c]);
    r.set(5 + c, b.wn[c]);
    r.set(7 + c, b.wb[c]);
    r.set(9 + c, b.wt[c]);
    r.set(11 + c, b.rd[c]);
  }
  r.set(13, (T)(bottom_parent(g, q) | (b.dx > 0) << 16));  // (below 2^17: exact in either type)
#pragma unroll
  for (int i = 0; i < PackedPair<T>::chunks; ++i)
    reinterpret_cast<typename PackedPair<T>::Chunk*>(A.w)[i * A.npairs + p] = r.c[i];
}

template <typename T>
__device__ __forceinline__ void bottom_setup(BottomPair<T>& q, const PackedPair<T>& r, int at) {
  q.wi = r.get(0);
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    q.wo[c] = r.get(1 + c);
    q.ws[c] = r.get(3 + c);
    q.wn[c] = r.get(5 + c);
    q.wb[c] = r.get(7 + c);
    q.wt[c] = r.get(9 + c);
    q.rd[c] = r.get(11 + c);
    q.b[c] = T(0);
  }
  const int info = (int)r.get(13);
  q.at = at;
  q.pk = info & 0xffff;
  q.dx = info >> 16 ? 1 : -1;
}

// n elements to LDS without registers in between, 16 bytes per lane (both
// pointers 16-byte aligned); complete after a wait for vmcnt and a barrier.
template <typename T>
__device__ __forceinline__ void copy_to_lds(T* dst, const T* src, int n, int nthreads) {
  const int wave = threadIdx.x & ~63, bytes = n * (int)sizeof(T);
  typedef const __attribute__((address_space(1))) void* gptr;
  typedef __attribute__((address_space(3))) void* lptr;
  char* d = reinterpret_cast<char*>(dst);
  const char* s = reinterpret_cast<const char*>(src);
  const int whole = bytes & ~15;
  for (int o = 16 * wave; o < whole; o += 16 * nthreads) {
    const int at = o + 16 * (int)(threadIdx.x & 63);
    if (at < whole) __builtin_amdgcn_global_load_lds((gptr)(s + at), (lptr)(d + o), 16, 0, 0);
  }
  for (int at = whole + (int)(threadIdx.x * sizeof(T)); at < bytes; at += nthreads * (int)sizeof(T))
    *reinterpret_cast<T*>(d + at) = *reinterpret_cast<const T*>(s + at);
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
// parent is pk; x: the coarse values in natural order.
template <typename T>
__device__ __forceinline__ T bottom_interp(const T* x, int pk, const Geom& gc, bool e) {
  asm volatile("" : "+v"(pk));  // (opaque: unpacked in each call, not kept unpacked)
  const int nat = pk & 511, dJ = ((pk >> 9) & 3) - 1, dK = ((pk >> 11) & 3) - 1;
  const int dI = e ? (pk >> 14) & 1 : -((pk >> 13) & 1);
  const int sJ = dJ * gc.nx, sK = dK * (gc.nx * gc.ny);
  T c[4], s[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const T* xi = x + nat + (u & 1 ? sJ : 0) + (u & 2 ? sK : 0);
    c[u] = xi[0];
    s[u] = xi[dI];
  }
  const T q3 = T(0.75), q1 = T(0.25), sk = dK == 0 ? T(-1) : T(1);
  const T p0 = q3 * (q3 * c[0] + q1 * s[0]) + q1 * (q3 * c[1] + q1 * s[1]);
  const T p1 = q3 * (q3 * c[2] + q1 * s[2]) + q1 * (q3 * c[3] + q1 * s[3]);
  return q3 * p0 + q1 * sk * p1;
}

// FMG false: one V-cycle from zero for the right side b0.  FMG true: the
// full multigrid cycle over these levels: b0 restricted (mean of 8) to every
// level, the coarsest solved, then on each finer level one V-cycle from the
// interpolated coarser solution; without b0 (the maps of a 4 x 4 x 4 level) the
// first MAP_CELLS workgroups run the V-cycle, the next ones the full multigrid
// cycle.  The result of the first bottom level goes to x0.  (Two
// instantiations, so that each inlines the V-cycle once.)
template <typename T, bool FMG>
__global__ __launch_bounds__(BottomShape<T>::threads) void k_vcycle_bottom(const BottomArgs<T> A) {
  constexpr int NT = BottomShape<T>::threads, NP0 = BottomShape<T>::pairs;
  __shared__ T lx[2][BOTTOM_LDS_X];
  __shared__ T part[2048];  // a pair's sum of residuals (or right sides) of the level being restricted
  __shared__ T lbc[512], lxc[512];  // right side (zeros beyond it) and solution of the coarsest level
  __shared__ __align__(16) T linv[BottomShape<T>::inv_lds * BottomShape<T>::inv_lds];
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
  // everything the launch reads is asked for before any of it is waited for
  const int ld = A.ld;
  const bool in_lds = nc <= BottomShape<T>::inv_lds, own_first = FMG && A.Afirst != A.Ainv;
  if (in_lds) copy_to_lds(linv, A.Ainv, nc * ld, NT);
  if (own_first) copy_to_lds(linv + nc * ld, A.Afirst, nc * ld, NT);
  PackedPair<T> f0[NP0], f1;
  T b0[NP0][2];
  const int unit = blockIdx.x % MAP_CELLS;
#pragma unroll
  for (int u = 0; u < NP0; ++u) {
    const int p = t + u * NT < np0 ? t + u * NT : 0;
    f0[u].load(A.w, A.npairs, A.poff[0] + p);
    b0[u][0] = A.b0 ? A.b0[2 * p] : T(2 * p == unit);
    b0[u][1] = A.b0 ? A.b0[2 * p + 1] : T(2 * p + 1 == unit);
  }
  // (chosen by value: indexed by lane, the arguments would be read from memory first)
  if (lev > 0) f1.load(A.w, A.npairs, (lev == 2 ? A.poff[2] : A.poff[1]) + p1);
  for (int c = t; c < BOTTOM_LDS_X; c += NT) lx[0][c] = lx[1][c] = T(0);
  if (t < 512) lbc[t] = T(0);
  BottomPair<T> q0[NP0], q1;
#pragma unroll
  for (int u = 0; u < NP0; ++u) {
    bottom_setup(q0[u], f0[u], A.xoff[0] + (t + u * NT < np0 ? t + u * NT : 0));
    q0[u].b[0] = q0[u].dx > 0 ? b0[u][1] : b0[u][0];
    q0[u].b[1] = q0[u].dx > 0 ? b0[u][0] : b0[u][1];
  }
  if (lev > 0) bottom_setup(q1, f1, (lev == 2 ? A.xoff[2] : A.xoff[1]) + p1);
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the copy to LDS
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
  // a level's solution in natural order, where the interpolation reads it
  auto natural = [&](const BottomPair<T>& q, int p) {
    const T v0 = lx[0][q.at], v1 = lx[1][q.at];
    lxc[2 * p] = q.dx > 0 ? v1 : v0;
    lxc[2 * p + 1] = q.dx > 0 ? v0 : v1;
  };
  // half-sweep of colour C (the last one of a level below the first: with its
  // solution in natural order): every pair's neighbour values are read before the
  // first is stored
  auto half = [&](int l, auto cc, bool last = false) {
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
      if (last) natural(q1, p1);
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
  auto coarsest = [&](const T* map) {
    T* x = lxc;
    if (in_lds) {
      // four or eight lanes per row, each every fourth or eighth column, U of
      // them per wait
      constexpr int U = 8;
      const int sh = 8 * nc <= NT ? 3 : 2, r = t >> sh, per = 1 << sh;
      if (r < nc) {
        T acc = T(0);
        for (int c0 = t & (per - 1); c0 < nc; c0 += per * U) {
          T a[U], b[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int c = c0 + u * per;
            a[u] = map[min(c, nc - 1) * ld + r];
            b[u] = lbc[c];
          }
#pragma unroll
          for (int u = 0; u < U; ++u) acc += a[u] * b[u];
        }
        acc += __shfl_xor(acc, 1, 64);
        acc += __shfl_xor(acc, 2, 64);
        if (sh == 3) acc += __shfl_xor(acc, 4, 64);
        if (!(t & (per - 1))) x[r] = acc;
      }
    } else {
      // A row per lane, the rows rounded up to whole waves, and the columns
      // dealt to the S groups of so many lanes that the workgroup holds (the
      // inverse is symmetric: consecutive rows read consecutive elements of a
      // column); U columns per wait.  One workgroup reads the whole inverse, so
      // the bytes a CU can have in flight bound it.  (Eight rows per wave with
      // the lanes across a row waited for eight loads at a time: V-cycle of 4158
      // cells and below, 462 in the coarsest, float64 80.6 -> 51.8 us, float32
      // 42.8 -> 32.5.)
      constexpr int U = 16;
      const int P = (nc + 63) & ~63, S = NT / P, h = (t >> 6) / (P >> 6), r = t - h * P;
      if (h < S) {
        const T* col = A.Ainv + min(r, nc - 1);
        T acc[4] = {T(0), T(0), T(0), T(0)};
        for (int c0 = h; c0 < nc; c0 += S * U) {
          T a[U];
#pragma unroll
          for (int u = 0; u < U; ++u) a[u] = col[(size_t)min(c0 + u * S, nc - 1) * ld];
#pragma unroll
          for (int u = 0; u < U; ++u) acc[u & 3] += c0 + u * S < nc ? a[u] * lbc[c0 + u * S] : T(0);
        }
        part[t] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
      }
      lds_barrier();
      if (t < nc) {
        T acc = T(0);
        for (int q = 0; q < S; ++q) acc += part[q * P + t];
        x[t] = acc;
      }
    }
    lds_barrier();
  };
  // x += P x_{l+1}, or x = P x_{l+1} when set; of the colours in cmask (1
  // red, 2 black): the colour that the next half-sweep overwrites without
  // reading it is left out
  auto prolong = [&](int l, bool set, int cmask) {
    const Geom gc = A.g[l + 1];
    each(l, [&](BottomPair<T>& q, int) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        if (!((cmask >> c) & 1)) continue;
        const bool e = (q.dx > 0) != (c == 1);
        const T v = bottom_interp(lxc, q.pk, gc, e);
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
    coarsest(linv);
    for (int l = L - 1; l >= l0; --l) {
      prolong(l, false, nu_post > 0 ? 1 : 3);
      for (int it = 0; it < nu_post; ++it) {
        half(l, BLACK);
        half(l, RED, l > 0 && it == nu_post - 1);
      }
      if (nu_post == 0 && l > 0) {
        each(l, [&](BottomPair<T>& q, int p) { natural(q, p); });
        lds_barrier();
      }
    }
  };

  if (!FMG) {
    cycle(0, false);
  } else {
    const bool full = A.b0 || blockIdx.x >= MAP_CELLS;
    if (full) {
      for (int l = 0; l < L; ++l) {  // right sides of every level
        each(l, [&](BottomPair<T>& q, int p) { part[p] = q.b[0] + q.b[1]; });
        lds_barrier();
        gather(l);
      }
      coarsest(own_first ? linv + nc * ld : linv);
    }
    for (int l = full ? L - 1 : 0; l >= 0; --l) {
      if (full) prolong(l, true, nu_pre > 0 ? 2 : 3);
      cycle(l, full);
    }
  }
#pragma unroll
  for (int u = 0; u < NP0; ++u) {
    const int p = t + u * NT;
    if (p < np0) {
      const T v0 = lx[0][q0[u].at], v1 = lx[1][q0[u].at];
      T* x0 = A.x0 + (size_t)blockIdx.x * MAP_LD<T>;
      x0[2 * p] = q0[u].dx > 0 ? v1 : v0;
      x0[2 * p + 1] = q0[u].dx > 0 ? v0 : v1;
    }
  }
}

}  // namespace gmg
