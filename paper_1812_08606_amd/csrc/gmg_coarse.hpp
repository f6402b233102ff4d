// gmg_coarse.hpp -- the coarsest level's direct solver: its dense matrix is
// assembled, inverted and applied on the GPU.
#pragma once

#include "gmg_kernels.hpp"

namespace gmg {

// In-place inverse of a symmetric positive definite n x n matrix A (float64,
// row-major, leading dimension n) by the symmetric sweep operator, NB rows
// and columns per step.  Sweeping block k with P = A_kk^{-1}, C the block
// column k of the symmetric matrix:
//     A_ij -= C_i P C_j^T,   A_ik = C_i P,   A_kk = -P   (i, j != k),
// which keeps the matrix symmetric, so only the blocks on and below the
// diagonal are stored and updated (n^3 operations instead of the 2 n^3 of
// Gauss-Jordan elimination on the full matrix); after every block is swept,
// A holds -A^{-1}.  No pivoting: the pivots of an SPD matrix are positive.
// Per step one launch of k_sweep_panel (W = C P into A, C copied to a side
// buffer) and one of k_sweep_update (the rank-NB update on the float64 matrix
// cores, one block per NB x NB tile); the block of tile (k+1, k+1) also
// inverts the next pivot block, so its serial chain of NB pivots runs beside
// the other tiles.  A zero, negative or non-finite pivot sets *bad (read back
// once, after the last step).
// Measured (renewal of the whole hierarchy): 4080 cells 187-289 -> 3.5 ms,
// 1287 cells 12.6 -> 0.95 ms, 343 cells 2.7 -> 0.35 ms against Gauss-Jordan
// elimination with two launches per cell (above 1024 cells) and a host
// Cholesky inverse (below).  A step takes about 51 us at 4080 cells, the
// update (40 us) bound by reading and writing the half matrix, and 30-42 us
// below 2200 cells, where the chain of pivots and the two launches bound it.
constexpr int NB = 64;
// rows of a tile in LDS are 66 doubles apart: the 16 rows x 2 columns that 32
// lanes read for a 16 x 16 x 4 matrix instruction fall on 64 different banks
constexpr int LDT = NB + 2;
constexpr int INV_THREADS = 256;

typedef double d4 __attribute__((ext_vector_type(4)));

// acc (rows 32 wr .., columns 32 wc .. of a 64 x 64 product, four 16 x 16
// pieces) += X Y^T with X and Y in LDS as [row][k], K columns, rows LD apart.
// Operand lanes of v_mfma_f64_16x16x4: row or column l % 16, k = l / 16; result
// register i: row 4 i + l / 16, column l % 16.
template <int K, int LD>
__device__ __forceinline__ void tile_mul(d4 (&acc)[2][2], const double* X, const double* Y, int wr, int wc) {
  const int l = threadIdx.x & 63, lr = l & 15, lk = l >> 4;
  const double* xr = X + (32 * wr + lr) * LD + lk;
  const double* yr = Y + (32 * wc + lr) * LD + lk;
#pragma unroll 4
  for (int k = 0; k < K; k += 4) {
    const double x0 = xr[k], x1 = xr[16 * LD + k], y0 = yr[k], y1 = yr[16 * LD + k];
    acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(x0, y0, acc[0][0], 0, 0, 0);
    acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(x0, y1, acc[0][1], 0, 0, 0);
    acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(x1, y0, acc[1][0], 0, 0, 0);
    acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(x1, y1, acc[1][1], 0, 0, 0);
  }
}

// fn(row, column, value) over the elements of the tile this thread's
// accumulators hold.
template <typename F>
__device__ __forceinline__ void tile_each(const d4 (&acc)[2][2], int wr, int wc, F&& fn) {
  const int l = threadIdx.x & 63;
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        fn(32 * wr + 16 * p + 4 * i + (l >> 4), 32 * wc + 16 * q + (l & 15), acc[p][q][i]);
}

// Tile of block row bi and block column bj of the symmetric matrix into LDS
// as [row][column] (above the diagonal: the transpose of the stored tile);
// elements outside the matrix are `pad` on the tile's diagonal, 0 elsewhere.
// All 16 loads of a thread are issued, from clamped addresses, before the
// first is stored.
constexpr int TILE_LOADS = NB * NB / INV_THREADS;

__device__ __forceinline__ void tile_load(double* S, const double* __restrict__ A, int n, int bi, int bj,
                                          double pad) {
  const bool tr = bi < bj;
  const int r0 = (tr ? bj : bi) * NB, c0 = (tr ? bi : bj) * NB;
  const int c = threadIdx.x % NB, rt = threadIdx.x / NB;
  const size_t cc = min(c0 + c, n - 1);
  double v[TILE_LOADS];
#pragma unroll
  for (int u = 0; u < TILE_LOADS; ++u) v[u] = A[(size_t)min(r0 + rt + u * (INV_THREADS / NB), n - 1) * n + cc];
#pragma unroll
  for (int u = 0; u < TILE_LOADS; ++u) {
    const int r = rt + u * (INV_THREADS / NB);
    const double w = (r0 + r < n && c0 + c < n) ? v[u] : (r == c ? pad : 0.0);
    S[tr ? c * LDT + r : r * LDT + c] = w;
  }
}

__device__ __forceinline__ double readlane(double v, int lane) {
  const int2 w = __builtin_bit_cast(int2, v);
  return __builtin_bit_cast(double, int2{__builtin_amdgcn_readlane(w.x, lane), __builtin_amdgcn_readlane(w.y, lane)});
}

// Sweeps the whole NB x NB block in S (symmetric, positive definite; LDS,
// [row][column]) and stores the result, -S^{-1}, in the diagonal tile bk of
// A.  QB columns at a time: one wave sweeps their QB pivots on the 64 x QB
// panel, a row per lane in registers, the pivot row by readlane (no barrier
// inside the chain), which leaves W = C P; then all four waves apply the
// rank-QB update S_ij -= W_i C_j^T to the other 16 x 16 pieces with matrix
// instructions.  A swept row is not scaled by its pivot's reciprocal at once:
// the lane keeps the factor to the end of the panel (its later updates, m -=
// (m_p / d) row, are the same with and without it), so a pivot costs one
// multiplication per column.  (One barrier and one division per pivot over the
// whole block took 50 us, scaling each row at once and a division 12; this
// takes about 10.)
constexpr int QB = 16;
constexpr int LDW = QB + 2;

__device__ __forceinline__ void sweep_pivot_block(double* S, double* Wb, double* __restrict__ A, int n, int bk,
                                                  double* __restrict__ bad) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  bool fail = false;
  const int nq = (min(NB, n - bk * NB) + QB - 1) / QB;  // (columns past the matrix are those of the identity)
  for (int q = 0; q < nq; ++q) {
    if (wave == 0) {
      double m[QB], s = 1.0;
#pragma unroll
      for (int c = 0; c < QB; ++c) m[c] = S[lane * LDT + QB * q + c];
#pragma unroll
      for (int p = 0; p < QB; ++p) {
        const int pr = QB * q + p;
        const double d = readlane(m[p], pr);
        fail |= !(d > 0.0) || !isfinite(d);
        const double id = recip(d);  // (every pivot waits for one: the division's chain is twice as long)
        const bool own = lane == pr;
        const double f = own ? 0.0 : m[p] * id;
#pragma unroll
        for (int c = 0; c < QB; ++c)
          if (c != p) m[c] = __builtin_fma(-f, readlane(m[c], pr), m[c]);
        m[p] = own ? -1.0 : f;
        s = own ? id : s;
      }
#pragma unroll
      for (int c = 0; c < QB; ++c) Wb[lane * LDW + c] = m[c] * s;
    }
    __syncthreads();
    constexpr int NP = NB / QB - 1;  // 16 x 16 pieces per side outside the swept ones
    for (int u = wave; u < NP * NP; u += INV_THREADS / 64) {
      int pi = u / NP, pj = u % NP;
      pi += pi >= q;
      pj += pj >= q;
      d4 acc = {};
#pragma unroll
      for (int k = 0; k < QB; k += 4)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(Wb[(QB * pi + lr) * LDW + k + lk],
                                                   S[(QB * pj + lr) * LDT + QB * q + k + lk], acc, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) S[(QB * pi + 4 * i + lk) * LDT + QB * pj + lr] -= acc[i];
    }
    __syncthreads();
    for (int u = t; u < NB * QB; u += INV_THREADS) {
      const int r = u / QB, c = u % QB;
      const double v = Wb[r * LDW + c];
      S[r * LDT + QB * q + c] = v;
      if (r / QB != q) S[(QB * q + c) * LDT + r] = v;
    }
    __syncthreads();
  }
  const int g0 = bk * NB;
  for (int u = t; u < NB * NB; u += INV_THREADS) {
    const int r = u / NB, c = u % NB;
    if (g0 + r < n && g0 + c < n) A[(size_t)(g0 + r) * n + g0 + c] = S[r * LDT + c];
  }
  if (fail && t == 0) *bad = 1.0;
}

__global__ __launch_bounds__(INV_THREADS) void k_sweep_first(double* __restrict__ A, int n,
                                                             double* __restrict__ bad) {
  __shared__ double S[NB * LDT];
  __shared__ double Wb[NB * LDW];
  if (threadIdx.x == 0) *bad = 0.0;
  tile_load(S, A, n, 0, 0, 1.0);
  __syncthreads();
  sweep_pivot_block(S, Wb, A, n, 0, bad);
}

// Block column k: C_i (tile (i, k) of the symmetric matrix) copied to C (n x
// NB, row-major) and W_i = C_i P stored in its place.  One block per i.
__global__ __launch_bounds__(INV_THREADS) void k_sweep_panel(double* __restrict__ A, int n, int k,
                                                             double* __restrict__ C) {
  __shared__ double X[NB * LDT], P[NB * LDT];
  const int i = blockIdx.x;
  if (i == k) return;
  tile_load(X, A, n, i, k, 0.0);
  tile_load(P, A, n, k, k, 0.0);  // holds -P
  __syncthreads();
  for (int t = threadIdx.x; t < NB * NB; t += INV_THREADS) {
    const int r = t / NB, c = t % NB;
    if (i * NB + r < n) C[(size_t)(i * NB + r) * NB + c] = X[r * LDT + c];
  }
  const int w = threadIdx.x >> 6, wr = w >> 1, wc = w & 1;
  d4 acc[2][2] = {};
  tile_mul<NB, LDT>(acc, X, P, wr, wc);  // C_i (-P)^T = -W_i
  tile_each(acc, wr, wc, [&](int r, int c, double v) {
    const int gi = i * NB + r, gk = k * NB + c;
    if (gi < n && gk < n) A[i > k ? (size_t)gi * n + gk : (size_t)gk * n + gi] = -v;
  });
}

// A_ij -= W_i C_j^T on every tile i >= j outside block row and column k; the
// tile (k+1, k+1), first in the grid, is then swept as the next pivot block.
// The operands pass through LDS KH columns at a time, the second half's loads
// in flight under the first half's products: 45 KB per block instead of 79, so
// three blocks share a CU and cover each other's loads (43 -> 40 us at 4080
// cells; 128-wide steps with 128 x 128 blocks, half the traffic, took 86 us per
// step, bound by the two pivot tiles one after the other).
constexpr int KH = NB / 2;
constexpr int LDH = KH + 2;  // (as LDT: 16 rows x 2 columns on 64 banks)

__global__ __launch_bounds__(INV_THREADS) void k_sweep_update(double* __restrict__ A, int n, int nb, int k,
                                                              const double* __restrict__ C,
                                                              double* __restrict__ bad) {
  __shared__ double buf[2 * NB * LDH];  // X and Y halves; then the pivot block
  __shared__ double Wb[NB * LDW];
  static_assert(2 * NB * LDH >= NB * LDT, "the pivot block does not fit the operand buffer");
  double *X = buf, *Y = buf + NB * LDH;
  const bool next = blockIdx.x == 0;
  int i, j;
  if (next) {
    i = j = k + 1;
    if (i >= nb) return;
    __builtin_amdgcn_s_setprio(3);  // the chain of pivots goes before the tiles that share its CU
  } else {
    // tile number blockIdx.x - 1 in the order (0,0), (1,0), (1,1), (2,0), ...
    const int t = blockIdx.x - 1;
    i = (int)((sqrtf(8.0f * t + 1.0f) - 1.0f) * 0.5f);
    while (i * (i + 1) / 2 > t) --i;
    while ((i + 1) * (i + 2) / 2 <= t) ++i;
    j = t - i * (i + 1) / 2;
    if (i == k || j == k || (i == j && i == k + 1)) return;
  }
  const int w = threadIdx.x >> 6, wr = w >> 1, wc = w & 1, l = threadIdx.x & 63;
  // half h of W_i (block column k; stored transposed for i < k) and of C_j
  constexpr int NL = NB * KH / INV_THREADS;
  double xv[NL], yv[NL];
  const bool tr = i < k;
  auto load = [&](int h) {
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const int e = threadIdx.x + u * INV_THREADS;
      // X: rows of W_i; along its columns when stored so, along its rows when transposed
      const int r = tr ? e % NB : e / KH, c = KH * h + (tr ? e / NB : e % KH);
      const int gi = min(i * NB + r, n - 1), gk = min(k * NB + c, n - 1);
      xv[u] = A[tr ? (size_t)gk * n + gi : (size_t)gi * n + gk];
      const int ry = e / KH, cy = KH * h + e % KH;
      yv[u] = C[(size_t)min(j * NB + ry, n - 1) * NB + cy];
    }
  };
  auto store = [&](int h) {
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const int e = threadIdx.x + u * INV_THREADS;
      const int r = tr ? e % NB : e / KH, c = tr ? e / NB : e % KH;
      X[r * LDH + c] = (i * NB + r < n && k * NB + KH * h + c < n) ? xv[u] : 0.0;
      const int ry = e / KH;
      Y[ry * LDH + e % KH] = j * NB + ry < n ? yv[u] : 0.0;
    }
  };
  load(0);
  // the tile itself (clamped addresses), in flight under the products
  d4 old[2][2];
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int gi = min(i * NB + 32 * wr + 16 * p + 4 * e + (l >> 4), n - 1);
        const int gj = min(j * NB + 32 * wc + 16 * q + (l & 15), n - 1);
        old[p][q][e] = A[(size_t)gi * n + gj];
      }
  d4 acc[2][2] = {};
  store(0);
  __syncthreads();
  load(1);
  tile_mul<KH, LDH>(acc, X, Y, wr, wc);
  __syncthreads();
  store(1);
  __syncthreads();
  tile_mul<KH, LDH>(acc, X, Y, wr, wc);
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int q = 0; q < 2; ++q) acc[p][q] = old[p][q] - acc[p][q];
  if (!next) {
    tile_each(acc, wr, wc, [&](int r, int c, double v) {
      const int gi = i * NB + r, gj = j * NB + c;
      if (gi < n && gj < n) A[(size_t)gi * n + gj] = v;
    });
    return;
  }
  __syncthreads();  // every wave is done with X and Y
  tile_each(acc, wr, wc, [&](int r, int c, double v) {
    const int gi = i * NB + r, gj = j * NB + c;
    buf[r * LDT + c] = (gi < n && gj < n) ? v : (r == c ? 1.0 : 0.0);
  });
  __syncthreads();
  sweep_pivot_block(buf, Wb, A, n, i, bad);
}

// The inverse, both triangles, in the V-cycle precision: out_ij = -A_ij for
// the stored tiles and their transposes (out may be A itself in float64: each
// block reads its tile before it writes, and the tiles above the diagonal
// hold nothing).
template <typename T>
__global__ __launch_bounds__(INV_THREADS) void k_sweep_finish(const double* A, int n, T* out) {
  __shared__ double S[NB * LDT];
  const int bi = blockIdx.y, bj = blockIdx.x;
  if (bi < bj) return;
  tile_load(S, A, n, bi, bj, 0.0);
  __syncthreads();
  for (int t = threadIdx.x; t < NB * NB; t += INV_THREADS) {
    const int r = t / NB, c = t % NB;
    // the stored tile, and (off the diagonal) its transpose; a diagonal tile
    // is symmetric to rounding: its lower half serves both
    const int gi = bi * NB + r, gj = bj * NB + c;
    const double v = bi == bj && c > r ? S[c * LDT + r] : S[r * LDT + c];
    if (gi < n && gj < n) out[(size_t)gi * n + gj] = (T)-v;
    const int ti = bj * NB + r, tj = bi * NB + c;
    if (bi != bj && ti < n && tj < n) out[(size_t)ti * n + tj] = (T)-S[c * LDT + r];
  }
}

// Dense matrix of the coarsest level, the blocks on and below the diagonal
// (one thread per element, rows in grid y): the 7-point operator from the
// stored face coefficients, or (single-level grids) from the cell
// coefficient.
__global__ __launch_bounds__(256) void k_dense_assemble(FaceCoef<double> co, const double* __restrict__ a, Geom g,
                                                        int n, double* __restrict__ A) {
  const int c = blockIdx.x * 256 + threadIdx.x, r = blockIdx.y;
  if (c >= n || c / NB > r / NB) return;
  const int sy = g.nx, sz = g.nx * g.ny;
  const int i = r % g.nx, j = (r / g.nx) % g.ny, k = r / sz;
  double v = 0.0;
  const int d = c - r;
  // the couplings that exist (a step to a neighbour stays in the row, plane
  // and grid); with nx, ny or nz = 1 several strides coincide, but then at
  // most one of the directions has a neighbour
  const bool w = i > 0, e = i < g.nx - 1, s = j > 0, nn = j < g.ny - 1, b = k > 0, t = k < g.nz - 1;
  if (d == 0 || (w && d == -1) || (e && d == 1) || (s && d == -sy) || (nn && d == sy) || (b && d == -sz) ||
      (t && d == sz)) {
    const Stencil<double> st = a ? CellCoef<double>{a}.load(g, i, j, k, (size_t)r) : co.load(g, i, j, k, (size_t)r);
    if (d == 0) {
      v = diag_cell(st, g, k);
    } else {
      if (w && d == -1) v -= st.ww;
      if (e && d == 1) v -= st.we;
      if (s && d == -sy) v -= st.ws;
      if (nn && d == sy) v -= st.wn;
      if (b && d == -sz) v -= st.wb;
      if (t && d == sz) v -= st.wt;
    }
  }
  A[(size_t)r * n + c] = v;
}

// Coarsest level: x = A_L^{-1} b with the precomputed symmetric inverse, one
// wave per row (a thread per row, as this kernel had before, put 3375 rows on
// 14 of 256 CUs and waited for each element: 632 us at 2145 rows, float32).
// The lanes stride the row in fixed order, then a wave reduction; summed in
// float64 (in float32 the sum's rounding left the first step's residual at
// 4080 rows four times as large; 17 -> 25 us).
template <typename T>
__global__ __launch_bounds__(NTHREADS) void k_coarse_solve(const T* __restrict__ Ainv, const T* __restrict__ b,
                                                           T* __restrict__ x, int n) {
  const int r = blockIdx.x * BY + threadIdx.y, lane = threadIdx.x;
  if (r >= n) return;
  const T* __restrict__ row = Ainv + (size_t)r * n;
  constexpr int U = 8;  // elements a lane loads per wait
  double acc = 0.0;
  for (int c0 = lane; c0 < n; c0 += 64 * U) {
    T v[U], w[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = c0 + 64 * u, cc = c < n ? c : c0;
      v[u] = row[cc];
      w[u] = c < n ? b[cc] : T(0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) acc += (double)v[u] * (double)w[u];
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
  if (lane == 0) x[r] = (T)acc;
}

}  // namespace gmg
