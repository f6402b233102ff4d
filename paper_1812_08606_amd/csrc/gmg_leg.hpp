// gmg_leg.hpp -- several half-sweeps of a small level in one launch, with the
// interpolation before them or the residual restriction after them.
#pragma once

#include "gmg_bottom.hpp"
#include "gmg_plan.hpp"

namespace gmg {

// On a level of 32^3 or 64^3 cells a half-sweep kernel takes about 4 us, of
// which the work is a fraction: the launch, one trip to memory and the drain
// set its time, and a visit of the level makes 12 to 14 such launches.  This
// kernel does a leg of the visit in one: a block owns a box of tx pairs x ty
// rows x tz planes, holds it with a halo in LDS (by colour) and the weights of
// its pairs in registers, as the bottom kernel does, and runs nh half-sweeps
// with LDS barriers between them.  The halo is recomputed rather than
// exchanged: half-sweep i (of 0 .. nh-1) updates the pairs within nh - 1 - i
// cells of the box (one more when the residual follows), so the halo is as
// deep as the half-sweeps are many.  Blocks read xin and write xout, another
// buffer.
//
// Measured against the per-sweep kernels, V(2,2): a visit of a 64^3 level in
// float32 is two launches of 10 us instead of 12 of 4 us, of a 32^3 level two
// of 6 to 9 us; 64^3 solve (both levels, full multigrid cycles) 1.29 -> 1.01
// ms, 128^3 time step 2.72 -> 2.33 ms, 256^3 gradient step 18.7 -> 16.5 ms.
// About 4 us of a launch are its start and the loads; then each half-sweep of
// 2048 pairs takes about 0.45 us, VALU and LDS bound.
//
// start: LEG_ZERO from x = 0; LEG_X from xin; LEG_ADD from xin + P xc;
// LEG_SET from P xc (xc the next level's iterate, P the trilinear
// prolongation).  Only the colour that the first half-sweep reads is loaded
// and interpolated.  bc: the mean over 8 children of the residual of the
// result, the next level's right side (null: none).
enum { LEG_ZERO = 0, LEG_X = 1, LEG_ADD = 2, LEG_SET = 3 };

template <typename T>
struct LegArgs {
  Geom g;
  FaceCoef<T> co;       // levels >= 1: stored faces, natural b and x
  const T* a;           // finest level: cell coefficient, colour-split B and x
  size_t hn;
  const T* xin;
  T* xout;
  const T* b;
  const double* u;      // finest level from x = 0: right side s u, s = *bscale (1 when null), stored into bout
  const double* bscale;
  T* bout;
  const T* xc;
  T* bc;
  int start, c1, nh;
  int tx, ty, tz;       // owned box: pairs, rows, planes
  int hx, hy;           // halo: pairs; rows and planes
};

// Weights and diagonals of the pair (m, j, k) of the finest level (cell
// coefficient, face = mean of the two cells; through a plate the cell's own
// coefficient, doubled by the mirrored ghost).
template <typename T>
__device__ __forceinline__ void pair_weights(BottomPair<T>& q, const T* __restrict__ a, const Geom& g, int m, int j,
                                             int k) {
  const int H = g.nx >> 1;
  const size_t c = cidx(g, 2 * m, j, k), sy = (size_t)g.nx, sz = (size_t)g.nx * g.ny;
  const T hx = (T)(0.5 * g.ihx2), hy = (T)(0.5 * g.ihy2), hz = (T)(0.5 * g.ihz2), pz = (T)(2.0 * g.ihz2);
  const bool hw = m > 0, he = m < H - 1, hs = j > 0, hn = j < g.ny - 1, bot = k == 0, top = k == g.nz - 1;
  const size_t cs = hs ? c - sy : c, cn = hn ? c + sy : c, cb = bot ? c : c - sz, ct = top ? c : c + sz;
  const T ac[2] = {a[c], a[c + 1]}, ao[2] = {a[hw ? c - 1 : c], a[he ? c + 2 : c + 1]};
  const T as[2] = {a[cs], a[cs + 1]}, an[2] = {a[cn], a[cn + 1]};
  const T ab[2] = {a[cb], a[cb + 1]}, at[2] = {a[ct], a[ct + 1]};
  const int par = (j + k) & 1;
  q.dx = par ? 1 : -1;
  q.wi = (ac[0] + ac[1]) * hx;
#pragma unroll
  for (int cc = 0; cc < 2; ++cc) {
    const bool e = par != cc;  // cell 2m + 1
    const T av = e ? ac[1] : ac[0];
    q.wo[cc] = (e ? he : hw) ? (av + (e ? ao[1] : ao[0])) * hx : T(0);
    q.ws[cc] = hs ? (av + (e ? as[1] : as[0])) * hy : T(0);
    q.wn[cc] = hn ? (av + (e ? an[1] : an[0])) * hy : T(0);
    q.wb[cc] = bot ? pz * av : (av + (e ? ab[1] : ab[0])) * hz;
    q.wt[cc] = top ? pz * av : (av + (e ? at[1] : at[0])) * hz;
    q.rd[cc] = recip(q.wi + q.wo[cc] + q.ws[cc] + q.wn[cc] + q.wb[cc] + q.wt[cc]);
  }
}

// P xc at cell 2m + e of row j, plane k (fine geometry g; xc natural).
template <typename T>
__device__ __forceinline__ T leg_interp(const T* __restrict__ xc, const Geom& g, int m, int j, int k, bool e) {
  const int NX = g.nx >> 1, NY = g.ny >> 1, NZ = g.nz >> 1;
  const int J = j >> 1, K = k >> 1;
  int J2 = J + (j & 1 ? 1 : -1), K2 = K + (k & 1 ? 1 : -1);
  if (J2 < 0 || J2 >= NY) J2 = J;
  T sk = T(1);
  if (K2 < 0 || K2 >= NZ) {
    K2 = K;
    sk = T(-1);
  }
  const int m2 = e ? min(m + 1, NX - 1) : max(m - 1, 0);
  T c[4], s[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const T* r = xc + ((size_t)(u & 2 ? K2 : K) * NY + (u & 1 ? J2 : J)) * NX;
    c[u] = r[m];
    s[u] = r[m2];
  }
  const T q3 = T(0.75), q1 = T(0.25);
  const T p0 = q3 * (q3 * c[0] + q1 * s[0]) + q1 * (q3 * c[1] + q1 * s[1]);
  const T p1 = q3 * (q3 * c[2] + q1 * s[2]) + q1 * (q3 * c[3] + q1 * s[3]);
  return q3 * p0 + q1 * sk * p1;
}

template <typename T, int PPT, bool FINE>
__global__ __launch_bounds__(LegShape<T>::threads) void k_leg(const LegArgs<T> A) {
  constexpr int NT = LegShape<T>::threads;
  __shared__ T lx[2][LegShape<T>::lds];
  __shared__ T part[LegShape<T>::own];
  const Tile tl = xcd_tile();
  const Geom g = A.g;
  const int t = threadIdx.x, H = g.nx >> 1;
  const int RX = A.tx + 2 * A.hx, RY = A.ty + 2 * A.hy, RZ = A.tz + 2 * A.hy;
  const int np = RX * RY * RZ;
  const int sy = RX, sz = RX * (RY + 2);
  const int M0 = tl.x * A.tx - A.hx, J0 = tl.y * A.ty - A.hy, K0 = tl.z * A.tz - A.hy;
  const int rad = A.nh - 1 + (A.bc ? 1 : 0);  // cells from the box that the first half-sweep updates
  const int co = 1 - A.c1;                    // the colour it reads
  for (int c = t; c < sz * (RZ + 2) + 2; c += NT) lx[0][c] = lx[1][c] = T(0);
  const double s = FINE && A.bscale ? *A.bscale : 1.0;
  BottomPair<T> q[PPT];
  T x[PPT];
  // q.pk: distance of the pair from the box in cells (steps through faces;
  // 255: outside the grid or not needed)
#pragma unroll
  for (int w = 0; w < PPT; ++w) {
    const int p = t + w * NT;
    const BottomAt at(p < np ? p : 0, RX, RY);
    const int m = M0 + at.m, j = J0 + at.j, k = K0 + at.k;
    const int dx = max(max(A.hx - at.m, at.m - (A.hx + A.tx - 1)), 0);
    const int dy = max(max(A.hy - at.j, at.j - (A.hy + A.ty - 1)), 0);
    const int dz = max(max(A.hy - at.k, at.k - (A.hy + A.tz - 1)), 0);
    const bool in = p < np && m >= 0 && m < H && j >= 0 && j < g.ny && k >= 0 && k < g.nz;
    const int dist = max(2 * dx - 1, 0) + dy + dz;
    q[w].pk = in && dist <= rad + 1 ? dist : 255;
    q[w].at = 1 + (at.k + 1) * sz + (at.j + 1) * sy + at.m;
    x[w] = T(0);
    if (q[w].pk <= rad) {
      const size_t c = cidx(g, 2 * m, j, k);
      const int par = (j + k) & 1;
      if constexpr (FINE) {
        pair_weights(q[w], A.a, g, m, j, k);
        if (A.u) {
          const double u0 = A.u[c], u1 = A.u[c + 1];
          const T b0 = (T)(u0 * s), b1 = (T)(u1 * s);
          q[w].b[0] = par ? b1 : b0;
          q[w].b[1] = par ? b0 : b1;
          if (dist == 0) {
            A.bout[c >> 1] = q[w].b[0];
            A.bout[A.hn + (c >> 1)] = q[w].b[1];
          }
        } else {
          q[w].b[0] = A.b[c >> 1];
          q[w].b[1] = A.b[A.hn + (c >> 1)];
        }
      } else {
        pair_weights(q[w], pair_faces(A.co, g, m, j, k), g, m, j, k);
        const T b0 = A.b[c], b1 = A.b[c + 1];
        q[w].b[0] = par ? b1 : b0;
        q[w].b[1] = par ? b0 : b1;
      }
    }
    if (A.start != LEG_ZERO && q[w].pk <= rad + 1) {
      const bool e = ((j + k) & 1) != co;  // the read colour's cell is 2m + 1
      const size_t c = cidx(g, 2 * m, j, k);
      if (A.start != LEG_SET) x[w] = FINE ? A.xin[(size_t)co * A.hn + (c >> 1)] : A.xin[c + e];
      if (A.start != LEG_X) x[w] += leg_interp(A.xc, g, m, j, k, e);
    }
    if (w & 1) __builtin_amdgcn_sched_barrier(0);  // the loads of two pairs at a time: registers
  }
  __syncthreads();
  if (A.start != LEG_ZERO) {
#pragma unroll
    for (int w = 0; w < PPT; ++w)
      if (q[w].pk <= rad + 1) lx[co][q[w].at] = x[w];
    lds_barrier();
  }
  auto half = [&](int r, auto cc) {
    constexpr int C = decltype(cc)::value;
    constexpr int G = PPT < 2 ? PPT : 2;  // pairs whose neighbours are read before the first is stored
#pragma unroll
    for (int w0 = 0; w0 < PPT; w0 += G) {
      BottomNbrs<T> v[G];
#pragma unroll
      for (int w = 0; w < G; ++w)
        if (w0 + w < PPT && q[w0 + w].pk <= r) v[w] = bottom_nbrs<C>(q[w0 + w], lx, sy, sz);
#pragma unroll
      for (int w = 0; w < G; ++w)
        if (w0 + w < PPT && q[w0 + w].pk <= r) bottom_update<C>(q[w0 + w], v[w], lx);
    }
    lds_barrier();
  };
  for (int i = 0; i < A.nh; ++i) {
    if ((A.c1 + i) & 1)
      half(rad - i, std::integral_constant<int, 1>{});
    else
      half(rad - i, std::integral_constant<int, 0>{});
  }
#pragma unroll
  for (int w = 0; w < PPT; ++w) {
    if (q[w].pk != 0) continue;
    const int p = t + w * NT;
    const BottomAt at(p, RX, RY);
    const T v0 = lx[0][q[w].at], v1 = lx[1][q[w].at];
    const size_t c = cidx(g, 2 * (M0 + at.m), J0 + at.j, K0 + at.k);
    if constexpr (FINE) {
      A.xout[c >> 1] = v0;
      A.xout[A.hn + (c >> 1)] = v1;
    } else {
      A.xout[c] = q[w].dx > 0 ? v1 : v0;
      A.xout[c + 1] = q[w].dx > 0 ? v0 : v1;
    }
    if (A.bc) {
      const BottomNbrs<T> n0 = bottom_nbrs<0>(q[w], lx, sy, sz), n1 = bottom_nbrs<1>(q[w], lx, sy, sz);
      part[((at.k - A.hy) * A.ty + (at.j - A.hy)) * A.tx + at.m - A.hx] =
          bottom_residual<0>(q[w], n0, v0) + bottom_residual<1>(q[w], n1, v1);
    }
  }
  if (A.bc) {
    lds_barrier();
    const int CY = A.ty >> 1, NY = g.ny >> 1, NZ = g.nz >> 1;
    for (int p = t; p < A.tx * CY * (A.tz >> 1); p += NT) {
      const BottomAt at(p, A.tx, CY);
      const int I = tl.x * A.tx + at.m, J = tl.y * CY + at.j, K = tl.z * (A.tz >> 1) + at.k;
      if (I >= H || J >= NY || K >= NZ) continue;
      const T* r = part + ((2 * at.k) * A.ty + 2 * at.j) * A.tx + at.m;
      A.bc[((size_t)K * NY + J) * H + I] =
          (r[0] + r[A.tx] + (r[A.ty * A.tx] + r[(A.ty + 1) * A.tx])) * T(0.125);
    }
  }
}

}  // namespace gmg
