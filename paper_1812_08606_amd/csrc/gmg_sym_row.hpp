// gmg_sym_row.hpp -- the fused symmetric red-black sweep of the finest level
// on rows of at most 128 x-pairs: a block spans the row.
#pragma once

#include "gmg_sym.hpp"

namespace gmg {

// k_sym_split (gmg_sym.hpp) for short rows.  Its 62-pair tiles fit a row of 64
// or 128 pairs badly (nx = 128: 64 of 124 lanes own pairs, nx = 256: 128 of
// 186) and start 4 bytes off a line; here a block spans the row with WX waves,
// so no lane is an x-halo and every row starts on a line.  Rows 0 and R-1 are
// a halo as there, the columns march z with the same rings, and the sweep's
// arithmetic is the same, face by face.  The x-neighbours outside the pair may
// lie in another wave: its coefficient and old value are read from the staged
// plane, its new colour-c1 value from the ring, and the outer x-face of the
// c2 cell, which k_sym_split takes from the adjacent lane, is formed from the
// staged coefficients one plane earlier.
// Bound by memory like k_sym_split, at short rows by the number of blocks and
// the halo rows (6 of 8 rows own cells with two waves in float32, 4 of 6 in
// float64).  Per symmetric sweep, two half-sweeps / k_sym_split / this kernel:
// 256^3 float64 167 / 140 / 104 us (28 B per cell, 4.5 TB/s), float32 69 / 78 /
// 62 us; 256 x 256 x 320 float64 210 / 174 / 126 us; 128^3 float32 17.8 / 18.3 /
// 14.0 us.
template <typename T, int WX>
struct SymRowShape {
  static constexpr int SX = 64 * WX;
  static constexpr int R = (sizeof(T) == 4 ? 16 : 12) / WX;
  static constexpr int IY = R - 2;
};

template <typename T, bool FIRST, bool SCALED, int WX>
__global__ __launch_bounds__((SymRowShape<T, WX>::SX * SymRowShape<T, WX>::R)) void k_sym_row(
    const T* __restrict__ Xin, T* __restrict__ Xout, T* __restrict__ B, const double* __restrict__ u,
    const double* __restrict__ bscale, const T* __restrict__ a, Geom g, size_t hn, int kc, int c1) {
  using T2 = typename Pair2<T>::type;
  using S = SymRowShape<T, WX>;
  constexpr int SX = S::SX, R = S::R, IY = S::IY;
  constexpr int NS = 2;              // planes of side values held in LDS
  __shared__ T2 sa[NS][R + 2][SX];  // a pairs of block rows -1 .. R (array rows 0 .. R+1)
  __shared__ T so[NS][R + 2][SX];   // old values of colour c2, same rows
  __shared__ T ring[4][R][SX];      // new c1 values of planes k-3 .. k (mod 4)
  __shared__ T2 ringw[4][R][SX];    // their south and north face weights, same planes
  const Tile tl = xcd_tile();
  const int H = g.nx >> 1;
  const int lane = threadIdx.x;  // and the pair
  const int r = sizeof(T) == 8 ? (int)__builtin_amdgcn_readfirstlane(threadIdx.y) : (int)threadIdx.y;
  const int m = lane;
  const int j = tl.y * IY + r - 1;
  const bool owner = m < H && j >= 0 && j < g.ny && r >= 1 && r < R - 1;
  const int lw = max(lane - 1, 0), le = min(lane + 1, SX - 1);
  const int c2 = 1 - c1;
  const size_t tz = (size_t)H * g.ny;
  const T hx = (T)(0.5 * g.ihx2), hy = (T)(0.5 * g.ihy2), hz = (T)(0.5 * g.ihz2), pz = (T)(2.0 * g.ihz2);
  const double s = SCALED ? *bscale : 1.0;
  const int k0 = tl.z * kc, k1 = min(g.nz, k0 + kc);
  // iterations kstart .. kend update c1 on plane k, c2 on plane k-1
  const int kstart = k0 - 1, kend = k1;
  // faces outside the pair: present when both cells lie in the grid (for
  // threads outside it, whose addresses are clamped to it, every such face
  // weight is zero)
  const bool hw = m > 0 && m < H, he = m < H - 1, hs = j > 0 && j < g.ny, hn_ = j >= 0 && j < g.ny - 1;
  // clamped (always valid) column of this thread, and of the row beyond the
  // block that rows 0 and R-1 stage (array row 0 or R+1)
  const int mm = min(m, H - 1), jj = min(max(j, 0), g.ny - 1);
  const size_t qcol = (size_t)jj * H + mm;
  const bool hrow = r == 0 || r == R - 1;
  const int jh = min(max(r == 0 ? j - 1 : j + 1, 0), g.ny - 1);
  const size_t qhcol = (size_t)jh * H + mm;
  const int arow = r == 0 ? 0 : R + 1;
  auto pl = [&](int k) { return min(max(k, 0), g.nz - 1); };
  // every array is addressed from plane kb, the lowest the block reads, with
  // per-lane byte offsets of the column (colour arrays: ST per pair; a and the
  // natural-layout u: two cells per pair) and a scalar offset per plane
  const int kb = pl(kstart - 1);
  const size_t pb = (size_t)kb * tz;  // first pair of plane kb
  constexpr uint32_t ST = sizeof(T);
  const size_t cbytes = (hn - pb) * ST, nbytes = 2 * (hn - pb) * ST;
  // (Xin is not read by the first sweep, u only by it)
  const auto rXo = buf_rsrc(FIRST ? nullptr : Xin + (size_t)c2 * hn + pb, FIRST ? 0 : cbytes);  // old colour c2
  const auto rY1 = buf_rsrc(Xout + (size_t)c1 * hn + pb, cbytes);
  const auto rY2 = buf_rsrc(Xout + (size_t)c2 * hn + pb, cbytes);
  const auto rB1 = buf_rsrc(B + (size_t)c1 * hn + pb, cbytes);
  const auto rB2 = buf_rsrc(B + (size_t)c2 * hn + pb, cbytes);
  const auto rA = buf_rsrc(a + 2 * pb, nbytes);
  const auto rU = buf_rsrc(FIRST ? u + 2 * pb : nullptr, FIRST ? 2 * (hn - pb) * sizeof(double) : 0);
  const uint32_t vq = (uint32_t)qcol * ST, vqh = (uint32_t)qhcol * ST;
  const uint32_t ptb = (uint32_t)tz * ST;  // bytes per plane of a colour array
  auto soff = [&](int k) { return (uint32_t)(k - kb) * ptb; };

  // e1c: RuntimeParity or the compile-time value of (c1 + j + p) % 2
  auto load = [&](int p, SymCol<T>& L, auto e1c) {
    const uint32_t so1 = soff(pl(p));
    const T2 av = buf_load_pair<T>(rA, 2 * vq, 2 * so1);
    L.a0 = av.x;
    L.a1 = av.y;
    if (!FIRST) {
      L.xo = buf_load<T>(rXo, vq, so1);
      L.b1 = buf_load<T>(rB1, vq, so1);
      L.b2 = buf_load<T>(rB2, vq, so1);
    } else {
      constexpr uint32_t W = sizeof(double) / ST;  // u bytes per colour-array byte, per cell pair
      const double u0d = buf_load<double>(rU, 2 * W * vq, 2 * W * so1);
      const double u1d = buf_load<double>(rU, 2 * W * vq + 8, 2 * W * so1);
      const T u0 = (T)(SCALED ? u0d * s : u0d), u1 = (T)(SCALED ? u1d * s : u1d);
      const int e1 = parity_of(e1c, (c1 + j + p) & 1);
      L.b1 = e1 ? u1 : u0;
      L.b2 = e1 ? u0 : u1;
      L.xo = T(0);
    }
    if (hrow) {
      const T2 hv = buf_load_pair<T>(rA, 2 * vqh, 2 * so1);
      L.ha0 = hv.x;
      L.ha1 = hv.y;
      L.hxo = FIRST ? T(0) : buf_load<T>(rXo, vqh, so1);
    }
  };
  auto stage = [&](int p, const SymCol<T>& L) {
    const int sl = p & (NS - 1);
    sa[sl][r + 1][lane] = T2{L.a0, L.a1};
    so[sl][r + 1][lane] = L.xo;
    if (hrow) {
      sa[sl][arow][lane] = T2{L.ha0, L.ha1};
      so[sl][arow][lane] = L.hxo;
    }
  };

  // registers: a of the pair on planes k-1 .. k+1, old c2 of the column on
  // k-1 .. k+1, new c1 of the column on k-3 .. k; right sides: c1 and c2 of
  // plane k (cb1, cb2), c2 of plane k-1 (pb2); face weights on plane k-1: the
  // inner x-face (wip) and the c2 cell's outer one (wo2p); top faces of the c1
  // cell on planes k-1 and k-2 (wtp, wtpp)
  T a0[3], a1[3], xo[3], c1n[4], cb1, cb2, pb2 = T(0);
  T wip = T(0), wo2p = T(0), wtp = T(0), wtpp = T(0);
#pragma unroll
  for (int t = 0; t < 4; ++t) c1n[t] = T(0);
  a0[0] = a1[0] = T(0);
  xo[0] = T(0);
  {
    SymCol<T> Lb, Lc;
    load(kstart - 1, Lb, RuntimeParity{});
    load(kstart, Lc, RuntimeParity{});
    a0[1] = Lb.a0;
    a1[1] = Lb.a1;
    xo[1] = Lb.xo;
    a0[2] = Lc.a0;
    a1[2] = Lc.a1;
    xo[2] = Lc.xo;
    cb1 = Lc.b1;
    cb2 = Lc.b2;
    stage(kstart, Lc);
  }
  lds_barrier();

  // iteration k: stage plane k+1, colour c1 on plane k, colour c2 on plane k-1
  auto iterate = [&](int k, const SymCol<T>& L, auto e1c) {
    a0[0] = a0[1];
    a1[0] = a1[1];
    a0[1] = a0[2];
    a1[1] = a1[2];
    a0[2] = L.a0;
    a1[2] = L.a1;
    xo[0] = xo[1];
    xo[1] = xo[2];
    xo[2] = L.xo;
    stage(k + 1, L);
    const int e1 = parity_of(e1c, (c1 + j + k) & 1);
    const int sl = k & (NS - 1);
    // the c1 cell is element e1 of the pair, its outer neighbour in the pair
    // on that side; the c2 cell's in the pair on the other side
    const int s1 = e1 ? le : lw, s2 = e1 ? lw : le;
    T v1, wb;
    {
      const T2 po = sa[sl][r + 1][s1], pq = sa[sl][r + 1][s2];
      const T2 ps = sa[sl][r][lane], pn = sa[sl][r + 2][lane];
      const bool top = k >= g.nz - 1, bot = k <= 0;
      const T acv = e1 ? a1[1] : a0[1], ain = e1 ? a0[1] : a1[1];
      const T abv = e1 ? a1[0] : a0[0], atv = e1 ? a1[2] : a0[2];
      const T wi = (acv + ain) * hx;
      const T wo = (e1 ? he : hw) ? (acv + (e1 ? po.x : po.y)) * hx : T(0);
      const T wo2 = (e1 ? hw : he) ? (ain + (e1 ? pq.y : pq.x)) * hx : T(0);
      const T ws = hs ? (acv + (e1 ? ps.y : ps.x)) * hy : T(0);
      const T wn = hn_ ? (acv + (e1 ? pn.y : pn.x)) * hy : T(0);
      wb = (acv + abv) * hz;
      const T wt = (acv + atv) * hz;
      const T dz1 = pz * acv;
      const T D1 = wi + wo + ws + wn + (!bot ? wb : dz1) + (!top ? wt : dz1);
      if (FIRST) {
        v1 = cb1 * recip(D1);
      } else {
        // (absent faces have zero weight and finite neighbour values)
        const T xs = so[sl][r][lane], xn = so[sl][r + 2][lane], xout = so[sl][r + 1][s1];
        const T off = wi * xo[1] + wo * xout + ws * xs + wn * xn + (!bot ? wb * xo[0] : T(0)) +
                      (!top ? wt * xo[2] : T(0));
        v1 = (cb1 + off) * recip(D1);
      }
      if (owner && k >= k0 && k < k1) {
        const uint32_t so1 = soff(k);
        buf_store<T>(v1, rY1, vq, so1);
        if (FIRST) {
          buf_store<T>(cb1, rB1, vq, so1);
          buf_store<T>(cb2, rB2, vq, so1);
        }
      }
      ringw[k & 3][r][lane] = T2{ws, wn};
      c1n[0] = c1n[1];
      c1n[1] = c1n[2];
      c1n[2] = c1n[3];
      c1n[3] = v1;
      ring[k & 3][r][lane] = v1;
      lds_barrier();
      // --- colour c2 on plane kk = k-1 (element e1 of the pair) ---
      const int kk = k - 1;
      if (owner && kk >= k0 && kk < k1) {
        const bool topk = kk == g.nz - 1, botk = kk == 0;
        const int rl = kk & 3;
        const T cov = ring[rl][r][s1];
        const T ys = ring[rl][r - 1][lane], yn = ring[rl][r + 1][lane];
        const T wsv = ringw[rl][r - 1][lane].y, wnv = ringw[rl][r + 1][lane].x;
        const T ac2 = e1 ? a1[0] : a0[0];
        const T D = wip + wo2p + wsv + wnv + (!botk ? wtpp : pz * ac2) + (!topk ? wb : pz * ac2);
        const T off = wip * c1n[2] + wo2p * cov + wsv * ys + wnv * yn + (!botk ? wtpp * c1n[1] : T(0)) +
                      (!topk ? wb * c1n[3] : T(0));
        buf_store<T>((pb2 + off) * recip(D), rY2, vq, soff(kk));
      }
      wtpp = wtp;
      wtp = wt;
      wip = wi;
      wo2p = wo2;
    }
    pb2 = cb2;
    cb1 = L.b1;
    cb2 = L.b2;
  };

  // two load buffers, four iterations per trip, as in k_sym_split; in float64
  // the loop is instantiated for both parities of the wave's row
  SymCol<T> L[2];
  auto run = [&](auto p0, auto p1) {
    load(kstart + 1, L[0], p1);
    for (int k = kstart; k <= kend; k += 4) {
#pragma unroll
      for (int t = 0; t < 4; t += 2) {
        load(k + t + 2, L[1], p0);
        if (k + t > kend) return;  // (an exit, not a break: no second path into the loop's back edge)
        iterate(k + t, L[0], p0);
        load(k + t + 3, L[0], p1);
        if (k + t + 1 > kend) return;
        iterate(k + t + 1, L[1], p1);
      }
    }
  };
  if constexpr (sizeof(T) == 8) {
    constexpr std::integral_constant<int, 0> P0{};
    constexpr std::integral_constant<int, 1> P1{};
    if ((c1 + j + kstart) & 1)
      run(P1, P0);
    else
      run(P0, P1);
  } else {
    run(RuntimeParity{}, RuntimeParity{});
  }
}

}  // namespace gmg
