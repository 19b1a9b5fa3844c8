// Schur solve by block cyclic reduction (Alg. 3), for pairs of TP = 1 to 4
// tiles, on the factor of k_bcr.hip / k_bcrn.hip:
//   forward   w_o = L_o^-1 r_o,  r_e -= X_R(o_l)' w_{o_l} + X_L(o_r)' w_{o_r},
//   border    s0 = s_b - sum_o Z_o'w_o,  w0 = T Lb^-1 s0,  u0 = -Lb^-T w0
//             (T = diag(-1 on the border's global rows, +1 on x_0)),
//   backward  u_o = L_o^-T (w_o - X_L u_L - X_R u_R - Z_o u0).
//
// A step is a chain of ceil(log2 P) dependent 16-vector products of some 0.3 us,
// so a launch or a round of memory per step is what costs.  The positions of a
// level are taken in groups of 2^lev: a workgroup eliminates all of its group
// but the first position (the separator) over lev levels, with all its tiles
// requested into registers at the start and the vectors in LDS, and hands the
// separators on to the next stage; a separator's terms of the group on its left
// are added where it is next read.  The last stage, with one group left, also
// eliminates the final pair, solves the border and starts the backward sweep;
// the groups then run backward, stage by stage.  A wave holds the tile row h of
// NP positions; tiles are loaded so that lane (i, g) holds four consecutive
// elements of row (of the transpose: column) i, so every product is four
// multiply-adds and one sum over g.
// Measured against one launch per level, a tail of the last 32 pairs and a
// launch for the blocks' part of the right-hand side, kernel time in us per
// solve: 7 pairs, border 8: 16.9 -> 8.3; 63 of 8 rows, border 22: 43 -> 21; 511 of
// 16 rows, border 32: 77 -> 37; 2189 of 2-8 rows, border 12: 96 -> 39; 511 of 4-32
// rows, border 64: 124 -> 68; 95 of 33-56 rows, border 24: 105 -> 70.  What is left
// is the launches and the tiles, which one compute unit loads twice in the last
// stage: with 32 positions there 21 us, with 8 9 us.
#include "bcr_geo.h"
#include "common.h"
#include "kernels.h"
#include "tile_chol.h"
#include "tile_ops.h"

#include <algorithm>

namespace ahlp {

namespace {

// NP positions per TP waves, 2^LEV positions at most in a group and 2^LLEV in
// the last stage's: 16 waves a workgroup, 12 for TP = 3.  TP = 4 needs more than
// 16 waves' registers: its groups have no waves of their own for the separator
// (OFF = 1: 12 waves), and the last stage takes two positions (8 waves).
template <int TP, int NP> struct Grp {
  static constexpr int TB = 16 * TP;
  static constexpr int LEV = TP == 1 ? (NP == 2 ? 5 : 4) : TP == 2 ? 3 : 2;
  static constexpr int LLEV = TP == 4 ? 1 : LEV;
  static constexpr int OFF = TP == 4 ? 1 : 0;
  static constexpr int GS = 1 << LEV;
  static constexpr int WAVES = (GS - OFF) * TP / NP, LWAVES = (1 << LLEV) * TP / NP;
};

template <int TP, int NP, int T0M> struct SolveLds {
  typedef Grp<TP, NP> G;
  double cl[G::GS * G::TB], cr[G::GS * G::TB];   // X_L'w, X_R'w by position
  double rv[G::GS * G::TB], wv[G::GS * G::TB];
  double uv[(G::GS + 1) * G::TB];
  double pb[16 * 16 * T0M];                // border partials by wave
  double u0[16 * T0M];
};

// where this wave stands: tile row h of the positions off + NP pg .. + NP - 1
template <int TP> struct Place {
  int wave, pg, h, lane, i16, off;
  __device__ __forceinline__ explicit Place(int o) {
    off = o;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    pg = wave / TP;
    h = wave % TP;
    lane = threadIdx.x & 63;
    i16 = lane & 15;
  }
};
__device__ __forceinline__ int level_of(int i) { return __builtin_ctz(i | 32); }

// lane (i, g) holds X(i, 4g .. 4g + 3) / X(4g .. 4g + 3, i)
__device__ __forceinline__ Op op_rows(const double* __restrict__ t) {
  const int lane = threadIdx.x & 63;
  Op o;
#pragma unroll
  for (int s = 0; s < 4; ++s) o.v[s] = t[(4 * (lane >> 4) + s) * TS + (lane & 15)];
  return o;
}
__device__ __forceinline__ Op op_cols(const double* __restrict__ t) {
  const int lane = threadIdx.x & 63;
  Op o;
#pragma unroll
  for (int s = 0; s < 4; ++s) o.v[s] = t[(lane & 15) * TS + 4 * (lane >> 4) + s];
  return o;
}
// acc + this lane's four products with the 16 values v in LDS; col_sum4 of it
// is the product's element lane % 16, in every lane
__device__ __forceinline__ double dot4(double acc, const Op& X, const double* v) {
  const double* p = v + 4 * ((threadIdx.x & 63) >> 4);
#pragma unroll
  for (int s = 0; s < 4; ++s) acc = fma(X.v[s], p[s], acc);
  return acc;
}

struct RowsOf { __device__ __forceinline__ Op operator()(const double* t) const { return op_rows(t); } };
struct ColsOf { __device__ __forceinline__ Op operator()(const double* t) const { return op_cols(t); } };

// whether the border tiles are requested only when the others are done with:
// with them the wider pairs' tiles don't fit the registers (128 of 16 waves, 168 of 12)
constexpr bool late_g(int tp, bool last) { return last ? tp == 2 || tp == 3 : tp == 4; }

// Right-hand side of pair j, element 16 h + lane % 16 (zero on the padding):
// the link rows' part and the blocks' parts of the two neighbouring blocks
template <int TP>
__device__ __forceinline__ double pair_rhs(const BcrSolveArgs& A, long long j, int h) {
  const int a = 16 * h + (threadIdx.x & 15);
  const BlockInfo &bl = A.blk[j], &br = A.blk[j + 1];
  return a < A.c.l[j] ? A.s[A.loff[j] + a] + (A.qn[bl.qoff + TS * bl.ktL + a] + A.qn[br.qoff + a]) : 0.0;
}

template <int TP, int NP, int T0M> struct FwdOps {
  Op li[NP][TP], xl[NP][TP], xr[NP][TP], g[NP][T0M];
  double r[NP], r0;   // right-hand sides; r0: the separator's where it has no slot
};

// Sum over this wave's lanes of a 16-vector's parts: the border sections of the
// blocks b0 .. b1 - 1 (subtracted) and the partials of earlier groups, shares
// taken by 16-lane rows
template <int TP, int T0M>
__device__ __forceinline__ void border_parts(const BcrSolveArgs& A, const Place<TP>& w, int rows,
                                             int b0, int b1, int nslots, double* acc) {
  const int t0 = A.c.t0, first = 4 * w.wave + (w.lane >> 4);
#pragma unroll
  for (int q = 0; q < T0M; ++q) acc[q] = 0.0;
  for (int b = b0 + first; b < b1; b += rows) {
    const BlockInfo& bi = A.blk[b];
    const double* src = A.qn + bi.qoff + TS * (bi.ktL + bi.ktR) + w.i16;
#pragma unroll
    for (int q = 0; q < T0M; ++q)
      if (16 * q + w.i16 < A.c.n0) acc[q] -= src[16 * q];
  }
#pragma unroll 4
  for (int s = first; s < nslots; s += rows)
#pragma unroll
    for (int q = 0; q < T0M; ++q)
      if (q < t0) acc[q] += A.pb[((long long)s * t0 + q) * 16 + w.i16];
}

// this wave's row of the right-hand side of position k of level lvl
template <int TP>
__device__ __forceinline__ double rhs_of(const BcrSolveArgs& A, int lvl, int k, const Place<TP>& w,
                                         const double* left) {
  const long long j = (long long)k << lvl, at = j * (16 * TP) + 16 * w.h + w.i16;
  if (lvl == 0) return pair_rhs<TP>(A, j, w.h);
  const double r = A.r[at];
  return k > 0 ? r - left[at] : r;
}

// Requests the forward tiles and the right-hand sides of this wave's positions.
// k0: position of the group's first at level lvl, n positions in all; last: the
// single group of the last stage, which eliminates its first position too.
template <int TP, int NP, int T0M>
__device__ __forceinline__ void fwd_load(const BcrSolveArgs& A, const Place<TP>& w, int lvl, int n,
                                         int k0, bool last, const double* left, FwdOps<TP, NP, T0M>& o) {
  typedef Geo<TP> G;
  const BcrArgs& c = A.c;
  o.r0 = w.off && w.pg == 0 ? rhs_of<TP>(A, lvl, k0, w, left) : 0.0;
#pragma unroll
  for (int sl = NP - 1; sl >= 0; --sl) {
    const int i = w.off + NP * w.pg + sl, k = k0 + i;
    const long long j = (long long)k << lvl;
    o.r[sl] = 0.0;
    if (k >= n) continue;
    o.r[sl] = rhs_of<TP>(A, lvl, k, w, left);
    if (i == 0 && !last) continue;
#pragma unroll
    for (int q = 0; q < TP; ++q)
      if (q <= w.h) o.li[sl][q] = op_rows(c.FLi + j * G::BLK + G::bt(w.h, q));
    if (i > 0) {
      const bool hr = k + (1 << level_of(i)) < n;
#pragma unroll
      for (int q = 0; q < TP; ++q) {
        o.xl[sl][q] = op_cols(c.FXL + j * G::BLK + G::bt(q, w.h));
        if (hr) o.xr[sl][q] = op_cols(c.FXR + j * G::BLK + G::bt(q, w.h));
      }
    }
  }
}
// the border tiles of the same positions, with op as op_rows or op_cols
template <int TP, int NP, int T0M, typename F>
__device__ __forceinline__ void load_g(const BcrSolveArgs& A, const Place<TP>& w, int lvl, int n, int k0,
                                       bool last, Op (&g)[NP][T0M], F op) {
#pragma unroll
  for (int sl = 0; sl < NP; ++sl) {
    const int i = w.off + NP * w.pg + sl, k = k0 + i;
    if (k >= n || (i == 0 && !last)) continue;
#pragma unroll
    for (int q = 0; q < T0M; ++q)
      if (q < A.c.t0) g[sl][q] = op(A.c.FGt + Geo<TP>::et((long long)k << lvl, q, w.h, A.c.t0));
  }
}

// w of position i from its right-hand side row r (other rows of the pair in
// the TP - 1 neighbouring waves); every wave of the workgroup calls it if TP > 1
template <int TP>
__device__ __forceinline__ void fwd_w(bool on, const Place<TP>& w, const Op* li, double r, double* rv,
                                      double* wv) {
  if (on) vec_put(rv + 16 * w.h, r);
  if constexpr (TP == 1) wave_order(); else lds_barrier();
  if (on) {
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < TP; ++q)
      if (q <= w.h) t = dot4(t, li[q], rv + 16 * q);
    vec_put(wv + 16 * w.h, col_sum4(t));
  }
  if constexpr (TP == 1) wave_order(); else lds_barrier();
}

// the levels of a group: after them o.r of position 0 holds its right-hand side
// less its own group's terms, and L.wv every eliminated position's w
template <int TP, int NP, int T0M>
__device__ __forceinline__ void fwd_levels(const Place<TP>& w, int n, int k0, int lev,
                                           FwdOps<TP, NP, T0M>& o, SolveLds<TP, NP, T0M>& L) {
  constexpr int TB = 16 * TP;
  for (int v = 0; v < lev; ++v) {
    const int d = 1 << v;
#pragma unroll
    for (int sl = 0; sl < NP; ++sl) {
      if (NP == 2 && (sl == 1) != (v == 0)) continue;   // odd positions at level 0, even ones later
      const int i = w.off + NP * w.pg + sl;
      const bool on = i > 0 && k0 + i < n && level_of(i) == v;
      fwd_w<TP>(on, w, o.li[sl], o.r[sl], L.rv + i * TB, L.wv + i * TB);
      if (on) {
        double a = 0.0, b = 0.0;
#pragma unroll
        for (int q = 0; q < TP; ++q) a = dot4(a, o.xl[sl][q], L.wv + i * TB + 16 * q);
        vec_put(L.cl + i * TB + 16 * w.h, col_sum4(a));
        if (k0 + i + d < n) {
#pragma unroll
          for (int q = 0; q < TP; ++q) b = dot4(b, o.xr[sl][q], L.wv + i * TB + 16 * q);
          vec_put(L.cr + i * TB + 16 * w.h, col_sum4(b));
        }
      }
    }
    lds_barrier();
#pragma unroll
    for (int sl = 0; sl < NP; ++sl) {
      const int i = w.off + NP * w.pg + sl;
      if (level_of(i) <= v || k0 + i >= n) continue;
      if (i > 0) o.r[sl] -= L.cr[(i - d) * TB + 16 * w.h + w.i16];
      if (k0 + i + d < n) o.r[sl] -= L.cl[(i + d) * TB + 16 * w.h + w.i16];
    }
    if (w.off && w.pg == 0 && k0 + d < n) o.r0 -= L.cl[d * TB + 16 * w.h + w.i16];
  }
}

// border partials Z'w of this wave's positions, with its share acc of the other
// parts, into L.pb
template <int TP, int NP, int T0M>
__device__ __forceinline__ void border_put(const BcrSolveArgs& A, const Place<TP>& w, int n, int k0,
                                           bool last, const FwdOps<TP, NP, T0M>& o, const double* acc,
                                           SolveLds<TP, NP, T0M>& L) {
#pragma unroll
  for (int q = 0; q < T0M; ++q) {
    if (q >= A.c.t0) continue;
    double t = acc[q];
#pragma unroll
    for (int sl = 0; sl < NP; ++sl) {
      const int i = w.off + NP * w.pg + sl;
      if (k0 + i < n && (i > 0 || last)) t = dot4(t, o.g[sl][q], L.wv + i * 16 * TP + 16 * w.h);
    }
    t = col_sum4(t);
    if (w.lane < 16) L.pb[w.wave * 16 * T0M + 16 * q + w.lane] = t;
  }
}
// element threadIdx.x of the waves' sum
template <int TP, int NP, int T0M>
__device__ __forceinline__ double border_sum(const SolveLds<TP, NP, T0M>& L) {
  const int waves = blockDim.x >> 6;
  double acc = 0.0;
#pragma unroll 16
  for (int v = 0; v < waves; ++v) acc += L.pb[v * 16 * T0M + threadIdx.x];
  return acc;
}

// One stage forward: group blockIdx.x of 2^lev positions at level lvl (n in all).
// left / left_out: a separator's terms of the group on its left, from the stage
// before and for the next (distinct arrays: the neighbour group still reads).
// The group's border partial goes to slot slot0 + blockIdx.x of A.pb.
template <int TP, int NP, int T0M>
__global__ __launch_bounds__((64 * Grp<TP, NP>::WAVES)) void k_bcrs_fwd(
    BcrSolveArgs A, int lvl, int n, int lev, int slot0, const double* left,
    double* left_out) {
  typedef Geo<TP> G;
  __shared__ SolveLds<TP, NP, T0M> L;
  const Place<TP> w(Grp<TP, NP>::OFF);
  const int k0 = blockIdx.x << lev, gs = 1 << lev;
  FwdOps<TP, NP, T0M> o;
  fwd_load<TP, NP, T0M>(A, w, lvl, n, k0, false, left, o);
  if (!late_g(TP, false)) load_g<TP, NP, T0M>(A, w, lvl, n, k0, false, o.g, RowsOf{});
  double acc[T0M];
  {   // the border sections of the blocks left of the group's pairs, and the very last
    const int b1 = lvl > 0 ? 0 : (k0 + gs >= n ? n + 1 : k0 + gs);
    border_parts<TP, T0M>(A, w, blockDim.x >> 4, k0, b1, 0, acc);
  }
  fwd_levels<TP, NP, T0M>(w, n, k0, lev, o, L);
  if (late_g(TP, false)) load_g<TP, NP, T0M>(A, w, lvl, n, k0, false, o.g, RowsOf{});
  border_put<TP, NP, T0M>(A, w, n, k0, false, o, acc, L);
  if (w.lane < 16) {
#pragma unroll
    for (int sl = 0; sl < NP; ++sl) {
      const int i = w.off + NP * w.pg + sl;
      const long long at = ((long long)(k0 + i) << lvl) * G::TB + 16 * w.h + w.lane;
      if (k0 + i >= n) continue;
      if (i > 0) A.w[at] = L.wv[i * G::TB + 16 * w.h + w.lane];
      else A.r[at] = o.r[sl];
    }
    if (w.off && w.pg == 0) A.r[((long long)k0 << lvl) * G::TB + 16 * w.h + w.lane] = o.r0;
    if (w.pg == 0 && k0 + gs < n) {
      double t = 0.0;
      for (int d = 1; d < gs; d *= 2) t += L.cr[(gs - d) * G::TB + 16 * w.h + w.lane];
      left_out[((long long)(k0 + gs) << lvl) * G::TB + 16 * w.h + w.lane] = t;
    }
  }
  lds_barrier();
  const int nbp = 16 * A.c.t0;
  if ((int)threadIdx.x < nbp) A.pb[(long long)(slot0 + blockIdx.x) * nbp + threadIdx.x] = border_sum<TP, NP, T0M>(L);
}

template <int TP, int NP, int T0M> struct BwdOps {
  Op li[NP][TP], xl[NP][TP], xr[NP][TP], g[NP][T0M];
  double t[NP];
  int len[NP];
  long long off[NP];
};

template <int TP, int NP, int T0M>
__device__ __forceinline__ void bwd_load(const BcrSolveArgs& A, const Place<TP>& w, int lvl, int n, int k0,
                                         bool last, BwdOps<TP, NP, T0M>& o) {
  typedef Geo<TP> G;
  const BcrArgs& c = A.c;
#pragma unroll
  for (int sl = 0; sl < NP; ++sl) {
    const int i = w.off + NP * w.pg + sl, k = k0 + i;
    const long long j = (long long)k << lvl;
    if (k >= n || (i == 0 && !last)) continue;
    if (!last) o.t[sl] = A.w[j * G::TB + 16 * w.h + w.i16];
    o.len[sl] = c.l[j];
    o.off[sl] = A.loff[j];
    if (i > 0) {
      const bool hr = k + (1 << level_of(i)) < n;
#pragma unroll
      for (int q = 0; q < TP; ++q) {
        o.xl[sl][q] = op_rows(c.FXL + j * G::BLK + G::bt(w.h, q));
        if (hr) o.xr[sl][q] = op_rows(c.FXR + j * G::BLK + G::bt(w.h, q));
      }
    }
#pragma unroll
    for (int q = 0; q < TP; ++q)
      if (q >= w.h) o.li[sl][q] = op_cols(c.FLi + j * G::BLK + G::bt(q, w.h));
  }
}

// u of position i from t = w - Z u0 and its neighbours' u (LDS, lvl as above);
// every wave of the workgroup calls it if TP > 1
template <int TP>
__device__ __forceinline__ void bwd_u(bool on, const BcrSolveArgs& A, const Place<TP>& w, long long j,
                                      const Op* li, const Op* xl, const Op* xr, const double* ul,
                                      const double* ur, double t, int len, long long off, bool keep,
                                      double* rv, double* uv) {
  if (on) {
    if (ul) {
      double a = 0.0;
#pragma unroll
      for (int q = 0; q < TP; ++q) a = dot4(a, xl[q], ul + 16 * q);
      if (ur)
#pragma unroll
        for (int q = 0; q < TP; ++q) a = dot4(a, xr[q], ur + 16 * q);
      t -= col_sum4(a);
    }
    vec_put(rv + 16 * w.h, t);
  }
  if constexpr (TP == 1) wave_order(); else lds_barrier();
  if (on) {
    double a = 0.0;
#pragma unroll
    for (int q = 0; q < TP; ++q)
      if (q >= w.h) a = dot4(a, li[q], rv + 16 * q);
    const double u = col_sum4(a);
    if (w.lane < 16) {
      const int e = 16 * w.h + w.lane;
      uv[e] = u;
      if (keep) A.up[j * (16 * TP) + e] = u;
      if (e < len) {
        A.u[off + e] = u;
        A.dyl[off + e] = u;
      }
    }
  }
}

template <int TP, int NP, int T0M>
__device__ __forceinline__ void bwd_levels(const BcrSolveArgs& A, const Place<TP>& w, int lvl, int n, int k0,
                                           int lev, bool keep, BwdOps<TP, NP, T0M>& o,
                                           SolveLds<TP, NP, T0M>& L) {
  constexpr int TB = 16 * TP;
  for (int v = lev - 1; v >= 0; --v) {
    const int d = 1 << v;
#pragma unroll
    for (int sl = 0; sl < NP; ++sl) {
      if (NP == 2 && (sl == 1) != (v == 0)) continue;
      const int i = w.off + NP * w.pg + sl;
      const bool on = i > 0 && k0 + i < n && level_of(i) == v;
      bwd_u<TP>(on, A, w, (long long)(k0 + i) << lvl, o.li[sl], o.xl[sl], o.xr[sl], L.uv + (i - d) * TB,
                k0 + i + d < n ? L.uv + (i + d) * TB : nullptr, o.t[sl], o.len[sl], o.off[sl], keep,
                L.rv + i * TB, L.uv + i * TB);
    }
    lds_barrier();
  }
}

// t = w - Z u0 of this wave's positions
template <int TP, int NP, int T0M>
__device__ __forceinline__ void bwd_border(const BcrSolveArgs& A, BwdOps<TP, NP, T0M>& o, const double* u0) {
#pragma unroll
  for (int sl = 0; sl < NP; ++sl) {
    double a = 0.0;
#pragma unroll
    for (int q = 0; q < T0M; ++q)
      if (q < A.c.t0) a = dot4(a, o.g[sl][q], u0 + 16 * q);
    o.t[sl] -= col_sum4(a);
  }
}

// One stage backward, the groups of k_bcrs_fwd
template <int TP, int NP, int T0M>
__global__ __launch_bounds__((64 * Grp<TP, NP>::WAVES)) void k_bcrs_bwd(BcrSolveArgs A, int lvl, int n, int lev) {
  typedef Geo<TP> G;
  __shared__ SolveLds<TP, NP, T0M> L;
  const Place<TP> w(Grp<TP, NP>::OFF);
  const int k0 = blockIdx.x << lev, gs = 1 << lev;
  BwdOps<TP, NP, T0M> o{};
  const int e = w.lane, b = w.wave == 0 ? 0 : gs;   // separators' u, u0
  const bool two = blockDim.x > 64;
  double us = 0.0, us2 = 0.0, u0v = 0.0;
  if (w.wave < 2 && e < G::TB && k0 + b < n) us = A.up[((long long)(k0 + b) << lvl) * G::TB + e];
  if (!two && e < G::TB && k0 + gs < n) us2 = A.up[((long long)(k0 + gs) << lvl) * G::TB + e];
  if (w.wave == 0 && e < 16 * A.c.t0) u0v = A.u0p[e];
  load_g<TP, NP, T0M>(A, w, lvl, n, k0, false, o.g, ColsOf{});
  if (!late_g(TP, false)) bwd_load<TP, NP, T0M>(A, w, lvl, n, k0, false, o);
  if (w.wave < 2 && e < G::TB) L.uv[b * G::TB + e] = us;
  if (!two && e < G::TB) L.uv[gs * G::TB + e] = us2;
  if (w.wave == 0 && e < 16 * T0M) L.u0[e] = u0v;
  lds_barrier();
  if (late_g(TP, false)) bwd_load<TP, NP, T0M>(A, w, lvl, n, k0, false, o);
  bwd_border<TP, NP, T0M>(A, o, L.u0);
  bwd_levels<TP, NP, T0M>(A, w, lvl, n, k0, lev, lvl > 0, o, L);
}

// The last stage: one group of n <= 2^LEV positions, its first included, then
// the border and the group's backward sweep.  nslots: border partials of the
// stages before.  The tiles of Lb^-1 are requested with the rest and put to LDS
// packed, lower tile (r, c) at r (r + 1) / 2 + c.
template <int TP, int NP, int T0M>
__global__ __launch_bounds__((64 * Grp<TP, NP>::LWAVES)) void k_bcrs_last(BcrSolveArgs A, int lvl, int n, int lev,
                                                                   int nslots, const double* left) {
  typedef Grp<TP, NP> R;
  constexpr int TB = R::TB, THREADS = 64 * R::LWAVES;
  constexpr int NLB = (T0M * (T0M + 1) / 2 * 256 + THREADS - 1) / THREADS;
  __shared__ SolveLds<TP, NP, T0M> L;
  __shared__ double lbi[T0M * (T0M + 1) / 2 * 256];
  __shared__ double s0[16 * T0M], w0[16 * T0M];
  const BcrArgs& c = A.c;
  const int t0 = c.t0, tid = threadIdx.x;
  const Place<TP> w(0);
  FwdOps<TP, NP, T0M> o;
  fwd_load<TP, NP, T0M>(A, w, lvl, n, 0, true, left, o);
  if (!late_g(TP, true)) load_g<TP, NP, T0M>(A, w, lvl, n, 0, true, o.g, RowsOf{});
  double lb[NLB], sb = 0.0, acc[T0M];
#pragma unroll
  for (int u = 0; u < NLB; ++u) {
    const int idx = tid + u * THREADS, tile = idx >> 8;
    int r = 0;
    while ((r + 1) * (r + 2) / 2 <= tile) ++r;
    const int cc = tile - r * (r + 1) / 2;
    lb[u] = r < t0 ? c.FLbi[(cc * t0 + r) * 256 + (idx & 255)] : 0.0;
  }
  if (tid < c.n0) sb = tid < c.ng ? A.s[A.nl + tid] : A.rhx0[tid - c.ng];
  border_parts<TP, T0M>(A, w, 4 * R::LWAVES, 0, lvl > 0 ? 0 : n + 1, nslots, acc);
  fwd_levels<TP, NP, T0M>(w, n, 0, lev, o, L);
  if (late_g(TP, true)) load_g<TP, NP, T0M>(A, w, lvl, n, 0, true, o.g, RowsOf{});
  const bool fin = w.pg == 0 && n > 0;   // the final pair
  fwd_w<TP>(fin, w, o.li[0], o.r[0], L.rv, L.wv);
  border_put<TP, NP, T0M>(A, w, n, 0, true, o, acc, L);
#pragma unroll
  for (int u = 0; u < NLB; ++u)
    if (tid + u * THREADS < t0 * (t0 + 1) / 2 * 256) lbi[tid + u * THREADS] = lb[u];
  BwdOps<TP, NP, T0M> b{};
  bwd_load<TP, NP, T0M>(A, w, lvl, n, 0, true, b);
  if (!late_g(TP, true)) load_g<TP, NP, T0M>(A, w, lvl, n, 0, true, b.g, ColsOf{});
#pragma unroll
  for (int sl = 0; sl < NP; ++sl) b.t[sl] = L.wv[(w.off + NP * w.pg + sl) * TB + 16 * w.h + w.i16];
  lds_barrier();
  if (tid < 16 * t0) s0[tid] = sb - border_sum<TP, NP, T0M>(L);
  lds_barrier();
  if (w.wave < t0) {
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < T0M; ++q)
      if (q <= w.wave) t = dot4(t, op_rows(lbi + (w.wave * (w.wave + 1) / 2 + q) * 256), s0 + 16 * q);
    t = col_sum4(t);
    if (w.lane < 16) w0[16 * w.wave + w.lane] = 16 * w.wave + w.lane < c.ng ? -t : t;
  }
  lds_barrier();
  if (late_g(TP, true)) load_g<TP, NP, T0M>(A, w, lvl, n, 0, true, b.g, ColsOf{});
  if (w.wave < t0) {
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < T0M; ++q)
      if (q >= w.wave && q < t0) t = dot4(t, op_cols(lbi + (q * (q + 1) / 2 + w.wave) * 256), w0 + 16 * q);
    t = -col_sum4(t);
    const int e = 16 * w.wave + w.lane;
    if (w.lane < 16) {
      L.u0[e] = t;
      A.u0p[e] = t;
      if (e < c.n0) A.u[A.nl + e] = t;
      if (e < c.ng) A.dyl[A.nl + e] = t;
    }
  }
  lds_barrier();
  bwd_border<TP, NP, T0M>(A, b, L.u0);
  bwd_u<TP>(fin, A, w, 0, b.li[0], nullptr, nullptr, nullptr, nullptr, b.t[0], b.len[0], b.off[0], lvl > 0,
            L.rv, L.uv);
  lds_barrier();
  bwd_levels<TP, NP, T0M>(A, w, lvl, n, 0, lev, lvl > 0, b, L);
}

int levels(int n) {   // ceil(log2 n)
  int v = 0;
  while ((1 << v) < n) ++v;
  return v;
}

// As few stages as the groups allow, the levels split evenly over them: the last
// stage, one compute unit that loads its tiles for both directions, gets the fewest,
// then the first, which has the most groups.
template <int TP, int NP, int T0M>
void solve_tp(hipStream_t st, const BcrSolveArgs& a) {
  typedef Grp<TP, NP> R;
  const int total = levels(a.c.P), before = total > R::LLEV ? total - R::LLEV : 0;
  const int stages = (before + R::LEV - 1) / R::LEV, ahead = total - std::min(total / (stages + 1), R::LLEV);
  int lvl = 0, n = a.c.P, slots = 0, lv[32], ln[32], lg[32];
  double* out[2] = {a.up, a.w};
  for (int s = 0; s < stages; ++s) {
    const int lev = (ahead - lvl) / (stages - s), groups = (n + (1 << lev) - 1) >> lev;
    lv[s] = lvl; ln[s] = n; lg[s] = lev;
    hipLaunchKernelGGL((k_bcrs_fwd<TP, NP, T0M>), dim3(groups), dim3(64 * ((1 << lev) - R::OFF) * TP / NP), 0, st, a, lvl, n, lev,
                       slots, out[(s + 1) & 1], out[s & 1]);
    slots += groups;
    lvl += lev;
    n = groups;
  }
  hipLaunchKernelGGL((k_bcrs_last<TP, NP, T0M>), dim3(1), dim3(64 * R::LWAVES), 0, st, a, lvl, n, levels(n), slots,
                     out[(stages + 1) & 1]);
  for (int s = stages - 1; s >= 0; --s)
    hipLaunchKernelGGL((k_bcrs_bwd<TP, NP, T0M>), dim3((ln[s] + (1 << lg[s]) - 1) >> lg[s]),
                       dim3(64 * ((1 << lg[s]) - R::OFF) * TP / NP), 0, st, a, lv[s], ln[s], lg[s]);
}

}  // namespace

// One tile a side: two positions a wave if the border's tiles leave the
// registers for it.
void launch_bcr_solve(hipStream_t st, const BcrSolveArgs& a) {
  if (a.c.tp == 2) solve_tp<2, 1, 4>(st, a);
  else if (a.c.tp == 3) solve_tp<3, 1, 4>(st, a);
  else if (a.c.tp == 4) solve_tp<4, 1, 4>(st, a);
  else if (a.c.t0 <= 2) solve_tp<1, 2, 2>(st, a);
  else solve_tp<1, 1, 4>(st, a);
}

}  // namespace ahlp
