// Block cyclic reduction of the Schur complement (a6) for link pairs of 17 to
// 64 rows: the odd-even reduction of the one-tile kernels (k_bcr.hip) with
// every pair padded to TP x TP tiles (TP = 2, 3 or 4, the widest pair's).  The
// elimination of a pair o with active neighbours L and R is the same,
//   T'_oo = L_o L_o',  X_L = L_o^-1 T'_oL,  X_R = L_o^-1 T'_oR,  Z = L_o^-1 E'_o,
//   T'_LL -= X_L'X_L,  T'_RR -= X_R'X_R,  T'_RL = -X_R'X_L,
//   E'_L -= X_L'Z,  E'_R -= X_R'Z.
// A level is two launches.  In the first a workgroup eliminates one odd pair:
// one wave after another factors the TP diagonal tiles (the chain, about 2 us
// a tile), all waves share the tile column below and the trailing update; then
// every wave takes whole columns of L_o^-1 [I, T'_oL, T'_oR, E'_o] by forward
// substitution in registers (an FP64 accumulator tile is laid out as the next
// product's B operand, so a column never leaves them).  The second updates the
// even pairs, one wave per tile.  A column's operands are requested before the
// factorization, so the step waits on memory once.  What bounds a level is
// the chain of TP tile factorizations and the two launches; the arithmetic of
// a whole reduction is below a MFMA-microsecond.
// Measured against what it replaced.  511 pairs of 4-32 rows, border 64, one
// wave per elimination and one launch per level: level 20.0 -> 10.2 + 7.8 us,
// solve step 11.5 -> 6.0 us forward and 7.3 -> 5.0 us backward.  95 pairs of
// 33-56 rows, border 24, a segmented chain of scalar eliminations: factor 8.4 ->
// 0.28 ms, solve 0.94 -> 0.10 ms.
//
// Storage (the BcrArgs arrays, sized for TP tiles per pair side):
//   BD[j], BC[j], FLi[o], FXL[o], FXR[o]   TP x TP tiles, tile (r, c) at c*TP + r
//   BEt[j], FGt[o]                         t0 x TP tiles, tile (q, c) at c*t0 + q
// Pair vectors r, w, up: 16 TP values per pair.
#include "bcr_border.h"
#include "common.h"
#include "kernels.h"
#include "tile_chol.h"
#include "tile_ops.h"

namespace ahlp {

namespace {

constexpr int MAXT0 = 4;               // border tiles (n0 <= 64)
constexpr int EW = 8;                  // waves of an eliminating workgroup
constexpr int MID_WAVES = 16;          // waves of the final-pair and border solve kernel
// LDS tiles have leading dimension 17 (one pad value per column), so the
// accumulator-layout and B-operand accesses of a 16-lane row group fall in
// distinct banks.
constexpr int PLD = TS + 1;
constexpr int PT = 16 * PLD;           // values per LDS tile

template <int TP> struct Geo {
  static constexpr int TB = 16 * TP, BLK = TP * TP * 256;
  __device__ static __forceinline__ int bt(int r, int c) { return (c * TP + r) * 256; }
  __device__ static __forceinline__ long long et(long long j, int q, int c, int t0) {
    return ((j * TP + c) * t0 + q) * 256;
  }
};

// a tile in accumulator layout, which is also the layout of the B operand of
// X * Y and of the A operand of X' * Y: element (4 s + lane / 16, lane % 16)
__device__ __forceinline__ Op op_load_b(const double* t) {
  const int lane = threadIdx.x & 63;
  const int idx = (lane & 15) * TS + (lane >> 4);
  Op o;
#pragma unroll
  for (int s = 0; s < 4; ++s) o.v[s] = t[idx + 4 * s];
  return o;
}
// acc + alpha * (product of register operands)
__device__ __forceinline__ d4 mm(d4 acc, const Op& a, const Op& b, double alpha) {
#pragma unroll
  for (int s = 0; s < 4; ++s) acc = mfma(alpha * a.v[s], b.v[s], acc);
  return acc;
}
__device__ __forceinline__ d4 as_acc(const Op& o) { return d4{o.v[0], o.v[1], o.v[2], o.v[3]}; }
__device__ __forceinline__ Op as_op(const d4& a) { return Op{{a[0], a[1], a[2], a[3]}}; }

// Working blocks from the assembled parts, one wave per tile: the diagonal
// (identity on the padding), the coupling T[j+1, j] and the border rows E_j'.
template <int TP>
__global__ __launch_bounds__(256) void k_bcrn_init(BcrArgs c) {
  typedef Geo<TP> G;
  const int per = 2 * TP * TP + TP * c.t0;
  const long long wt = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (wt >= (long long)c.P * per) return;
  const int j = (int)(wt / per), kind = (int)(wt % per), lj = c.l[j];
  if (kind < TP * TP) {
    const int r = kind % TP, cc = kind / TP;
    acc_store(c.BD + (long long)j * G::BLK + G::bt(r, cc),
              acc_load_exact(c.Td + c.tdoff[j] + 16 * r + 16LL * cc * lj, lj - 16 * r,
                             lj - 16 * cc, lj, r == cc));
  } else if (kind < 2 * TP * TP) {
    if (j + 1 < c.P) {
      const int t = kind - TP * TP, r = t % TP, cc = t / TP, ln = c.l[j + 1];
      acc_store(c.BC + (long long)j * G::BLK + G::bt(r, cc),
                acc_load_exact(c.To + c.tooff[j] + 16 * r + 16LL * cc * ln, ln - 16 * r,
                               lj - 16 * cc, ln, false));
    }
  } else {
    const int t = kind - 2 * TP * TP, q = t % c.t0, cc = t / c.t0;
    acc_store(c.BEt + G::et(j, q, cc, c.t0),
              acc_load_exact_t(c.E + c.eoff[j] + 16LL * q * lj + 16 * cc,
                               min(16, c.n0 - 16 * q), lj - 16 * cc, lj));
  }
}

// Eliminates the odd position k = 2 blockIdx.x + 1 of level lvl (n active
// pairs), or with n = 1 the final pair 0 (no neighbours).
template <int TP>
__global__ __launch_bounds__(64 * EW, 2) void k_bcrn_elim(BcrArgs c, int lvl, int n) {
  typedef Geo<TP> G;
  constexpr int NT = TP * (TP + 1) / 2;
  __shared__ double B[NT * PT];    // working diagonal -> L, lower tiles (r, c) at r (r + 1) / 2 + c
  __shared__ double Ld[TP * PT];   // inverted diagonal tiles
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int t0 = c.t0;
  const bool fin = n == 1;
  const int k = fin ? 0 : 2 * blockIdx.x + 1;
  const long long s = 1LL << lvl, o = k * s, L = (k - 1) * s;
  const bool hasR = k + 1 < n;
  auto tl = [](int r, int cc) { return (r * (r + 1) / 2 + cc) * PT; };
  for (int t = wave; t < NT; t += EW) {
    int r = 0;
    while ((r + 1) * (r + 2) / 2 <= t) ++r;
    op_store<PLD>(B + t * PT, op_load(c.BD + o * G::BLK + G::bt(r, t - r * (r + 1) / 2)));
  }
  // column tasks: TP columns of L^-1, TP of X_L, TP of X_R, t0 of Z
  const int ntask = 3 * TP + t0;
  auto load_task = [&](int t, Op* b) {
    const int kind = t / TP, cc = t % TP;
#pragma unroll
    for (int r = 0; r < TP; ++r) {
      b[r] = Op{};
      if (kind == 0) {
        if (r == cc) {
#pragma unroll
          for (int q = 0; q < 4; ++q) b[r].v[q] = (4 * q + (lane >> 4) == (lane & 15)) ? 1.0 : 0.0;
        }
      } else if (kind == 1) {
        if (!fin) b[r] = op_load_b(c.BC + L * G::BLK + G::bt(r, cc));
      } else if (kind == 2) {
        if (hasR) b[r] = op_load(c.BC + o * G::BLK + G::bt(cc, r));   // of the transposed coupling
      } else {
        b[r] = op_load(c.BEt + G::et(o, t - 3 * TP, r, t0));          // of E_o, stored transposed
      }
    }
  };
  auto skipped = [&](int t) { return (t / TP == 1 && fin) || (t / TP == 2 && !hasR); };
  Op b[TP];
  int task = wave;
  if (task < ntask && !skipped(task)) load_task(task, b);
  const double thr = c.thrT[o];
  __syncthreads();
  int cnt = 0;
#pragma unroll
  for (int p = 0; p < TP; ++p) {
    if (wave == 0) cnt += wave_chol_tile<double, PLD>(B + tl(p, p), B + tl(p, p), Ld + p * PT, thr, nullptr);
    if (p + 1 == TP) break;
    __syncthreads();
    if (wave >= 1 && wave < TP - p) {   // rows p + 1 .. TP - 1
      const int r = p + wave;
      const d4 a = mma_xyt<PLD>(acc_zero(), B + tl(r, p), Ld + p * PT, 1.0);
      wave_order();
      acc_store<PLD>(B + tl(r, p), a);
    }
    __syncthreads();
    // trailing tiles; tile (p + 1, p + 1), the next to be factored, by wave 0
    int u = 0;
#pragma unroll
    for (int r = p + 1; r < TP; ++r)
#pragma unroll
      for (int cc = p + 1; cc <= r; ++cc, ++u)
        if (u % EW == wave) {
          const d4 a = mma_xyt<PLD>(acc_load<PLD>(B + tl(r, cc)), B + tl(r, p), B + tl(cc, p), -1.0);
          wave_order();
          acc_store<PLD>(B + tl(r, cc), a);
        }
    // the other tiles are read after the next step's first barrier
    wave_order();
  }
  __syncthreads();
  for (;;) {
    if (task < ntask && !skipped(task)) {
      // x_r = L_rr^-1 (b_r - sum_q L_rq x_q)
      Op x[TP];
#pragma unroll
      for (int r = 0; r < TP; ++r) {
        d4 a = as_acc(b[r]);
#pragma unroll
        for (int q = 0; q < r; ++q) a = mm(a, op_load<PLD>(B + tl(r, q)), x[q], -1.0);
        x[r] = as_op(mm(acc_zero(), op_load<PLD>(Ld + r * PT), as_op(a), 1.0));
      }
      const int kind = task / TP, cc = task % TP;
#pragma unroll
      for (int r = 0; r < TP; ++r) {
        if (kind == 0) acc_store(c.FLi + o * G::BLK + G::bt(r, cc), as_acc(x[r]));
        else if (kind == 1) acc_store(c.FXL + o * G::BLK + G::bt(r, cc), as_acc(x[r]));
        else if (kind == 2) acc_store(c.FXR + o * G::BLK + G::bt(r, cc), as_acc(x[r]));
        else op_store(c.FGt + G::et(o, task - 3 * TP, r, t0), x[r]);   // Z' from Z
      }
    }
    task += EW;
    if (task >= ntask) break;
    if (!skipped(task)) load_task(task, b);
  }
  if (threadIdx.x == 0 && cnt) atomicAdd(&c.info->pivots, cnt);
}

// Updates of the even pairs of a level from their eliminated neighbours, one
// wave per tile: the lower diagonal tiles, the new coupling to the next even
// pair, the border rows.
template <int TP>
__global__ __launch_bounds__(256) void k_bcrn_update(BcrArgs c, int lvl, int n) {
  typedef Geo<TP> G;
  constexpr int ND = TP * (TP + 1) / 2;
  const int t0 = c.t0, per = ND + TP * TP + TP * t0;
  const int wt = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  const int k = 2 * (wt / per), t = wt % per;
  if (k >= n) return;
  const long long s = 1LL << lvl, e = k * s, ol = (k - 1) * s, orr = (k + 1) * s;
  const bool hl = k >= 1, hr = k + 1 < n, hrr = k + 2 < n;
  const double* XRl = c.FXR + ol * G::BLK;
  const double* XLr = c.FXL + orr * G::BLK;
  Op a1[TP], b1[TP], a2[TP], b2[TP];
  if (t < ND) {
    int r = 0;
    while ((r + 1) * (r + 2) / 2 <= t) ++r;
    const int cc = t - r * (r + 1) / 2;
    double* D = c.BD + e * G::BLK + G::bt(r, cc);
    d4 acc = acc_load(D);
#pragma unroll
    for (int p = 0; p < TP; ++p) {
      if (hl) { a1[p] = op_load_b(XRl + G::bt(p, r)); b1[p] = op_load_b(XRl + G::bt(p, cc)); }
      if (hr) { a2[p] = op_load_b(XLr + G::bt(p, r)); b2[p] = op_load_b(XLr + G::bt(p, cc)); }
    }
#pragma unroll
    for (int p = 0; p < TP; ++p) if (hl) acc = mm(acc, a1[p], b1[p], -1.0);
#pragma unroll
    for (int p = 0; p < TP; ++p) if (hr) acc = mm(acc, a2[p], b2[p], -1.0);
    acc_store(D, acc);
  } else if (t < ND + TP * TP) {
    if (!hr || !hrr) return;
    const int r = (t - ND) % TP, cc = (t - ND) / TP;
    const double* XRr = c.FXR + orr * G::BLK;
    d4 acc = acc_zero();
#pragma unroll
    for (int p = 0; p < TP; ++p) { a1[p] = op_load_b(XRr + G::bt(p, r)); b1[p] = op_load_b(XLr + G::bt(p, cc)); }
#pragma unroll
    for (int p = 0; p < TP; ++p) acc = mm(acc, a1[p], b1[p], -1.0);
    acc_store(c.BC + e * G::BLK + G::bt(r, cc), acc);
  } else {
    const int q = (t - ND - TP * TP) % t0, cc = (t - ND - TP * TP) / t0;
    double* Et = c.BEt + G::et(e, q, cc, t0);
    d4 acc = acc_load(Et);
#pragma unroll
    for (int p = 0; p < TP; ++p) {
      if (hl) { a1[p] = op_load(c.FGt + G::et(ol, q, p, t0)); b1[p] = op_load_b(XRl + G::bt(p, cc)); }
      if (hr) { a2[p] = op_load(c.FGt + G::et(orr, q, p, t0)); b2[p] = op_load_b(XLr + G::bt(p, cc)); }
    }
#pragma unroll
    for (int p = 0; p < TP; ++p) if (hl) acc = mm(acc, a1[p], b1[p], -1.0);
#pragma unroll
    for (int p = 0; p < TP; ++p) if (hr) acc = mm(acc, a2[p], b2[p], -1.0);
    acc_store(Et, acc);
  }
}

// ----------------------------------------------------------------- solve
// Forward: w_o = L_o^-1 r_o, r_e -= X_R(o_l)' w_{o_l} + X_L(o_r)' w_{o_r};
// backward: u_o = L_o^-T (w_o - X_L u_L - X_R u_R - Z_o u0).  A workgroup of TP
// waves per pair, wave h for the pair's tile row h; a step's tiles are all
// requested before the first product.

// element 16 h + lane % 16 of pair j's vector at level lvl (level 0: the
// exact right-hand side, zero on the padding)
template <int TP>
__device__ __forceinline__ double rvecn(const BcrSolveArgs& A, int lvl, long long j, int h) {
  const int i = 16 * h + (threadIdx.x & 15);
  if (lvl == 0) return i < A.c.l[j] ? A.s[A.loff[j] + i] : 0.0;
  return A.r[j * (16 * TP) + i];
}
// border partials Z_o' w of the border tiles q = h, h + TP, ... (w in LDS)
template <int TP>
__device__ __forceinline__ void border_partial(const BcrSolveArgs& A, long long o, int h,
                                               const double* w) {
  const BcrArgs& c = A.c;
  const int lane = threadIdx.x & 63;
  for (int q = h; q < c.t0; q += TP) {
    Op g[TP];
#pragma unroll
    for (int p = 0; p < TP; ++p) g[p] = op_load(c.FGt + Geo<TP>::et(o, q, p, c.t0));
    double acc = 0.0;
#pragma unroll
    for (int p = 0; p < TP; ++p) acc += op_mv(g[p], w + 16 * p);
    if (lane < 16) A.pb[(o * c.t0 + q) * 16 + lane] = acc;
  }
}

template <int TP>
__global__ __launch_bounds__(64 * TP) void k_bcrn_fwd(BcrSolveArgs A, int lvl, int n) {
  typedef Geo<TP> G;
  const BcrArgs& c = A.c;
  __shared__ double vl[G::TB], vr[G::TB], wl[G::TB], wr[G::TB];
  const int lane = threadIdx.x & 63;
  const int h = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int k = 2 * blockIdx.x;
  const long long s = 1LL << lvl, e = k * s, ol = (k - 1) * s, orr = (k + 1) * s;
  const bool hl = k >= 1, hr = k + 1 < n;
  double acc = rvecn<TP>(A, lvl, e, h);
  Op ll[TP], lr[TP], xl[TP], xr[TP];
#pragma unroll
  for (int q = 0; q < TP; ++q) {
    if (hl && q <= h) ll[q] = op_load(c.FLi + ol * G::BLK + G::bt(h, q));
    if (hr && q <= h) lr[q] = op_load(c.FLi + orr * G::BLK + G::bt(h, q));
    if (hl) xl[q] = op_load(c.FXR + ol * G::BLK + G::bt(q, h));
    if (hr) xr[q] = op_load(c.FXL + orr * G::BLK + G::bt(q, h));
  }
  if (hl) vec_put(vl + 16 * h, rvecn<TP>(A, lvl, ol, h));
  if (hr) vec_put(vr + 16 * h, rvecn<TP>(A, lvl, orr, h));
  lds_barrier();
  if (hl) {
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < TP; ++q)
      if (q <= h) t += op_mv(ll[q], vl + 16 * q);
    vec_put(wl + 16 * h, t);
  }
  if (hr) {
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < TP; ++q)
      if (q <= h) t += op_mv(lr[q], vr + 16 * q);
    vec_put(wr + 16 * h, t);
    if (lane < 16) A.w[orr * G::TB + 16 * h + lane] = t;
  }
  lds_barrier();
  if (hl)
#pragma unroll
    for (int q = 0; q < TP; ++q) acc -= op_mtv(xl[q], wl + 16 * q, nullptr);
  if (hr) {
#pragma unroll
    for (int q = 0; q < TP; ++q) acc -= op_mtv(xr[q], wr + 16 * q, nullptr);
    border_partial<TP>(A, orr, h, wr);
  }
  if (lane < 16) A.r[e * G::TB + 16 * h + lane] = acc;
}

// u_o from w_o, the neighbours' u (L, R < 0: no such neighbour) and u0 (LDS),
// by waves h = 0 .. TP - 1 (waves beyond only take the barrier); v: 16 TP
// values of LDS
template <int TP>
__device__ __forceinline__ void bwdn_pair(const BcrSolveArgs& A, long long o, long long L,
                                          long long R, const double* u0, double* ua, double* ub,
                                          double* v) {
  typedef Geo<TP> G;
  const BcrArgs& c = A.c;
  const int lane = threadIdx.x & 63;
  const int h = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Op li[TP];
  double t = 0.0;
  if (h < TP) {
    Op xl[TP], xr[TP], g[MAXT0];
#pragma unroll
    for (int q = 0; q < TP; ++q) {
      if (L >= 0) xl[q] = op_load(c.FXL + o * G::BLK + G::bt(h, q));
      if (R >= 0) xr[q] = op_load(c.FXR + o * G::BLK + G::bt(h, q));
      if (q >= h) li[q] = op_load(c.FLi + o * G::BLK + G::bt(q, h));
    }
#pragma unroll
    for (int q = 0; q < MAXT0; ++q)
      if (q < c.t0) g[q] = op_load(c.FGt + G::et(o, q, h, c.t0));
    t = A.w[o * G::TB + 16 * h + (lane & 15)];
    // every wave keeps its own copies of the neighbours' vectors
    double* a = ua + h * G::TB;
    double* b = ub + h * G::TB;
    if (lane < G::TB) {
      if (L >= 0) a[lane] = A.up[L * G::TB + lane];
      if (R >= 0) b[lane] = A.up[R * G::TB + lane];
    }
    wave_order();
#pragma unroll
    for (int q = 0; q < TP; ++q) {
      if (L >= 0) t -= op_mv(xl[q], a + 16 * q);
      if (R >= 0) t -= op_mv(xr[q], b + 16 * q);
    }
#pragma unroll
    for (int q = 0; q < MAXT0; ++q)
      if (q < c.t0) t -= op_mtv(g[q], u0 + 16 * q, nullptr);
    vec_put(v + 16 * h, t);
  }
  lds_barrier();
  if (h < TP) {
    double u = 0.0;
#pragma unroll
    for (int q = 0; q < TP; ++q)
      if (q >= h) u += op_mtv(li[q], v + 16 * q, nullptr);
    if (lane < 16) {
      A.up[o * G::TB + 16 * h + lane] = u;
      if (16 * h + lane < c.l[o]) A.u[A.loff[o] + 16 * h + lane] = u;
    }
  }
}

template <int TP>
__global__ __launch_bounds__(64 * TP) void k_bcrn_bwd(BcrSolveArgs A, int lvl, int n) {
  __shared__ double ua[TP * 16 * TP], ub[TP * 16 * TP], v[16 * TP], u0[16 * MAXT0];
  for (int i = threadIdx.x; i < 16 * A.c.t0; i += blockDim.x) u0[i] = A.u0p[i];
  lds_barrier();
  const int k = 2 * blockIdx.x + 1;
  const long long s = 1LL << lvl;
  bwdn_pair<TP>(A, k * s, (k - 1) * s, k + 1 < n ? (k + 1) * s : -1, u0, ua, ub, v);
}

// The final pair forward (w_0 = L_0^-1 r_0 and its border partial), the
// border solve, the final pair backward.  lvl: the level after the last
// reduction (where pair 0's right-hand side is).
template <int TP>
__global__ __launch_bounds__(64 * MID_WAVES) void k_bcrn_mid(BcrSolveArgs A, int lvl) {
  typedef Geo<TP> G;
  const BcrArgs& c = A.c;
  __shared__ double ua[TP * G::TB], ub[TP * G::TB], vl[G::TB], w[G::TB], sc[16];
  __shared__ double part[64 * MID_WAVES];
  __shared__ double s0[16 * MAXT0], w0[16 * MAXT0], u0[16 * MAXT0];
  const int lane = threadIdx.x & 63;
  const int h = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (h < TP) vec_put(vl + 16 * h, rvecn<TP>(A, lvl, 0, h));
  __syncthreads();
  if (h < TP) {
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < TP; ++q)
      if (q <= h) t += op_mv(op_load(c.FLi + G::bt(h, q)), vl + 16 * q);
    vec_put(w + 16 * h, t);
    if (lane < 16) A.w[16 * h + lane] = t;
  }
  __syncthreads();
  if (h < TP) border_partial<TP>(A, 0, h, w);
  __syncthreads();
  bcr_border_solve(A, c.FLbi, false, part, s0, w0, u0, sc);
  bwdn_pair<TP>(A, 0, -1, -1, u0, ua, ub, vl);
}

template <int TP>
void reduce_tp(hipStream_t st, const BcrArgs& c) {
  const long long tiles = (long long)c.P * (2 * TP * TP + TP * c.t0);
  hipLaunchKernelGGL(k_bcrn_init<TP>, dim3((unsigned)((tiles + 3) / 4)), dim3(256), 0, st, c);
  const int per = TP * (TP + 1) / 2 + TP * TP + TP * c.t0;
  int n = c.P, lvl = 0;
  for (; n > 1; ++lvl, n = (n + 1) / 2) {
    hipLaunchKernelGGL(k_bcrn_elim<TP>, dim3(n / 2), dim3(64 * EW), 0, st, c, lvl, n);
    hipLaunchKernelGGL(k_bcrn_update<TP>, dim3(((n + 1) / 2 * per + 3) / 4), dim3(256), 0, st, c, lvl, n);
  }
  hipLaunchKernelGGL(k_bcrn_elim<TP>, dim3(1), dim3(64 * EW), 0, st, c, 0, 1);
}

template <int TP>
void solve_tp(hipStream_t st, const BcrSolveArgs& a) {
  int n = a.c.P, lvl = 0;
  for (; n > 1; ++lvl, n = (n + 1) / 2)
    hipLaunchKernelGGL(k_bcrn_fwd<TP>, dim3((n + 1) / 2), dim3(64 * TP), 0, st, a, lvl, n);
  hipLaunchKernelGGL(k_bcrn_mid<TP>, dim3(1), dim3(64 * MID_WAVES), 0, st, a, lvl);
  for (int lv = lvl - 1; lv >= 0; --lv) {
    int nl = a.c.P;
    for (int v = 0; v < lv; ++v) nl = (nl + 1) / 2;
    hipLaunchKernelGGL(k_bcrn_bwd<TP>, dim3(nl / 2), dim3(64 * TP), 0, st, a, lv, nl);
  }
}

}  // namespace

void launch_bcrn_reduce(hipStream_t st, const BcrArgs& c) {
  if (c.P <= 0) return;
  if (c.tp == 2) reduce_tp<2>(st, c);
  else if (c.tp == 3) reduce_tp<3>(st, c);
  else reduce_tp<4>(st, c);
}

void launch_bcrn_solve(hipStream_t st, const BcrSolveArgs& a) {
  if (a.c.tp == 2) solve_tp<2>(st, a);
  else if (a.c.tp == 3) solve_tp<3>(st, a);
  else solve_tp<4>(st, a);
}

}  // namespace ahlp
