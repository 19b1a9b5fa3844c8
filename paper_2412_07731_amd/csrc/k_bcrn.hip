// Block cyclic reduction of the Schur complement (a6) for link pairs of 17 to
// 64 rows: the odd-even reduction of the one-tile kernels (k_bcr.hip) with
// every pair padded to TP x TP tiles (TP = 2, 3 or 4, the widest pair's).  The
// elimination of a pair o with active neighbours L and R is the same,
//   T'_oo = L_o L_o',  X_L = L_o^-1 T'_oL,  X_R = L_o^-1 T'_oR,  Z = L_o^-1 E'_o,
//   T'_LL -= X_L'X_L,  T'_RR -= X_R'X_R,  T'_RL = -X_R'X_L,
//   E'_L -= X_L'Z,  E'_R -= X_R'Z.
// A level is two launches.  In the first a workgroup eliminates one odd pair:
// one wave after another factors the TP diagonal tiles (the chain, 1.3 us
// a tile), all waves share the tile column below and the trailing update; then
// every wave takes whole columns of L_o^-1 [I, T'_oL, T'_oR, E'_o] by forward
// substitution in registers (an FP64 accumulator tile is laid out as the next
// product's B operand, so a column never leaves them).  The second updates the
// even pairs, one wave per tile.  A column's operands are requested before the
// factorization, so the step waits on memory once.  What bounds a level is
// the chain of TP tile factorizations and the two launches; the arithmetic of
// a whole reduction is below a MFMA-microsecond.
// Measured against what it replaced.  511 pairs of 4-32 rows, border 64, one
// wave per elimination and one launch per level: level 20.0 -> 10.2 + 7.8 us.
// 95 pairs of 33-56 rows, border 24, a segmented chain of scalar eliminations:
// factor 8.4 -> 0.28 ms.
#include "bcr_geo.h"
#include "common.h"
#include "kernels.h"
#include "tile_chol.h"
#include "tile_ops.h"

namespace ahlp {

namespace {

constexpr int MAXT0 = 4;               // border tiles (n0 <= 64)
constexpr int EW = 8;                  // waves of an eliminating workgroup
// LDS tiles have leading dimension 17 (one pad value per column), so the
// accumulator-layout and B-operand accesses of a 16-lane row group fall in
// distinct banks.
constexpr int PLD = TS + 1;
constexpr int PT = 16 * PLD;           // values per LDS tile

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
    if (wave == 0) cnt += wave_chol_tile<double, PLD, false, false>(B + tl(p, p), nullptr, Ld + p * PT, thr);
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

}  // namespace

void launch_bcrn_reduce(hipStream_t st, const BcrArgs& c) {
  if (c.P <= 0) return;
  if (c.tp == 2) reduce_tp<2>(st, c);
  else if (c.tp == 3) reduce_tp<3>(st, c);
  else reduce_tp<4>(st, c);
}

}  // namespace ahlp
