// Block cyclic reduction of the Schur complement (a6) for link pairs of at
// most 16 rows and at most 64 linking variables (wider pairs: k_bcrn.hip,
// which shares the border kernels below).
//
// The assembled Schur complement is S = [T E; E' S00] with T block
// tridiagonal over the P link pairs (App. A) and E, S00 the x_0 border.  T is
// eliminated by odd-even reduction: at level v the active pairs are
// j = k 2^v (k = 0 .. n_v - 1); the pairs at odd positions k are eliminated
// all at once (each is coupled only to its two active neighbours), which
// updates the even ones and couples neighbouring even pairs; the evens form
// level v + 1.  This is the elimination of Alg. 3 of the Schur solve in a
// symmetric permutation of T that turns its dependent chain of P steps into
// ceil(log2 P) levels of independent steps.  For an eliminated pair o with
// active neighbours L (left) and R (right):
//   T'_oo = L_o L_o',  X_L = L_o^-1 T'_oL,  X_R = L_o^-1 T'_oR,  Z = L_o^-1 E'_o
//   T'_LL -= X_L'X_L,  T'_RR -= X_R'X_R,  T'_RL = -X_R'X_L,
//   E'_L -= X_L'Z,  E'_R -= X_R'Z,  S00 - sum over all pairs of Z'Z.
// The border Schur complement S00 - E'T^-1 E is negative definite (the
// system is quasi-definite) and is factorized as -(S00 - sum Z'Z) = Lb Lb'.
//
// Storage: 16x16 column-major tiles per pair j, padded with the identity.
//   BD[j], BC[j], BEt[j][q]   working diagonal, coupling T'[next active, j]
//                             and border rows (transposed, t0 tiles)
//   FLi[o], FXL[o], FXR[o]    L_o^-1, X_L, X_R of the eliminated pair o
//   FGt[o][q]                 Z' of pair o (t0 tiles), the final pair included
//   FLbi                      inverse of the border factor Lb, tiles (r, c) at c*t0 + r
//
// What a level costs is a chain: the factor of a 16x16 tile (1 us), its products
// and the updates, a few hundred cycles each; a launch or a round of memory per
// level costs more than that.  So a workgroup takes a group of 2^lev neighbouring
// positions into LDS and eliminates all of them but the first (the separator)
// over lev levels: the factors one wave each, then the products and then the
// updates as one tile per wave, while four waves that have no factor sum Z'Z of
// the level before.  A group leaves its separator's updated tiles in BD, BC, BEt
// and a record of what the next stage adds: the sum of its Z'Z (with its child
// groups' sums) and its terms of the next group's separator.  The last stage, one
// group, eliminates its first position too and factorizes the border.  A group's
// tiles must fit in LDS: 16 positions with a border of up to one tile, 8 with up
// to four.
// Measured against a launch per level, a single workgroup for the last 16 pairs
// through memory and three launches for the border, kernel time in us per
// factorization: 7 pairs, border 8: 37 -> 20; 63 pairs, border 22: 93 -> 49; 511
// pairs, border 32: 115 -> 73; 2189 pairs, border 12: 128 -> 83.  A level takes 5000
// to 6000 cycles, 3000 of them the factor; a stage another 5 us for its first round
// of memory and the first fetch of its instructions.
//
// Every sum is taken in a fixed order.  The solve is in k_bcrs.hip.
#include "bcr_plan.h"
#include "common.h"
#include "kernels.h"
#include "tile_chol.h"
#include "tile_ops.h"
#include <algorithm>

namespace ahlp {

namespace {

constexpr int BT_MAXT0 = 4;      // border tiles (n0 <= 64)
constexpr int FW = 8;            // waves of a group's workgroup
constexpr int ZW = 4;            // its last waves, which sum Z'Z
// LDS tiles are column-major with leading dimension 17: accumulator-layout
// writes and B-operand reads walk a tile by columns across the lanes, which
// with 16 would put 16 lanes in one bank
constexpr int PLD = TS + 1, PTE = TS * PLD;
struct T4 { double v[4]; };   // a tile as a matrix operand
// the same operations on padded LDS tiles (element col 16 + row at col 17 + row)
__device__ __forceinline__ int pe(int e) { return e + (e >> 4); }
__device__ __forceinline__ void acc_store_l(double* t, const d4& a) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int r = 0; r < 4; ++r) t[pe(acc_index<double>(lane, r))] = a[r];
}
__device__ __forceinline__ T4 ld_a_l(const double* t) {
  const int lane = threadIdx.x & 63;
  T4 o;
#pragma unroll
  for (int s = 0; s < 4; ++s) o.v[s] = t[pe(64 * s + lane)];
  return o;
}
__device__ __forceinline__ T4 ld_b_l(const double* t) {
  const int lane = threadIdx.x & 63;
  const int idx = (lane & 15) * TS + (lane >> 4);
  T4 o;
#pragma unroll
  for (int s = 0; s < 4; ++s) o.v[s] = t[pe(idx + 4 * s)];
  return o;
}
__device__ __forceinline__ void tile_copy_l(double* __restrict__ dst, const double* src) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int s = 0; s < 4; ++s) dst[64 * s + lane] = src[pe(64 * s + lane)];
}
// acc + alpha * (product with the given operands)
__device__ __forceinline__ d4 mm(d4 acc, const T4& a, const T4& b, double alpha) {
#pragma unroll
  for (int s = 0; s < 4; ++s) acc = mfma(alpha * a.v[s], b.v[s], acc);
  return acc;
}


// ---------------------------------------------------------------- factor
int border_low(int t0) { return t0 * (t0 + 1) / 2; }
// positions of a group with this border
int group_size(int t0) { return t0 <= 1 ? 16 : 8; }
size_t group_smem(int t0) {
  return ((size_t)group_size(t0) * (2 + t0) + (1 + t0) + FW) * PTE * sizeof(double);
}

// Group blockIdx.x of 2^lev positions at level lvl (n positions in all); LAST:
// the only one, down to the final pair and the border.  Records, one per group,
// at c.s00part: Z'Z (lower tiles, row by row), then the terms of the next
// separator's diagonal and border tiles.  slot0: this stage's first, prev: that
// of the stage before.  LAST with n = 0 is the border alone, its record prev
// holding only the sum of Z'Z (if kids).
// Code that runs for the first time costs its size (about a cycle per two bytes),
// so all factors of the kernel, the border's included, are the same instructions:
// the steps are lev levels, then in the last stage the final pair and the border's
// t0 tile columns.
template <int GS, bool LAST>
__global__ __launch_bounds__(64 * FW) void k_bcr_group(BcrArgs c, int lvl, int n, int lev, int slot0, int prev,
                                                     int kids) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ double s_thr[GS + 1];
  touch_args(c.l, c.Td, c.thrT, c.FLi, c.s00part, lvl, kids);
  double* lds = reinterpret_cast<double*>(smem_raw);
  const int t0 = c.t0, per = 2 + t0, nz = t0 * (t0 + 1) / 2, lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int gs = 1 << lev, k0 = LAST ? 0 : (int)blockIdx.x << lev;
  const bool right = !LAST && k0 + gs < n;    // there is a next separator
  const long long rec = (long long)(LAST && n == 0 ? nz : nz + 1 + t0) * 256;
  const int inv = per == 2 ? 32769 : per == 3 ? 21846 : per == 4 ? 16385 : per == 5 ? 13108 : 10923;
  auto div_per = [&](int t) { return (t * inv) >> 16; };   // t / per for t < 2^12
  auto tile = [&](int i, int kind) { return lds + (i * per + kind) * PTE; };   // 0: D, 1: C, 2 + q: E_q
  double* sep = lds + GS * per * PTE;                                          // next separator's D, E_q
  double* scr = sep + (1 + t0) * PTE;                                          // a tile per wave

  // The group's tiles, NT of the waves' turns: where they are by lane (one wait for
  // the offsets), then all of them (one wait), then to LDS.  Element (a, b) at
  // src + a sa + b sb for a < rows, b < cols; more: the separator's terms of the
  // group on its left.
  constexpr int NT = 48 / FW;
  unsigned long long my_src = 0, my_more = 0;
  int my_sa = 1, my_sb = 16, my_rows = 16, my_cols = 16;
  {
    const int t = wave + FW * lane, i = div_per(t), kind = t - i * per, k = k0 + i;
    const double* src = nullptr;
    if (lane < NT && i < gs && k < n && !(kind == 1 && k + 1 >= n)) {
      const long long j = (long long)k << lvl;
      if (lvl == 0) {
        const long long off = (kind == 0 ? c.tdoff : kind == 1 ? c.tooff : c.eoff)[j];
        const PairTile p = pair_tile(kind, c.l[j], kind == 1 ? c.l[j + 1] : 0, c.n0, off);
        src = (kind == 0 ? c.Td : kind == 1 ? c.To : c.E) + p.off;
        my_sa = p.sa; my_sb = p.sb; my_rows = p.rows; my_cols = p.cols;
      } else {
        src = kind == 0 ? c.BD + j * 256 : kind == 1 ? c.BC + j * 256 : c.BEt + (j * t0 + kind - 2) * 256;
        if (k > 0 && kind != 1)
          my_more = (unsigned long long)(c.s00part + (prev + k - 1) * rec + (nz + (kind == 0 ? 0 : kind - 1)) * 256);
      }
    }
    my_src = (unsigned long long)src;
  }
  const auto lane_ptr = [](unsigned long long p, int u) {
    return reinterpret_cast<const double*>(
        (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)p, u) |
        (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(p >> 32), u) << 32);
  };
  double v[NT][4], add[NT][4];
  const int a15 = lane & 15, b15 = lane >> 4;
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    const double* src = lane_ptr(my_src, u);
    if (!src) continue;
    const int sa = __builtin_amdgcn_readlane(my_sa, u), sb = __builtin_amdgcn_readlane(my_sb, u);
    const int rows = __builtin_amdgcn_readlane(my_rows, u), cols = __builtin_amdgcn_readlane(my_cols, u);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int b = 4 * s + b15;
      v[u][s] = src[tile_at(sa, sb, rows, cols, a15, b)];
    }
    const double* more = lane_ptr(my_more, u);
    if (more)
#pragma unroll
      for (int s = 0; s < 4; ++s) add[u][s] = more[64 * s + lane];
  }
  if ((int)threadIdx.x < gs && k0 + (int)threadIdx.x < n)
    s_thr[threadIdx.x] = c.thrT[(long long)(k0 + threadIdx.x) << lvl];
  for (int e = threadIdx.x; e < (1 + t0) * PTE; e += blockDim.x) sep[e] = 0.0;
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    const int t = wave + FW * u;
    if (t >= GS * per || !lane_ptr(my_src, u)) continue;
    const int rows = __builtin_amdgcn_readlane(my_rows, u), cols = __builtin_amdgcn_readlane(my_cols, u);
    const bool diag = t == div_per(t) * per, more = lane_ptr(my_more, u) != nullptr;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int b = 4 * s + b15;
      double x = a15 < rows && b < cols ? v[u][s] : 0.0;
      if (more) x += add[u][s];
      lds[t * PTE + pe(64 * s + lane)] = diag && b == a15 && b >= cols ? 1.0 : x;
    }
  }
  lds_barrier();

  // Z'Z: the last ZW waves share its tiles, or with one tile the pairs
  d4 zz[3] = {acc_zero(), acc_zero(), acc_zero()};
  const int zw = wave - (FW - ZW);
  auto zz_tile = [&](int z) { return nz == 1 ? (z == 0 ? 0 : nz) : zw + ZW * z; };
  // of the positions i0, i0 + step, ..: those eliminated together
  auto zz_level = [&](int i0, int step) {
    if (zw < 0) return;
    int u = 0;
    for (int i = i0; i < gs && k0 + i < n; i += step, ++u) {
      if (nz == 1 && u % ZW != zw) continue;
#pragma unroll
      for (int z = 0; z < 3; ++z) {
        const int t = zz_tile(z);
        if (t >= nz) continue;
        const int q = t >= 6 ? 3 : t >= 3 ? 2 : t >= 1 ? 1 : 0, q2 = t - q * (q + 1) / 2;
        zz[z] = mm(zz[z], ld_a_l(tile(i, 2 + q)), ld_a_l(tile(i, 2 + q2)), 1.0);
      }
    }
  };
  if (zw >= 0) {   // the child groups' sums
    if (lvl > 0) kids = min(n, k0 + gs) - k0;
#pragma unroll
    for (int z = 0; z < 3; ++z) {
      const int t = zz_tile(z);
      if (t >= nz) continue;
#pragma unroll 4
      for (int g = nz == 1 ? zw : 0; g < kids; g += nz == 1 ? ZW : 1)
        zz[z] += acc_load(c.s00part + (prev + k0 + g) * rec + t * 256);
    }
  }
  // their sum over the waves where those shared the pairs: to the first of them
  auto zz_finish = [&]() {
    if (nz != 1) return;
    lds_barrier();
    if (zw >= 0) acc_store_l(scr + wave * PTE, zz[0]);
    lds_barrier();
    if (zw == 0)
      for (int w = 1; w < ZW; ++w)
#pragma unroll
        for (int s = 0; s < 4; ++s) zz[0][s] += scr[(wave + w) * PTE + pe(acc_index<double>(lane, s))];
  };
  auto zz_store = [&](double* dst) {
    if (zw < 0 || (nz == 1 && zw > 0)) return;
#pragma unroll
    for (int z = 0; z < 3; ++z)
      if (zz_tile(z) < nz) acc_store(dst + zz_tile(z) * 256, zz[z]);
  };

  // the border's tiles, over the group's once those are done with: B (r, c) at
  // c t0 + r, its inverse X and the inverted diagonal tiles Ld
  double* B = lds + nz * PTE;
  double* X = B + t0 * t0 * PTE;
  double* Ld = X + t0 * t0 * PTE;
  const unsigned long long neg = LAST ? (c.ng >= 64 ? ~0ull : ((1ull << c.ng) - 1ull)) : 0ull;
  const int fin = LAST && n > 0 ? 1 : 0, first_b = lev + fin, steps = first_b + (LAST ? t0 : 0);
  int cnt = 0;
  for (int v0 = 0; v0 < steps; ++v0) {
    const int p = v0 - first_b;                       // border: the tile column
    const bool border = LAST && p >= 0, last_pair = LAST && v0 == lev && fin;
    const int d = last_pair || border ? gs : 1 << v0, nel = last_pair || border ? 1 : gs / (2 * d);
    if (LAST && p == 0) {
      // all pairs are eliminated: the last one's Z'Z and the border's tiles,
      // B = -(S00 - sum Z'Z), the identity on the padding
      if (fin) zz_level(0, gs);
      zz_finish();
      lds_barrier();
      zz_store(lds);
      lds_barrier();
      const int n0 = c.n0;
      for (int idx = threadIdx.x; idx < 256 * t0 * t0; idx += blockDim.x) {
        const int tl = idx >> 8, e = idx & 255, r1 = tl % t0, c1 = tl / t0;
        const int i = 16 * r1 + (e & 15), j = 16 * c1 + (e >> 4);
        if (r1 < c1) continue;
        double b = (i == j) ? 1.0 : 0.0;
        if (i < n0 && j < n0) b = -(c.S00[i + j * n0] - lds[(r1 * (r1 + 1) / 2 + c1) * 256 + e]);
        B[tl * PTE + pe(e)] = b;
      }
      lds_barrier();
      if (wave == 0) {
        double md = 0.0;
        if (lane < n0) md = fabs(B[((lane >> 4) * t0 + (lane >> 4)) * PTE + (lane & 15) * (PLD + 1)]);
        for (int off = 32; off > 0; off >>= 1) md = fmax(md, __shfl_xor(md, off));
        if (lane == 0) s_thr[GS] = PIVOT_REL * md;
        wave_order();
      }
    }
    auto pos = [&](int w) { return last_pair ? 0 : d * (2 * w + 1); };
    if (wave < nel) {
      const int i = pos(wave);
      if (border || k0 + i < n) {
        double* D = border ? B + (p * t0 + p) * PTE : tile(i, 0);
        double* Li = border ? Ld + p * PTE : scr + wave * PTE;
        const double thr = s_thr[border ? GS : i];
        const unsigned np = border ? (unsigned)((neg >> (16 * p)) & 0xFFFFull) : 0u;
        cnt += wave_chol_tile<double, PLD, LAST, false>(D, nullptr, Li, thr, np);
        if (!border) tile_copy_l(c.FLi + ((long long)(k0 + i) << lvl) * 256, Li);
      }
    } else if (v0 > 0 && !border) {
      zz_level(last_pair ? gs / 2 : d / 2, last_pair ? gs : d);
    }
    lds_barrier();
    if (border) {
      const unsigned np = (unsigned)((neg >> (16 * p)) & 0xFFFFull);
      const int rr = p + 1 + wave;
      if (rr < t0) {   // L_rp = B_rp L_pp^-T S_p
        double* t = B + (p * t0 + rr) * PTE;
        d4 x = mm(acc_zero(), ld_a_l(t), ld_a_l(Ld + p * PTE), 1.0);
        if ((np >> a15) & 1u) x = -x;
        wave_order();
        acc_store_l(t, x);
      }
      lds_barrier();
      int u = 0;
      for (int r1 = p + 1; r1 < t0; ++r1)
        for (int c1 = p + 1; c1 <= r1; ++c1, ++u) {
          if (u % FW != wave) continue;
          double* t = B + (c1 * t0 + r1) * PTE;
          d4 x;
#pragma unroll
          for (int s = 0; s < 4; ++s) x[s] = t[pe(acc_index<double>(lane, s))];
          const T4 l = ld_a_l(B + (p * t0 + r1) * PTE), m = ld_a_l(B + (p * t0 + c1) * PTE);
#pragma unroll
          for (int s = 0; s < 4; ++s)
            x = mfma(((np >> (4 * s + (lane >> 4))) & 1u) ? l.v[s] : -l.v[s], m.v[s], x);
          acc_store_l(t, x);
        }
      lds_barrier();
      continue;
    }
    // X_L to the place of D, X_R to that of the coupling, Z' to that of E'
    for (int t = wave; t < nel * per; t += FW) {
      const int w = div_per(t), kind = t - w * per, i = pos(w);
      if (k0 + i >= n || (kind == 1 && k0 + i + d >= n) || (last_pair && kind < 2)) continue;
      const long long o = (long long)(k0 + i) << lvl;
      const T4 li = ld_a_l(scr + w * PTE);
      T4 x, y;
      double* dst;
      if (kind == 0) {
        x = li;
        y = ld_b_l(tile(i - d, 1));
        dst = c.FXL + o * 256;
      } else if (kind == 1) {
        x = li;
        y = ld_a_l(tile(i, 1));
        dst = c.FXR + o * 256;
      } else {
        x = ld_a_l(tile(i, kind));
        y = li;
        dst = c.FGt + (o * t0 + kind - 2) * 256;
      }
      const d4 z = mm(acc_zero(), x, y, 1.0);
      acc_store_l(tile(i, kind), z);
      acc_store(dst, z);
    }
    lds_barrier();
    if (!last_pair) {
      // the remaining positions, and last the next separator
      const int ne = nel + (right ? 1 : 0);
      for (int t = wave; t < ne * per; t += FW) {
        const int w = div_per(t), kind = t - w * per, i = 2 * d * w;
        const bool next = w == nel;
        if (k0 + i >= n) continue;
        const bool hl = i > 0, hr = !next && k0 + i + d < n;
        double* dst = !next ? tile(i, kind) : sep + (kind == 0 ? 0 : kind - 1) * PTE;
        d4 x = acc_zero();
        if (kind != 1)
#pragma unroll
          for (int s = 0; s < 4; ++s) x[s] = dst[pe(acc_index<double>(lane, s))];
        // kind 0: D - X_R'X_R - X_L'X_L, 1: -X_R'X_L, 2 + q: E'_q - Z'X_R - Z'X_L
        if (hl && kind != 1) {
          const T4 y = ld_b_l(tile(i - d, 1));
          x = mm(x, kind == 0 ? y : ld_a_l(tile(i - d, kind)), y, -1.0);
        }
        if (kind == 1 && !(hr && k0 + i + 2 * d < n)) continue;
        if (hr) {
          const T4 y = ld_b_l(tile(i + d, 0));
          x = mm(x, kind == 0 ? y : kind == 1 ? ld_b_l(tile(i + d, 1)) : ld_a_l(tile(i + d, kind)), y, -1.0);
        }
        acc_store_l(dst, x);
      }
      lds_barrier();
    }
  }
  if (lane == 0 && cnt) atomicAdd(&c.info->pivots, cnt);
  if constexpr (!LAST) {
    zz_level(gs / 2, gs);
    zz_finish();
    double* R = c.s00part + (slot0 + blockIdx.x) * rec;
    zz_store(R);
    const long long j = (long long)k0 << lvl;
    for (int t = wave; t < per; t += FW) {
      if (t == 1 && !right) continue;
      tile_copy_l(t == 0 ? c.BD + j * 256 : t == 1 ? c.BC + j * 256 : c.BEt + (j * t0 + t - 2) * 256, tile(0, t));
    }
    if (right)
      for (int t = wave; t < 1 + t0; t += FW) tile_copy_l(R + (nz + t) * 256, sep + t * PTE);
  } else if (wave < t0) {
    // the inverse of the border's factor, a tile column a wave
    const int cc = wave;
    for (int r1 = 0; r1 < t0; ++r1) {
      double* x = X + (cc * t0 + r1) * PTE;
      if (r1 > cc) {
        d4 a = acc_zero();
        for (int q = cc; q < r1; ++q)
          a = mm(a, ld_a_l(B + (q * t0 + r1) * PTE), ld_b_l(q == cc ? Ld + cc * PTE : X + (cc * t0 + q) * PTE), 1.0);
        acc_store_l(scr + wave * PTE, a);
        wave_order();
        const d4 y = mm(acc_zero(), ld_a_l(Ld + r1 * PTE), ld_b_l(scr + wave * PTE), -1.0);
        wave_order();
        acc_store_l(x, y);
        wave_order();
      }
      double* dst = c.FLbi + (cc * t0 + r1) * 256;
      if (r1 >= cc) tile_copy_l(dst, r1 == cc ? Ld + cc * PTE : x);
      else
#pragma unroll
        for (int s = 0; s < 4; ++s) dst[64 * s + lane] = 0.0;
    }
  }
}

// Partial sums of Z_j'Z_j = FGt_j FGt_j' (lower tiles) over contiguous chunks of
// pairs, one wave per (chunk, border tile (q, q2)), for pairs of several tiles.
// Pair j's tile (q, c) of FGt is at (j tp + c) t0 + q, so u = j tp + c runs over a
// chunk's tiles in order.
__global__ __launch_bounds__(64) void k_bcr_s00_partial(BcrArgs c, int chunk) {
  const int t0 = c.t0, nz = t0 * (t0 + 1) / 2;
  const int part = blockIdx.x / nz, t = blockIdx.x % nz;
  const int q = t >= 6 ? 3 : t >= 3 ? 2 : t >= 1 ? 1 : 0, q2 = t - q * (q + 1) / 2;
  const long long u0 = (long long)part * chunk * c.tp;
  const long long u1 = (long long)min(c.P, (part + 1) * chunk) * c.tp;
  const double* __restrict__ G = c.FGt;
  d4 acc = acc_zero();
#pragma unroll 4
  for (long long u = u0; u < u1; ++u)
    acc = mma_xyt(acc, G + (u * t0 + q) * 256, G + (u * t0 + q2) * 256, 1.0);
  acc_store(c.s00part + ((long long)part * nz + t) * 256, acc);
}

// Sum of the chunk partials, one thread per element, chunks in order; the
// sum goes after the nparts partials.
__global__ __launch_bounds__(256) void k_bcr_s00_sum(BcrArgs c, int nparts) {
  const int n = c.t0 * (c.t0 + 1) / 2 * 256;
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n) return;
  const double* src = c.s00part + idx;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  int pp = 0;
#pragma unroll 4
  for (; pp + 4 <= nparts; pp += 4)
    for (int u = 0; u < 4; ++u) acc[u] += src[(long long)(pp + u) * n];
  for (; pp < nparts; ++pp) acc[0] += src[(long long)pp * n];
  c.s00part[(long long)nparts * n + idx] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// The stages of P pairs: as few as the groups allow, the levels before the last
// split evenly, the fewer first, where there are most groups to fill the chip.
struct Stages { int count, lvl[32], n[32], lev[32], slot[33]; };   // the last stage at index count
Stages make_stages(int P, int t0) {
  Stages s{};
  int most = 0, total = 0, lvl = 0, n = P;
  while ((1 << most) < group_size(t0)) ++most;
  while ((1 << total) < P) ++total;
  const int before = std::max(0, total - most);
  s.count = (before + most - 1) / most;
  for (int v = 0; v < s.count; ++v) {
    s.lvl[v] = lvl;
    s.n[v] = n;
    s.lev[v] = (before - lvl) / (s.count - v);
    n = (n + (1 << s.lev[v]) - 1) >> s.lev[v];
    s.slot[v + 1] = s.slot[v] + n;
    lvl += s.lev[v];
  }
  s.lvl[s.count] = lvl;
  s.n[s.count] = n;
  s.lev[s.count] = total - lvl;
  return s;
}

template <int GS>
void reduce_groups(hipStream_t st, const BcrArgs& c) {
  const Stages s = make_stages(c.P, c.t0);
  const size_t smem = group_smem(c.t0);
  for (int v = 0; v < s.count; ++v)
    hipLaunchKernelGGL((k_bcr_group<GS, false>), dim3(s.slot[v + 1] - s.slot[v]), dim3(64 * FW), smem, st, c,
                       s.lvl[v], s.n[v], s.lev[v], s.slot[v], v ? s.slot[v - 1] : 0, 0);
  const int v = s.count;
  hipLaunchKernelGGL((k_bcr_group<GS, true>), dim3(1), dim3(64 * FW), smem, st, c, s.lvl[v], s.n[v], s.lev[v],
                     0, v ? s.slot[v - 1] : 0, 0);
}

}  // namespace

int bcr_tiles(int lmax, int n0) {
  if (n0 > 16 * BT_MAXT0) return 0;
  return lmax <= 16 ? 1 : (lmax + 15) / 16;
}

long long bcr_part_doubles(int P, int t0, int tp, int nparts) {
  if (tp >= 2) return (long long)(nparts + 1) * std::max(border_low(t0), 1) * 256;
  const Stages s = make_stages(P, t0);
  return (long long)std::max(s.slot[s.count], 1) * (border_low(t0) + 1 + t0) * 256;
}

void launch_bcr_factor(hipStream_t st, const BcrArgs& c, int nparts, int chunk) {
  if (c.tp < 2) {
    if (group_size(c.t0) == 16) reduce_groups<16>(st, c);
    else reduce_groups<8>(st, c);
    return;
  }
  launch_bcrn_reduce(st, c);
  if (c.n0 > 0) {
    if (nparts > 0) {
      const int nz = border_low(c.t0);
      hipLaunchKernelGGL(k_bcr_s00_partial, dim3(nparts * nz), dim3(64), 0, st, c, chunk);
      hipLaunchKernelGGL(k_bcr_s00_sum, dim3(nz), dim3(256), 0, st, c, nparts);
    }
    // (the tiles' layout of a group of 8 holds any border)
    hipLaunchKernelGGL((k_bcr_group<8, true>), dim3(1), dim3(64 * FW), group_smem(BT_MAXT0), st, c, 0, 0, 0, 0,
                       nparts, nparts > 0 ? 1 : 0);
  }
}

void set_bcr_smem_limits() {
  const auto set = [](const void* f, size_t bytes) {
    hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  };
  set((const void*)k_bcr_group<16, false>, group_smem(1));
  set((const void*)k_bcr_group<16, true>, group_smem(1));
  set((const void*)k_bcr_group<8, false>, group_smem(BT_MAXT0));
  set((const void*)k_bcr_group<8, true>, group_smem(BT_MAXT0));
}

}  // namespace ahlp
