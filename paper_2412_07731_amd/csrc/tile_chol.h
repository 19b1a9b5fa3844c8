// Cholesky factor and its inverse for one 16x16 tile, computed by one wave.
//
// Column elimination without pivoting of the stacked [P; I], P = L_u D L_u': the
// upper part becomes U' = L_u D, the lower one L_u^-T.  Scaling column j by
// 1/sqrt(d_j) gives L and L^-T of the Cholesky factor P = L L'.  A pivot
// d_j <= thr is replaced by a huge value (the pivot rule) and counted.
//
// The 16 pivots are a chain, and what bounds it is the instructions a wave issues
// per pivot.  So the columns go in panels of four: the panel's four columns are
// copied to every 16-lane row (lane % 16 = the tile's row), where a pivot costs a
// row broadcast, its reciprocal, a product and the few columns right of it in the
// panel; the columns right of the panel follow by one 16x16x4 product for each of
// the two parts.  P is symmetric, so its multipliers m_j = u_j / d_j and its
// columns u_j are both operands, and the lower part takes the same multipliers.
// An accumulator lane holds elements (acc_row, lane % 16) of a part's transpose:
// of P the same element by symmetry, of the lower part those of L^-1 itself.
// One wave, tile in LDS: 3090 cycles (2920 without L) against 4280 of a step for
// every pivot over the whole tile, as the FP32 tile is (below).
#pragma once

#include "common.h"

namespace ahlp {

__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// workgroup barrier that orders LDS accesses only: the waves' global stores
// stay in flight across it
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// value of lane J of each 16-lane row, in every lane of that row
// (row_newbcast writes every lane, so the move needs no old value; it is the
// one DPP control with a 64-bit move, one instruction for a double)
template <int J>
__device__ __forceinline__ double row_bcast(double v) {
  const long long x = __builtin_bit_cast(long long, v);
  const long long y = __builtin_amdgcn_mov_dpp(x, 0x150 + J, 0xF, 0xF, false);
  return __builtin_bit_cast(double, y);
}
template <int J>
__device__ __forceinline__ float row_bcast(float v) {
  union { float f; int i; } u, o;
  u.f = v;
  o.i = __builtin_amdgcn_mov_dpp(u.i, 0x150 + J, 0xF, 0xF, false);
  return o.f;
}

// The four row groups of v (lanes 16K..16K+15), each in every row group: lane l of
// out[K] is v of lane 16K + l%16.  Swaps on the VALU (permlane16 pairs rows 0/1
// and 2/3, permlane32 the half waves), no permute through the LDS pipe.
__device__ __forceinline__ void rowgroups_u32(unsigned v, unsigned (&out)[4]) {
  const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);   // [r0 r0 r2 r2], [r1 r1 r3 r3]
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const auto b = __builtin_amdgcn_permlane32_swap(a[h], a[h], false, false);
    out[h] = b[0];
    out[2 + h] = b[1];
  }
}
// Columns 4 B .. 4 B + 3 of an accumulator tile's transpose: lane l of p[j] is
// element (4 B + j, l % 16) of the tile.
template <int B>
__device__ __forceinline__ void panel_columns(const d4& a, double (&p)[4]) {
  union { double d; unsigned i[2]; } u;
  u.d = a[B];
  unsigned lo[4], hi[4];
  rowgroups_u32(u.i[0], lo);
  rowgroups_u32(u.i[1], hi);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    u.i[0] = lo[j];
    u.i[1] = hi[j];
    p[j] = u.d;
  }
}

// -a / p for the multipliers, with q = -a r for the reciprocal estimate r of p: its
// error e = 1 - p r taken out as r (1 + e + e^2), which leaves e^3.
__device__ __forceinline__ double div_by(double q, double p, double r) {
  const double e = fma(-p, r, 1.0);
  return fma(q, fma(e, e, e), q);
}
// 1 / sqrt(p): the estimate y corrected by its error, y (1 + e / 2 + 3 e^2 / 8) for
// e = 1 - p y^2
__device__ __forceinline__ double rsqrt_of(double p) {
  const double y = __builtin_amdgcn_rsq(p);
  const double e = fma(-p * y, y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}

// What lane (i, g) keeps of a panel's pivots j: the entries with j = g of u (the
// columns of P), x (of the lower part), m (the multipliers) and d (the pivots).
struct PanelSel { double u, x, m, d; };

// Pivot J of panel J / 4: p, x its columns of the two parts (lane % 16 = row i).
// Rows down to J get multipliers too: what they change is not read again (the
// finished rows of P, and rows of L^-1 that are out).  RULE: with the pivot rule;
// SG: signed (quasi-definite) form, where column J's pivot must have the sign of
// its bit in neg (set: negative), the rule then applying to the pivot times that
// sign.
template <int J, bool SG, bool RULE>
__device__ __forceinline__ void chol_pivot(double (&p)[4], double (&x)[4], PanelSel& k, int g, double thr,
                                           unsigned neg) {
  constexpr int j = J & 3;
  const double d = row_bcast<J>(p[j]);
  const double r = __builtin_amdgcn_rcp(d);
  double m = div_by(-p[j] * r, d, r);
  if constexpr (RULE) {
    const double tj = SG && ((neg >> J) & 1u) ? -1.0 : 1.0;
    if (!((SG ? tj * d : d) > thr)) m = -p[j] * (tj * (1 / PIVOT_BIG));
  }
#pragma unroll
  for (int c = j + 1; c < 4; ++c) p[c] = fma(m, row_bcast<J>(p[c]), p[c]);
  if constexpr (j < 3) x[j + 1] = fma(x[j], row_bcast<J + 1>(m), x[j + 1]);
  if constexpr (j < 2) x[j + 2] = fma(x[j], row_bcast<(j < 2 ? J + 2 : J)>(m), x[j + 2]);
  if constexpr (j < 1) x[j + 3] = fma(x[j], row_bcast<(j < 1 ? J + 3 : J)>(m), x[j + 3]);
  const bool mine = j == 0 || g == j;
  k.u = mine ? p[j] : k.u;
  k.x = mine ? x[j] : k.x;
  k.m = mine ? m : k.m;
  k.d = mine ? d : k.d;
}

// Panel B of the tile in s, with e the transpose of the lower part.  Writes the
// panel's rows of L^-1 to Li and, if WL, leaves its columns of L in l (lane (i, g):
// element (i, 4 B + g)).
template <int B, int LD, bool SG, bool WL, bool RULE>
__device__ __forceinline__ void chol_panel(d4& s, d4& e, double* Li, double (&l)[4], int i, int g, double thr,
                                           int& cnt, unsigned neg) {
  double p[4], x[4];
  PanelSel k;
  panel_columns<B>(s, p);
  if constexpr (B == 0) {
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] = i == j ? 1.0 : 0.0;
  } else {
    panel_columns<B>(e, x);
  }
  chol_pivot<4 * B, SG, RULE>(p, x, k, g, thr, neg);
  chol_pivot<4 * B + 1, SG, RULE>(p, x, k, g, thr, neg);
  chol_pivot<4 * B + 2, SG, RULE>(p, x, k, g, thr, neg);
  chol_pivot<4 * B + 3, SG, RULE>(p, x, k, g, thr, neg);
  if constexpr (B < 3) {
    s = mfma(k.m, k.u, s);
    e = mfma(k.m, k.x, e);
  }
  // the pivot of this row group's column by the rule
  const int c = 4 * B + g;
  const bool minus = SG && ((neg >> c) & 1u);
  const double d = minus ? -k.d : k.d;
  const bool bad = !(d > thr);
  cnt += __builtin_popcountll(__ballot(bad) & 0x0001000100010001ull);
  const double sc = rsqrt_of(RULE && bad ? PIVOT_BIG : d);
  Li[i * LD + c] = k.x * sc;
  if constexpr (WL) l[B] = i >= c ? k.u * (minus ? -sc : sc) : 0.0;   // SG: times the column's sign
}

template <int LD, bool SG, bool WL, bool RULE>
__device__ __forceinline__ int chol_panels(const double* P, double* Li, double (&l)[4], double thr, unsigned neg) {
  const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
  d4 s, e;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int c = acc_row<double>(lane, r);
    s[r] = P[c * LD + i];
    e[r] = c == i ? 1.0 : 0.0;
  }
  int cnt = 0;
  chol_panel<0, LD, SG, WL, RULE>(s, e, Li, l, i, g, thr, cnt, neg);
  chol_panel<1, LD, SG, WL, RULE>(s, e, Li, l, i, g, thr, cnt, neg);
  chol_panel<2, LD, SG, WL, RULE>(s, e, Li, l, i, g, thr, cnt, neg);
  chol_panel<3, LD, SG, WL, RULE>(s, e, Li, l, i, g, thr, cnt, neg);
  return cnt;
}

// The FP32 tile: a step for every pivot over the whole tile, the two parts in one
// 16x16 array C (U = D L_u' on and above the diagonal, L_u^-1 below it: step j
// zeroes column j of U exactly where the other part gets its first nonzero there).
// Lane l holds row i = l%16, columns 4g..4g+3 (g = l/16); row j reaches its lanes by
// a row broadcast, the multiplier of row i from lane (i, j/4) by two cross-row
// swaps.  Refinement on FP32 factors may end where the factors' rounding lets it, so
// FP32 keeps this order of operations; a replaced pivot is infinite, 1 / inf = 0.
template <int K>
__device__ __forceinline__ float rowgroup_bcast(float v) {
  unsigned o[4];
  rowgroups_u32(__builtin_bit_cast(unsigned, v), o);
  return __builtin_bit_cast(float, o[K]);
}
__device__ __forceinline__ float lane_bcast(float v, int src) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), src));
}
template <int J>
__device__ __forceinline__ void chol_steps_f32(float (&a)[4], int i, int g, double thr, int& cnt, float& mypiv) {
  if constexpr (J < 16) {
    float p = lane_bcast(a[J & 3], J + 16 * (J >> 2));
    if (!((double)p > thr)) {
      p = (float)PIVOT_BIG;
      ++cnt;
    }
    const float rp = 1.0f / p;
    if (i == J) mypiv = p;
    // a_iJ from lane (i, J/4); row J from lane J of this lane's 16-lane row
    const float aij = rowgroup_bcast<J / 4>(a[J & 3]);
    float rj[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) rj[r] = row_bcast<J>(a[r]);
    const float m = (i > J) ? aij * rp : 0.0f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float u = a[r] - m * rj[r];
      // column J of a row below the pivot: 0 - m * 1
      a[r] = (r == (J & 3) && g == (J >> 2) && i > J) ? 0.0f - m : u;
    }
    chol_steps_f32<J + 1>(a, i, g, thr, cnt, mypiv);
  }
}
template <int LD>
__device__ __forceinline__ int chol_tile_f32(const float* P, float* L, float* Li, double thr) {
  const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
  float a[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) a[r] = P[(4 * g + r) * LD + i];
  int cnt = 0;
  float mypiv = 1.0f;
  chol_steps_f32<0>(a, i, g, thr, cnt, mypiv);
  const float s = 1.0f / (float)sqrt((double)mypiv);
  wave_order();   // every lane has read P before L (which may alias it) is written
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int c = 4 * g + r;
    const float e = c < i ? a[r] : (c == i ? 1.0f : 0.0f);
    L[i * LD + c] = (c >= i) ? a[r] * s : 0.0f;
    Li[c * LD + i] = e * s;
  }
  wave_order();
  return cnt;
}

// P: input tile (column-major with leading dimension LD, LDS or global, both
// triangles).  Li receives the inverse of the lower factor and, if WL, L (may
// alias P) the factor itself, upper parts zero, both column-major with leading
// dimension LD.  Returns the number of replaced pivots (all lanes).  SG: the
// signed factorization of a quasi-definite tile, P = L S L' with S = diag(-1
// where neg has the column's bit, +1 elsewhere); with D the elimination's
// pivots, L = L1 |D|^(1/2).
// The rule costs a pivot five instructions on the chain and is seldom applied, so
// an FP64 tile is factorized without it first, and again with it if any pivot falls
// under it (ONCE: with it at once, half the code, for kernels whose registers the
// two don't fit: the panels of six tiles a wave, 240 against 218 us, and of two).
template <typename T, int LD = TS, bool SG = false, bool WL = true, bool ONCE = false>
__device__ __forceinline__ int wave_chol_tile(const T* P, T* L, T* Li, double thr, unsigned neg = 0) {
  const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
  if constexpr (sizeof(T) == 4) {
    static_assert(!SG, "FP32 has no signed form");
    return chol_tile_f32<LD>(P, L, Li, thr);
  } else {
    double l[4];
    int cnt = ONCE ? 1 : chol_panels<LD, SG, WL, false>(P, Li, l, thr, neg);
    if (cnt) cnt = chol_panels<LD, SG, WL, true>(P, Li, l, thr, neg);   // the same in all lanes
    wave_order();   // every lane has read P before L (which may alias it) is written
    if constexpr (WL)
#pragma unroll
      for (int r = 0; r < 4; ++r) L[(4 * r + g) * LD + i] = l[r];
    wave_order();
    return cnt;
  }
}

}  // namespace ahlp
