// The link columns B_i' (a1): the rows of the bordered blocks below M_i, and
// F_i D_i F_i'.  A launch of their own (k_link), or workgroups among those of a
// small dense SYRK, which writes other tiles.
#pragma once
#include "common.h"
#include "kernels.h"

namespace ahlp {

// One workgroup per (block, tile row of the link columns).  Writes B_i' =
// [F_i D_i A_i' ; C_i'] into the bordered rows and F_i D_i F_i' (FP64) into the
// Schur-contribution tiles, F_i being block i's part of its two link pairs
// and of the global rows.  These rows are sparse (compressed rows, sorted
// columns), so the products are gathers rather than GEMMs.
// Tile row rr of block b's link columns, by 256 threads (t = 0..255).
template <typename T>
__device__ __forceinline__ void link_tile_row(const BlockInfo& b, int rr, int t, int nb,
                                              const double* __restrict__ A,
                                              const double* __restrict__ C,
                                              const int* __restrict__ lptr,
                                              const int* __restrict__ lcol,
                                              const double* __restrict__ lval,
                                              const double* __restrict__ Dp,
                                              T* __restrict__ LB, double* __restrict__ PQ) {
  const int r = b.mt + rr;
  const int ql = t & 15, al = t >> 4;
  const int q = TS * rr + ql;
  int qi;
  bool real;
  const int sec = link_section(b, q, &qi, nb, &real);
  const bool is_row = link_is_row(b, sec, qi);
  int p0 = 0, p1 = 0;
  if (real && is_row) {
    p0 = lptr[b.csr_off + q];
    p1 = lptr[b.csr_off + q + 1];
  }
  // LINK_CB column tiles at a time, their gathers independent so that they
  // are all in flight together; the sparse row is walked once per chunk
  constexpr int LINK_CB = 8;
  for (int c0 = 0; c0 < b.mt; c0 += LINK_CB) {
    double v[LINK_CB];
#pragma unroll
    for (int u = 0; u < LINK_CB; ++u) v[u] = 0.0;
    if (real && is_row) {
      for (int e = p0; e < p1; ++e) {
        const int j = lcol[e];
        const double coef = lval[e] * Dp[b.dpoff + j];
        const double* col = A + a_tile(b, 0, j >> 4) + (j & 15) * TS + al;
#pragma unroll
        for (int u = 0; u < LINK_CB; ++u) {
          const int c = c0 + u;
          if (c < b.mt && TS * c + al < b.m) v[u] += coef * col[(long long)c * b.nt * TE];
        }
      }
    } else if (real) {
      const int qc = qi - b.ng;   // column of C_i
      const double* col = C + c_tile(b, 0, qc >> 4) + (qc & 15) * TS + al;
#pragma unroll
      for (int u = 0; u < LINK_CB; ++u) {
        const int c = c0 + u;
        if (c < b.mt && TS * c + al < b.m) v[u] = col[(long long)c * b.kc0 * TE];
      }
    }
#pragma unroll
    for (int u = 0; u < LINK_CB; ++u)
      if (c0 + u < b.mt) LB[lb_tile(b, r, c0 + u) + t] = (T)v[u];
  }
  // F D F' for tiles (rr, cc), cc <= rr
  for (int cc = 0; cc <= rr; ++cc) {
    const int q2 = TS * cc + al;
    int qi2;
    bool real2;
    const int sec2 = link_section(b, q2, &qi2, nb, &real2);
    double v = 0.0;
    if (real && real2 && is_row && link_is_row(b, sec2, qi2)) {
      int e1 = p0, e2 = lptr[b.csr_off + q2];
      const int e2end = lptr[b.csr_off + q2 + 1];
      while (e1 < p1 && e2 < e2end) {
        const int j1 = lcol[e1], j2 = lcol[e2];
        if (j1 == j2) {
          v += lval[e1] * Dp[b.dpoff + j1] * lval[e2];
          ++e1; ++e2;
        } else if (j1 < j2) {
          ++e1;
        } else {
          ++e2;
        }
      }
    }
    PQ[pq_tile(b, rr, cc) + t] = v;
  }
}

// Units of eight workgroups, a multiple of the XCDs, so that the SYRK's keep
// theirs: every lc.every-th of the launch is the link columns', lc.units in
// all.  Returns the SYRK's workgroup, or ~ that of the link columns.
__device__ __forceinline__ int link_split(int w, const LinkCols& lc) {
  const int u = w >> 3, k = u / lc.every;
  if (k < lc.units && u % lc.every == lc.every - 1) return ~(8 * k + (w & 7));
  return 8 * (u - min(k, lc.units)) + (w & 7);
}

// item w of the link columns, by 256 threads
template <typename T>
__device__ __forceinline__ void link_cols(const BlockInfo* __restrict__ blk, const LinkCols& lc, int w,
                                          int t, const double* __restrict__ Dp, T* __restrict__ LB) {
  if (w >= lc.n) return;
  const int2 it = lc.items[w];
  link_tile_row<T>(blk[it.x], it.y, t, lc.nb, lc.A, lc.C, lc.lptr, lc.lcol, lc.lval, Dp, LB, lc.PQ);
}

// Workgroups of a launch with nitems of the SYRK's and lc's link columns; sets
// lc.units and lc.every.
inline int link_grid(int nitems, LinkCols& lc) {
  const int su = (nitems + 7) / 8;
  lc.units = (lc.n + 7) / 8;
  lc.every = lc.units > 0 ? (su + lc.units) / lc.units : su + 1;
  return 8 * (su + lc.units);
}

}  // namespace ahlp
