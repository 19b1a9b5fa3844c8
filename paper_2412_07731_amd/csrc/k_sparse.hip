// Sparse passes over the constraint blocks (a7/a8): products with [A_i | C_i]
// and its transpose that read only the nonzeros.
//
// The blocks of a time-block LP are handed over dense but mostly hold zeros
// (10% nonzeros in the benchmark shape, fewer in real models).  A pass over
// the dense tiles is bound by HBM (537 MB for 512 blocks of 256 x 512: 83 us at
// 6.4 TB/s), so where it is shorter the passes read a compressed copy instead,
// built on the device once at create: for every tile row (16 rows of [A_i |
// C_i]) and every tile column (16 columns) the nonzeros of its 16 lines in
// groups of 64, lane l of a group holding element l / 16 of line l % 16's next
// four, so that a wave reads a group as one 512-byte and one 128-byte access
// (FP64 value, 16-bit index).  Lines are padded to the longest of their 16.  The
// block's part of the vector is staged in LDS, where the gathers are free of
// the caches' line granularity, and the next chunk of a slice is requested
// while one is summed.  512 blocks of 256 x 512 at 10% nonzeros: row pass 83 ->
// 19 us (one vector), 126 -> 24 us (three); column pass with C_i 104 -> 29 us.
// sparse_setup in the host driver states when the copy is used.
#include "common.h"
#include "kernels.h"
#include "link_rows.h"

namespace ahlp {

namespace {

// Nonzeros of 16 lines (one thread each) into the slice's groups, in
// ascending order; the rest of the groups is zero.
struct SpPut {
  double* val;
  unsigned short* idx;
  long long base;
  int line, q;
  __device__ __forceinline__ void put(double v, int i) {
    const long long at = (base + (q >> 2)) * 64 + (q & 3) * 16 + line;
    val[at] = v;
    idx[at] = (unsigned short)i;
    ++q;
  }
};

__global__ __launch_bounds__(256) void k_sp_fill_rows(const BlockInfo* __restrict__ blk,
                                                      const int2* __restrict__ rowtiles, int nrt,
                                                      const double* __restrict__ A,
                                                      const double* __restrict__ C,
                                                      const long long* __restrict__ off,
                                                      double* __restrict__ val,
                                                      unsigned short* __restrict__ idx) {
  const int t = blockIdx.x * 16 + (threadIdx.x >> 4), r = threadIdx.x & 15;
  if (t >= nrt) return;
  const int2 rt = rowtiles[t];
  const BlockInfo b = blk[rt.x];
  SpPut p{val, idx, off[t], r, 0};
  for (int c = 0; c < TS * b.nt; ++c) {
    const double v = A[a_tile(b, rt.y, c >> 4) + (c & 15) * TS + r];
    if (v != 0.0) p.put(v, c);
  }
  for (int c = 0; c < TS * b.kc0; ++c) {
    const double v = C[c_tile(b, rt.y, c >> 4) + (c & 15) * TS + r];
    if (v != 0.0) p.put(v, TS * b.nt + c);
  }
  while (p.q < 4 * (int)(off[t + 1] - off[t])) p.put(0.0, 0);
}

__global__ __launch_bounds__(256) void k_sp_fill_cols(const BlockInfo* __restrict__ blk,
                                                      const int2* __restrict__ coltiles, int nct,
                                                      const double* __restrict__ A,
                                                      const double* __restrict__ C,
                                                      const long long* __restrict__ off,
                                                      double* __restrict__ val,
                                                      unsigned short* __restrict__ idx) {
  const int t = blockIdx.x * 16 + (threadIdx.x >> 4), c = threadIdx.x & 15;
  if (t >= nct) return;
  const int2 ct = coltiles[t];
  const BlockInfo b = blk[ct.x];
  SpPut p{val, idx, off[t], c, 0};
  for (int r = 0; r < TS * b.mt; ++r) {
    const double* tile = ct.y < b.nt ? A + a_tile(b, r >> 4, ct.y) : C + c_tile(b, r >> 4, ct.y - b.nt);
    const double v = tile[c * TS + (r & 15)];
    if (v != 0.0) p.put(v, r);
  }
  while (p.q < 4 * (int)(off[t + 1] - off[t])) p.put(0.0, 0);
}

// SP_U groups of a slice, requested together (past its end g1: zeros, no
// load).  A pass requests the next chunk before it works on the one at hand,
// the first before the vector is staged.
constexpr int SP_U = 8;
struct SpChunk {
  double a[SP_U];
  int i[SP_U];
  __device__ __forceinline__ void load(const double* __restrict__ val,
                                       const unsigned short* __restrict__ idx, long long g,
                                       long long g1) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int u = 0; u < SP_U; ++u) {
      a[u] = 0.0;
      i[u] = 0;
      if (g + u < g1) {
        a[u] = __builtin_nontemporal_load(val + (g + u) * 64 + lane);
        i[u] = __builtin_nontemporal_load(idx + (g + u) * 64 + lane);
      }
    }
  }
  // sums over the chunk's groups for NV vectors in LDS (vector k at v + k ld)
  template <int NV>
  __device__ __forceinline__ void dot(long long g, long long g1, const double* v, int ld,
                                      double* acc) const {
#pragma unroll
    for (int u = 0; u < SP_U; ++u)
      if (g + u < g1)
#pragma unroll
        for (int k = 0; k < NV; ++k) acc[k] += a[u] * v[k * ld + i[u]];
  }
};

// The slices t0 + w, t0 + w + 4, ... below t1 of one wave: fn(t, acc) gets each
// slice's sums (every lane the one of line lane % 16).  staged() fills the LDS.
template <int NV, class Stage, class Fn>
__device__ __forceinline__ void sp_slices(const double* __restrict__ val,
                                          const unsigned short* __restrict__ idx,
                                          const long long* __restrict__ off, int t0, int t1, int w,
                                          const double* v, int ld, Stage staged, Fn fn) {
  int t = t0 + w;
  long long g = 0, g1 = 0;
  SpChunk c;
  if (t < t1) {
    g = off[t];
    g1 = off[t + 1];
    c.load(val, idx, g, g1);
  }
  staged();
  double acc[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) acc[k] = 0.0;
  while (t < t1) {
    // the next chunk: of this slice, or the first of the wave's next one
    long long gn = g + SP_U, g1n = g1;
    int tn = t;
    if (gn >= g1) {
      tn = t + 4;
      if (tn < t1) {
        gn = off[tn];
        g1n = off[tn + 1];
      }
    }
    SpChunk n;
    if (tn < t1) n.load(val, idx, gn, g1n);
    c.dot<NV>(g, g1, v, ld, acc);
    if (tn != t) {
#pragma unroll
      for (int k = 0; k < NV; ++k) acc[k] = col_sum4(acc[k]);
      fn(t, acc);
#pragma unroll
      for (int k = 0; k < NV; ++k) acc[k] = 0.0;
    }
    c = n;
    t = tn;
    g = gn;
    g1 = g1n;
  }
}

// Row pass as k_rows_nv, out_k = base_k + alpha_k (A_i v_k [+ C_i v_k,0]): one
// item (a few tile rows of a block) per workgroup, a tile row per wave at a
// time.  A vector that does not take the x_0 columns has zeros staged there.
template <int NV>
__global__ __launch_bounds__(256) void k_sp_rows(const BlockInfo* __restrict__ blk, const SpMat sp,
                                                 long long d0off, RowsArgs ra, const LinkArgs la) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* v = reinterpret_cast<double*>(smem_raw);
  if ((int)blockIdx.x < la.wgs) return link_rows(blk, la, blockIdx.x);
  const int4 it = sp.row_items[blockIdx.x - la.wgs];   // block, first tile row, end, slice of the first
  const BlockInfo b = blk[it.x];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int na = TS * b.nt, ld = na + TS * b.kc0;
  auto staged = [&]() {
#pragma unroll
    for (int k = 0; k < NV; ++k)
      for (int c = threadIdx.x; c < ld; c += 256)
        v[k * ld + c] = c < na ? ra.v[k][b.dpoff + c] : (ra.with_C[k] ? ra.v[k][d0off + c - na] : 0.0);
    __syncthreads();
  };
  sp_slices<NV>(sp.rval, sp.ridx, sp.roff, it.w, it.w + it.z - it.y, wave, v, ld, staged,
                [&](int t, const double* acc) {
    if (lane >= 16) return;
    const int row = TS * (it.y + t - it.w) + lane;
    const bool in = row < b.m;
    double prev = 0.0;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      double base = 0.0;
      if (ra.chain[k]) base = prev;
      else if (ra.base[k] && in) base = ra.base[k][b.yoff + row];
      const double o = in ? base + ra.alpha[k] * acc[k] : 0.0;
      prev = o;
      if (ra.padded[k]) ra.out[k][b.voff + row] = o;
      else if (in) ra.out[k][b.yoff + row] = o;
    }
  });
}

// Column pass as k_cols and k_ccols in one: the first nt tile columns of a
// block are A_i's, the others C_i's, whose sums go to part.
__global__ __launch_bounds__(256) void k_sp_cols(const BlockInfo* __restrict__ blk, const SpMat sp,
                                                 const double* __restrict__ yp, const ColsArgs ca) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* y = reinterpret_cast<double*>(smem_raw);
  const int4 it = sp.col_items[blockIdx.x];
  const BlockInfo b = blk[it.x];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  auto staged = [&]() {
    for (int r = threadIdx.x; r < TS * b.mt; r += 256) y[r] = yp[b.voff + r];
    __syncthreads();
  };
  sp_slices<1>(sp.cval, sp.cidx, sp.coff, it.w, it.w + it.z - it.y, wave, y, 0, staged,
               [&](int t, const double* acc) {
    if (lane >= 16) return;
    const int K = it.y + t - it.w;
    double g = acc[0];
    if (K >= b.nt) {
      const int col = TS * (K - b.nt) + lane;
      if (col < ca.n0) ca.part[(long long)it.x * ca.n0 + col] = g;
      return;
    }
    const int col = TS * K + lane;
    if (col >= b.n) return;
    for (int e = ca.cptr[b.csc_off + col]; e < ca.cptr[b.csc_off + col + 1]; ++e)
      g += ca.cval[e] * ca.yL[ca.crow[e]];
    const long long o = b.xoff + col;
    if (ca.gout) ca.gout[o] = g;
    double x = g;
    if (ca.mode == 1) x = ca.cvec[o] - g - ca.zvec[o];
    else if (ca.mode == 2) x = ca.Dp[b.dpoff + col] * (g - ca.cvec[o]);
    if (ca.out) ca.out[o] = x;
    if (ca.dzv.dz) ca.dzv.dz[o] = (ca.dzv.rz[o] - ca.dzv.zs[o] * x) / ca.dzv.xs[o];
  });
}

}  // namespace

void launch_sp_fill(hipStream_t st, const BlockInfo* blk, const int2* rowtiles, int nrt,
                    const int2* coltiles, int nct, const double* A, const double* C,
                    const SpMat& sp) {
  hipLaunchKernelGGL(k_sp_fill_rows, dim3((nrt + 15) / 16), dim3(256), 0, st, blk, rowtiles, nrt, A, C,
                     sp.roff, sp.rval, sp.ridx);
  hipLaunchKernelGGL(k_sp_fill_cols, dim3((nct + 15) / 16), dim3(256), 0, st, blk, coltiles, nct, A, C,
                     sp.coff, sp.cval, sp.cidx);
}

void launch_sp_rows(hipStream_t st, const BlockInfo* blk, const SpMat& sp, long long d0off,
                    const RowsArgs& ra, const LinkArgs& la) {
  const size_t sh = (size_t)ra.nv * sp.max_cols * sizeof(double);
  const dim3 g(sp.nrow_items + la.wgs), b(256);
  if (ra.nv == 1) hipLaunchKernelGGL(k_sp_rows<1>, g, b, sh, st, blk, sp, d0off, ra, la);
  else if (ra.nv == 2) hipLaunchKernelGGL(k_sp_rows<2>, g, b, sh, st, blk, sp, d0off, ra, la);
  else hipLaunchKernelGGL(k_sp_rows<3>, g, b, sh, st, blk, sp, d0off, ra, la);
}

void launch_sp_cols(hipStream_t st, const BlockInfo* blk, const SpMat& sp, const double* yp,
                    const ColsArgs& ca) {
  hipLaunchKernelGGL(k_sp_cols, dim3(sp.ncol_items), dim3(256), (size_t)sp.max_rows * sizeof(double), st,
                     blk, sp, yp, ca);
}

}  // namespace ahlp
