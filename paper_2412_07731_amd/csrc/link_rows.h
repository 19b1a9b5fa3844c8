// The dual rows after the blocks, out = base + alpha (F xp [+ F0 x0]), by workgroups
// of 256 threads: beside a row pass or alone.
#pragma once

#include "common.h"
#include "kernels.h"

namespace ahlp {

// Workgroup wg of la.wgs: the global rows first, one each, their entries kept as one
// compressed row over the padded x: each thread a fixed strided share, then a fixed
// tree.  Then the link rows, a pair a wave: row a of pair j is
// base + alpha (FR_j xp_j + FL_j xp_{j+1} [+ F0 x0]).
__device__ __forceinline__ void link_rows(const BlockInfo* __restrict__ blk, const LinkArgs& la, int wg) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (wg < la.ng) {
    const int k = wg;
    __shared__ double sh[4];
    double v = 0.0;
    const int e1 = la.gptr[k + 1];
    for (int e = la.gptr[k] + threadIdx.x; e < e1; e += 256) v += la.gval[e] * la.xp[la.gidx[e]];
    if (la.F0 && la.x0)
      for (int c = threadIdx.x; c < la.n0; c += 256) v += la.F0[(la.nl + k) * la.n0 + c] * la.x0[c];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if (lane == 0) sh[wave] = v;
    __syncthreads();
    if (threadIdx.x == 0)
      la.out[la.nl + k] = (la.base ? la.base[la.nl + k] : 0.0) + la.alpha * (((sh[0] + sh[1]) + sh[2]) + sh[3]);
    return;
  }
  const int step = 4 * (la.wgs - la.ng);
  for (int j = 4 * (wg - la.ng) + wave; j < la.P; j += step) {
    const BlockInfo &bl = blk[j], &br = blk[j + 1];
    const int l = la.lsz[j];
    for (int a = lane; a < l; a += 64) {
      double s = 0.0;
      const int qr = TS * bl.ktL + a;   // right section of block j
      for (int e = la.lptr[bl.csr_off + qr]; e < la.lptr[bl.csr_off + qr + 1]; ++e)
        s += la.lval[e] * la.xp[bl.dpoff + la.lcol[e]];
      for (int e = la.lptr[br.csr_off + a]; e < la.lptr[br.csr_off + a + 1]; ++e)
        s += la.lval[e] * la.xp[br.dpoff + la.lcol[e]];
      if (la.F0L && la.x0)
        for (int c = 0; c < la.n0; ++c) s += la.F0L[(la.loff[j] + a) * la.n0 + c] * la.x0[c];
      const long long o = la.loff[j] + a;
      la.out[o] = (la.base ? la.base[o] : 0.0) + la.alpha * s;
    }
  }
}

}  // namespace ahlp
