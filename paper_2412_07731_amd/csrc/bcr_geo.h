// Tile layout of the block cyclic reduction's arrays (BcrArgs) for pairs of
// TP x TP tiles and a border of t0 tiles, shared by the reduction (k_bcr.hip,
// k_bcrn.hip) and the solve (k_bcrs.hip):
//   BD[j], BC[j], FLi[o], FXL[o], FXR[o]   TP x TP tiles, tile (r, c) at c*TP + r
//   BEt[j], FGt[o]                         t0 x TP tiles, tile (q, c) at c*t0 + q
// Pair vectors r, w, up: 16 TP values per pair.
#pragma once

#include "common.h"

namespace ahlp {

template <int TP> struct Geo {
  static constexpr int TB = 16 * TP, BLK = TP * TP * 256;
  __device__ static __forceinline__ int bt(int r, int c) { return (c * TP + r) * 256; }
  __device__ static __forceinline__ long long et(long long j, int q, int c, int t0) {
    return ((j * TP + c) * t0 + q) * 256;
  }
};

}  // namespace ahlp
