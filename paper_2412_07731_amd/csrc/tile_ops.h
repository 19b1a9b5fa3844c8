// One-wave operations on 16x16 FP64 tiles (column-major, 256 doubles) and on
// 16-vectors, built on the 16x16x4 FP64 MFMA.
//
// Operand layout of v_mfma_f64_16x16x4f64: for the s-th of four K-steps lane l
// supplies A(l%16, 4s + l/16) and B(4s + l/16, l%16); for a column-major tile X
// these are X[64 s + l] (A = X) and X[(l%16)*16 + 4s + l/16] (B = X).  The
// accumulator holds element (acc_row(l, r), l%16) in register r.
//
// The tile helpers take the leading dimension LD as a template argument
// (default 16, a dense 256-value tile).  LDS tiles with LD = 17 pad each
// column by one value: the accumulator-layout and B-operand accesses then
// spread the 16 lanes of a row group over distinct banks, where LD = 16 puts
// them all in one.  A padded tile takes 16 * 17 values.
#pragma once

#include "common.h"
#include "tile_chol.h"

namespace ahlp {

struct Op { double v[4]; };   // a tile as an A operand: element 64 s + lane

// offset of element (i, j) of a tile with leading dimension LD
template <int LD = TS>
__device__ __forceinline__ int tix(int i, int j) { return j * LD + i; }

template <int LD = TS>
__device__ __forceinline__ Op op_load(const double* t) {
  const int lane = threadIdx.x & 63;
  Op o;
#pragma unroll
  for (int s = 0; s < 4; ++s) o.v[s] = t[tix<LD>(lane & 15, 4 * s + (lane >> 4))];
  return o;
}
template <int LD = TS>
__device__ __forceinline__ void op_store(double* t, const Op& o) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int s = 0; s < 4; ++s) t[tix<LD>(lane & 15, 4 * s + (lane >> 4))] = o.v[s];
}
__device__ __forceinline__ d4 acc_zero() { return d4{0.0, 0.0, 0.0, 0.0}; }
template <int LD = TS>
__device__ __forceinline__ d4 acc_load(const double* t) {
  const int lane = threadIdx.x & 63;
  d4 a;
#pragma unroll
  for (int r = 0; r < 4; ++r) a[r] = t[tix<LD>(acc_row<double>(lane, r), lane & 15)];
  return a;
}
template <int LD = TS>
__device__ __forceinline__ void acc_store(double* t, d4 a) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int r = 0; r < 4; ++r) t[tix<LD>(acc_row<double>(lane, r), lane & 15)] = a[r];
}
// padded tile of an exact column-major block (rows x cols, leading dimension
// ld); identity on the padded part of the diagonal if diag
__device__ __forceinline__ d4 acc_load_exact(const double* src, int rows, int cols, int ld,
                                             bool diag) {
  const int lane = threadIdx.x & 63;
  d4 a;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = acc_row<double>(lane, r), j = lane & 15;
    double v = 0.0;
    if (i < rows && j < cols) v = src[i + j * ld];
    else if (diag && i == j) v = 1.0;
    a[r] = v;
  }
  return a;
}
// transposed padded tile: element (i, j) = src[j + i*ld], i < rows, j < cols
__device__ __forceinline__ d4 acc_load_exact_t(const double* src, int rows, int cols, int ld) {
  const int lane = threadIdx.x & 63;
  d4 a;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = acc_row<double>(lane, r), j = lane & 15;
    a[r] = (i < rows && j < cols) ? src[j + i * ld] : 0.0;
  }
  return a;
}
// acc += alpha X Y'
template <int LD = TS>
__device__ __forceinline__ d4 mma_xyt(d4 acc, const double* X, const double* Y, double alpha) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int o = tix<LD>(lane & 15, 4 * s + (lane >> 4));
    acc = mfma(alpha * X[o], Y[o], acc);
  }
  return acc;
}
__device__ __forceinline__ void vec_put(double* dst, double y) {
  const int lane = threadIdx.x & 63;
  if (lane < 16) dst[lane] = y;
}
}  // namespace ahlp
