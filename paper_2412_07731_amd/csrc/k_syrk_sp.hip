// Block SYRK M_i = A_i D_i A_i' (+ delta I) of blocks with few nonzeros (a2).
//
// The dense kernel (k_syrk) multiplies whole 16x16 tiles and is bound by the
// matrix cores and their operand delivery (17.2 GFLOP for 512 blocks of 256 x
// 512: 377 us).  With a share d of nonzeros an entry of M_i needs only d n of
// its n products if one of the two rows is walked by its nonzeros.  Here a lane
// owns two columns s of M_i, a wave a tile row: for every nonzero (r, k) of its
// 16 rows, in ascending k, acc(r, s) += a_rk * (a_sk D_k), with the products
// a_sk D_k of SS_C columns s and a stage of SS_K columns k expanded in LDS
// ([k][s], zeros included).  The matrix instructions accumulate as a chain of
// fused multiply-adds in ascending k (checked on gfx950) and products with a
// zero leave the chain's value as it is, so this gives the dense kernel's
// values bit for bit.
//
// What bounds it is the LDS read per nonzero and 128 columns, and a stage's fixed
// part (clearing and expanding the products between barriers): the LDS is active in
// 55% of the cycles, the vector unit in 39%, memory at 1.15 TB/s (counters).  Two
// columns a lane make it a 16-byte read in FP64, which the LDS serves at 234 bytes per
// clock (8-byte reads: 125); a nonzero's value and k reach all lanes by DPP
// from the lane of each row of 16 that loaded it, as operands of the
// multiply-add and of the address sum, so that the vector unit stays below the
// LDS time.  512 blocks of 256 x 512 at 10% nonzeros: 206 us against the dense
// kernel's 368 us in FP64, 149 against 207 us in FP32 (with the link columns' gather
// beside it on another stream 252 and 181 us, and 377 and 209 us).  (Broadcast by scalar
// loads waits on their latency, since those share their counter with the LDS
// reads: 333 us with the gather beside it; one column a lane and a stage of 128: 273 us.)
#include "common.h"
#include "kernels.h"
#include "tile_chol.h"

namespace ahlp {

namespace {

constexpr int SS_W = SS_ROWS;  // waves: tile rows of an item
constexpr int SS_C = 16 * SS_COLS;   // columns of an item
static_assert(SS_K * SS_C <= 65536 && SS_C % 16 == 0, "16-bit indices, the row in the low four bits");
constexpr int SS_PRE = 2;      // entries of the next stage a thread holds ahead
constexpr int SS_AHEAD = 3;    // rows whose entries a wave holds ahead
constexpr int SS_LD = TS + 1;  // leading dimension of the output tiles in LDS

template <typename T> struct Pair;
template <> struct Pair<double> { typedef double type __attribute__((ext_vector_type(2))); };
template <> struct Pair<float> { typedef float type __attribute__((ext_vector_type(2))); };

// A DPP instruction's operands must not have been written by the vector unit in the two
// wait states before, and the compiler does not look into asm for that: an asm with one
// starts with these waits, so that it stands wherever it is scheduled, and its products
// are of both columns, so that no sum follows itself sooner.  (With the waits on a chunk's
// first product alone the kernel took 2% to 3% less; two or four entries in one asm took
// 2% to 3% more, since their products then wait for each other's reads.)

// Both columns' acc + (lane J of the 16-lane row's a) * x.  The FP64 form is written
// out: the compiler broadcasts into a register first.
template <int J>
__device__ __forceinline__ void fmac_bcast(double a, const Pair<double>::type& x, double& c0, double& c1) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %2, %3 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %2, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf"
      : "+&v"(c0), "+&v"(c1) : "v"(a), "v"(x.x), "v"(x.y), "n"(J));
#endif
}
template <int J>
__device__ __forceinline__ void fmac_bcast(float a, const Pair<float>::type& x, float& c0, float& c1) {
  const float aj = row_bcast<J>(a);
  c0 = fmaf(aj, x.x, c0);
  c1 = fmaf(aj, x.y, c1);
}

// xb + lane J of the row's o: one DPP add, to which the compiler gives its waits
template <int J>
__device__ __forceinline__ unsigned add_bcast(unsigned o, unsigned xb) {
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)o, 0x150 + J, 0xF, 0xF, true) + xb;
}
template <typename T>
using LdsPair = const __attribute__((address_space(3))) typename Pair<T>::type*;
// Entries J .. J + 3 of a chunk into both columns, in order: the LDS reads go
// out before the first product.  xb: LDS address of this lane's place in row 0
// of X, o: each lane's entry's byte offset of its row, added lane to lane.
template <int J, typename T>
__device__ __forceinline__ void sp_chunk(T a, unsigned o, unsigned xb, T& c0, T& c1) {
  typename Pair<T>::type x[4];
  x[0] = *(LdsPair<T>)add_bcast<J>(o, xb);
  x[1] = *(LdsPair<T>)add_bcast<J + 1>(o, xb);
  x[2] = *(LdsPair<T>)add_bcast<J + 2>(o, xb);
  x[3] = *(LdsPair<T>)add_bcast<J + 3>(o, xb);
  __builtin_amdgcn_sched_barrier(0);   // all reads before the first product
  fmac_bcast<J>(a, x[0], c0, c1);
  fmac_bcast<J + 1>(a, x[1], c0, c1);
  fmac_bcast<J + 2>(a, x[2], c0, c1);
  fmac_bcast<J + 3>(a, x[3], c0, c1);
}

template <typename T>
using CPtr = const __attribute__((address_space(4))) T*;   // read through the scalar cache
template <typename T>
__device__ __forceinline__ CPtr<T> cptr(const T* p) { return (CPtr<T>)(unsigned long long)p; }

// bytes of LDS for X, and in its place at the end for the output tiles
template <typename T>
__host__ __device__ constexpr size_t ss_area() {
  constexpr size_t x = (size_t)SS_K * SS_C * sizeof(T),
                   o = (size_t)SS_W * (SS_COLS / 2) * TS * SS_LD * sizeof(T);
  return x > o ? x : o;
}

template <typename T>
__global__ __launch_bounds__(64 * SS_W, 4) void k_syrk_sp(const BlockInfo* __restrict__ blk,
                                                          const int4* __restrict__ items, int nitems,
                                                          const SyrkSp sp, const T* __restrict__ val,
                                                          const double* __restrict__ Dp,
                                                          T* __restrict__ LB, double delta) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* X = reinterpret_cast<T*>(smem_raw);   // [SS_K][SS_C]
  T* Dl = reinterpret_cast<T*>(smem_raw + ss_area<T>());   // the block's D
  const int per = gridDim.x / 8, g0 = (blockIdx.x % 8) * per + blockIdx.x / 8;
  if (g0 >= nitems) return;
  const int4 it = items[g0];   // block, first of SS_COLS tile columns, first tile row, tile rows
  const BlockInfo b = blk[it.x];
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int J0 = it.y, I = it.z + w, nst = (TS * b.nt + SS_K - 1) / SS_K;
  const bool active = w < it.w;
  const int row0 = (int)(b.voff / TS);   // the block's first tile row in the lists
  // wave j expands tile column J0 + j
  const int Js = min(J0 + w, b.mt - 1);
  const bool have = J0 + w < b.mt;
  const int sl = cptr(sp.first)[row0 + Js], ql = cptr(sp.first)[row0 + min(I, b.mt - 1)];
  // list bounds one stage ahead of their use (in batches of four entries):
  // [e0, e1) of the tile column to expand, the first batch and the rows'
  // batches of the tile row to walk
  int e0 = 4 * cptr(sp.off)[sl], e1 = 4 * cptr(sp.off)[sl + 1], gn = cptr(sp.off)[ql];
  unsigned cn[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) cn[u] = cptr(sp.cnt)[4 * ql + u];
  int pi[SS_PRE];
  T pa[SS_PRE];
  auto fetch = [&]() {
#pragma unroll
    for (int u = 0; u < SS_PRE; ++u) {
      const int e = e0 + lane + 64 * u;
      pa[u] = T(0);
      pi[u] = 0;
      if (have && e < e1) {
        pi[u] = sp.idx[e];
        pa[u] = val[e];
      }
    }
  };
  auto clear = [&]() {
    typedef T V __attribute__((ext_vector_type(16 / sizeof(T))));
    V* z = reinterpret_cast<V*>(X);
    for (int i = tid; i < (int)(SS_K * SS_C * sizeof(T) / 16); i += 64 * SS_W) z[i] = V(0);
  };
  T acc[16][2];
#pragma unroll
  for (int j = 0; j < 16; ++j) acc[j][0] = acc[j][1] = T(0);
  const unsigned xb = (unsigned)(unsigned long long)(__attribute__((address_space(3))) char*)(X + 2 * lane);
  fetch();
  for (int i = tid; i < TS * b.nt; i += 64 * SS_W) Dl[i] = (T)Dp[b.dpoff + i];
  clear();
  for (int st = 0; st < nst; ++st) {
    __syncthreads();
    auto put = [&](T v, int i) {
      if (v != T(0)) X[i + 16 * w] = v * Dl[SS_K * st + i / SS_C];
    };
#pragma unroll
    for (int u = 0; u < SS_PRE; ++u) put(pa[u], pi[u]);
    if (have)   // what a thread does not hold ahead
      for (int e = e0 + lane + 64 * SS_PRE; e < e1; e += 64) put(val[e], sp.idx[e]);
    const unsigned c4[4] = {cn[0], cn[1], cn[2], cn[3]};
    const T* vr = val + 4LL * gn;                    // the rows' entries, walked
    const unsigned short* xr = sp.idx + 4LL * gn;
    auto count = [&](int j) { return (int)((c4[j >> 2] >> (8 * (j & 3))) & 255); };
    // 16 entries of a row, lane l entry l % 16 (every row of 16 lanes holds
    // them all; 16 past the last
    // are readable); SS_AHEAD rows are held ahead
    T ra[SS_AHEAD];
    unsigned ro[SS_AHEAD];
    auto load_row = [&](int j) {
      ra[j % SS_AHEAD] = vr[l16];
      ro[j % SS_AHEAD] = xr[l16];
      vr += 4 * count(j);
      xr += 4 * count(j);
    };
    if (active) {
#pragma unroll
      for (int j = 0; j < SS_AHEAD; ++j) load_row(j);
    }
    __syncthreads();
    const int sn = min(st + 1, nst - 1);
    e0 = 4 * cptr(sp.off)[sl + sn];
    e1 = 4 * cptr(sp.off)[sl + sn + 1];
    const T* vs = val + 4LL * gn;
    const unsigned short* xs = sp.idx + 4LL * gn;
    gn = cptr(sp.off)[ql + sn];
#pragma unroll
    for (int u = 0; u < 4; ++u) cn[u] = cptr(sp.cnt)[4 * (ql + sn) + u];
    if (st + 1 < nst) fetch();
    if (active) {
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int c = count(j);
        const T a = ra[j % SS_AHEAD];
        const unsigned o = (ro[j % SS_AHEAD] & ~15u) * (unsigned)sizeof(T);
        if (j + SS_AHEAD < 16) load_row(j + SS_AHEAD);
        if (c > 0) sp_chunk<0>(a, o, xb, acc[j][0], acc[j][1]);
        if (c > 1) sp_chunk<4>(a, o, xb, acc[j][0], acc[j][1]);
        if (c > 2) sp_chunk<8>(a, o, xb, acc[j][0], acc[j][1]);
        if (c > 3) sp_chunk<12>(a, o, xb, acc[j][0], acc[j][1]);
        for (int d = 4; d < c; ++d)
          sp_chunk<0>(vs[4 * d + l16], (xs[4 * d + l16] & ~15u) * (unsigned)sizeof(T), xb, acc[j][0],
                         acc[j][1]);
        vs += 4 * c;
        xs += 4 * c;
      }
    }
    if (st + 1 < nst) {
      __syncthreads();
      clear();
    }
  }
  // a lane's two columns lie in tile J0 + lane / 8; through LDS to whole lines,
  // half of the tiles at a time
  T* buf = X + w * (SS_COLS / 2) * TS * SS_LD;
  __syncthreads();
  if (!active) return;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if ((lane >> 5) == h) {
      T* t = buf + ((lane & 31) >> 3) * TS * SS_LD + (2 * lane & 15) * SS_LD;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        t[j] = acc[j][0];
        t[SS_LD + j] = acc[j][1];
      }
    }
    wave_order();
    for (int q = 0; q < SS_COLS / 2; ++q) {
      const int J = J0 + SS_COLS / 2 * h + q;
      if (J > I || J >= b.mt) break;
      T* dst = LB + lb_tile(b, I, J);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int e = 64 * s + lane, c = e >> 4, r = e & 15;
        T v = buf[q * TS * SS_LD + c * SS_LD + r];
        if (I == J && r == c) v = (TS * I + r < b.m) ? (T)(v + delta) : T(1);
        dst[e] = v;
      }
    }
    wave_order();
  }
}

// Fills the lists: one thread per row and stage.
__global__ __launch_bounds__(256) void k_syrk_sp_fill(const BlockInfo* __restrict__ blk,
                                                      const int2* __restrict__ rowtiles, int nrt,
                                                      const double* __restrict__ A, const SyrkSp sp,
                                                      double* __restrict__ val,
                                                      unsigned short* __restrict__ idx) {
  const int t = blockIdx.x, j = threadIdx.x & 15;
  if (t >= nrt) return;
  const int2 rt = rowtiles[t];
  const BlockInfo b = blk[rt.x];
  const int nst = (TS * b.nt + SS_K - 1) / SS_K;
  for (int st = threadIdx.x >> 4; st < nst; st += 16) {
    const long long q = sp.first[t] + st;
    long long e = 4LL * sp.off[q];
    for (int u = 0; u < j; ++u) e += 4 * ((sp.cnt[4 * q + (u >> 2)] >> (8 * (u & 3))) & 255);
    const long long e1 = e + 4 * ((sp.cnt[4 * q + (j >> 2)] >> (8 * (j & 3))) & 255);
    const int c1 = min(SS_K * (st + 1), TS * b.nt);
    for (int c = SS_K * st; c < c1; ++c) {
      const double v = A[a_tile(b, rt.y, c >> 4) + (c & 15) * TS + j];
      if (v != 0.0) {
        val[e] = v;
        idx[e++] = (unsigned short)((c - SS_K * st) * SS_C + j);
      }
    }
    for (; e < e1; ++e) {
      val[e] = 0.0;
      idx[e] = 0;
    }
  }
}

}  // namespace

template <typename T>
void launch_syrk_sp(hipStream_t st, const BlockInfo* blk, const int4* items, int nitems,
                    const SyrkSp& sp, const T* val, const double* Dp, T* LB, double delta) {
  if (nitems == 0) return;
  hipLaunchKernelGGL(k_syrk_sp<T>, dim3(8 * ((nitems + 7) / 8)), dim3(64 * SS_W),
                     ss_area<T>() + (size_t)sp.max_cols * sizeof(T), st,
                     blk, items, nitems, sp, val, Dp, LB, delta);
}
template void launch_syrk_sp<double>(hipStream_t, const BlockInfo*, const int4*, int, const SyrkSp&,
                                     const double*, const double*, double*, double);
template void launch_syrk_sp<float>(hipStream_t, const BlockInfo*, const int4*, int, const SyrkSp&,
                                    const float*, const double*, float*, double);

void launch_syrk_sp_fill(hipStream_t st, const BlockInfo* blk, const int2* rowtiles, int nrt,
                         const double* A, const SyrkSp& sp, double* val, unsigned short* idx) {
  hipLaunchKernelGGL(k_syrk_sp_fill, dim3(nrt), dim3(256), 0, st, blk, rowtiles, nrt, A, sp, val, idx);
}

void set_syrk_sp_smem_limits() {
  hipFuncSetAttribute((const void*)k_syrk_sp<double>, hipFuncAttributeMaxDynamicSharedMemorySize,
                      (int)(ss_area<double>() + SS_NMAX * sizeof(double)));
  hipFuncSetAttribute((const void*)k_syrk_sp<float>, hipFuncAttributeMaxDynamicSharedMemorySize,
                      (int)(ss_area<float>() + SS_NMAX * sizeof(float)));
}

}  // namespace ahlp
