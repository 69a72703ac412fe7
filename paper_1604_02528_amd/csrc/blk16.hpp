// 16 x 16 blocks held by one wavefront, and the lane broadcasts their serial
// parts run on (device factorization and normalization).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>
#include <utility>

#include "scalar.hpp"
#include "tile.hpp"

namespace selinv {

// ---------------------------------------------------------------------------
// 16 x 16 blocks.  A block of S (rows i of one 16-row strip, columns j of
// another) is held by one wavefront as register v of lane l = S(l % 16, 4 v +
// l / 16): its transpose in the MFMA result layout, which is the A-operand
// layout of the block and the B-operand layout of its transpose at the same
// time.  Everything below works on transposed blocks, so that a product's
// result is the next product's operand without any data movement:
//   W^T = M S^T (M = L_kk^{-1}, W = L D),  L^T = D^{-1} W^T,
//   S(i, j)^T -= L(j, k) W(i, k)^T          (M and L(j, k) conjugated if Hermitian)
// ---------------------------------------------------------------------------
template <typename T> struct Blk {
  d4 p[Planes<T>::P];
};

__device__ __forceinline__ double blk_get(const Blk<double> &b, int v) { return b.p[0][v]; }
__device__ __forceinline__ cplx blk_get(const Blk<cplx> &b, int v) { return cplx{b.p[0][v], b.p[1][v]}; }
__device__ __forceinline__ void blk_set(Blk<double> &b, int v, double x) { b.p[0][v] = x; }
__device__ __forceinline__ void blk_set(Blk<cplx> &b, int v, cplx x) {
  b.p[0][v] = x.re;
  b.p[1][v] = x.im;
}
template <typename T> __device__ __forceinline__ Blk<T> blk_zero() {
  Blk<T> b;
#pragma unroll
  for (int p = 0; p < Planes<T>::P; ++p) b.p[p] = d4{0.0, 0.0, 0.0, 0.0};
  return b;
}

// acc += A B for 16 x 16 operands in the layout above, over the first 4 nv
// contraction indices (complex: four real products)
template <typename T>
__device__ __forceinline__ void blk_mma(const Blk<T> &a, const Blk<T> &b, Blk<T> &acc, int nv = 4) {
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    if (v < nv) {
      acc.p[0] = mfma16(a.p[0][v], b.p[0][v], acc.p[0]);
      if constexpr (Planes<T>::P == 2) {
        acc.p[1] = mfma16(a.p[0][v], b.p[1][v], acc.p[1]);
        acc.p[0] = mfma16(-a.p[1][v], b.p[1][v], acc.p[0]);
        acc.p[1] = mfma16(a.p[1][v], b.p[0][v], acc.p[1]);
      }
    }
  }
}

// acc += A B, the product summed by itself first: the sums' roundings are then
// of the update's size, and acc rounds once for 16 contraction indices (in the
// accumulator it rounds 16 times at acc's own size).
template <typename T> __device__ __forceinline__ void blk_mma_add(const Blk<T> &a, const Blk<T> &b, Blk<T> &acc) {
  Blk<T> u = blk_zero<T>();
  blk_mma<T>(a, b, u);
#pragma unroll
  for (int p = 0; p < Planes<T>::P; ++p) acc.p[p] += u.p[p];
}

// A block in LDS, plane p at q[p * stride]: element v * 64 + lane, so that
// reads and writes of a register are contiguous.
template <typename T> __device__ __forceinline__ Blk<T> blk_from_lds(const double *q, int stride) {
  const int lane = threadIdx.x & 63;
  Blk<T> b;
#pragma unroll
  for (int p = 0; p < Planes<T>::P; ++p)
#pragma unroll
    for (int v = 0; v < 4; ++v) b.p[p][v] = q[p * stride + v * 64 + lane];
  return b;
}
template <typename T> __device__ __forceinline__ void blk_to_lds(const Blk<T> &b, double *q, int stride) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int p = 0; p < Planes<T>::P; ++p)
#pragma unroll
    for (int v = 0; v < 4; ++v) q[p * stride + v * 64 + lane] = b.p[p][v];
}

__device__ __forceinline__ void st_off(double *base, uint32_t b, double v) {
  *reinterpret_cast<SELINV_GAS double *>(reinterpret_cast<SELINV_GAS char *>(gw(base)) + b) = v;
}
__device__ __forceinline__ void st_off(cplx *base, uint32_t b, cplx v) {
  SELINV_GAS char *q = reinterpret_cast<SELINV_GAS char *>(gw(base)) + b;
  *reinterpret_cast<SELINV_GAS double *>(q) = v.re;
  *reinterpret_cast<SELINV_GAS double *>(q + 8) = v.im;
}
// The order of a strip's rows over the lanes for blocks that are added to the
// ancestors' panels (see blk_atomic): complex rows are dealt to even and odd
// lanes, row t / 2 + 8 (t % 2) to lane t.
template <typename T> __device__ __forceinline__ int strip_row(int t) {
  return Planes<T>::P == 2 ? (t >> 1) + 8 * (t & 1) : t;
}

// This lane's row of a block, opaque: the addresses below are cheap to form
// and cost registers when kept from a block's load to its store.
__device__ __forceinline__ int blk_row() {
  int r = threadIdx.x & 15;
  asm("" : "+v"(r));
  return r;
}
// Rows [0, rows) and columns [0, cols) of a 16 x 16 block at Q (wave-uniform,
// leading dimension ld); zeros outside (read from Q's first element).
// STRIP: rows in the order of strip_row.
template <typename T, bool STRIP = false>
__device__ __forceinline__ Blk<T> blk_load(const T *Q, int ld, int rows, int cols) {
  const int r = STRIP ? strip_row<T>(blk_row()) : blk_row(), g = (threadIdx.x & 63) >> 4;
  T v[4];
#pragma unroll
  for (int q = 0; q < 4; ++q)
    v[q] = ld_off(Q, ((uint32_t)((4 * q + g) * ld + r) & opaque_mask32(r < rows && 4 * q + g < cols)) * (uint32_t)sizeof(T));
  Blk<T> b;
#pragma unroll
  for (int q = 0; q < 4; ++q) blk_set(b, q, masked(v[q], opaque_mask(r < rows && 4 * q + g < cols)));
  return b;
}
template <typename T, bool STRIP = false>
__device__ __forceinline__ void blk_store(const Blk<T> &b, T *Q, int ld, int rows, int cols) {
  const int r = STRIP ? strip_row<T>(blk_row()) : blk_row(), g = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (r < rows && 4 * q + g < cols) st_off(Q, (uint32_t)((4 * q + g) * ld + r) * (uint32_t)sizeof(T), blk_get(b, q));
}

// Component-wise select (a select of whole complex values goes through memory).
__device__ __forceinline__ double pick(bool c, double a, double b) { return c ? a : b; }
__device__ __forceinline__ cplx pick(bool c, cplx a, cplx b) { return cplx{c ? a.re : b.re, c ? a.im : b.im}; }

// LDS ordering inside one wavefront.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

template <class F, int... I> __device__ __forceinline__ void static_for(F f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}

// Lane broadcasts inside a row of 16 lanes (row_newbcast, the one DPP form of
// 64-bit operations): acc += w[lane L of the row] y in one instruction.  The
// compiler does not look into these for hazards: a DPP read needs two wait
// states after its source was written, which bcast16 supplies and fmac16
// gets by following a bcast16 of the same source.
template <int L> __device__ __forceinline__ double bcast16(double w) {
  double r;
  asm("s_nop 1\n\tv_mov_b64_dpp %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf" : "=v"(r) : "v"(w), "n"(L));
  return r;
}
template <int L> __device__ __forceinline__ cplx bcast16(cplx w) { return cplx{bcast16<L>(w.re), bcast16<L>(w.im)}; }
template <int L> __device__ __forceinline__ void fmac16(double &acc, double w, double y) {
  asm("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(w), "v"(y), "n"(L));
}

// quad_perm moves between neighbouring lanes.
template <int CTRL> __device__ __forceinline__ int32_t quad(int32_t v) {
  return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, false);
}
template <int CTRL> __device__ __forceinline__ double quad(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)quad<CTRL>((int32_t)(uint32_t)u), hi = (uint32_t)quad<CTRL>((int32_t)(u >> 32));
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// u added to the entries of an ancestor's column: row i0 + strip_row(lane % 16)
// at base[pos], where k <= row < c.  Complex: the two lanes of a pair hold
// rows m and m + 8 of the strip; they exchange one plane each, and both add to
// row m, then both to row m + 8, so that one instruction covers eight whole
// entries in a row (real and imaginary parts by themselves touch every cache
// line twice; the atomics bound the updates of narrow nodes).
__device__ __forceinline__ void blk_atomic(double *base, int32_t pos, int i0, int k, int c, double u) {
  const int i = i0 + (threadIdx.x & 15);
  if (i < c && k <= i) unsafeAtomicAdd(base + pos, u);
}
__device__ __forceinline__ void blk_atomic(cplx *base, int32_t pos, int i0, int k, int c, cplx u) {
  const int odd = threadIdx.x & 1, i = i0 + ((threadIdx.x & 15) >> 1);
  const double other = quad<0xb1>(odd ? u.re : u.im);  // [1, 0, 3, 2]
  const int32_t pa = quad<0xa0>(pos), pb = quad<0xf5>(pos);  // [0, 0, 2, 2], [1, 1, 3, 3]
  double *q = reinterpret_cast<double *>(base) + odd;
  if (i < c && k <= i) unsafeAtomicAdd(q + 2 * (int64_t)pa, odd ? other : u.re);
  if (i + 8 < c && k <= i + 8) unsafeAtomicAdd(q + 2 * (int64_t)pb, odd ? u.im : other);
}

template <int L> __device__ __forceinline__ void fmac16_t(double &acc, double w, double y) { fmac16<L>(acc, w, y); }
template <int L> __device__ __forceinline__ void fmac16_t(cplx &acc, cplx w, cplx y) {
  fmac16<L>(acc.re, w.re, y.re);
  fmac16<L>(acc.im, w.re, y.im);
  fmac16<L>(acc.re, w.im, -y.im);
  fmac16<L>(acc.im, w.im, y.re);
}
// The two wait states between a write of v and its broadcasts.
__device__ __forceinline__ void dpp_source(double &v) { asm("s_nop 1" : "+v"(v)); }
__device__ __forceinline__ void dpp_source(cplx &v) { asm("s_nop 1" : "+v"(v.re), "+v"(v.im)); }

}  // namespace selinv
