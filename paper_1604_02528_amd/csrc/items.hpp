// Work items of the selected-inversion traversal (device code shared by the
// forward and adjoint kernels): the dense X_{C,C} gather, the GEMM-1 tile with
// its fused share of GEMM-2, the split-tile reduction and the diagonal-block
// tile.  See plan.hpp for the item vocabulary.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "blk16.hpp"
#include "plan.hpp"
#include "scalar.hpp"
#include "tile.hpp"

namespace selinv {

// ---------------------------------------------------------------------------
// Work items
// ---------------------------------------------------------------------------
template <typename T> struct Ctx {
  const DevPlan *pl;
  const T *Lp;  // normalized panels of this matrix
  T *Xp;        // selected inverse of this matrix
  T *Pp;        // GEMM-2 partial products of this matrix
  T *Gp;        // dense X_{C,C} buffers of this matrix
  T *Yp;        // partial GEMM-1 tiles of this matrix (split nodes)
};

// The same from a record (wave-uniform values, kept in scalar registers).
__device__ __forceinline__ int64_t uniform64(int64_t v) {
  const uint32_t lo = uniform((int32_t)(uint32_t)v), hi = uniform((int32_t)(v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ NodeInfo uniform(const NodeInfo &a) {
  NodeInfo n = a;
  n.K = uniform(a.K);
  n.s = uniform(a.s);
  n.c = uniform(a.c);
  n.ldg = uniform(a.ldg);
  n.split = uniform(a.split);
  n.kchunk = uniform(a.kchunk);
  n.defer2 = uniform(a.defer2);
  n.glow = uniform(a.glow);
  n.off = uniform64(a.off);
  n.rp = uniform64(a.rp);
  n.goff = uniform64(a.goff);
  n.poff = uniform64(a.poff);
  n.yoff = uniform64(a.yoff);
  n.np = uniform(a.np);
  n.g2 = uniform(a.g2);
  return n;
}

// NodeInfo from the plan's node tables (the persistent schedule and the
// adjoint, whose items carry only the node index).
__device__ __forceinline__ NodeInfo node_info(const DevPlan &pl, int K) {
  NodeInfo n;
  n.K = K;
  n.s = uniform(gp(pl.node_s)[K]);
  n.c = uniform(gp(pl.node_c)[K]);
  n.ldg = uniform(gp(pl.node_ldg)[K]);
  n.split = uniform(gp(pl.node_split)[K]);
  n.kchunk = uniform(gp(pl.node_kchunk)[K]);
  n.defer2 = n.glow = 0;
  n.off = uniform64(gp(pl.node_off)[K]);
  n.rp = uniform64(gp(pl.node_rowptr)[K]);
  n.goff = uniform64(gp(pl.node_goff)[K]);
  n.poff = uniform64(gp(pl.node_poff)[K]);
  n.yoff = uniform64(gp(pl.node_yoff)[K]);
  n.np = (n.c + 63) / 64;
  n.g2 = 0;
  return n;
}

__device__ __forceinline__ void atomic_add_t(double *p, double v) { unsafeAtomicAdd(p, v); }
__device__ __forceinline__ void atomic_add_t(cplx *p, cplx v) {
  double *q = reinterpret_cast<double *>(p);
  unsafeAtomicAdd(q, v.re);
  unsafeAtomicAdd(q + 1, v.im);
}

// The 64 x 64 tile in LDS (rows i0.., columns k0.. of C(K) x C(K), lower part)
// added to the ancestors' entries of S_{C,C} in a panel-layout array, with
// f(value, diagonal) applied: the positions of all of a thread's elements
// first, then the adds.
// Complex entries: neighbouring lanes take the two planes of one entry, so
// that an atomic instruction covers whole cache lines.
template <typename T, class F>
__device__ __forceinline__ void scatter_lower(const DevPlan &pl, int64_t rp, int c, int i0, int k0, const double *smem,
                                              T *base, F f) {
  constexpr int P = Planes<T>::P, Q = 64 * 64 / NT;
  const int lane = threadIdx.x & 63, w = uniform((int)(threadIdx.x >> 6)), p = P == 2 ? lane & 1 : 0;
  int64_t col[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) col[q] = uniform64(gp(pl.kcol)[rp + min(k0 + w + 4 * q, c - 1)]);
#pragma unroll
  for (int h = 0; h < P; ++h) {
    const int i = lane / P + 64 / P * h, ig = i0 + i;
    int32_t pos[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int kg = k0 + w + 4 * q;
      pos[q] = gp(pl.posarr)[(gp(pl.kpos)[rp + min(kg, c - 1)] + ig) & opaque_mask(ig < c && kg < c && ig >= kg)];
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int kg = k0 + w + 4 * q;
      if (ig < c && kg < c && ig >= kg)
        unsafeAtomicAdd(reinterpret_cast<double *>(base + col[q] + pos[q]) + p,
                        f(smem[p * 64 * PITCH + (w + 4 * q) * PITCH + i], ig == kg));
    }
  }
}

// Block (a, b), a >= b, of X_{C,C} for a node with a dense buffer G (column
// major, leading dimension ldg): element (i, k), i >= k, is the lower-part
// entry Src[kcol[k] + posarr[kpos[k] + i]] of the ancestor owning column k
// (Src: the X panels, or any array in the same panel layout); it is written
// to G(i, k) and G(k, i) (conjugated in a Hermitian plan; in an LU plan G(k, i)
// is the entry at the same position of the second panel set, X^T).  Lanes run
// along i (one column k per wave and step) for the gather and the G(i, k)
// stores; the mirror stores go through an LDS transpose so that they are
// contiguous too.
// MAYBE_LU = false: for kernels that never run an LU plan.
template <typename T, bool MAYBE_LU>
__device__ void do_gtile(const Ctx<T> &cx, const NodeInfo &nd, int a, int b, double *smem, int64_t *rt, const T *Src) {
  const DevPlan &pl = *cx.pl;
  const int c = uniform(nd.c);
  const int64_t rp = nd.rp;
  const int ldg = nd.ldg;
  T *G = cx.Gp + nd.goff;
  const int i0 = a * 64, k0 = b * 64;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  constexpr int Q = 64 * 64 / NT;
  // three dependent rounds: the gather tables of the block's 64 columns (into
  // LDS), the positions of all of a thread's elements, then their values.
  // Element q of a thread: row i = i0 + lane, column k = k0 + w + 4 q.
  if (threadIdx.x < 64) {
    const int k = k0 + threadIdx.x;
    const int64_t kq = k < c ? k : 0;
    rt[threadIdx.x] = gp(pl.kcol)[rp + kq];
    rt[64 + threadIdx.x] = gp(pl.kpos)[rp + kq];
  }
  lds_barrier();
  const int i = i0 + lane;
  int32_t pos[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int kl = w + 4 * q, k = k0 + kl;
    pos[q] = gp(pl.posarr)[(rt[64 + kl] + i) & opaque_mask(i < c && k < c && i >= k)];
  }
  T v[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int kl = w + 4 * q, k = k0 + kl;
    v[q] = Mem<false>::ld(Src + ((rt[kl] + (int64_t)pos[q]) & opaque_mask(i < c && k < c && i >= k)));
  }
  const bool lu = MAYBE_LU && uniform(pl.half > 0 ? 1 : 0) != 0;
  if (lu) {  // the mirror values: the same positions of the X^T set
    T u[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int kl = w + 4 * q, k = k0 + kl;
      u[q] = Mem<false>::ld(Src + pl.half + ((rt[kl] + (int64_t)pos[q]) & opaque_mask(i < c && k < c && i >= k)));
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int kl = w + 4 * q, k = k0 + kl;
      const bool ok = i < c && k < c && i >= k;
      lds_put<T>(smem, lane, kl, masked(u[q], opaque_mask(ok)));
      if (ok) Mem<false>::st(G + (int64_t)k * ldg + i, masked(v[q], opaque_mask(ok)));
    }
  } else {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int kl = w + 4 * q, k = k0 + kl;
      const bool ok = i < c && k < c && i >= k;
      const T x = masked(v[q], opaque_mask(ok));
      lds_put<T>(smem, lane, kl, x);  // tile[i][k] at smem[k * PITCH + i]
      if (ok) Mem<false>::st(G + (int64_t)k * ldg + i, x);
    }
  }
  lds_barrier();
  // mirror: G(k, i) = tile[i][k] (its conjugate if Hermitian; the X^T entry
  // in an LU plan), lanes along k; a lower-only buffer keeps the mirrors of
  // diagonal blocks alone
  const double cs = lu ? 1.0 : pl.csign;
  if (uniform(nd.glow != 0 && a != b ? 0 : 1)) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int e = threadIdx.x + NT * q;
      const int kl = e & 63, il = e >> 6, i = i0 + il, k = k0 + kl;
      if (i < c && k < c && i > k) Mem<false>::st(G + (int64_t)i * ldg + k, cj(lds_get<T>(smem, il, kl), cs));
    }
  }
  lds_barrier();
}

// Store -acc (a 64 x 64 tile of X_{C,K} = -X_{C,C} Lhat) into X, rows 64a..
// of C(K) and columns 64b.. of K, through LDS so that the stores coalesce.
template <typename T, bool COH>
__device__ void store_xtile(const Ctx<T> &cx, const NodeInfo &nd, int a, int b, const Acc<T> &acc, double *smem) {
  const DevPlan &pl = *cx.pl;
  const int s = nd.s, c = nd.c, ld = s + c;
  const int64_t off = nd.off;
  const int i0 = a * 64, j0 = b * 64;
  acc_to_lds<T>(acc, smem);
  lds_barrier();
  for (int e = threadIdx.x; e < 64 * 64; e += NT) {
    const int i = e & 63, j = e >> 6;
    if (i0 + i < c && j0 + j < s)
      Mem<COH>::st(cx.Xp + off + (int64_t)(j0 + j) * ld + s + i0 + i, SOps<T>::scale(-1.0, lds_get<T>(smem, i, j)));
  }
  lds_barrier();
}

// R[p][j * PITCH + x] = (Ls^T acc)(x, j) for a 64 x 64 block: Ls holds
// Lhat[tile rows i, 64 columns x] as Ls[p][i * PITCH + x] (already in LDS,
// barrier done); acc is a 64 x 64 GEMM-1 tile in the accumulator layout,
// which is the MFMA B-operand layout for a contraction over the tile rows
// (register v of a 16 x 16 block holds rows 4v..4v+3 of lanes l / 16).  R
// overwrites Ls; ends with a barrier.  The 64 columns x run in parts of
// 16 XB (all 64 for FP64, 16 for complex, whose three product chains per
// block take more registers): R's columns of a part overwrite Ls's, which
// only that part reads.  Complex products take three real chains (see
// Acc3M), or four where G3 is false.
template <typename T, bool G3 = true>
__device__ void gemm2_block(const Acc<T> &acc, double *Ls) {
  constexpr int P = Planes<T>::P, C = P == 2 && G3 ? 3 : P;  // accumulators of a block
  constexpr int XB = P == 1 ? 4 : 1;                   // 16-column blocks per part
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int wi = w & 1, wj = w >> 1;
#pragma unroll 1
  for (int h = 0; h < 4 / XB; ++h) {
    d4 pacc[C][XB][2];
#pragma unroll
    for (int q = 0; q < C; ++q)
#pragma unroll
      for (int xb = 0; xb < XB; ++xb)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj) pacc[q][xb][bj] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int k4 = 0; k4 < 4; ++k4) {
        const int row = 32 * wi + 16 * bi + 4 * k4 + (lane >> 4);
#pragma unroll
        for (int xb = 0; xb < XB; ++xb) {
          const int x = 16 * (XB * h + xb) + (lane & 15);
          if constexpr (P == 1) {
            const double af = Ls[row * PITCH + x];
#pragma unroll
            for (int bj = 0; bj < 2; ++bj) pacc[0][xb][bj] = mfma16(af, acc.v[0][bi][bj][k4], pacc[0][xb][bj]);
          } else {
            const double a0 = Ls[row * PITCH + x], a1 = Ls[64 * PITCH + row * PITCH + x];
#pragma unroll
            for (int bj = 0; bj < 2; ++bj) {
              const double b0 = acc.v[0][bi][bj][k4], b1 = acc.v[1][bi][bj][k4];
              pacc[0][xb][bj] = mfma16(a0, b0, pacc[0][xb][bj]);
              if constexpr (C == 3) {
                pacc[1][xb][bj] = mfma16(a1, b1, pacc[1][xb][bj]);
                pacc[2][xb][bj] = mfma16(a0 + a1, b0 + b1, pacc[2][xb][bj]);
              } else {
                pacc[1][xb][bj] = mfma16(a0, b1, pacc[1][xb][bj]);
                pacc[0][xb][bj] = mfma16(-a1, b1, pacc[0][xb][bj]);
                pacc[1][xb][bj] = mfma16(a1, b0, pacc[1][xb][bj]);
              }
            }
          }
        }
      }
    lds_barrier();
    // sum the two row halves (wi = 0, 1) into R's columns of this part
    double *R = Ls;
    for (int part = 0; part < 2; ++part) {
      if (wi == part) {
#pragma unroll
        for (int xb = 0; xb < XB; ++xb)
#pragma unroll
          for (int bj = 0; bj < 2; ++bj) {
            d4 out[P];
            if constexpr (C == 3) {
              out[0] = pacc[0][xb][bj] - pacc[1][xb][bj];
              out[1] = pacc[2][xb][bj] - pacc[0][xb][bj] - pacc[1][xb][bj];
            } else {
#pragma unroll
              for (int p = 0; p < P; ++p) out[p] = pacc[p][xb][bj];
            }
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
              for (int v = 0; v < 4; ++v) {
                const int x = 16 * (XB * h + xb) + 4 * v + (lane >> 4);
                const int j = 32 * wj + 16 * bj + (lane & 15);
                double &r = R[p * 64 * PITCH + j * PITCH + x];
                r = part == 0 ? out[p][v] : r + out[p][v];
              }
          }
      }
      lds_barrier();
    }
  }
}

// Row tile a's share of GEMM-2 (Alg. 1 step 4): P_a[:, 64b..] = Lhat[rows of
// tile a, :]^T Y[tile a, 64b..] = -(Lhat_a^T acc) (^H in a Hermitian plan;
// Uhat_{K,C} of the U^T panel set in place of Lhat^T in an LU plan),
// written to the partial buffer (column-major s x s per row tile); rows
// 64qb .. 64qe - 1 of P_a only.  PF: load the next 64 columns of Lhat while
// the current block is multiplied (off in kernels that rely on occupancy
// instead, so that the prefetch registers do not cost a workgroup per CU).
template <typename T, bool COH, bool PF = true, bool G3 = true>
__device__ void gemm2_partial(const Ctx<T> &cx, const NodeInfo &nd, int a, int b, const Acc<T> &acc, double *smem,
                              int qb = 0, int qe = 1 << 20) {
  constexpr int P = Planes<T>::P;
  const DevPlan &pl = *cx.pl;
  const int s = nd.s, c = nd.c, ld = s + c;
  const int64_t off = nd.off;
  const int i0 = a * 64, j0 = b * 64;
  const int64_t pbase = nd.poff + (int64_t)a * s * s;
  double *Ls = smem;  // Lhat[i0 .. i0+63, q0 .. q0+63] as Ls[p][i * PITCH + x]
  // the next 64 columns of Lhat are loaded while the current block is multiplied
  T lv[64 * 64 / NT];
  auto load_l = [&](int q0) {
#pragma unroll
    for (int q = 0; q < 64 * 64 / NT; ++q) {
      const int e = threadIdx.x + NT * q;
      const int i = e & 63, x = e >> 6;
      lv[q] = gload(cx.Lp + pl.half + off + (((int64_t)(q0 + x) * ld + s + i0 + i) & opaque_mask(i0 + i < c && q0 + x < s)));
    }
  };
  const int qend = min(s, qe * 64);
  const double cs = pl.csign;
  if (PF) load_l(qb * 64);
  for (int q0 = qb * 64; q0 < qend; q0 += 64) {
    if (!PF) load_l(q0);
#pragma unroll
    for (int q = 0; q < 64 * 64 / NT; ++q) {
      const int e = threadIdx.x + NT * q;
      const int i = e & 63, x = e >> 6;
      const T v = cj(masked(lv[q], opaque_mask(i0 + i < c && q0 + x < s)), cs);
#pragma unroll
      for (int p = 0; p < P; ++p) Ls[p * 64 * PITCH + i * PITCH + x] = Planes<T>::get(v, p);
    }
    lds_barrier();
    if (PF && q0 + 64 < qend) load_l(q0 + 64);
    gemm2_block<T, G3>(acc, Ls);
    // P = Lhat^T Y = -(Lhat^T acc)
    const double *R = Ls;
    for (int e = threadIdx.x; e < 64 * 64; e += NT) {
      const int x = e & 63, j = e >> 6;
      if (q0 + x < s && j0 + j < s)
        Mem<COH>::st(cx.Pp + pbase + (int64_t)(j0 + j) * s + q0 + x, SOps<T>::scale(-1.0, lds_get<T>(R, x, j)));
    }
    lds_barrier();
  }
}

// GEMM-1 tile, rows 64a.. and columns 64b.. of X_{C,K} (Alg. 1 step 3):
//   acc = X_{C,C}[tile rows, k] Lhat_{C,K}[k, tile columns], k in this part's
// share of [0, c).  A node without an R phase stores Y = -acc into X and its
// row tile's share of GEMM-2 (step 4); otherwise acc is stored as a partial
// tile (a split node's parts, or the one part of a node whose GEMM-2 shares
// are cut into R items).
template <typename T, bool COH>
__device__ void do_ytile(const Ctx<T> &cx, const NodeInfo &nd, int a, int bp, double *smem, int64_t *rt) {
  const DevPlan &pl = *cx.pl;
  const int s = uniform(nd.s), c = uniform(nd.c), ld = s + c;
  const int64_t off = nd.off, rp = nd.rp;
  const int64_t goff = nd.goff;
  const int b = bp & 0xffff, part = bp >> 16;
  const int parts = uniform(nd.split), kchunk = uniform(nd.kchunk);
  const int kb = part * kchunk, ke = min(c, kb + kchunk);
  const int i0 = a * 64, j0 = b * 64;
  Acc<T> acc;
  if (uniform(goff >= 0 ? 1 : 0)) {  // X_{C,C} already gathered into the dense buffer
    constexpr int TK = DenseTK<T>::TK;
    const T *G = static_cast<const T *>(cx.Gp) + goff;
    LoadDenseA<T, TK> la{G, nd.ldg, c, ke, i0};
    LoadDenseB<T, TK> lb{cx.Lp, off, ld, s, ke, j0, s};
    gemm_dense<T>(kb, ke, la, lb, smem, acc);
  } else {
    if (threadIdx.x < 64) {
      const int ig = i0 + threadIdx.x;
      rt[threadIdx.x] = gp(pl.kcol)[rp + (ig < c ? ig : 0)];
      rt[64 + threadIdx.x] = gp(pl.kpos)[rp + (ig < c ? ig : 0)];
    }
    lds_barrier();
    LoadGather<T, COH> la{cx.Xp, pl.kcol + rp, pl.kpos + rp, pl.posarr, rt, rt + 64, c, ke, i0};
    la.cs = pl.csign;
    LoadPanelK<T, false> lb{cx.Lp, off, ld, s, 0, ke, j0, s};
    gemm_tile<T>(kb, ke, la, lb, smem, acc);
  }
  if (nd.yoff < 0) {
    store_xtile<T, COH>(cx, nd, a, b, acc, smem);
    if (!uniform(nd.defer2)) gemm2_partial<T, COH>(cx, nd, a, b, acc, smem);
    return;
  }
  // partial tile of a node with an R phase: Ypart[part] (column-major c x s)
  T *Y = static_cast<T *>(cx.Yp) + nd.yoff + (int64_t)part * c * s;
  acc_to_lds<T>(acc, smem);
  lds_barrier();
  for (int e = threadIdx.x; e < 64 * 64; e += NT) {
    const int i = e & 63, j = e >> 6;
    if (i0 + i < c && j0 + j < s) Mem<COH>::st(Y + (int64_t)(j0 + j) * c + i0 + i, lds_get<T>(smem, i, j));
  }
  lds_barrier();
}

// The gathered GEMM-1 tile of the level schedule's k_ygather: do_ytile without
// the dense-buffer form, and (up) the tile of an LU plan's upper part, rows
// 64a.. and columns 64b.. of X_{K,C}^T = -(X_{C,C})^T Uhat^T, gathered with the
// two X panel sets exchanged and stored into the second (it has no GEMM-2
// share: A^{-1}_{K,K} needs only X_{C,K}).
template <typename T>
__device__ __forceinline__ void do_ygather(const Ctx<T> &cx, const NodeInfo &nd, int a, int bp, bool up, double *smem,
                                           int64_t *rt) {
  const DevPlan &pl = *cx.pl;
  const int s = nd.s, c = nd.c, ld = s + c;
  const int64_t rp = nd.rp;
  const int b = bp & 0xffff, part = bp >> 16;
  const int kb = part * nd.kchunk, ke = min(c, kb + nd.kchunk);
  const int i0 = a * 64, j0 = b * 64;
  if (threadIdx.x < 64) {
    const int ig = i0 + threadIdx.x;
    rt[threadIdx.x] = gp(pl.kcol)[rp + (ig < c ? ig : 0)];
    rt[64 + threadIdx.x] = gp(pl.kpos)[rp + (ig < c ? ig : 0)];
  }
  lds_barrier();
  // LU plans: X_{C,C}'s upper part from the X^T panel set; the upper tiles
  // exchange the two sets (X_{C,C} transposed) and read Uhat^T
  const int64_t hs = up ? pl.half : 0;
  LoadGather<T, false> la{cx.Xp + hs, pl.kcol + rp, pl.kpos + rp, pl.posarr, rt, rt + 64, c, ke, i0};
  la.cs = pl.csign;
  la.du = up ? -pl.half : pl.half;
  LoadPanelK<T, false> lb{cx.Lp + hs, nd.off, ld, s, 0, ke, j0, s};
  Acc<T> acc;
  gemm_tile<T>(kb, ke, la, lb, smem, acc);
  acc_to_lds<T>(acc, smem);
  lds_barrier();
  if (nd.yoff < 0) {  // Y = -acc into X_{C,K} (up: the second set)
    T *X = cx.Xp + hs + nd.off + s;
    for (int e = threadIdx.x; e < 64 * 64; e += NT) {
      const int i = e & 63, j = e >> 6;
      if (i0 + i < c && j0 + j < s) gstore(X + (int64_t)(j0 + j) * ld + i0 + i, SOps<T>::scale(-1.0, lds_get<T>(smem, i, j)));
    }
    if (!up && !nd.defer2) {
      lds_barrier();
      gemm2_partial<T, false, Planes<T>::P == 1>(cx, nd, a, b, acc, smem);
    }
  } else {  // partial tile Ypart[part] (column-major c x s)
    T *Y = static_cast<T *>(cx.Yp) + nd.yoff + (int64_t)part * c * s;
    for (int e = threadIdx.x; e < 64 * 64; e += NT) {
      const int i = e & 63, j = e >> 6;
      if (i0 + i < c && j0 + j < s) gstore(Y + (int64_t)(j0 + j) * c + i0 + i, lds_get<T>(smem, i, j));
    }
  }
}

// Rows i0 .. i0 + 63, columns [j0, j1) of X_{C,K} from a split node's partial tiles.
template <typename T>
__device__ __forceinline__ void sum_columns(const Ctx<T> &cx, const NodeInfo &nd, int i0, int j0, int j1) {
  const int s = nd.s, c = nd.c, parts = nd.split;
  constexpr int U = 4, PB = 4 / Planes<T>::P;  // columns of a wavefront, parts per round trip
  const int i = i0 + (int)(threadIdx.x & 63), w = uniform((int)(threadIdx.x >> 6));
  const uint32_t row = (uint32_t)(i < c ? i : 0) * (uint32_t)sizeof(T);
  const T *Y = static_cast<const T *>(cx.Yp) + nd.yoff;
  T *X = cx.Xp + nd.off + s + i;
  for (int j = j0 + w; j < j1; j += U * (NT / 64)) {
    T sum[U];
#pragma unroll
    for (int u = 0; u < U; ++u) sum[u] = zero_of<T>();
    for (int p0 = 0; p0 < parts; p0 += PB) {
      T v[PB][U];
#pragma unroll
      for (int p = 0; p < PB; ++p)
#pragma unroll
        for (int u = 0; u < U; ++u)
          v[p][u] = ld_off(Y + ((int64_t)min(p0 + p, parts - 1) * s + min(j + u * (NT / 64), j1 - 1)) * c, row);
#pragma unroll
      for (int p = 0; p < PB; ++p) {
        if (p > 0 && p0 + p >= parts) break;
#pragma unroll
        for (int u = 0; u < U; ++u) sum[u] += v[p][u];
      }
    }
    if (i < c)
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (j + u * (NT / 64) < j1) gstore(X + (int64_t)(j + u * (NT / 64)) * (s + c), SOps<T>::scale(-1.0, sum[u]));
  }
}

// Sum of a split node's partial tiles (a, b) into X, then the row tile's share
// of GEMM-2 (the step-3 and step-4 work that an unsplit tile does itself).
// With br = b | r << 16 | rq << 24 and rq > 1, the tile's GEMM-2 share is cut
// into rq items by rows of P_a: item r computes 64-row blocks [r nq / rq,
// (r + 1) nq / rq) of the nq = ceil(s / 64), and item 0 alone stores the tile.
// Every item sums the parts in the same order, so the result is the same.
template <typename T, bool COH, bool PF = true>
__device__ void do_rtile(const Ctx<T> &cx, const NodeInfo &nd, int a, int br, double *smem) {
  const DevPlan &pl = *cx.pl;
  const int s = uniform(nd.s), c = uniform(nd.c);
  const int b = br & 0xffff, r = (br >> 16) & 0xff, rq = max(1, br >> 24);
  const int nq = (s + 63) / 64, qb = uniform(r * nq / rq), qe = uniform((r + 1) * nq / rq);
  const int parts = uniform(nd.split);
  const T *Y = static_cast<const T *>(cx.Yp) + nd.yoff;
  const int i0 = a * 64, j0 = b * 64;
  if constexpr (!COH) {
    if (uniform(nd.g2)) {  // the sum alone: columns [64 r / rq, 64 (r + 1) / rq) of the tile
      sum_columns<T>(cx, nd, i0, j0 + 64 * r / rq, min(s, j0 + 64 * (r + 1) / rq));
      return;
    }
  }
  constexpr int Q = 64 * 64 / NT;
  T sum[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) sum[q] = zero_of<T>();
  // the loads of PB parts are issued together; the sum runs over p in order
  constexpr int PB = 2 / Planes<T>::P;
  for (int p0 = 0; p0 < parts; p0 += PB) {
    T v[PB][Q];
#pragma unroll
    for (int pp = 0; pp < PB; ++pp) {
      const int64_t pbase = (int64_t)min(p0 + pp, parts - 1) * c * s;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int e = threadIdx.x + NT * q;
        const int i = e & 63, j = e >> 6;
        v[pp][q] = Mem<COH>::ld(Y + pbase + (((int64_t)(j0 + j) * c + i0 + i) & opaque_mask(i0 + i < c && j0 + j < s)));
      }
    }
#pragma unroll
    for (int pp = 0; pp < PB; ++pp) {
      const int64_t m = opaque_mask(p0 + pp < parts);
#pragma unroll
      for (int q = 0; q < Q; ++q) sum[q] += masked(v[pp][q], m);
    }
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int e = threadIdx.x + NT * q;
    const int i = e & 63, j = e >> 6;
    lds_put<T>(smem, i, j, masked(sum[q], opaque_mask(i0 + i < c && j0 + j < s)));
  }
  lds_barrier();
  // into the accumulator layout of the MFMA tile
  constexpr int P = Planes<T>::P;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int wi = w & 1, wj = w >> 1;
  Acc<T> acc;
#pragma unroll
  for (int p = 0; p < P; ++p)
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int bj = 0; bj < 2; ++bj)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int i = 32 * wi + 16 * bi + 4 * v + (lane >> 4);
          const int j = 32 * wj + 16 * bj + (lane & 15);
          acc.v[p][bi][bj][v] = smem[p * 64 * PITCH + j * PITCH + i];
        }
  lds_barrier();
  if (r == 0) store_xtile<T, COH>(cx, nd, a, b, acc, smem);
  gemm2_partial<T, COH, PF>(cx, nd, a, b, acc, smem, qb, qe);
}

// The GEMM-2 share of a tile whose GEMM-1 item stored Y = X_{C,K} (rows 64a..,
// columns 64b..) without it: the tile is read back from X into the
// accumulator layout (acc = -Y) and gemm2_partial computes 64-row blocks
// [qb, qe) of P_a, with br = b | r << 16 | rq << 24 as for do_rtile.
template <typename T, bool COH, bool PF = true>
__device__ void do_ptile(const Ctx<T> &cx, const NodeInfo &nd, int a, int br, double *smem) {
  const int s = uniform(nd.s), c = uniform(nd.c), ld = s + c;
  const int b = br & 0xffff, r = (br >> 16) & 0xff, rq = max(1, br >> 24);
  const int nq = (s + 63) / 64, qb = uniform(r * nq / rq), qe = uniform((r + 1) * nq / rq);
  const int i0 = a * 64, j0 = b * 64;
  const T *Y = cx.Xp + nd.off + s;
  constexpr int Q = 64 * 64 / NT;
  T v[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int e = threadIdx.x + NT * q;
    const int i = e & 63, j = e >> 6;
    v[q] = Mem<COH>::ld(Y + (((int64_t)(j0 + j) * ld + i0 + i) & opaque_mask(i0 + i < c && j0 + j < s)));
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int e = threadIdx.x + NT * q;
    const int i = e & 63, j = e >> 6;
    lds_put<T>(smem, i, j, SOps<T>::scale(-1.0, masked(v[q], opaque_mask(i0 + i < c && j0 + j < s))));
  }
  lds_barrier();
  constexpr int P = Planes<T>::P;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int wi = w & 1, wj = w >> 1;
  Acc<T> acc;
#pragma unroll
  for (int p = 0; p < P; ++p)
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int bj = 0; bj < 2; ++bj)
#pragma unroll
        for (int vv = 0; vv < 4; ++vv) {
          const int i = 32 * wi + 16 * bi + 4 * vv + (lane >> 4);
          const int j = 32 * wj + 16 * bj + (lane & 15);
          acc.v[p][bi][bj][vv] = smem[p * 64 * PITCH + j * PITCH + i];
        }
  lds_barrier();
  gemm2_partial<T, COH, PF>(cx, nd, a, b, acc, smem, qb, qe);
}

// GEMM-1 tile of a node with a dense X_{C,C} buffer: the level schedule runs
// these in k_ydense (dense loaders only, so fewer registers than the general
// item kernel: two workgroups per CU).  An unsplit tile goes to X and then, in
// a node whose GEMM-2 is not a product of its own (k_gemm2_dense), adds its
// GEMM-2 share from the registers; a 128 x 128 tile leaves that share to
// ITEM_P items, and a split contraction writes partial tiles that ITEM_R items
// sum.
// LU plans: up (an ITEM_YU tile) takes X_{K,C}^T = -(X_{C,C})^T Uhat^T from
// the transposed full buffer and the second panel sets.
template <typename T>
__device__ __forceinline__ void do_ytile_dense(const Ctx<T> &cx, const NodeInfo &nd, int a, int bp, bool up,
                                               double *smem) {
  const int s = uniform(nd.s), c = uniform(nd.c), ld = s + c;
  const int b = bp & 0xffff, part = bp >> 16;
  const int kchunk = uniform(nd.kchunk);
  const int kb = part * kchunk, ke = min(c, kb + kchunk);
  const int i0 = a * 64, j0 = b * 64;
  constexpr int TK = DenseTK<T>::TK;
  const int64_t hs = up ? cx.pl->half : 0;
  const T *G = static_cast<const T *>(cx.Gp) + nd.goff;
  // a lower-only buffer (see the plan) mirrors the stages right of the
  // diagonal block; a full one (LU) reads as is, or transposed for up
  const int kmir = nd.glow ? i0 + 64 : up ? 0 : 1 << 30;
  LoadDenseASym<T, TK> la{G, nd.ldg, c, ke, i0, uniform(kmir)};
  la.cs = cx.pl->csign;
  LoadDenseB<T, TK> lb{cx.Lp + hs, nd.off, ld, s, ke, j0, s};
  Acc<T> acc;
  gemm_dense_il<T, true>(kb, ke, la, lb, smem, acc);  // complex: three real product chains
  acc_to_lds<T>(acc, smem);
  lds_barrier();
  if (nd.yoff < 0) {  // Y = -acc into X_{C,K} (LU up: the second set)
    T *X = cx.Xp + hs + nd.off + s;
    for (int e = threadIdx.x; e < 64 * 64; e += NT) {
      const int i = e & 63, j = e >> 6;
      if (i0 + i < c && j0 + j < s) gstore(X + (int64_t)(j0 + j) * ld + i0 + i, SOps<T>::scale(-1.0, lds_get<T>(smem, i, j)));
    }
    // the row tile's GEMM-2 share (Alg. 1 step 4) from the tile still in
    // registers, unless the plan runs it elsewhere (the LU upper part has none)
    if (!up && !uniform(nd.defer2)) {
      lds_barrier();
      gemm2_partial<T, false, Planes<T>::P == 1>(cx, nd, a, b, acc, smem);
    }
  } else {  // partial tile Ypart[part] (column-major c x s)
    T *Y = static_cast<T *>(cx.Yp) + nd.yoff + (int64_t)part * c * s;
    for (int e = threadIdx.x; e < 64 * 64; e += NT) {
      const int i = e & 63, j = e >> 6;
      if (i0 + i < c && j0 + j < s) gstore(Y + (int64_t)(j0 + j) * c + i0 + i, lds_get<T>(smem, i, j));
    }
  }
}

// GEMM-2 tile: rows 64 a .. and columns 64 b .. of P = Lhat^T X_{C,K} over the
// row range `part` of np (LU: Uhat X_{C,K}), into the node's partial product
// `part`.  Both operands run along the contraction.
template <typename T>
__device__ __forceinline__ void do_gemm2(const Ctx<T> &cx, const NodeInfo &nd, int a, int b, int part, double *smem) {
  const int s = uniform(nd.s), c = uniform(nd.c), ld = s + c;
  const int nr = (c + 63) / 64, ct = 64 * ((nr + nd.np - 1) / nd.np);  // rows of a range
  const int kb = part * ct, ke = min(c, kb + ct);
  constexpr int TK = DenseTK<T>::TK;
  LoadDenseBC<T, TK> la{cx.Lp + cx.pl->half, nd.off, ld, s, ke, 64 * a, s};
  la.cs = cx.pl->csign;
  LoadDenseB<T, TK> lb{cx.Xp, nd.off, ld, s, ke, 64 * b, s};
  Acc<T> acc;
  gemm_dense_il<T, true>(kb, ke, la, lb, smem, acc);
  acc_to_lds<T>(acc, smem);
  lds_barrier();
  T *P = cx.Pp + nd.poff + (int64_t)part * s * s;
  for (int e = threadIdx.x; e < 64 * 64; e += NT) {
    const int x = e & 63, j = e >> 6;
    if (64 * a + x < s && 64 * b + j < s) gstore(P + (int64_t)(64 * b + j) * s + 64 * a + x, lds_get<T>(smem, x, j));
  }
}

// Blocks (a, b) and (b, a), a >= b, of sym(Src - sum_r P_r) into Dst, where
// Src and Dst are s x s column-major with leading dimensions sld and dld and
// P_r are the node's np partial products.
template <typename T, bool COH>
__device__ void dtile_core(const Ctx<T> &cx, const NodeInfo &nd, int a, int b, double *smem, const T *Dti, int sld, T *Xkk,
                           int dld) {
  const int s = nd.s;
  const int nr = nd.np;
  const int64_t pb = nd.poff;
  const int64_t ss = (int64_t)s * s;
  const int a0 = a * 64, b0 = b * 64;
  double *Sab = smem, *Sba = smem + tile_doubles<T>();
  // T[a0 + i, b0 + j] into Sab[i][j] and T[b0 + i, a0 + j] into Sba[i][j].
  // Each thread owns 16 elements of each block, taken in two halves of 8;
  // for every row tile the 16 loads of a half are issued together.
  constexpr int Q = 64 * 64 / NT, QH = Q / 2;
  const int ie = threadIdx.x & 63, jb = threadIdx.x >> 6;  // element (ie, jb + 4 q)
  for (int h = 0; h < 2; ++h) {
    T sab[QH], sba[QH];
    int64_t mab[QH], mba[QH];
#pragma unroll
    for (int q = 0; q < QH; ++q) {
      const int j = jb + 4 * (QH * h + q);
      sab[q] = zero_of<T>();
      sba[q] = zero_of<T>();
      mab[q] = opaque_mask(a0 + ie < s && b0 + j < s);
      mba[q] = opaque_mask(b0 + ie < s && a0 + j < s);
    }
    // two row tiles per round trip: their 32 loads are issued together
    for (int r = 0; r < nr; r += 2) {
      const T *pr0 = cx.Pp + pb + r * ss;
      const T *pr1 = cx.Pp + pb + min(r + 1, nr - 1) * ss;
      const int64_t m1 = opaque_mask(r + 1 < nr);
      T la0[QH], lb0[QH], la1[QH], lb1[QH];
#pragma unroll
      for (int q = 0; q < QH; ++q) {
        const int j = jb + 4 * (QH * h + q);
        la0[q] = Mem<COH>::ld(pr0 + (((int64_t)(b0 + j) * s + a0 + ie) & mab[q]));
        lb0[q] = Mem<COH>::ld(pr0 + (((int64_t)(a0 + j) * s + b0 + ie) & mba[q]));
        la1[q] = Mem<COH>::ld(pr1 + (((int64_t)(b0 + j) * s + a0 + ie) & mab[q]));
        lb1[q] = Mem<COH>::ld(pr1 + (((int64_t)(a0 + j) * s + b0 + ie) & mba[q]));
      }
#pragma unroll
      for (int q = 0; q < QH; ++q) {
        sab[q] += la0[q] + masked(la1[q], m1);
        sba[q] += lb0[q] + masked(lb1[q], m1);
      }
    }
#pragma unroll
    for (int q = 0; q < QH; ++q) {
      const int j = jb + 4 * (QH * h + q);
      const T dab = gload(Dti + (((int64_t)(b0 + j) * sld + a0 + ie) & mab[q]));
      const T dba = gload(Dti + (((int64_t)(a0 + j) * sld + b0 + ie) & mba[q]));
      lds_put<T>(Sab, ie, j, masked(dab - sab[q], mab[q]));
      lds_put<T>(Sba, ie, j, masked(dba - sba[q], mba[q]));
    }
  }
  lds_barrier();
  // x(i, j) = (T[a0+i, b0+j] + T[b0+j, a0+i]) / 2 (the second term conjugated
  // in a Hermitian plan); keep it in Sab
  const double cs = cx.pl->csign;
  T xv[64 * 64 / NT];
#pragma unroll
  for (int q = 0; q < 64 * 64 / NT; ++q) {
    const int e = threadIdx.x + NT * q;
    const int i = e & 63, j = e >> 6;
    xv[q] = SOps<T>::scale(0.5, lds_get<T>(Sab, i, j) + cj(lds_get<T>(Sba, j, i), cs));
  }
  lds_barrier();
#pragma unroll
  for (int q = 0; q < 64 * 64 / NT; ++q) {
    const int e = threadIdx.x + NT * q;
    lds_put<T>(Sab, e & 63, e >> 6, xv[q]);
  }
  lds_barrier();
  for (int e = threadIdx.x; e < 64 * 64; e += NT) {
    const int i = e & 63, j = e >> 6;
    if (a0 + i < s && b0 + j < s) Mem<COH>::st(Xkk + (int64_t)(b0 + j) * dld + a0 + i, lds_get<T>(Sab, i, j));
    if (a != b && b0 + i < s && a0 + j < s)
      Mem<COH>::st(Xkk + (int64_t)(a0 + j) * dld + b0 + i, cj(lds_get<T>(Sab, j, i), cs));
  }
  lds_barrier();
}

// The same as dtile_core for the column slab [b0 + kDSlabW sl, b0 +
// kDSlabW (sl + 1)) of block (a, b) only (and the matching row slab of block
// (b, a)): with a quarter of the elements per thread, the loads of several row
// tiles' partials are in flight together, and two LDS slabs are all it needs
// (rows of the second one a pitch of kDSlabW + 1 apart: it is read by columns).
constexpr int kDSlabP = kDSlabW + 1;
template <typename T> __device__ __forceinline__ constexpr int dslab_elems() { return 64 * kDSlabW + 64 * kDSlabP; }
template <typename T>
__device__ void dtile_slab(const Ctx<T> &cx, const NodeInfo &nd, int a, int b, int sl, T *smem, const T *Dti, int sld, T *Xkk,
                           int dld) {
  constexpr int W = kDSlabW, WP = kDSlabP, QE = 64 * W / NT;
  constexpr int R = Planes<T>::P == 1 ? 4 : 2;  // row tiles per round trip
  const DevPlan &pl = *cx.pl;
  const int s = nd.s;
  const int nr = uniform(nd.np);
  const int64_t pb = nd.poff;
  const int64_t ss = (int64_t)s * s;
  const int a0 = a * 64, b0 = b * 64 + sl * W;
  // element q of a thread: (i, j) = (e % 64, e / 64) of the (a, b) slab, and
  // (j', i') = (e % W, e / W) of the (b, a) slab, e = threadIdx.x + NT q
  uint32_t oab[QE], oba[QE];  // byte offsets in an s x s block
  T sab[QE], sba[QE];
#pragma unroll
  for (int q = 0; q < QE; ++q) {
    const int e = threadIdx.x + NT * q;
    const int ia = e % 64, ja = e / 64, jb = e % W, ib = e / W;
    oab[q] = ((uint32_t)((b0 + ja) * s + a0 + ia) & opaque_mask32(a0 + ia < s && b0 + ja < s)) * (uint32_t)sizeof(T);
    oba[q] = ((uint32_t)((a0 + ib) * s + b0 + jb) & opaque_mask32(b0 + jb < s && a0 + ib < s)) * (uint32_t)sizeof(T);
    sab[q] = zero_of<T>();
    sba[q] = zero_of<T>();
  }
  for (int r = 0; r < nr; r += R) {
    T la[R][QE], lb[R][QE];
#pragma unroll
    for (int rr = 0; rr < R; ++rr) {
      const T *pr = cx.Pp + pb + min(r + rr, nr - 1) * ss;
#pragma unroll
      for (int q = 0; q < QE; ++q) {
        la[rr][q] = ld_off(pr, oab[q]);
        lb[rr][q] = ld_off(pr, oba[q]);
      }
    }
#pragma unroll
    for (int rr = 0; rr < R; ++rr) {
      if (rr > 0 && r + rr >= nr) break;
#pragma unroll
      for (int q = 0; q < QE; ++q) {
        sab[q] += la[rr][q];
        sba[q] += lb[rr][q];
      }
    }
  }
  T *Sab = smem;            // [i + 64 j]
  T *Sba = Sab + 64 * W;    // [j' + WP i']
#pragma unroll
  for (int q = 0; q < QE; ++q) {
    const int e = threadIdx.x + NT * q;
    const int ia = e % 64, ja = e / 64, jb = e % W, ib = e / W;
    const int64_t mab = opaque_mask(a0 + ia < s && b0 + ja < s), mba = opaque_mask(b0 + jb < s && a0 + ib < s);
    const T dab = ld_off(Dti, ((uint32_t)((b0 + ja) * sld + a0 + ia) & (uint32_t)mab) * (uint32_t)sizeof(T));
    const T dba = ld_off(Dti, ((uint32_t)((a0 + ib) * sld + b0 + jb) & (uint32_t)mba) * (uint32_t)sizeof(T));
    sab[q] = masked(dab - sab[q], mab);
    sba[q] = masked(dba - sba[q], mba);
    Sab[e] = sab[q];
    Sba[jb + WP * ib] = sba[q];
  }
  lds_barrier();
  if (uniform(pl.half > 0 ? 1 : 0)) {
    // LU plan: no symmetrization.  X_KK's slabs into the L half, their
    // transposes into the U^T half (entry (r, q) = X(q, r)).
    T *Xu = Xkk + pl.half;
#pragma unroll
    for (int q = 0; q < QE; ++q) {
      const int e = threadIdx.x + NT * q;
      const int ia = e % 64, ja = e / 64, jb = e % W, ib = e / W;
      if (a0 + ia < s && b0 + ja < s) {
        const int64_t o = (int64_t)(b0 + ja) * dld + a0 + ia;
        gstore(Xkk + o, sab[q]);
        gstore(Xu + o, Sba[ja + WP * ia]);
      }
      if (a != b && b0 + jb < s && a0 + ib < s) {
        const int64_t o = (int64_t)(a0 + ib) * dld + b0 + jb;
        gstore(Xkk + o, sba[q]);
        gstore(Xu + o, Sab[ib + 64 * jb]);
      }
    }
    lds_barrier();
    return;
  }
  // x(i, j) = (T[a0 + i, b0 + j] + T[b0 + j, a0 + i]) / 2 (the second term
  // conjugated in a Hermitian plan), kept in Sab (each thread its own elements)
  const double cs = pl.csign;
#pragma unroll
  for (int q = 0; q < QE; ++q) {
    const int e = threadIdx.x + NT * q;
    const int ia = e % 64, ja = e / 64;
    const T x = SOps<T>::scale(0.5, sab[q] + cj(Sba[ja + WP * ia], cs));
    Sab[e] = x;
    if (a0 + ia < s && b0 + ja < s) gstore(Xkk + (int64_t)(b0 + ja) * dld + a0 + ia, x);
  }
  lds_barrier();
  if (a != b) {
#pragma unroll
    for (int q = 0; q < QE; ++q) {
      const int e = threadIdx.x + NT * q;
      const int jb = e % W, ib = e / W;
      if (b0 + jb < s && a0 + ib < s) gstore(Xkk + (int64_t)(a0 + ib) * dld + b0 + jb, cj(Sab[ib + 64 * jb], cs));
    }
  }
  lds_barrier();
}

// Blocks (a, b) and (b, a), a >= b, of X_KK = sym(Dt^{-1} - sum_r P_r)
// (Alg. 1 step 4 and the symmetrization of Section 2.3).
template <typename T, bool COH>
__device__ void do_dtile(const Ctx<T> &cx, const NodeInfo &nd, int a, int b, double *smem) {
  const DevPlan &pl = *cx.pl;
  const int ld = nd.s + nd.c;
  const int64_t off = nd.off;
  // top block of the normalized panel = Dt^{-1}; top block of the X panel.
  // b carries the slab number + 1 in its high half for slab items.
  if (b >> 16)
    dtile_slab<T>(cx, nd, a, b & 0xffff, (b >> 16) - 1, reinterpret_cast<T *>(smem), cx.Lp + off, ld, cx.Xp + off, ld);
  else
    dtile_core<T, COH>(cx, nd, a, b, smem, cx.Lp + off, ld, cx.Xp + off, ld);
}

// A whole node with c <= 64 and s <= 64 in one workgroup (Alg. 1 steps 3-4
// and the symmetrization of Section 2.3), in three dependent rounds of
// memory reads (and Dt^{-1} at the end): (1) the row tables of C(K) and Lhat; (2) the panel
// positions of X_{C,C} (the column tables of X_{C,C} are the row tables:
// both index C(K)); (3) the values of X_{C,C}.  GEMM-1, GEMM-2 and the
// diagonal block then run from LDS; nothing goes through the partial buffer.
template <typename T, bool COH>
__device__ void do_stile(const Ctx<T> &cx, const NodeInfo &nd, double *smem, int64_t *rt) {
  constexpr int P = Planes<T>::P, TK = Planes<T>::TK;
  constexpr int Q = 64 * 64 / NT;
  const DevPlan &pl = *cx.pl;
  const int s = uniform(nd.s), c = uniform(nd.c), ld = s + c;
  const int64_t off = nd.off, rp = nd.rp;
  // round 1: row tables into LDS; Lhat (c x s) straight into the B planes of
  // the four GEMM-1 stages (B(k, x) = Lhat(k, x): plane [kk][x] of stage k / TK)
  if (threadIdx.x < 64) {
    const int ig = threadIdx.x < c ? threadIdx.x : 0;
    rt[threadIdx.x] = gp(pl.kcol)[rp + ig];
    rt[64 + threadIdx.x] = gp(pl.kpos)[rp + ig];
  }
  {
    T lv[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int e = threadIdx.x + NT * q;
      const int i = e & 63, j = e >> 6;
      lv[q] = gload(cx.Lp + off + ((((int64_t)j * ld + s + i) & opaque_mask(i < c && j < s))));
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int e = threadIdx.x + NT * q;
      const int i = e & 63, j = e >> 6;
      const T l = masked(lv[q], opaque_mask(i < c && j < s));
      double *stgb = smem + (i / TK) * stage_doubles<T>() + P * TK * PITCH + (i % TK) * PITCH + j;
#pragma unroll
      for (int p = 0; p < P; ++p) stgb[p * TK * PITCH] = Planes<T>::get(l, p);
    }
  }
  lds_barrier();
  Acc<T> acc;
  acc_zero<T>(acc);
  if (c > 0) {
    // round 2: positions of X_{C,C}(i, k): lower part (i >= k) through column
    // k's table, upper part through row i's table; element e -> (i = e & 63, k = e >> 6)
    int32_t pos[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int e = threadIdx.x + NT * q;
      const int i = e & 63, k = e >> 6;
      const int64_t okm = opaque_mask(i < c && k < c);
      const int64_t lm = opaque_mask(i >= k);
      const int64_t pidx = (((rt[64 + k] + i) & lm) | ((rt[64 + i] + k) & ~lm)) & okm;
      pos[q] = gp(pl.posarr)[pidx];
    }
    // round 3: the values (panel column bases read again from LDS)
    T gv[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int e = threadIdx.x + NT * q;
      const int i = e & 63, k = e >> 6;
      const int64_t lm = opaque_mask(i >= k);
      const int64_t base = (rt[k] & lm) | (rt[i] & ~lm);
      gv[q] = Mem<COH>::ld(cx.Xp + ((base + (int64_t)pos[q]) & opaque_mask(i < c && k < c)));
    }
    // GEMM-1 from LDS: four stages of TK contraction indices, A = X_{C,C}
    // (upper part conjugated in a Hermitian plan), B = Lhat
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int e = threadIdx.x + NT * q;
      const int i = e & 63, k = e >> 6;
      const T g = cj(masked(gv[q], opaque_mask(i < c && k < c)), i < k ? pl.csign : 1.0);
      double *stg = smem + (k / TK) * stage_doubles<T>() + (k % TK) * PITCH + i;
#pragma unroll
      for (int p = 0; p < P; ++p) stg[p * TK * PITCH] = Planes<T>::get(g, p);  // A plane [kk][i]
    }
    lds_barrier();
#pragma unroll
    for (int st = 0; st < 64 / TK; ++st) stage_compute<T>(smem + st * stage_doubles<T>(), acc);
    // Lhat back out of the B planes before store_xtile reuses the stages
    T lv[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int e = threadIdx.x + NT * q;
      const int i = e & 63, x = e >> 6;
      lv[q] = Planes<T>::from(smem + (i / TK) * stage_doubles<T>() + P * TK * PITCH + (i % TK) * PITCH + x,
                              TK * PITCH);
    }
    lds_barrier();
    // Y = -acc into X_{C,K}
    store_xtile<T, COH>(cx, nd, 0, 0, acc, smem);
    // Lhat (conjugated if Hermitian) into LDS as Ls[p][i * PITCH + x], then R = Lhat^T acc
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int e = threadIdx.x + NT * q;
      const int i = e & 63, x = e >> 6;
      const T l = cj(lv[q], pl.csign);
#pragma unroll
      for (int p = 0; p < P; ++p) smem[p * 64 * PITCH + i * PITCH + x] = Planes<T>::get(l, p);
    }
    lds_barrier();
    gemm2_block<T>(acc, smem);  // R[p][j * PITCH + x] = (Lhat^T acc)(x, j) = -(Lhat^T Y)(x, j)
  } else {
#pragma unroll
    for (int e = threadIdx.x; e < 64 * 64; e += NT) lds_put<T>(smem, e >> 6, e & 63, zero_of<T>());
    lds_barrier();
  }
  // T = Dt^{-1} - Lhat^T Y = Dt^{-1} + R; X_KK = (T + T^T) / 2.  Dt^{-1} is
  // read only now: holding it through both products costs registers.
  double *Tt = smem + tile_doubles<T>();
  T dv[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int e = threadIdx.x + NT * q;
    const int i = e & 63, j = e >> 6;
    dv[q] = gload(cx.Lp + off + ((((int64_t)j * ld + i) & opaque_mask(i < s && j < s))));
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int e = threadIdx.x + NT * q;
    const int i = e & 63, j = e >> 6;
    const T d = masked(dv[q], opaque_mask(i < s && j < s));
    lds_put<T>(Tt, i, j, d + lds_get<T>(smem, i, j));
  }
  lds_barrier();
  const double cs = pl.csign;
  for (int e = threadIdx.x; e < 64 * 64; e += NT) {
    const int i = e & 63, j = e >> 6;
    if (i < s && j < s)
      Mem<COH>::st(cx.Xp + off + (int64_t)j * ld + i,
                   SOps<T>::scale(0.5, lds_get<T>(Tt, i, j) + cj(lds_get<T>(Tt, j, i), cs)));
  }
  lds_barrier();
}

// A whole small node (c <= CM <= kTinyCF, s <= SM <= kTinyS) of one matrix in one
// wavefront, for the level schedule.  Three dependent memory rounds: the
// record, then the byte offsets of X_{C,C} in the panel array (host table:
// c x c row-major, then padding), Lhat and Dt^{-1}, then the X_{C,C} values.
// Lane (i, grp) holds X_{C,C}(i, k) for k = grp + G u; the partial sums of
// X_{C,C} Lhat over the G lane groups are combined with a fixed butterfly, so
// the result does not depend on timing.  LDS blocks are CM x SM, a row's SM
// entries together and zero past c and s, so that every product reads without
// a branch and many reads are in flight (a branch on j < s around each read
// waited for it alone: a launch of complex nodes with 32 < c <= 64, 32 shifts of
// 30^3, took 188 us, now 77).  HERM: a Hermitian plan (conjugate
// transposes).
//   Y = -X_{C,C} Lhat (stored into X_{C,K});  T = Dt^{-1} - Lhat^T Y;
//   X_{K,K} = (T + T^T) / 2                      (Alg. 1, Eqs. (2.9)-(2.10))

// Lhat (or Uhat^T) from its lanes' registers (entry e = lane + 64 q: k = e % CM, j = e / CM) into LDS.
template <int CM, int SM> constexpr int tiny_ql() { return CM * SM >= 64 ? CM * SM / 64 : 1; }
template <typename T, int CM, int SM>
__device__ __forceinline__ void tiny_load(const TinyRec &r, int lane, const T *L, T (&lv)[tiny_ql<CM, SM>()]) {
#pragma unroll
  for (int q = 0; q < tiny_ql<CM, SM>(); ++q) {
    const int e = lane + 64 * q, k = e % CM, j = e / CM;
    lv[q] = gload(L + r.off + ((j * (r.s + r.c) + r.s + k) & opaque_mask(k < r.c && j < r.s)));
  }
}
template <typename T, int CM, int SM>
__device__ __forceinline__ void tiny_put(const TinyRec &r, int lane, const T (&lv)[tiny_ql<CM, SM>()], T *ls) {
#pragma unroll
  for (int q = 0; q < tiny_ql<CM, SM>(); ++q) {
    const int e = lane + 64 * q, k = e % CM, j = e / CM;
    if (CM * SM >= 64 || e < CM * SM) ls[k * SM + j] = masked(lv[q], opaque_mask(k < r.c && j < r.s));
  }
}

// X_KK = sym(Dt^{-1} + Lhat^T ys), entry (x, y) on lane x + 8 y.
template <typename T, int SM, bool HERM>
__device__ __forceinline__ void tiny_diag(const TinyRec &r, int x, int y, T dxy, T dyx, const T *ls, const T *ys, T *X) {
  constexpr double cs = HERM ? -1.0 : 1.0;
  if (x < r.s && y < r.s) {
    T rxy = zero_of<T>(), ryx = zero_of<T>();
    for (int q0 = 0; q0 < r.c; q0 += 8)
#pragma unroll
      for (int q = q0; q < q0 + 8; ++q) {
        rxy += cj(ls[q * SM + x], cs) * ys[q * SM + y];
        ryx += cj(ls[q * SM + y], cs) * ys[q * SM + x];
      }
    X[r.off + y * (r.s + r.c) + x] = SOps<T>::scale(0.5, (dxy + rxy) + cj(dyx + ryx, cs));
  }
}

template <typename T, int CM, int SM, bool HERM>
__device__ __forceinline__ void do_tiny(const TinyRec &r, int lane, const uint32_t *toff, const T *L, T *X, T *ls, T *ys) {
  constexpr int G = 64 / CM, U = CM / G;
  const int i = lane % CM, grp = lane / CM;
  const int s = r.s, c = r.c;
  const int64_t ld = s + c;
  const uint32_t *tb = toff + r.tbl;
  // round 2: the offsets of this lane's X_{C,C}(i, k); Lhat; Dt^{-1}(x, y), (y, x)
  const uint32_t rowb = 4u * ((uint32_t)(i * c + grp) & opaque_mask32(i < c));
  uint32_t o[U];
#pragma unroll
  for (int u = 0; u < U; ++u) o[u] = ld_off(tb, rowb + 4u * (G * u));
  T lv[tiny_ql<CM, SM>()];
  tiny_load<T, CM, SM>(r, lane, L, lv);
  const int x = lane % kTinyS, y = lane / kTinyS;
  const int64_t dm = opaque_mask(x < s && y < s);
  const T dxy = gload(L + r.off + ((y * ld + x) & dm)), dyx = gload(L + r.off + ((x * ld + y) & dm));
  // round 3: the values (bit 0 of an offset: the entry is read conjugated,
  // Hermitian plans only; the bits are kept packed so that the offsets die here)
  T xv[U];
  uint32_t cbits = 0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if constexpr (HERM) {
      xv[u] = ld_off(X, o[u] & ~1u);
      cbits |= (o[u] & 1u) << u;
    } else {
      xv[u] = ld_off(X, o[u]);
    }
  }
  tiny_put<T, CM, SM>(r, lane, lv, ls);
  wave_lds_fence();
  T acc[SM];
#pragma unroll
  for (int j = 0; j < SM; ++j) acc[j] = zero_of<T>();
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int k = grp + G * u;
    T g = masked(xv[u], opaque_mask(i < c && k < c));
    if constexpr (HERM) g = cj(g, ((cbits >> u) & 1u) ? -1.0 : 1.0);
#pragma unroll
    for (int j = 0; j < SM; ++j) acc[j] += g * ls[k * SM + j];
  }
#pragma unroll
  for (int m = CM; m < 64; m <<= 1)
#pragma unroll
    for (int j = 0; j < SM; ++j) acc[j] += shfl_xor_t(acc[j], m);
  if (grp == 0) {
#pragma unroll
    for (int j = 0; j < SM; ++j) {
      if (j < s && i < c) X[r.off + j * ld + s + i] = SOps<T>::scale(-1.0, acc[j]);
      ys[i * SM + j] = masked(acc[j], opaque_mask(i < c));  // (0 times an infinite entry of Lhat past c)
    }
  }
  wave_lds_fence();
  tiny_diag<T, SM, HERM>(r, x, y, dxy, dyx, ls, ys, X);
}

// The same for 32 < c <= kTinyCF: lane i holds row i of X_{C,C}, and the
// contraction runs in two halves of 32 columns so that one half's offsets and
// one half's values are in registers at a time.  Four dependent rounds: the
// record; Lhat, Dt^{-1} and the first half's offsets; the first half's values
// with the second half's offsets; the second half's values.  HERM: a Hermitian
// plan (bit 0 of an offset marks an entry read conjugated; the diagonal block
// takes Lhat^H and the conjugate transpose).
__device__ __forceinline__ void hold(double &x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void hold(cplx &x) {
  hold(x.re);
  hold(x.im);
}
template <typename T, int SM, bool HERM = false>
__device__ __forceinline__ void do_tiny64(const TinyRec &r, int lane, const uint32_t *toff, const T *L, T *X, T *ls, T *ys) {
  constexpr int H = kTinyCF / 2, CM = kTinyCF;
  const int i = lane;
  const int s = r.s, c = r.c;
  const int64_t ld = s + c;
  const uint32_t *tb = toff + r.tbl;
  T lv[tiny_ql<CM, SM>()];
  tiny_load<T, CM, SM>(r, lane, L, lv);
  const int x = i % kTinyS, y = i / kTinyS;
  const int64_t dm = opaque_mask(x < s && y < s);
  const T dxy = gload(L + r.off + ((y * ld + x) & dm)), dyx = gload(L + r.off + ((x * ld + y) & dm));
  const uint32_t rowb = 4u * ((uint32_t)(i * c) & opaque_mask32(i < c));
  uint32_t o[H];
  T xv[H], acc[SM];
#pragma unroll
  for (int j = 0; j < SM; ++j) acc[j] = zero_of<T>();
#pragma unroll
  for (int u = 0; u < H; ++u) o[u] = ld_off(tb, rowb + 4u * u);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    uint32_t cbits = 0;
#pragma unroll
    for (int u = 0; u < H; ++u) {
      if constexpr (HERM) {
        xv[u] = ld_off(X, o[u] & ~1u);
        cbits |= (o[u] & 1u) << u;
      } else {
        xv[u] = ld_off(X, o[u]);
      }
    }
    if (h == 0) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < H; ++u) o[u] = ld_off(tb, rowb + 4u * (H + u));
      tiny_put<T, CM, SM>(r, lane, lv, ls);
      wave_lds_fence();
    }
    constexpr int UB = 16 / Planes<T>::P / (SM / 4);  // rows of Lhat in flight
#pragma unroll
    for (int u0 = 0; u0 < H; u0 += UB) {
      // these reads stay behind the previous products (all of them in front
      // of all products took 2000 spilled registers)
      int at = (H * h + u0) * SM;
      asm volatile("" : "+s"(at));
#pragma unroll
      for (int u = u0; u < u0 + UB; ++u) {
        T g = masked(xv[u], opaque_mask(i < c && H * h + u < c));
        if constexpr (HERM) g = cj(g, ((cbits >> u) & 1u) ? -1.0 : 1.0);
#pragma unroll
        for (int j = 0; j < SM; ++j) acc[j] += g * ls[at + (u - u0) * SM + j];
      }
#pragma unroll
      for (int j = 0; j < SM; ++j) hold(acc[j]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int j = 0; j < SM; ++j) {
    if (j < s && i < c) X[r.off + j * ld + s + i] = SOps<T>::scale(-1.0, acc[j]);
    ys[i * SM + j] = masked(acc[j], opaque_mask(i < c));  // (0 times an infinite entry of Lhat past c)
  }
  wave_lds_fence();
  tiny_diag<T, SM, HERM>(r, x, y, dxy, dyx, ls, ys, X);
}

// A whole small node of an LU plan (c <= CM, s <= SM) in one wavefront, as
// do_tiny for both panel sets: lane (i, grp) holds X_{C,C}(i, k) and X_{C,C}(k, i)
// for k = grp + G u (the table gives the first; the second is the same
// position of the other set, half8 bytes away), 16 of each at a time, and
// accumulates X_{C,C} Lhat and (X_{C,C})^T Uhat^T.
//   X_{C,K} = -X_{C,C} Lhat, X_{K,C}^T = -(X_{C,C})^T Uhat^T,
//   X_KK = Dt^{-1} - Uhat X_{C,K}, stored into the first set and transposed into the second
template <int CM, int SM>
__device__ __forceinline__ void do_tiny_lu(const TinyRec &r, int lane, const uint32_t *toff, int64_t half, const double *L,
                                           double *X, double *ls, double *us, double *ys) {
  constexpr int G = 64 / CM, U = CM / G, UC = U < 16 ? U : 16;
  const int i = lane % CM, grp = lane / CM;
  const int s = r.s, c = r.c;
  const int64_t ld = s + c;
  const uint32_t *tb = toff + r.tbl;
  const uint32_t rowb = 4u * ((uint32_t)(i * c + grp) & opaque_mask32(i < c)), half8 = (uint32_t)(8 * half);
  uint32_t o[UC];
#pragma unroll
  for (int u = 0; u < UC; ++u) o[u] = ld_off(tb, rowb + 4u * (G * u));
  double lv[tiny_ql<CM, SM>()], uv[tiny_ql<CM, SM>()];
  tiny_load<double, CM, SM>(r, lane, L, lv);
  tiny_load<double, CM, SM>(r, lane, L + half, uv);
  const int x = lane % kTinyS, y = lane / kTinyS;
  const double dxy = gload(L + r.off + ((y * ld + x) & opaque_mask(x < s && y < s)));
  tiny_put<double, CM, SM>(r, lane, lv, ls);
  tiny_put<double, CM, SM>(r, lane, uv, us);
  wave_lds_fence();
  double al[SM], au[SM];
#pragma unroll
  for (int j = 0; j < SM; ++j) al[j] = au[j] = 0.0;
#pragma unroll
  for (int u0 = 0; u0 < U; u0 += UC) {
    if (G * u0 >= c) break;
    double xl[UC], xu[UC];
#pragma unroll
    for (int u = 0; u < UC; ++u) {
      const int k = grp + G * (u0 + u);
      const uint32_t ok = opaque_mask32(i < c && k < c);
      xl[u] = ld_off(X, o[u] & ok);
      xu[u] = ld_off(X, (i >= k ? o[u] + half8 : o[u] - half8) & ok);
    }
    if (u0 + UC < U) {
#pragma unroll
      for (int u = 0; u < UC; ++u) o[u] = ld_off(tb, rowb + 4u * (G * (u0 + UC + u)));
    }
#pragma unroll
    for (int u = 0; u < UC; ++u) {
      const int k = grp + G * (u0 + u);
      const int64_t m = opaque_mask(i < c && k < c);
      const double a = masked(xl[u], m), b = masked(xu[u], m);
#pragma unroll
      for (int j = 0; j < SM; ++j) {
        al[j] += a * ls[k * SM + j];
        au[j] += b * us[k * SM + j];
      }
      if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // bounds the reads in flight
    }
  }
#pragma unroll
  for (int m = CM; m < 64; m <<= 1)
#pragma unroll
    for (int j = 0; j < SM; ++j) {
      al[j] += shfl_xor_t(al[j], m);
      au[j] += shfl_xor_t(au[j], m);
    }
  if (grp == 0) {
#pragma unroll
    for (int j = 0; j < SM; ++j) {
      if (j < s && i < c) {
        gstore(X + r.off + j * ld + s + i, -al[j]);
        gstore(X + half + r.off + j * ld + s + i, -au[j]);
      }
      ys[i * SM + j] = masked(al[j], opaque_mask(i < c));
    }
  }
  wave_lds_fence();
  if (x < s && y < s) {
    double t = 0.0;  // (added to Dt^{-1} at the end: one rounding at its size)
    for (int q0 = 0; q0 < c; q0 += 8)
#pragma unroll
      for (int q = q0; q < q0 + 8; ++q) t += us[q * SM + x] * ys[q * SM + y];
    t += dxy;
    gstore(X + r.off + y * ld + x, t);
    gstore(X + half + r.off + x * ld + y, t);
  }
}

// Any item of a symmetric plan (an LU plan's run in kernels of their own types).
// Inlined into the kernels, so that the node record stays in scalar registers
// (a call would pass it through the stack).
template <typename T, bool COH>
__device__ __forceinline__ void do_item(const Ctx<T> &cx, const Item &item, const NodeInfo &nd, double *smem,
                                        int64_t *rt) {
  const Item it = uniform(item);
  if (it.type == ITEM_G) {
    do_gtile<T, false>(cx, nd, it.a, it.b, smem, rt, cx.Xp);
  } else if (it.type == ITEM_Y) {
    do_ytile<T, COH>(cx, nd, it.a, it.b, smem, rt);
  } else if (it.type == ITEM_R) {
    do_rtile<T, COH>(cx, nd, it.a, it.b, smem);
  } else if (it.type == ITEM_P) {
    do_ptile<T, COH>(cx, nd, it.a, it.b, smem);
  } else if (it.type == ITEM_D) {
    do_dtile<T, COH>(cx, nd, it.a, it.b, smem);
  } else {  // ITEM_S: the whole node (c <= 64, s <= 64) in this workgroup
    do_stile<T, COH>(cx, nd, smem, rt);
  }
}

}  // namespace selinv
