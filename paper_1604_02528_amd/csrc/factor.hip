// Numeric factorization on the GPU: unpivoted supernodal LDL^T of B = P A P^T
// (LDL^H for a Hermitian A: the transposed factor of every product below is
// conjugated, Section 2.3).
//
// The paper takes its factors from an external solver that permutes
// symmetrically and does no dynamic pivoting (Section 4); this is the
// library's device producer of that input, in the panel layout the rest of
// the path reads (strict lower L_KK, D_K on the diagonal, L_{C,K} below).
// Right-looking supernodal form, etree depth by depth, the deepest first
// (every descendant of K is complete before K starts):
//
//   small  a whole node with s <= 16 and c <= 64 in one wavefront, or c <= 128 in
//          four (the lower depths hold little else)
//   diag   S_KK = L_KK D_K L_KK^T of a block of at most kFacCols columns, its
//          16 x 16 blocks in the registers of one workgroup
//   lc     the rows below that block, by block forward substitution with the
//          16 x 16 inverses the diag kernel left (one wavefront per 16 rows)
//   inner  a node wider than kFacCols: the update of its remaining columns,
//          then diag and lc again for those
//   schur  S_{C,C} -= L_{C,K} D_K L_{C,K}^T on the lower block pairs of C(K),
//          scattered into the ancestors' panels through the same index maps
//          the selected inversion gathers through (Eq. (newset)), with FP64
//          atomic adds: siblings of one depth update shared ancestors, so the
//          summation order (and the last bits) may vary from run to run.
//
// A last kernel sums log D_jj per matrix (log det B, Section 2.3) in a fixed
// order.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <utility>

#include "blk16.hpp"
#include "items.hpp"
#include "plan.hpp"
#include "scalar.hpp"
#include "tile.hpp"

namespace selinv {

hipError_t launch_scatter(const DevPlan &pl, const DevPlan *dpl, bool cplx_, const void *vals, void *panel,
                          hipStream_t st);

namespace {

__device__ __forceinline__ bool finite_nonzero(double d) { return d != 0.0 && isfinite(d); }
__device__ __forceinline__ bool finite_nonzero(cplx d) {
  return (d.re != 0.0 || d.im != 0.0) && isfinite(d.re) && isfinite(d.im);
}

// Rows 4 v + l / 16 of a transposed block times dl[4 v + l / 16] (planes `stride` apart).
template <typename T> __device__ __forceinline__ Blk<T> blk_scale_rows(const Blk<T> &b, const double *dl, int stride) {
  const int g = (threadIdx.x & 63) >> 4;
  Blk<T> o;
#pragma unroll
  for (int v = 0; v < 4; ++v) blk_set(o, v, blk_get(b, v) * Planes<T>::from(dl + 4 * v + g, stride));
  return o;
}
// The operand -L(j, k) (conjugated if Hermitian) of the updates.
template <typename T> __device__ __forceinline__ Blk<T> blk_neg_cj(const Blk<T> &b, double cs) {
  Blk<T> o;
  o.p[0] = -b.p[0];
  if constexpr (Planes<T>::P == 2) o.p[1] = -cs * b.p[1];
  return o;
}

// Lanes 0 .. 15 of v on lanes 0 .. 15 and 16 .. 31 (and 32 .. 47 on the rest).
__device__ __forceinline__ double even_row(double v) {
  asm("s_nop 1" : "+v"(v));  // v may come from an fmac16
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)u, hi = (uint32_t)(u >> 32);
  const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
  const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
  return __builtin_bit_cast(double, ((uint64_t)b[0] << 32) | a[0]);
}
__device__ __forceinline__ cplx even_row(cplx v) { return cplx{even_row(v.re), even_row(v.im)}; }

// 1 / d.  The pivots' reciprocals are one serial chain per node, so the usual
// range takes the hardware estimate and two Newton steps (r += r (1 - d r),
// each doubling the correct bits) instead of a full division.  recip_ok says
// afterwards whether that held: out of range, zero and non-finite pivots all
// leave a result whose exponent is beyond the limits.
__device__ __forceinline__ double fast_recip(double d) {
  double r = __builtin_amdgcn_rcp(d);
  r = fma(fma(-d, r, 1.0), r, r);
  return fma(fma(-d, r, 1.0), r, r);
}
__device__ __forceinline__ cplx fast_recip(cplx d) {
  const double r = fast_recip(fma(d.re, d.re, d.im * d.im));
  const cplx q{d.re * r, -d.im * r};  // r rounds three times: one more step q += q (1 - d q)
  const cplx e{fma(-d.re, q.re, fma(d.im, q.im, 1.0)), -fma(d.re, q.im, d.im * q.re)};
  return cplx{fma(q.re, e.re, fma(-q.im, e.im, q.re)), fma(q.re, e.im, fma(q.im, e.re, q.im))};
}
// x / d from di = 1 / d
__device__ __forceinline__ double fast_quot(double x, double d, double di) {
  const double y = x * di;
  return fma(fma(-y, d, x), di, y);
}
__device__ __forceinline__ cplx fast_quot(cplx x, cplx, cplx di) { return x * di; }
__device__ __forceinline__ uint32_t exponent_of(double v) {
  return (uint32_t)(__builtin_bit_cast(uint64_t, v) >> 52) & 0x7ffu;
}
__device__ __forceinline__ bool recip_ok(double di) { return exponent_of(di) - 523u < 1000u; }
__device__ __forceinline__ bool recip_ok(cplx di) {
  return max(exponent_of(di.re), exponent_of(di.im)) - 783u < 480u;  // the squared modulus is in range too
}

// x -= w[lane Q of the row] y; sg: the sign of the imaginary part of w (conj(w_q) on the lanes of S if Hermitian)
template <int Q> __device__ __forceinline__ void ldl_step(double &x, double w, double ny) { fmac16<Q>(x, w, ny); }
struct NegY {
  cplx ny, sy;  // -y and sg y
};
template <int Q> __device__ __forceinline__ void ldl_step(cplx &x, cplx w, const NegY &y) {
  fmac16<Q>(x.re, w.re, y.ny.re);
  fmac16<Q>(x.im, w.re, y.ny.im);
  fmac16<Q>(x.re, w.im, y.sy.im);
  fmac16<Q>(x.im, w.im, -y.sy.re);
}
__device__ __forceinline__ double neg_y(double y, double) { return -y; }
__device__ __forceinline__ NegY neg_y(cplx y, double sg) { return NegY{cplx{-y.re, -y.im}, cplx{sg * y.re, sg * y.im}}; }

// The rows of ldl16 in LDS: before it, row r of S (lower part) at [17 r + k] and
// column q of the identity at [17 (16 + q) + p]; afterwards L and D, and M(p, q),
// in their places, and 1 / D_j at [kLdlD + j]; planes kLdlLds apart.
constexpr int kLdlD = 32 * 17;
constexpr int kLdlLds = kLdlD + 16;
template <typename T> __device__ __forceinline__ void lds_set(double *q, T v) {
#pragma unroll
  for (int p = 0; p < Planes<T>::P; ++p) q[p * kLdlLds] = Planes<T>::get(v, p);
}
template <typename T> __device__ __forceinline__ T lds_at(const double *q) { return Planes<T>::from(q, kLdlLds); }
// A block of w < 16 columns is padded with the identity.
template <typename T> __device__ __forceinline__ void ldl16_stage(const Blk<T> &b, int w, double *ls) {
  const int r = threadIdx.x & 15, g = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int c = 4 * v + g;
    const T id = pick(r == c, SOps<T>::one(), zero_of<T>());
    lds_set<T>(ls + 17 * r + c, pick(r < w && c <= r, blk_get(b, v), id));
    lds_set<T>(ls + 17 * (16 + r) + c, id);
  }
  wave_lds_fence();
}
template <typename T> __device__ __forceinline__ void ldl16_put(const T (&x)[16], T dinv, double *ls) {
  const int lane = threadIdx.x & 63;
  if (lane < 32) {
#pragma unroll
    for (int k = 0; k < 16; ++k) lds_set<T>(ls + 17 * lane + k, x[k]);
  }
  if (lane < 16) lds_set<T>(ls + kLdlD + lane, dinv);
}

// Unpivoted LDL^T (LDL^H) of one 16 x 16 diagonal block and the inverse of
// its L, by one wavefront: lane r < 16 has row r of S (lower part), lane
// 16 + q column q of the identity (lanes 32 .. 63 are not used).  Step j needs
// the same update on both:
// row r:  S(r, q) -= L(r, j) W(q, j),  column q:  M(p, q) -= L(p, j) M(j, q),
// i.e. x[q] -= w_q (x[j] / d_j) with w_q = S(q, j) of lane q.  The updates of
// an entry are summed by themselves in x and meet the entry, read from LDS, when
// its column's step comes: one rounding at the entry's size (the entry in x
// itself would take one or, complex, two per step).  The columns of the padding
// are skipped in fours.
// Row r becomes L(r, 0 .. r - 1) and D_r, column q M(:, q), and lane j < 16
// gets 1 / D_j.  False when a pivot is outside the range of the fast
// reciprocal (x is then undefined).
// One wavefront issues at most an instruction every four cycles, so what
// counts in this serial chain is their number: a column of S is copied to the
// lanes of M once, a broadcast and its multiply-add are one instruction, and
// there is no branch per column (with scalar lane reads and branches a block
// took 4.7 us of the 128-column kernel's 39 us, FP64).
template <typename T>
__device__ __forceinline__ bool ldl16(const double *ls, T (&x)[16], int w, double cs, T &dinv) {
  const int lane = threadIdx.x & 63;
  const double *row = ls + 17 * (lane & 31);
  const double sg = lane < 16 ? cs : 1.0;
  dinv = SOps<T>::one();
#pragma unroll
  for (int k = 0; k < 16; ++k) x[k] = zero_of<T>();
  T next = lds_at<T>(row);
  static_for(
      [&](auto bc) {
        constexpr int b = decltype(bc)::value;
        if (b == 0 || 4 * b < w) {
          static_for(
              [&](auto jc) {
                constexpr int j = 4 * b + decltype(jc)::value;
                const T xj = next + x[j];
                if constexpr (j < 15) next = lds_at<T>(row + j + 1);
                const T ww = even_row(xj);
                const T d = bcast16<j>(ww), di = fast_recip(d);
                const T y = fast_quot(xj, d, di);
                const auto ny = neg_y(y, sg);
                static_for(
                    [&](auto qc) {
                      constexpr int q = decltype(qc)::value + j + 1;
                      ldl_step<q>(x[q], ww, ny);
                    },
                    std::make_integer_sequence<int, 15 - j>{});
                int ln = lane;
                asm("" : "+v"(ln));  // the lane masks are made here: kept from step to step they spill
                x[j] = pick((unsigned)(ln - j - 1) < (unsigned)(15 - j), y, xj);
                dinv = pick(ln == j, di, dinv);
              },
              std::make_integer_sequence<int, 4>{});
        } else {
#pragma unroll
          for (int k = 4 * b; k < 4 * b + 4; ++k) x[k] = lds_at<T>(row + k);
        }
      },
      std::make_integer_sequence<int, 4>{});
  return __ballot(lane < 16 && !recip_ok(dinv)) == 0;
}

// The same in LDS, with full divisions, for the blocks ldl16 turns down.  A
// zero or non-finite pivot is recorded (column first + j).
template <typename T>
__device__ __forceinline__ void ldl16_wide_range(double *ls, int w, double cs, int64_t first, unsigned long long *ferr) {
  const int lane = threadIdx.x & 63, row = lane & 31;
  const double sg = row < 16 ? cs : 1.0;
  if (lane < 16) lds_set<T>(ls + kLdlD + lane, SOps<T>::one());
#pragma unroll 1
  for (int j = 0; j < w; ++j) {
    wave_lds_fence();
    const T d = lds_at<T>(ls + 18 * j);
    if (!finite_nonzero(d) && lane == 0) atomicMin(ferr, (unsigned long long)(first + j));
    const T di = SOps<T>::div(SOps<T>::one(), d);
    const T y = SOps<T>::div(lds_at<T>(ls + 17 * row + j), d);
#pragma unroll 1
    for (int q = j + 1; q < 16; ++q) {
      const T v = lds_at<T>(ls + 17 * row + q) - cj(lds_at<T>(ls + 17 * q + j), sg) * y;
      if (lane < 32) lds_set<T>(ls + 17 * row + q, v);
    }
    wave_lds_fence();
    if (lane > j && lane < 16) lds_set<T>(ls + 17 * lane + j, y);
    if (lane == 0) lds_set<T>(ls + kLdlD + j, di);
  }
}

// Both of them, on a staged block.
template <typename T>
__device__ __forceinline__ void ldl16_block(int w, double cs, double *ls, int64_t first, unsigned long long *ferr) {
  T x[16], dinv;
  const bool ok = ldl16<T>(ls, x, w, cs, dinv);
  wave_lds_fence();
  if (ok)
    ldl16_put<T>(x, dinv, ls);
  else
    ldl16_wide_range<T>(ls, w, cs, first, ferr);
  wave_lds_fence();
}

// M as the A operand of W^T = M S^T (conjugated if Hermitian).
template <typename T> __device__ __forceinline__ Blk<T> ldl16_m(const double *q, double cs) {
  const int r = threadIdx.x & 15, g = (threadIdx.x & 63) >> 4;
  Blk<T> m;
#pragma unroll
  for (int v = 0; v < 4; ++v) blk_set(m, v, cj(Planes<T>::from(q + 17 * (16 + 4 * v + g) + r, kLdlLds), cs));
  return m;
}
// L and D into the panel (lower triangle only).
template <typename T> __device__ __forceinline__ void ldl16_store(const double *ls, T *Q, int ld, int w) {
  const int r = blk_row(), g = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int v = 0; v < 4; ++v)
    if (r < w && 4 * v + g <= r)
      st_off(Q, (uint32_t)((4 * v + g) * ld + r) * (uint32_t)sizeof(T), lds_at<T>(ls + 17 * r + 4 * v + g));
}

// ---------------------------------------------------------------------------
// Whole nodes with s <= 16 and c <= kFacSmallC in one wavefront: the diagonal
// block, L_{C,K} one 16-row strip at a time, and every 16 x 16 block of the
// update of S_{C,C} from registers.  These nodes are most of the tree and
// have almost no arithmetic: what bounds them is the launches and the
// dependent rounds of loads (record -> panel and row tables -> positions), so
// one launch does everything and a CU holds many nodes at once (four launches
// on 64 x 64 tiles before; 31 x 31 FP64 grid: 0.27 -> 0.07 ms for its ten depths;
// 16 Hermitian 30^3 matrices, the lower 13 depths: 10.5 -> 1.7 ms, where the
// atomics of nodes with c near 64 bound it: 1.9 ms with the two planes of an
// entry added by separate instructions, 1.1 with whole entries, see blk_atomic).
// ---------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(64, 2) k_fac_small(const DevPlan *__restrict__ plp, T *Pall, const FacNode *recs,
                                                  int32_t count, unsigned long long *ferr) {
  constexpr int P = Planes<T>::P, NST = kFacSmallC / 16;
  const DevPlan &pl = *plp;
  __shared__ double ls[P * kLdlLds];
  __shared__ int64_t rcol[16 * NST], rpos[16 * NST];
  const int64_t gidx = blockIdx.x;
  const int64_t l = gidx / count;
  const FacNode nd = recs[gidx - l * count];
  const int s = uniform(nd.s), c = uniform(nd.c), ld = s + c;
  T *Pl = Pall + l * pl.panel_elems;
  T *Q = Pl + nd.off;
  const int lane = threadIdx.x, r = strip_row<T>(lane & 15), g = lane >> 4;
  const double cs = pl.csign;
  const int kq = min(lane, c - 1);
  const int64_t kc = c > 0 ? gp(pl.kcol)[nd.rp + kq] : 0, kp = c > 0 ? gp(pl.kpos)[nd.rp + kq] : 0;
  const Blk<T> dg = blk_load<T>(Q, ld, s, s);
  Blk<T> wb[NST];
#pragma unroll
  for (int i = 0; i < NST; ++i)
    if (16 * i < c) wb[i] = blk_load<T, true>(Q + s + 16 * i, ld, c - 16 * i, s);
  rcol[lane] = kc;
  rpos[lane] = kp;
  wave_lds_fence();
  // positions of the update's elements in strip j's columns, loaded one strip
  // ahead (the first while the diagonal block is factored)
  int32_t pos[2][NST][4];
  auto load_pos = [&](int j) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int kg = 16 * j + strip_row<T>(4 * v + g);
      const int64_t rp = rpos[kg];
#pragma unroll
      for (int i = 0; i < NST; ++i) {
        const int ig = 16 * i + r;
        if (i >= j && 16 * i < c) pos[j & 1][i][v] = gp(pl.posarr)[(rp + ig) & opaque_mask(ig < c && ig >= kg)];
      }
    }
  };
  load_pos(0);
  ldl16_stage<T>(dg, s, ls);
  ldl16_block<T>(s, cs, ls, nd.first, ferr + l);
  ldl16_store<T>(ls, Q, ld, s);
  const int nv = (s + 3) / 4;
  const Blk<T> m = ldl16_m<T>(ls, cs);
#pragma unroll
  for (int i = 0; i < NST; ++i) {
    if (16 * i >= c) break;
    Blk<T> w = blk_zero<T>();
    blk_mma<T>(m, wb[i], w, nv);
    wb[i] = w;
    blk_store<T, true>(blk_scale_rows<T>(w, ls + kLdlD, kLdlLds), Q + s + 16 * i, ld, c - 16 * i, s);
  }
#pragma unroll
  for (int j = 0; j < NST; ++j) {
    if (16 * j >= c) break;
    if (j + 1 < NST && 16 * (j + 1) < c) load_pos(j + 1);
    const Blk<T> lj = blk_neg_cj<T>(blk_scale_rows<T>(wb[j], ls + kLdlD, kLdlLds), cs);
    int64_t col[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) col[v] = rcol[16 * j + strip_row<T>(4 * v + g)];
#pragma unroll
    for (int i = j; i < NST; ++i) {
      if (16 * i >= c) break;
      Blk<T> u = blk_zero<T>();
      blk_mma<T>(lj, wb[i], u, nv);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int kg = 16 * j + strip_row<T>(4 * v + g);
        blk_atomic(Pl + col[v], pos[j & 1][i][v], 16 * i, kg, c, blk_get(u, v));
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// The same for kFacSmallC < c <= kFacMidC by four wavefronts: one factors the
// diagonal block, each forms every fourth strip of W and -L in LDS and takes
// every fourth pair of strips of the update (one wavefront for all of it held
// 360 registers and waited for one strip's positions after another: 30 to 36
// us a launch on the 40^3 FP64 Laplacian, now 10 to 22).
template <typename T>
__global__ void __launch_bounds__(NT, 2) k_fac_mid(const DevPlan *__restrict__ plp, T *Pall, const FacNode *recs,
                                                int32_t count, unsigned long long *ferr) {
  constexpr int P = Planes<T>::P, NST = kFacMidC / 16, W = NT / 64, NP = NST * (NST + 1) / 2, LP = NST * 256;
  const DevPlan &pl = *plp;
  __shared__ double ls[P * kLdlLds], wp[P * LP], lp[P * LP];
  __shared__ int64_t rcol[kFacMidC], rpos[kFacMidC];
  const int64_t gidx = blockIdx.x;
  const int64_t l = gidx / count;
  const FacNode nd = recs[gidx - l * count];
  const int s = uniform(nd.s), c = uniform(nd.c), ld = s + c;
  T *Pl = Pall + l * pl.panel_elems;
  T *Q = Pl + nd.off;
  const int wv = uniform((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63, r = strip_row<T>(lane & 15), g = lane >> 4;
  const double cs = pl.csign;
  if (threadIdx.x < kFacMidC) {
    const int kq = min((int)threadIdx.x, c - 1);
    rcol[threadIdx.x] = gp(pl.kcol)[nd.rp + kq];
    rpos[threadIdx.x] = gp(pl.kpos)[nd.rp + kq];
  }
  Blk<T> dg;
  if (wv == 0) dg = blk_load<T>(Q, ld, s, s);
  Blk<T> sb[NST / W];
#pragma unroll
  for (int q = 0; q < NST / W; ++q) {
    const int i = wv + W * q;
    if (16 * i < c) sb[q] = blk_load<T, true>(Q + s + 16 * i, ld, c - 16 * i, s);
  }
  lds_barrier();
  // pair e = wv + W q of strips (i, j), i >= j, row by row
  int pi[(NP + W - 1) / W], pj[(NP + W - 1) / W];
  int32_t pos[(NP + W - 1) / W][4];
#pragma unroll
  for (int q = 0; q < (NP + W - 1) / W; ++q) {
    int j = wv + W * q, i = 0;
    while (j > i) j -= ++i;
    pi[q] = uniform(i);
    pj[q] = uniform(j);
    if (16 * pi[q] >= c) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int ig = 16 * pi[q] + r, kg = 16 * pj[q] + strip_row<T>(4 * v + g);
      pos[q][v] = gp(pl.posarr)[(rpos[kg] + ig) & opaque_mask(ig < c && ig >= kg)];
    }
  }
  if (wv == 0) {
    ldl16_stage<T>(dg, s, ls);
    ldl16_block<T>(s, cs, ls, nd.first, ferr + l);
    ldl16_store<T>(ls, Q, ld, s);
  }
  lds_barrier();
  const int nv = (s + 3) / 4;
  const Blk<T> m = ldl16_m<T>(ls, cs);
#pragma unroll
  for (int q = 0; q < NST / W; ++q) {
    const int i = wv + W * q;
    if (16 * i >= c) break;
    Blk<T> w = blk_zero<T>();
    blk_mma<T>(m, sb[q], w, nv);
    const Blk<T> lo = blk_scale_rows<T>(w, ls + kLdlD, kLdlLds);
    blk_to_lds<T>(w, wp + 256 * i, LP);
    blk_to_lds<T>(blk_neg_cj<T>(lo, cs), lp + 256 * i, LP);
    blk_store<T, true>(lo, Q + s + 16 * i, ld, c - 16 * i, s);
  }
  lds_barrier();
#pragma unroll
  for (int q = 0; q < (NP + W - 1) / W; ++q) {
    if (16 * pi[q] >= c) break;
    Blk<T> u = blk_zero<T>();
    blk_mma<T>(blk_from_lds<T>(lp + 256 * pj[q], LP), blk_from_lds<T>(wp + 256 * pi[q], LP), u, nv);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int kg = 16 * pj[q] + strip_row<T>(4 * v + g);
      blk_atomic(Pl + rcol[kg], pos[q][v], 16 * pi[q], kg, c, blk_get(u, v));
    }
  }
}

// ---------------------------------------------------------------------------
// Unpivoted LDL^T of a diagonal block of at most kFacCols = 128 columns (a
// whole node's, or one column block of a wider node), one workgroup of eight
// wavefronts.  The lower 16 x 16 blocks stay in registers: wavefront i owns
// diagonal block i and up to four of the others.  Step k: the owner of
// block (k, k) factors and inverts it (ldl16); the blocks below become W^T =
// M S^T and L^T = D^{-1} W^T and go to LDS; every block right of the panel
// takes its rank-16 update.  The next diagonal block is updated and factored
// before its owner's other blocks.  What bounds it is the serial chain of the
// ldl16 steps: 27 us (FP64) and 56 us (complex) for 128 columns; 19.9 -> 0.90 ms
// of diagonal blocks a factorization on the 40^3 FP64 Laplacian, 15.9 -> 1.2 ms
// on 16 Hermitian 30^3 matrices; the form before updated the block in global memory, one
// thread an element, 1.3 ms (FP64) and 1.7 ms (complex) for 256 columns.
// The inverses M_k (operand layout) and 1 / D go to `fin` for k_fac_lc.
// ---------------------------------------------------------------------------
constexpr int kFacWaves = kFacCols / 16;  // wavefronts, and 16-column blocks, of k_fac_diag
constexpr int kFacOff = kFacWaves * (kFacWaves - 1) / 2;
constexpr int kFacSlots = (kFacOff + kFacWaves - 1) / kFacWaves;

template <typename T>
__global__ void __launch_bounds__(64 * kFacWaves, 2)
    k_fac_diag(const DevPlan *__restrict__ plp, T *Pall, const FacNode *recs, int32_t count, unsigned long long *ferr) {
  constexpr int P = Planes<T>::P, NB = kFacWaves, LP = NB * 256;  // LP: doubles of one plane of a panel
  const DevPlan &pl = *plp;
  __shared__ double lp[P * LP], wp[P * LP];  // -L(i, k) (conjugated if Hermitian) and W(i, k), block i at 256 i
  __shared__ double ls[P * kLdlLds];
  const int64_t gidx = blockIdx.x;
  const int64_t l = gidx / count;
  const FacNode nd = recs[gidx - l * count];
  const int s = uniform(nd.s), ld = uniform(nd.ld), nb = (s + 15) / 16;
  T *Q = Pall + l * pl.panel_elems + nd.off;
  T *F = reinterpret_cast<T *>(pl.finv) + l * pl.fin_elems + nd.fin;
  const int wv = uniform((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const double cs = pl.csign;
  int bi[kFacSlots], bj[kFacSlots];  // the wavefront's other blocks, listed column by column
#pragma unroll
  for (int q = 0; q < kFacSlots; ++q) {
    int e = wv + NB * q, j = 0;
    while (j < NB - 1 && e >= NB - 1 - j) e -= NB - 1 - j, ++j;
    const bool in = j < NB - 1 && j + 1 + e < nb;
    bi[q] = uniform(in ? j + 1 + e : -1);
    bj[q] = uniform(in ? j : -1);
  }
  Blk<T> dg = blk_zero<T>(), ob[kFacSlots];
  if (wv < nb) dg = blk_load<T>(Q + (int64_t)(16 * wv) * ld + 16 * wv, ld, s - 16 * wv, s - 16 * wv);
#pragma unroll
  for (int q = 0; q < kFacSlots; ++q)
    if (bi[q] >= 0) ob[q] = blk_load<T>(Q + (int64_t)(16 * bj[q]) * ld + 16 * bi[q], ld, s - 16 * bi[q], 16);
  // L, D, M and 1 / D of diagonal block kk, from LDS
  auto store_diag = [&](int kk) {
    ldl16_store<T>(ls, Q + (int64_t)(16 * kk) * ld + 16 * kk, ld, min(16, s - 16 * kk));
    const Blk<T> m = ldl16_m<T>(ls, cs);
    T *Fk = F + kFacFin * kk;
#pragma unroll
    for (int v = 0; v < 4; ++v) gstore(Fk + 64 * v + lane, blk_get(m, v));
    if (lane < 16) gstore(Fk + 256 + lane, Planes<T>::from(&ls[kLdlD + lane], kLdlLds));
  };
  for (int k = 0; k < nb; ++k) {
    if (k > 0) {  // panel k - 1
      lds_barrier();
      const int kk = k - 1;
#pragma unroll
      for (int q = 0; q < kFacSlots; ++q)
        if (bj[q] == kk) {
          Blk<T> w = blk_zero<T>();
          blk_mma<T>(ldl16_m<T>(ls, cs), ob[q], w);
          const Blk<T> lo = blk_scale_rows<T>(w, ls + kLdlD, kLdlLds);
          blk_to_lds<T>(w, wp + 256 * bi[q], LP);
          blk_to_lds<T>(blk_neg_cj<T>(lo, cs), lp + 256 * bi[q], LP);
          blk_store<T>(lo, Q + (int64_t)(16 * kk) * ld + 16 * bi[q], ld, s - 16 * bi[q], 16);
        }
      if (wv == kk) store_diag(kk);
      lds_barrier();
      if (wv >= k && wv < nb)
        blk_mma_add<T>(blk_from_lds<T>(lp + 256 * wv, LP), blk_from_lds<T>(wp + 256 * wv, LP), dg);
    }
    if (wv == k) {
      const int w = min(16, s - 16 * k);
      ldl16_stage<T>(dg, w, ls);
      ldl16_block<T>(w, cs, ls, nd.first + 16 * k, ferr + l);
    }
    if (k > 0) {
#pragma unroll
      for (int q = 0; q < kFacSlots; ++q)
        if (bj[q] >= k)
          blk_mma_add<T>(blk_from_lds<T>(lp + 256 * bj[q], LP), blk_from_lds<T>(wp + 256 * bi[q], LP), ob[q]);
    }
  }
  wave_lds_fence();
  if (wv == nb - 1) store_diag(nb - 1);  // its own wavefront wrote it
}

// The rows below a diagonal block of at most kFacCols columns, in place: L =
// S L_KK^{-T} D^{-1} (L_KK^{-H} if Hermitian) by block forward substitution,
// one wavefront per 16 rows with its up to eight 16 x 16 blocks in registers:
//   W(:, k)^T = M_k S(:, k)^T, L(:, k)^T = D_k^{-1} W(:, k)^T,
//   S(:, j)^T -= L(j, k) W(:, k)^T for j > k.
// The four wavefronts of a workgroup share the step's operands (M_k and L(j,
// k)) through LDS, two buffers deep: the loads of step k + 2 are in flight
// while step k is multiplied.  No inverse of the whole L_KK is formed, and no
// column waits for another workgroup.  Bound by the chain of eight steps where
// few rows are left, else by MFMA: 40^3 FP64, inverse and product 2.4 ms a
// factorization before, 0.6 ms now; 16 Hermitian 30^3 matrices 8.0 -> 1.5 ms.
template <typename T>
__global__ void __launch_bounds__(NT, 2)
    k_fac_lc(const DevPlan *__restrict__ plp, T *Pall, const FacNode *recs, const int2 *rblocks, int32_t nrb) {
  constexpr int P = Planes<T>::P, NB = kFacWaves, LP = NB * 256;
  const DevPlan &pl = *plp;
  __shared__ double buf[2][P * LP];  // M_k at 256 k, -L(j, k) at 256 j, j > k
  __shared__ double dl[NB][P * 16];
  const int64_t gidx = blockIdx.x;
  const int64_t l = gidx / nrb;
  const int2 rb = rblocks[gidx - l * nrb];
  const FacNode nd = recs[uniform(rb.x)];
  const int s = uniform(nd.s), c = uniform(nd.c), ld = uniform(nd.ld), nb = (s + 15) / 16;
  T *Q = Pall + l * pl.panel_elems + nd.off;
  const T *F = reinterpret_cast<const T *>(pl.finv) + l * pl.fin_elems + nd.fin;
  const int wv = uniform((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const double cs = pl.csign;
  const int i0 = uniform(rb.y) * 64 + 16 * wv;
  T *R = Q + s + (i0 < c ? i0 : 0);  // the wavefront's 16 rows
  const int rows = i0 < c ? c - i0 : 0;
  Blk<T> sb[NB];
#pragma unroll
  for (int k = 0; k < NB; ++k)
    if (k < nb) sb[k] = blk_load<T>(R + (int64_t)(16 * k) * ld, ld, rows, s - 16 * k);
  if (threadIdx.x < 16 * NB) {
    const int k = threadIdx.x / 16;
    const T d = gload(F + (k < nb ? kFacFin * k + 256 + r : 256));
#pragma unroll
    for (int p = 0; p < P; ++p) dl[k][16 * p + r] = Planes<T>::get(d, p);
  }
  // thread t of the workgroup: element t of every 256-element block of a step
  T st[NB];
  auto load = [&](int k) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      if (j == k) st[j] = gload(F + kFacFin * k + (int)threadIdx.x);
      if (j > k && j < nb)
        st[j] = gload(Q + (((int64_t)(16 * k + 4 * wv + g) * ld + 16 * j + r) & opaque_mask(16 * j + r < s)));
    }
  };
  auto put = [&](int k) {
    double *b = buf[k & 1];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      if (j < k || j >= nb) continue;
      T v = st[j];
      if (j > k) {
        v = masked(v, opaque_mask(16 * j + r < s));
        v = cj(SOps<T>::scale(-1.0, v), cs);
      }
#pragma unroll
      for (int p = 0; p < P; ++p) b[p * LP + 256 * j + (int)threadIdx.x] = Planes<T>::get(v, p);
    }
  };
  load(0);
  put(0);
  if (nb > 1) load(1);
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    if (k >= nb) break;
    lds_barrier();
    const double *b = buf[k & 1];
    Blk<T> w = blk_zero<T>();
    blk_mma<T>(blk_from_lds<T>(b + 256 * k, LP), sb[k], w);
    if (k + 1 < nb) put(k + 1);
    if (k + 2 < nb) load(k + 2);
    blk_store<T>(blk_scale_rows<T>(w, dl[k], 16), R + (int64_t)(16 * k) * ld, ld, rows, s - 16 * k);
#pragma unroll
    for (int j = k + 1; j < NB; ++j)
      if (j < nb) blk_mma_add<T>(blk_from_lds<T>(b + 256 * j, LP), w, sb[j]);
  }
}

// ---------------------------------------------------------------------------
// Updates L D L^T on 64 x 64 tiles.
// ---------------------------------------------------------------------------

// B(k, x) = D_k M[k ld + i0 + x] (M conjugated if Hermitian): the pivots come
// from LDS and multiply the loaded values where these go to LDS, so that the
// loads stay in flight (a product at the load site waits for each of them).
template <typename T, int TK> struct FacLoadB : LoadDenseAIl<T, TK> {
  const T *D;  // LDS
  double cs;
  __device__ __forceinline__ FacLoadB(const T *M, int ld, int rows, int kend, int x0, const T *D_, double cs_)
      : LoadDenseAIl<T, TK>(M, ld, rows, kend, x0), D(D_), cs(cs_) {}
  __device__ __forceinline__ void store_bf(double *stg, int plane_off, int k0, const DVals<T, TK> &v) const {
#pragma unroll
    for (int m = 0; m < this->E; ++m) {
      const int k = min(k0 + this->kq + (NT / 64) * m, this->kend - 1);
      const T x = masked(cj(v.v[m], cs) * D[k], this->mask(k0, m));
#pragma unroll
      for (int p = 0; p < Planes<T>::P; ++p) stg[(plane_off + p) * TK * PITCH + this->slot(k0, m)] = Planes<T>::get(x, p);
    }
  }
};

// Tile (a, b), a >= b, of the update L D L^T of the rows below a column block,
// subtracted from
//   INNER:  the node's own columns behind a column block of kFacCols (the rows
//           and columns of the tile count from the block's end; columns
//           >= kFacCols / no atomics, the tiles of a launch are disjoint);
//   else:   the ancestors' entries of S_{C,C} (lower part: C-local rows i >= k)
//           over all columns of the node, with atomic adds.
// MFMA-bound on wide nodes, by the atomics on narrow ones.  Branch-free
// interleaved stages at two workgroups a CU; complex products in the
// four-product form: the 3M form's imaginary part carries an error of the real
// parts' size, which a nearly real pivot's imaginary part would show.  16 Hermitian
// 30^3 matrices: 12.7 ms of updates (nodes beyond the single-wavefront ones) ->
// 8.1 ms (5.5 in the 3M form).
template <typename T, bool INNER>
__global__ void __launch_bounds__(NT, 2)
    k_fac_update(const DevPlan *__restrict__ plp, T *Pall, const FacNode *recs, const int4 *tiles, int32_t ntiles) {
  const DevPlan &pl = *plp;
  constexpr int TK = DenseTK<T>::TK;
  constexpr int kStages = 2 * dense_stage_doubles<T, TK>();
  __shared__ double smem[kStages > tile_doubles<T>() ? kStages : tile_doubles<T>()];
  __shared__ T dls[INNER ? kFacCols : 256];
  const int64_t gidx = blockIdx.x;
  const int64_t l = gidx / ntiles;
  const int4 tl = tiles[gidx - l * ntiles];
  const int i0 = uniform(tl.y) * 64, k0 = uniform(tl.z) * 64;
  int s, c, ld, nc;  // contraction length, rows, leading dimension, columns of the target
  T *Pl = Pall + l * pl.panel_elems;
  T *Q;
  int64_t rp = 0;
  if constexpr (INNER) {
    const FacNode nd = recs[uniform(tl.x)];
    s = uniform(nd.s);
    c = uniform(nd.c);
    ld = uniform(nd.ld);
    nc = uniform(nd.rest);
    Q = Pl + nd.off;
  } else {
    const int K = uniform(tl.x);
    s = uniform(gp(pl.node_s)[K]);
    c = uniform(gp(pl.node_c)[K]);
    ld = s + c;
    nc = c;
    Q = Pl + gp(pl.node_off)[K];
    rp = gp(pl.node_rowptr)[K];
  }
  for (int k = threadIdx.x; k < s; k += NT) dls[k] = gload(Q + (int64_t)k * (ld + 1));
  lds_barrier();
  LoadDenseAIl<T, TK> la(Q + s, ld, c, s, i0);
  FacLoadB<T, TK> lb(Q + s, ld, nc, s, k0, dls, pl.csign);
  Acc<T> acc;
  gemm_dense_il<T, false>(0, s, la, lb, smem, acc);  // complex: four products (see above)
  acc_to_lds<T>(acc, smem);
  lds_barrier();
  const int i = threadIdx.x & 63, w = uniform((int)(threadIdx.x >> 6)), ig = i0 + i;
  constexpr int QN = 64 * 64 / NT;
  if constexpr (INNER) {
    T *R = Q + (int64_t)s * (ld + 1);
    T v[QN];
#pragma unroll
    for (int q = 0; q < QN; ++q) {
      const int kg = k0 + w + 4 * q;
      v[q] = gload(R + (((int64_t)kg * ld + ig) & opaque_mask(ig < c && kg < nc && ig >= kg)));
    }
#pragma unroll
    for (int q = 0; q < QN; ++q) {
      const int kg = k0 + w + 4 * q;
      if (ig < c && kg < nc && ig >= kg) gstore(R + (int64_t)kg * ld + ig, v[q] - lds_get<T>(smem, i, w + 4 * q));
    }
  } else {
    scatter_lower<T>(pl, rp, c, i0, k0, smem, Pl, [](double v, bool) { return -v; });
  }
}

__global__ void k_fac_init(unsigned long long *ferr, int64_t batch) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < batch) ferr[i] = ~0ull;
}

// log det B = sum_j log D_jj per matrix: the sum of the principal logarithms
// of the pivots (real part log |d|, imaginary part arg d; pi per negative
// pivot of a real matrix).  Workgroup q of a matrix takes pivots [q, q + 1)
// kLdetSpan and leaves its sum, reduced in a fixed order; the host adds the sums in
// order when it reads them.  Bound by the logarithms' arithmetic: one
// workgroup for a whole matrix took 215 us for 64,000 pivots.
template <typename T>
__global__ void __launch_bounds__(NT) k_fac_logdet(const DevPlan *__restrict__ plp, const T *Pall, double *out, int32_t nq) {
  constexpr int U = 4;
  static_assert(kLdetSpan % (NT * U) == 0, "whole rounds of loads");
  const DevPlan &pl = *plp;
  __shared__ double sr[NT], si[NT];
  const int64_t l = blockIdx.x / nq, q = blockIdx.x - l * nq;
  const T *P = Pall + l * pl.panel_elems;
  const int64_t jend = min((q + 1) * kLdetSpan, pl.n);
  double re = 0.0, im = 0.0;
  for (int64_t j0 = q * kLdetSpan + threadIdx.x; j0 < jend; j0 += NT * U) {
    T d[U];
#pragma unroll
    for (int u = 0; u < U; ++u) d[u] = gload(P + gp(pl.dpos)[min(j0 + NT * u, jend - 1)]);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (j0 + NT * u >= jend) break;
      if constexpr (Planes<T>::P == 1) {
        re += log(fabs(d[u]));
        if (d[u] < 0) im += M_PI;
      } else {
        re += log(hypot(d[u].re, d[u].im));
        im += atan2(d[u].im, d[u].re);
      }
    }
  }
  sr[threadIdx.x] = re;
  si[threadIdx.x] = im;
  __syncthreads();
  for (int h = NT / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) {
      sr[threadIdx.x] += sr[threadIdx.x + h];
      si[threadIdx.x] += si[threadIdx.x + h];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[2 * (int64_t)blockIdx.x] = sr[0];
    out[2 * (int64_t)blockIdx.x + 1] = si[0];
  }
}

template <typename T>
hipError_t factor_impl(const DevPlan &pl, const DevPlan *dpl, const FactorAux &fa, const void *values, void *panels,
                       hipStream_t st) {
  T *P = reinterpret_cast<T *>(panels);
  hipError_t e = launch_scatter(pl, dpl, sizeof(T) == 16, values, panels, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_fac_init, dim3((unsigned)((pl.batch + 255) / 256)), dim3(256), 0, st, pl.ferr, pl.batch);
  const unsigned B = (unsigned)pl.batch;
  for (int q = 0; q < fa.nlev; ++q) {
    const FacLevel &lv = fa.lev[q];
    if (lv.small_n > 0)
      hipLaunchKernelGGL(k_fac_small<T>, dim3(lv.small_n * B), dim3(64), 0, st, dpl, P, fa.nodes + lv.small_b,
                         lv.small_n, pl.ferr);
    if (lv.mid_n > 0)
      hipLaunchKernelGGL(k_fac_mid<T>, dim3(lv.mid_n * B), dim3(NT), 0, st, dpl, P, fa.nodes + lv.mid_b, lv.mid_n,
                         pl.ferr);
    for (int h = 0; h < 2; ++h) {  // column block h of the nodes
      if (lv.diag_n[h] > 0)
        hipLaunchKernelGGL(k_fac_diag<T>, dim3(lv.diag_n[h] * B), dim3(64 * kFacWaves), 0, st, dpl, P,
                           fa.nodes + lv.diag_b[h], lv.diag_n[h], pl.ferr);
      if (lv.rb_n[h] > 0)
        hipLaunchKernelGGL(k_fac_lc<T>, dim3(lv.rb_n[h] * B), dim3(NT), 0, st, dpl, P, fa.nodes,
                           fa.rblocks + lv.rb_b[h], lv.rb_n[h]);
      if (h == 0 && lv.inner_n > 0)
        hipLaunchKernelGGL((k_fac_update<T, true>), dim3(lv.inner_n * B), dim3(NT), 0, st, dpl, P, fa.nodes,
                           fa.tiles + lv.inner_b, lv.inner_n);
    }
    if (lv.tiles_n > 0)
      hipLaunchKernelGGL((k_fac_update<T, false>), dim3(lv.tiles_n * B), dim3(NT), 0, st, dpl, P, fa.nodes,
                         fa.tiles + lv.tiles_b, lv.tiles_n);
  }
  const int32_t nq = (int32_t)ldet_parts(pl.n);
  hipLaunchKernelGGL(k_fac_logdet<T>, dim3(B * nq), dim3(NT), 0, st, dpl, P, pl.fldet, nq);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_factor(const DevPlan &pl, const DevPlan *dpl, const FactorAux &fa, bool cplx_, const void *values,
                         void *panels, hipStream_t st) {
  return cplx_ ? factor_impl<cplx>(pl, dpl, fa, values, panels, st)
               : factor_impl<double>(pl, dpl, fa, values, panels, st);
}

}  // namespace selinv
