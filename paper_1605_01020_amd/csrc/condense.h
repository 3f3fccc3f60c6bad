// Shared declarations of the condensation translation units.
#pragma once

#include <algorithm>

#include "common.h"

namespace iedg {

// One segment: E elements of one size with their inputs and outputs.
template <typename T>
struct CondenseArgs {
  int E, n, t;
  const double *A, *B, *C, *D, *F;
  T *LU, *U12, *L21, *Ke;
  int32_t* perm;
  double *w, *r;
  DeviceStatus* status;
};

// The elements one launch sequence condenses, all of one size (n, t): item i
// is element i of `a`, or element items[i].y of segs[items[i].x] (device
// arrays) when items is not null.
template <typename T>
struct CondenseWork {
  CondenseArgs<T> a;
  const CondenseArgs<T>* segs;
  const int2* items;
  int count;
  int n, t;
  // the panels' inverses do not fit the elements' Ke blocks (small t)
  int self;
};

// Condenses every item of w: sub-panel width lw (8 or 16), panel width ct
// (64, or 128 in FP32 storage).  Each is defined in the translation unit of
// its precision.
hipError_t condense_run_f64(const CondenseWork<double>& w, int lw, int ct, hipStream_t s);
hipError_t condense_run_f32(const CondenseWork<float>& w, int lw, int ct, hipStream_t s);
hipError_t condense_run_bf16(const CondenseWork<float>& w, int lw, int ct, hipStream_t s);

// The panel launches of one precision (condense_panel.hip).  c0: first column
// of the panel the inverse belongs to; [cb, ce): the columns factored, at most
// 64; right: columns of the panel's right half still to come (left half of a
// 128-wide panel), else 0.
template <typename T>
hipError_t condense_panel(const CondenseWork<T>& w, int lw, int c0, int cb, int ce, int right, hipStream_t s);

// Untuned sub-panel width for elements of n local dofs and t trace dofs: 16,
// but 8 for FP64 elements with more than 512 rows of A or of C and for FP32
// ones with more than 1536 or 512.  512 elements, 8 against 16 wide: FP64
// n = 160 0.67 / 0.66 ms, n = 540 7.9 / 7.8, n = 1280 50.0 / 49.8, and n = 2500,
// where a thread's rows of 16 FP64 columns are spilled, 301 / 326; FP32 n = 540
// 5.5 / 4.9, n = 1280 29.7 / 25.6, and n = 2500 162 / 141, where the tuned table
// takes 16.
inline int default_leaf_width(size_t elem_bytes, int n, int t) {
  const int qa = (n + 511) / 512, qc = (t + 511) / 512;
  const int q = (qa <= 1 && qc <= 1) ? 2 : (qa <= 3 && qc <= 1) ? 4 : 7;
  return (elem_bytes == 8 ? q <= 2 : q <= 4) ? 16 : 8;
}

// Untuned panel width: 128 columns for FP32 storage (FP32 or BF16
// operands) and elements of at least 1024 local dofs, else 64 (the only
// width FP64 storage is built for).  A wider panel halves the launches and
// reads of L and costs the update between its halves: 512 elements, 64 against
// 128 wide, FP32 n = 540 4.9 / 5.5 ms, n = 1280 25.6 / 25.6, n = 2500 148 / 141;
// BF16 4.1 / 4.3, 20.0 / 18.4, 114 / 92.
inline int default_panel_width(size_t elem_bytes, int n) {
  return elem_bytes == 4 && n >= 1024 ? 128 : 64;
}

// Largest n and t the panel kernels are built for: 4 rows of [A; C] per
// thread at 1024 threads, and 16-bit row indices in LDS.
constexpr int kCondenseMaxN = 5 * 512, kCondenseMaxT = 2 * 512;
static_assert(kCondenseMaxN + kCondenseMaxT <= 4 * 1024, "rows per thread of the panel kernels");

// ---- scratch for a panel's inverse -----------------------------------------
// L_pp^{-1} of the current panel as up to three 64 x 64 row-major blocks: rows
// and columns [0, 64), rows [64, 128) x columns [0, 64), rows and columns
// [64, 128).  It lives in the element's Ke block, which nothing else touches
// before the Schur complement is written; elements whose Ke is smaller form
// the inverse again where it is used (CondenseWork::self).
constexpr int kInvBlock = 64 * 64;
inline bool inverse_fits(int n, int t, int ct) {
  return (size_t)t * t >= (size_t)(std::min(n, ct) > 64 ? 3 : 1) * kInvBlock;
}

// ---- device side: one element of the work -----------------------------------
template <typename T>
struct Elem {
  int n, t, N;
  const double *A, *B, *C, *D, *F;
  T *LU, *U12, *L21, *Ke;
  int32_t* perm;
  double *w, *r;
  DeviceStatus* status;
  int id;

  // Rows are pivot positions: position p < n lives in physical row perm[p]
  // of A, B, F, LU, U12 and w.
  __device__ __forceinline__ T* lrow(int p, int phys) const {
    return p < n ? LU + (size_t)phys * n : L21 + (size_t)(p - n) * n;
  }
};

template <typename T>
__device__ __forceinline__ Elem<T> condense_elem(const CondenseWork<T>& wk, int it) {
  CondenseArgs<T> a;
  int e = it;
  if (wk.items) {
    const int2 w = wk.items[it];
    a = wk.segs[w.x];
    e = w.y;
  } else {
    a = wk.a;
  }
  const int n = wk.n, t = wk.t;
  const size_t nn = (size_t)n * n, nt = (size_t)n * t, tt = (size_t)t * t;
  Elem<T> el;
  el.n = n; el.t = t; el.N = n + t;
  el.A = a.A + e * nn; el.B = a.B + e * nt; el.C = a.C + e * nt; el.D = a.D + e * tt;
  el.F = a.F ? a.F + (size_t)e * n : nullptr;
  el.LU = a.LU + e * nn; el.U12 = a.U12 + e * nt; el.L21 = a.L21 + e * nt; el.Ke = a.Ke + e * tt;
  el.perm = a.perm + (size_t)e * n;
  el.w = a.w ? a.w + (size_t)e * n : nullptr;
  el.r = a.r ? a.r + (size_t)e * t : nullptr;
  el.status = a.status;
  el.id = e;
  return el;
}

// Tile kernels: block -> (item, tile).  Workgroups go to the 8 XCDs in turn
// by block index, so that every tile of an item (and the next launch's tiles of
// it) runs on one XCD and shares operands in its L2.  Consecutive tiles on
// consecutive XCDs measured no better for few items either, down to one: 1, 8,
// 64 FP64 elements of n = 540 1.737, 1.737, 2.152 ms against 1.750, 1.752,
// 2.172, BF16 of n = 2500 10.06, 10.60, 17.9 against 10.2, 10.8, 18.9.
template <typename T>
__device__ __forceinline__ bool condense_locate(const CondenseWork<T>& wk, int tiles, int& it, int& tile) {
  const int b = blockIdx.x, s = b >> 3;
  it = (s / tiles) * 8 + (b & 7);
  tile = s % tiles;
  return it < wk.count;
}
template <typename T>
inline dim3 condense_grid(const CondenseWork<T>& wk, int tiles) {
  return dim3((unsigned)((wk.count + 7) / 8 * 8 * tiles));
}

// ---- growing L_pp^{-1} where L may hold infinities or NaN -----------------------
// As grow_inverse, for an element without a pivot: the zeros of whole blocks
// would spread them to rows that do not depend on them, so every entry takes
// the products of the triangles alone, in the same order.
template <typename T>
__device__ __forceinline__ void grow_inverse_entries(T* Li, int LS, const T* Lb, T* Y, int kp, int sw) {
  int tid = threadIdx.x, nt = blockDim.x;
  asm volatile("" : "+v"(tid));  // (cold: nothing of it is computed ahead and kept)
#pragma unroll 1
  for (int o = tid; o < sw * kp; o += nt) {
    const int i = o / kp, k = o % kp;
    T acc = T(0);
#pragma unroll 1
    for (int m = k; m < kp; ++m) acc = fma(Lb[i * 64 + m], Li[m * LS + k], acc);
    Y[i * 64 + k] = acc;
  }
  if (tid < sw)
#pragma unroll 1
    for (int i = tid; i < sw; ++i) {
      T acc = i == tid ? T(1) : T(0);
#pragma unroll 1
      for (int m = tid; m < i; ++m) acc = fma(-Lb[i * 64 + kp + m], Li[(kp + m) * LS + kp + tid], acc);
      Li[(kp + i) * LS + kp + tid] = acc;
    }
  __syncthreads();
#pragma unroll 1
  for (int o = tid; o < sw * kp; o += nt) {
    const int i = o / kp, k = o % kp;
    T acc = T(0);
#pragma unroll 1
    for (int m = 0; m <= i; ++m) acc = fma(Li[(kp + i) * LS + kp + m], Y[m * 64 + k], acc);
    Li[(kp + i) * LS + k] = -acc;
  }
  __syncthreads();
}

// ---- growing L_pp^{-1} ---------------------------------------------------
// Rows kp .. kp+sw of the inverse of a unit lower triangle from rows 0 .. kp
// of it (Li, stride LS, zero above the diagonal and in rows >= kp) and the
// triangle's rows kp .. kp+sw (Lb, LW x 64, strictly lower part):
//   inv = [L11^{-1} 0; -L22^{-1} L21 L11^{-1}  L22^{-1}].
// Every product is an ascending chain of fused multiply-adds (the MFMA sums
// its four products in that order, measured against fma), zeros aside.  L22 is
// inverted by one wave as a chain of rank-one MFMAs on the identity, each with
// one nonzero k, while others form L21 L11^{-1}: in vector registers its rows
// would cost more than the rest of the growth.  Y: LW x 64 of LDS.  Called by
// every thread; ends with a barrier.
// odd (uniform): L may hold infinities or NaN; grow_inverse_entries then.
template <typename T, int LW>
__device__ __forceinline__ void grow_inverse(T* Li, int LS, const T* Lb, T* Y, int kp, int sw, bool odd) {
  typedef Mfma<T> MF;
  if (__builtin_expect(odd, 0)) {
    grow_inverse_entries<T>(Li, LS, Lb, Y, kp, sw);
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lg = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
  const int kb = (kp + 15) / 16;  // column blocks of the finished part (at most 4)
  for (int b = wv; b < kb; b += nw) {
    typename MF::acc_t acc = MF::zero();
    // (kp is a multiple of 4; rows kp .. are written below by another wave
    // before the barrier, so none of them may be read here)
    for (int m = 0; m < kp; m += 4) {
      const T av = li < sw ? Lb[li * 64 + m + lg] : T(0);
      acc = MF::mac(av, Li[(m + lg) * LS + 16 * b + li], acc);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = MF::row(lane, v);
      if (row < LW) Y[row * 64 + 16 * b + li] = acc[v];
    }
  }
  if (wv == nw - 1) {
    // L22^{-1}: row i takes -L[i][m] (row m) for m = 0 .. i-1 in turn
    typename MF::acc_t acc;
    T av[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int m = MF::row(lane, v);  // this lane group's row in register v
      acc[v] = m == li ? T(1) : T(0);
      av[v] = (m < sw && li < sw && li > m) ? -Lb[li * 64 + kp + m] : T(0);
    }
#pragma unroll
    for (int m = 0; m < LW; ++m) {
      const int v = sizeof(T) == 4 ? m & 3 : m >> 2, g = sizeof(T) == 4 ? m >> 2 : m & 3;  // MF::row(16 g, v) == m
      acc = MF::mac(lg == g ? av[v] : T(0), lg == g ? acc[v] : T(0), acc);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = MF::row(lane, v);
      if (row < sw && li < sw) Li[(kp + row) * LS + kp + li] = acc[v];
    }
  }
  __syncthreads();
  for (int b = wv; b < kb; b += nw) {
    typename MF::acc_t acc = MF::zero();
#pragma unroll
    for (int m = 0; m < LW; m += 4) {
      // rows and columns at and past sw: not stored, and zero
      const T av = (li < sw && m + lg < sw) ? Li[(kp + li) * LS + kp + m + lg] : T(0);
      const T bv = m + lg < sw ? Y[(m + lg) * 64 + 16 * b + li] : T(0);
      acc = MF::mac(av, bv, acc);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = MF::row(lane, v), col = 16 * b + li;
      if (row < sw && col < kp) Li[(kp + row) * LS + col] = -acc[v];
    }
  }
  __syncthreads();
}

// The bottom-left block of a 128-wide panel's inverse, -L22^{-1} (L21 L11^{-1}):
// inv11 (64 x 64, stride s1) and inv22 (wr x wr in a 64 x 64 block, stride s2)
// are the halves' inverses, l21(i, k) reads L21.  Y: 64 x 65 of LDS; out:
// 64 x 64, rows >= wr zero.  odd: as for grow_inverse, entry by entry.  Called by
// every thread; ends with a barrier.
template <typename T, typename F>
__device__ __forceinline__ void inverse_offdiag(const T* inv11, int s1, const T* inv22, int s2, int wr, F l21, T* Y,
                                                T* out, bool odd) {
  typedef Mfma<T> MF;
  if (__builtin_expect(odd, 0)) {
#pragma unroll 1
    for (int o = threadIdx.x; o < 64 * wr; o += blockDim.x) {
      const int i = o >> 6, k = o & 63;
      T acc = T(0);
#pragma unroll 1
      for (int m = k; m < 64; ++m) acc = fma(l21(i, m), inv11[m * s1 + k], acc);
      Y[i * 65 + k] = acc;
    }
    __syncthreads();
#pragma unroll 1
    for (int o = threadIdx.x; o < 64 * 64; o += blockDim.x) {
      const int i = o >> 6, k = o & 63;
      T acc = T(0);
#pragma unroll 1
      for (int m = 0; m <= i && i < wr; ++m) acc = fma(inv22[i * s2 + m], Y[m * 65 + k], acc);
      out[o] = -acc;
    }
    __syncthreads();
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lg = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
  for (int b = wv; b < 16; b += nw) {
    const int ib = b >> 2, kb = b & 3;
    T av[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) av[q] = 16 * ib + li < wr ? l21(16 * ib + li, 4 * q + lg) : T(0);
    typename MF::acc_t acc = MF::zero();
#pragma unroll
    for (int q = 0; q < 16; ++q) acc = MF::mac(av[q], inv11[(4 * q + lg) * s1 + 16 * kb + li], acc);
#pragma unroll
    for (int v = 0; v < 4; ++v) Y[(16 * ib + MF::row(lane, v)) * 65 + 16 * kb + li] = acc[v];
  }
  __syncthreads();
  for (int b = wv; b < 16; b += nw) {
    const int ib = b >> 2, kb = b & 3;
    typename MF::acc_t acc = MF::zero();
    for (int m = 0; m < 16 * (ib + 1); m += 4)
      acc = MF::mac(inv22[(16 * ib + li) * s2 + m + lg], Y[(m + lg) * 65 + 16 * kb + li], acc);
#pragma unroll
    for (int v = 0; v < 4; ++v) out[(16 * ib + MF::row(lane, v)) * 64 + 16 * kb + li] = -acc[v];
  }
  __syncthreads();
}

}  // namespace iedg
