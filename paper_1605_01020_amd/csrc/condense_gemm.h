#pragma once
// Element static condensation on gfx950 (section 2.2.1, eq. LS): the tile
// kernels and the launch sequence.  Included by one translation unit per
// precision (condense_<p>.hip); the panel factorisation is condense_panel.hip.
//
// Per element the bordered matrix  M = [A B F; C D 0]  (N = n + t rows,
// NC = N + 1 columns with F) is reduced by n steps of Gaussian elimination
// with partial pivoting over the rows of A.  After those steps
//   rows of A:  unit-lower L and U of P A, U12 = L^{-1} P B, w = L^{-1} P F
//   rows of C:  L21 = C U^{-1},  Ke = D - L21 U12,  r = -L21 w
// so the trailing block is the Schur complement D - C A^{-1} B of eq. LS.
//
// Row interchanges never move data: pivot position i of P A lives in the
// physical row perm[i] of every A-row-indexed array (A itself, LU, U12, w),
// and only the row map is updated when a pivot is chosen.
//
// Schedule: every phase of a panel step is a launch of its own over all
// elements, in Crout order, panels of CT = 64 or (FP32 storage) 128 columns:
//   for each panel [c0, c1):
//     1. condense_col:   M[c0:, c0:c1] = in - L[c0:, :c0] U[:c0, c0:c1]
//     2. condense_panel: the panel is factored (a 128-wide one as two halves
//        of 64 with one update, condense_col with HALF = 1, between them); its
//        L^{-1} goes to scratch
//     3. condense_row:   U[c0:c1, c1:] = L_pp^{-1} (in - L[c0:c1, :c0] U[:c0, c1:])
//   4. condense_schur: M[n:, n:] = in - L21 U12
// One workgroup per element for the whole elimination would leave the chip
// to whichever phase each element is in: its panels wait on their chain of
// pivots with one workgroup a CU, the matrix cores idle meanwhile, fewer
// elements than CUs leave CUs idle, and the last round of elements too.  As
// launches, the products of every element spread over all CUs in tiles, and
// the panels, which need few registers and little LDS on their own, share
// them.  Crout order reads every input once, in its FP64 form, straight into
// the accumulators, and writes every output once.  Whole condensation, one
// workgroup an element -> launches: 64 FP64 elements of n = 540 4.59 -> 2.19 ms,
// 864 FP32 elements of n = 1280 67.1 -> 44.1 ms (panel columns 14.6, panel rows
// 14.4, panels 8.2, Schur block 5.2 ms), 216 BF16 elements of n = 2500 62.9 ->
// 42.7 ms.
//
// BF16 operand mode: the operands of 1, 3 and 4 are rounded to BF16 once, as
// they enter LDS; accumulation, panels and storage stay FP32.
#include "condense.h"

namespace iedg {

constexpr int GT = 256;  // threads per workgroup of the tile kernels (4 waves)

// Round to nearest even FP32 -> BF16 (bit pattern); NaN stays NaN.
__device__ __forceinline__ unsigned to_bf16(float f) {
  const unsigned u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
  return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

typedef short bf16x4 __attribute__((ext_vector_type(4)));

// ---- the tile engine --------------------------------------------------------
// acc += (-L) U over k for a workgroup's TM x TN tile, operands through LDS in
// slabs of KC, the next slab's loads in flight in registers while one is
// multiplied.  Every entry takes its products in ascending k, four (BF16: 16)
// per MFMA, so neither the tile shape nor the order of the phases shows in the
// result.  Waves are 2 x 2, or with COLS all along columns (each wave then
// holds every row of its columns, which the panel-row triangular solve needs).
//
// What bounds it: the matrix cores (FP32: 105 TFLOP/s of 155 where K is long,
// 112 in the Schur block), and for short K the inputs, read in 1 KB pieces of
// rows at 3 TB/s (the first panel's columns, which have no product).  BF16
// (216 elements of n = 2500): the operands' reads from beyond the L2, 3.7 TB/s
// for the whole of the panel columns, vector instructions issuing 31% of the
// time and the matrix cores busy 12%.  L is read a row at a time with rows far apart, so a slab is as deep as a
// cache line is long, 32 in FP32 (16 deep, two slabs in LDS, left waves
// waiting 58% of the time and the matrix cores busy 48%) and 16 in FP64 (32
// deep costs a wave a SIMD: 512 elements of n = 1280 54.2 ms, 49.5 ms 16 deep).
// One slab in LDS, and the next in registers.
//
// LDS, MM = 0: slabs k-major, A at As[k][row ^ swizzle(k)], B at
// Bs[k][col ^ 16 (k & 3)]: the four k of a fragment read then lie in
// different banks, and so do the k of a vector write.  MM = 1: BF16,
// row-major with KC k per row, k group g = k / 4 of a row at g ^ 2 (row / 4 % 4):
// a fragment is one 8-byte read.
template <typename T, int MM, int TM, int TN, bool COLS>
struct Tile {
  static constexpr int KC = sizeof(T) == 8 ? 16 : 32;  // slab depth
  static constexpr int WR = COLS ? 1 : 2, WC = 4 / WR;
  static constexpr int WM = TM / WR, WN = TN / WC, RB = WM / 16, CB = WN / 16;
  static constexpr int V = 16 / sizeof(T);            // values per 16-byte vector
  static constexpr int AL = TM * KC / (V * GT);       // A vectors per thread and slab
  static constexpr int BC = MM ? TN / 64 : 8 / (int)sizeof(T);  // B columns per load
  static constexpr int BL = TN * KC / (BC * GT);      // B loads per thread and slab
  static constexpr int ES = MM ? 2 : (int)sizeof(T);  // bytes per LDS value
  static constexpr int STAGE = KC * (TM + TN) * ES;   // bytes
  static_assert(AL >= 1 && BL >= 1 && (MM == 0 || BL == 8), "tile shape");

  typedef typename Mfma<T>::acc_t acc_t;
  typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
  typedef T bvec __attribute__((ext_vector_type(BC)));

  // Operand addresses (global: pointers read from a segment in memory would
  // make generic loads, which also hold up LDS reads).  A: row pointers at
  // this thread's k.  B: this thread's column, bytes between rows.  rhs: that
  // column is the right-hand side, read from w (FP64): 8 bytes a row like any
  // column of a tile that may hold it, converted on the way to LDS.
  typedef const __attribute__((address_space(1))) T* gptr;
  typedef const __attribute__((address_space(1))) vec* gvec;
  typedef const __attribute__((address_space(1))) bvec* gbvec;
  typedef const __attribute__((address_space(1))) char* gbytes;
  struct Ops {
    gptr a[AL];
    gbytes b;
    unsigned bstride;
    bool rhs;
    // columns of m (stride columns a row) from j; column `width` is w, where
    // there is one, and columns past the last read column 0 (never stored)
    __device__ __forceinline__ void columns(const T* m, int stride, int j, int width, const double* wcol) {
      rhs = wcol && j == width;
      b = rhs ? (gbytes)wcol : (gbytes)(m + (j < width ? j : 0));
      bstride = rhs ? 8 : stride * (int)sizeof(T);
    }
  };

  static __device__ __forceinline__ int a_row(int q) { return (threadIdx.x + q * GT) / (KC / V); }
  static __device__ __forceinline__ int a_k() { return V * (threadIdx.x % (KC / V)); }
  static __device__ __forceinline__ int b_col() { return BC * (threadIdx.x % (TN / BC)); }
  static __device__ __forceinline__ int b_k(int q) {
    return MM ? 4 * (threadIdx.x / (TN / BC) + 4 * (q >> 2)) + (q & 3) : threadIdx.x / (TN / BC) + q * (GT / (TN / BC));
  }

  static __device__ __forceinline__ int swizzle(int k) { return 16 * ((k ^ (k >> 2)) & 3) ^ 8 * ((k >> 4) & 1); }
  struct Slab {
    vec a[AL];
    bvec b[BL];
  };
  // Raw loads only: nothing waits for a value before it is stored to LDS.
  // TAIL: K is a multiple of 4 but not of KC (past it k = 0 is read, and
  // masked on the way to LDS).
  template <bool TAIL>
  static __device__ __forceinline__ void load(const Ops& o, const unsigned short* sp, int k0, int K, Slab& s) {
    unsigned pr[BL];
#pragma unroll
    for (int q = 0; q < BL; ++q) {
      const int k = k0 + b_k(q);
      pr[q] = sp[!TAIL || k < K ? k : 0];
    }
    const int ka = !TAIL || k0 + a_k() < K ? k0 : 0;
#pragma unroll
    for (int q = 0; q < AL; ++q) s.a[q] = *(gvec)(o.a[q] + ka);
#pragma unroll
    for (int q = 0; q < BL; ++q) s.b[q] = *(gbvec)(o.b + (size_t)pr[q] * o.bstride);
  }
  template <bool TAIL>
  static __device__ __forceinline__ void store(const Ops& o, unsigned char* stage, Slab& s, int k0, int K) {
    if constexpr (sizeof(bvec) == 8 && sizeof(T) == 4) {
      if (o.rhs)
#pragma unroll
        for (int q = 0; q < BL; ++q) s.b[q][0] = (T)__hiloint2double(__float_as_int(s.b[q][1]), __float_as_int(s.b[q][0]));
    }
    if constexpr (TAIL) {
      if (k0 + a_k() >= K)
#pragma unroll
        for (int q = 0; q < AL; ++q) s.a[q] = vec(T(0));
#pragma unroll
      for (int q = 0; q < BL; ++q)
        if (k0 + b_k(q) >= K) s.b[q] = bvec(T(0));
    }
    if constexpr (MM == 0) {
      T* As = reinterpret_cast<T*>(stage);
      T* Bs = As + KC * TM;
#pragma unroll
      for (int q = 0; q < AL; ++q)
#pragma unroll
        for (int i = 0; i < V; ++i) {
          const int k = a_k() + i;
          As[k * TM + (a_row(q) ^ swizzle(k))] = -s.a[q][i];  // L enters negated
        }
#pragma unroll
      for (int q = 0; q < BL; ++q) {
        const int k = b_k(q);
        *reinterpret_cast<bvec*>(Bs + k * TN + (b_col() ^ (16 * (k & 3)))) = s.b[q];
      }
    } else {
      unsigned* As = reinterpret_cast<unsigned*>(stage);
      unsigned* Bs = As + KC * TM / 2;
#pragma unroll
      for (int q = 0; q < AL; ++q) {
        const int row = a_row(q), g = (a_k() >> 2) ^ (((row >> 2) & 3) << 1);
        uint2 v;
        v.x = to_bf16(-s.a[q][0]) | (to_bf16(-s.a[q][1]) << 16);
        v.y = to_bf16(-s.a[q][2]) | (to_bf16(-s.a[q][3]) << 16);
        *reinterpret_cast<uint2*>(As + row * (KC / 2) + 2 * g) = v;
      }
#pragma unroll
      for (int c = 0; c < BC; ++c) {
        const int col = b_col() + c, sw = ((col >> 2) & 3) << 1;
#pragma unroll
        for (int q = 0; q < BL; q += 4) {
          const int g = (b_k(q) >> 2) ^ sw;
          uint2 v;
          v.x = to_bf16(s.b[q][c]) | (to_bf16(s.b[q + 1][c]) << 16);
          v.y = to_bf16(s.b[q + 2][c]) | (to_bf16(s.b[q + 3][c]) << 16);
          *reinterpret_cast<uint2*>(Bs + col * (KC / 2) + 2 * g) = v;
        }
      }
    }
  }
  static __device__ __forceinline__ void mma(const unsigned char* stage, int wr0, int wc0, acc_t (&acc)[RB][CB]) {
    const int lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
    if constexpr (MM == 0) {
      const T* As = reinterpret_cast<const T*>(stage) + lg * TM + wr0;
      const T* Bs = reinterpret_cast<const T*>(stage) + KC * TM + lg * TN + li;
#pragma unroll
      for (int ks = 0; ks < KC / 4; ++ks) {
        // two k-steps' fragments at a time: all of a slab's would not fit
        // beside the accumulators and the next slab's loads
        if (ks % 2 == 0) __builtin_amdgcn_sched_barrier(0);
        T av[RB], bv[CB];
        // (wr0 is a multiple of 64: the swizzle stays inside 64 rows)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) av[rb] = As[4 * ks * TM + 64 * (rb >> 2) + 16 * ((rb ^ ks ^ lg) & 3) + (li ^ (8 * (ks >> 2)))];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) bv[cb] = Bs[4 * ks * TN + ((wc0 + 16 * cb) ^ (16 * lg))];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int cb = 0; cb < CB; ++cb) acc[rb][cb] = Mfma<T>::mac(av[rb], bv[cb], acc[rb][cb]);
      }
    } else {
      const unsigned* As = reinterpret_cast<const unsigned*>(stage) + (wr0 + li) * (KC / 2);
      const unsigned* Bs = reinterpret_cast<const unsigned*>(stage) + KC * TM / 2 + (wc0 + li) * (KC / 2);
#pragma unroll
      for (int ks = 0; ks < KC / 16; ++ks) {
        const int g = (4 * ks + lg) ^ ((li >> 2) << 1);
        bf16x4 av[RB], bv[CB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) av[rb] = *reinterpret_cast<const bf16x4*>(As + 16 * rb * (KC / 2) + 2 * g);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) bv[cb] = *reinterpret_cast<const bf16x4*>(Bs + 16 * cb * (KC / 2) + 2 * g);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int cb = 0; cb < CB; ++cb)
            acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(av[rb], bv[cb], acc[rb][cb], 0, 0, 0);
      }
    }
  }
  // acc += (-L) U for k in [0, K), K > 0; sp[k]: physical row of U's row k.
  // lds: one slab.  Starts with every thread past the last use of lds.
  template <bool TAIL>
  static __device__ __forceinline__ void product(const Ops& o, const unsigned short* sp, int K, unsigned char* lds,
                                                 int wr0, int wc0, acc_t (&acc)[RB][CB]) {
    Slab s;
    load<TAIL>(o, sp, 0, K, s);
    for (int k0 = 0; k0 < K; k0 += KC) {
      store<TAIL>(o, lds, s, k0, K);
      __syncthreads();
      if (k0 + KC < K) load<TAIL>(o, sp, k0 + KC, K, s);
      mma(lds, wr0, wc0, acc);
      __syncthreads();
    }
  }
};

// v as a value the compiler cannot follow: what is computed from it after the
// slab loop is not computed before it and carried through it in registers.
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Between the row blocks of a tile's inputs.  FP32 storage: two row blocks'
// FP64 inputs in flight, as more would set the kernel's registers (and so the
// waves a SIMD holds) by its first microseconds.
template <typename T>
__device__ __forceinline__ void input_step(int rb) {
  if (sizeof(T) == 4 && rb % 2 == 0) __builtin_amdgcn_sched_barrier(0);
}

// Row map of a launch in LDS: sp[k] for U's rows (positions kb .. kb+K-1) and
// rp[i] for the tile's rows (positions r0 .. r0+TM-1, of A).
template <int TM>
__device__ __forceinline__ void load_row_map(const int32_t* perm, bool identity, int n, int kb, int K, int r0,
                                             unsigned short* sp, unsigned short* rp) {
  for (int i = threadIdx.x; i < K; i += GT) sp[i] = (unsigned short)perm[kb + i];
  if (r0 >= 0)
    for (int i = threadIdx.x; i < TM; i += GT)
      rp[i] = (unsigned short)(r0 + i < n ? (identity ? r0 + i : perm[r0 + i]) : 0);
  __syncthreads();
}

// ---- 1. panel columns, and the update between a panel's halves --------------
// HALF = 0: M[r0:, c0:c1] = in - L[r0:, :c0] U[:c0, c0:c1], rows from c0.
// HALF = 1: M[r0:, cm:c1] -= L[r0:, c0:cm] U[c0:cm, cm:c1], rows from cm =
//   c0 + 64, FP32 operands in every operand mode.
// c0, c1: columns written; kb: first k; rows from c0 on.
template <typename T, int MM, int TN, int HALF>
__global__ __launch_bounds__(GT, sizeof(T) == 8 ? 2 : 3) void condense_col_kernel(CondenseWork<T> wk, int tiles, int c0, int c1,
                                                                               int kb) {
  typedef Tile<T, MM, 128, TN, false> TL;
  extern __shared__ __align__(16) unsigned char lds[];
  int it, tile;
  if (!condense_locate(wk, tiles, it, tile)) return;
  const Elem<T> el = condense_elem(wk, it);
  const int n = el.n, K = c0 - kb, r0 = c0 + 128 * tile;
  unsigned short* rp = reinterpret_cast<unsigned short*>(lds + TL::STAGE);
  unsigned short* sp = rp + 128;
  load_row_map<128>(el.perm, c0 == 0, n, kb, K, r0, sp, rp);
  int lane = threadIdx.x & 63;
  const int li = lane & 15;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr0 = (wv % TL::WR) * TL::WM, wc0 = (wv / TL::WR) * TL::WN;

  typename TL::acc_t acc[TL::RB][TL::CB];
#pragma unroll
  for (int rb = 0; rb < TL::RB; ++rb) {
    input_step<T>(rb);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = wr0 + 16 * rb + Mfma<T>::row(lane, v), row = r0 + i;
      if constexpr (HALF) {
        const T* src = el.lrow(min(row, el.N - 1), rp[i]) + c0;
#pragma unroll
        for (int cb = 0; cb < TL::CB; ++cb) {
          const int j = wc0 + 16 * cb + li;
          acc[rb][cb][v] = (row < el.N && c0 + j < c1) ? src[j] : T(0);
        }
      } else {
        const double* src = (row < n ? el.A + (size_t)rp[i] * n : el.C + (size_t)(min(row, el.N - 1) - n) * n) + c0;
#pragma unroll
        for (int cb = 0; cb < TL::CB; ++cb) {
          const int j = wc0 + 16 * cb + li;
          acc[rb][cb][v] = (row < el.N && c0 + j < c1) ? (T)src[j] : T(0);
        }
      }
    }
  }
  if (K > 0) {
    typename TL::Ops o;
#pragma unroll
    for (int q = 0; q < TL::AL; ++q) {
      const int i = TL::a_row(q), row = min(r0 + i, el.N - 1);
      o.a[q] = (typename TL::gptr)(el.lrow(row, rp[i]) + kb + TL::a_k());
    }
    o.columns(el.LU + c0, n, TL::b_col(), c1 - c0, nullptr);
    TL::template product<false>(o, sp, K, lds, wr0, wc0, acc);
  }
  lane = opaque(lane);
#pragma unroll
  for (int rb = 0; rb < TL::RB; ++rb)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = wr0 + 16 * rb + Mfma<T>::row(lane, v), row = r0 + i;
      if (row < el.N) {
        T* dst = el.lrow(row, rp[i]) + c0;
#pragma unroll
        for (int cb = 0; cb < TL::CB; ++cb) {
          const int j = wc0 + 16 * cb + li;
          if (c0 + j < c1) dst[j] = acc[rb][cb][v];
        }
      }
    }
}

// ---- 3. panel rows with the triangular solve on the accumulators -------------
// Tiles 0 .. tiles0-1 cover columns [c1, n) of U, the others the t columns of
// U12 and, at column t, the right-hand side w.
// SELF: L_pp^{-1} is formed here from the panel's L instead of read.
// The solve takes L_pp^{-1} in 16 x 16 blocks from LDS (over the slab, which is
// done by then): read from memory where needed, block by block, its latency
// was most of the kernel's time in the first panels.
template <typename T, int CT>
struct InvBlocks {
  static constexpr int NB = CT / 16, COUNT = NB * (NB + 1) / 2;  // on and below the diagonal
  static constexpr size_t BYTES = sizeof(T) * 256 * COUNT;
  static __device__ __forceinline__ int at(int ib, int rb) { return (ib * (ib + 1) / 2 + rb) * 256; }
  // entry (r, c) of a block: runs of four columns swizzled by the row, so
  // that a fragment's lanes fall into different banks
  static __device__ __forceinline__ int entry(int r, int c) {
    return r * 16 + (c ^ (4 * (sizeof(T) == 4 ? (r >> 2) & 3 : (r >> 1) & 3)));
  }
  // inv: 64 x 64 blocks as the panel kernel writes them (memory or LDS); only
  // the wp rows of the panel's own are there
  static __device__ __forceinline__ void stage(const T* inv, T* dst, int wp) {
    typedef T vec4 __attribute__((ext_vector_type(4)));
    for (int o = threadIdx.x; o < COUNT * 64; o += GT) {
      const int b = o >> 6, r = (o >> 2) & 15, c = 4 * (o & 3);
      int ib = 0;
      while ((ib + 1) * (ib + 2) / 2 <= b) ++ib;
      if (16 * ib >= wp) break;
      const int rb = b - ib * (ib + 1) / 2;
      const vec4 v = *reinterpret_cast<const vec4*>(inv + ((ib >> 2) + (rb >> 2)) * kInvBlock + (16 * (ib & 3) + r) * 64 +
                                                    16 * (rb & 3) + c);
      *reinterpret_cast<vec4*>(dst + b * 256 + entry(r, c)) = v;
    }
    __syncthreads();
  }
};

template <typename T, int MM, int CT>
constexpr int row_slab() {
  return std::max<int>(Tile<T, MM, CT, 128, true>::STAGE, (int)InvBlocks<T, CT>::BYTES);
}

template <typename T, int MM, int CT, int LW, bool SELF>
__global__ __launch_bounds__(GT, sizeof(T) == 8 ? 2 : 3) void condense_row_kernel(CondenseWork<T> wk, int tiles, int tiles0,
                                                                               int c0, int c1) {
  constexpr int TN = 128;
  typedef Tile<T, MM, CT, TN, true> TL;
  typedef Mfma<T> MF;
  extern __shared__ __align__(16) unsigned char lds[];
  int it, tile;
  if (!condense_locate(wk, tiles, it, tile)) return;
  const Elem<T> el = condense_elem(wk, it);
  const int n = el.n, t = el.t, wp = c1 - c0, tid = threadIdx.x;
  const bool seg = tile >= tiles0;  // columns of U12 and w
  const int j0 = seg ? TN * (tile - tiles0) : c1 + TN * tile;
  const int width = seg ? t : n, jl = seg && el.F ? t + 1 : width;
  if (j0 >= jl) return;
  unsigned short* rp = reinterpret_cast<unsigned short*>(lds + row_slab<T, MM, CT>());
  unsigned short* sp = rp + CT;
  load_row_map<CT>(el.perm, false, n, 0, c0, c0, sp, rp);
  int lane = tid & 63;
  const int li = lane & 15;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wc0 = wv * TL::WN;
  const T* inv = el.Ke;
  if constexpr (SELF) {
    // as the panel kernel grows it, from the stored L
    T* Li = reinterpret_cast<T*>(lds + row_slab<T, MM, CT>() + 2 * ((CT + c0 + 7) & ~7));
    T* Lb = Li + (CT == 128 ? 3 : 1) * kInvBlock;
    T* Y = Lb + LW * 64;
    for (int i = tid; i < (CT == 128 ? 3 : 1) * kInvBlock; i += GT) Li[i] = T(0);
    __syncthreads();
    bool odd = false;  // an infinity or NaN in L (of an element without a pivot)
    for (int h = 0; h < wp; h += 64)
      for (int kp = 0; kp < min(64, wp - h); kp += LW) {
        const int sw = min(LW, min(64, wp - h) - kp);
        for (int o = tid; o < sw * (kp + sw); o += GT) {
          const int i = o / (kp + sw), k = o % (kp + sw);
          const T l = k < kp + i ? el.LU[(size_t)rp[h + kp + i] * n + c0 + h + k] : T(0);
          odd |= !isfinite(l);
          Lb[i * 64 + k] = l;
        }
        odd = __syncthreads_or(odd);
        grow_inverse<T, LW>(h ? Li + 2 * kInvBlock : Li, 64, Lb, Y, kp, sw, odd);
      }
    if (CT == 128 && wp > 64)
      inverse_offdiag<T>(Li, 64, Li + 2 * kInvBlock, 64, wp - 64,
                         [&](int i, int k) __attribute__((always_inline)) {
                           return el.LU[(size_t)rp[64 + i] * n + c0 + k];
                         },
                         Y, Li + kInvBlock, odd);
    inv = Li;
  }

  typename TL::acc_t acc[TL::RB][TL::CB];
  const double* in = seg ? el.B : el.A;
#pragma unroll
  for (int rb = 0; rb < TL::RB; ++rb) {
    input_step<T>(rb);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = 16 * rb + MF::row(lane, v);
      const size_t pr = rp[i];
#pragma unroll
      for (int cb = 0; cb < TL::CB; ++cb) {
        const int j = j0 + wc0 + 16 * cb + li;
        T x = T(0);
        if (i < wp && j < jl) x = (T)(j < width ? in[pr * width + j] : el.F[pr]);
        acc[rb][cb][v] = x;
      }
    }
  }
  if (c0 > 0) {
    typename TL::Ops o;
#pragma unroll
    for (int q = 0; q < TL::AL; ++q) o.a[q] = (typename TL::gptr)(el.LU + (size_t)rp[min(TL::a_row(q), wp - 1)] * n + TL::a_k());
    o.columns(seg ? el.U12 : el.LU, width, j0 + TL::b_col(), width, jl > width ? el.w : nullptr);
    TL::template product<false>(o, sp, c0, lds, 0, wc0, acc);
    lane = opaque(lane);
    // rows of a narrow last panel past its end met other rows' L
#pragma unroll
    for (int rb = 0; rb < TL::RB; ++rb)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (16 * rb + MF::row(lane, v) >= wp)
#pragma unroll
          for (int cb = 0; cb < TL::CB; ++cb) acc[rb][cb][v] = T(0);
  }
  typedef InvBlocks<T, CT> IB;
  T* ib_lds = reinterpret_cast<T*>(lds);
  IB::stage(inv, ib_lds, wp);
#pragma unroll
  for (int ib = TL::RB - 1; ib >= 0; --ib) {
    if (16 * ib >= wp) continue;
    typename MF::acc_t nacc[TL::CB];
#pragma unroll
    for (int cb = 0; cb < TL::CB; ++cb) nacc[cb] = MF::zero();
#pragma unroll
    for (int rb = 0; rb <= ib; ++rb) {
      const T* blk = ib_lds + IB::at(ib, rb);
      T av[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) av[v] = blk[IB::entry(li, MF::row(lane, v))];
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int cb = 0; cb < TL::CB; ++cb) nacc[cb] = MF::mac(av[v], acc[rb][cb][v], nacc[cb]);
    }
#pragma unroll
    for (int cb = 0; cb < TL::CB; ++cb) acc[ib][cb] = nacc[cb];
  }
#pragma unroll
  for (int rb = 0; rb < TL::RB; ++rb)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = 16 * rb + MF::row(lane, v);
      if (i < wp) {
        const size_t pr = rp[i];
        T* dst = (seg ? el.U12 : el.LU) + pr * width;
#pragma unroll
        for (int cb = 0; cb < TL::CB; ++cb) {
          const int j = j0 + wc0 + 16 * cb + li;
          if (j < width) dst[j] = acc[rb][cb][v];
          else if (j < jl) el.w[pr] = (double)acc[rb][cb][v];
        }
      }
    }
}

// ---- 4. Schur block ---------------------------------------------------------
template <typename T, int MM, int TN>
__global__ __launch_bounds__(GT, sizeof(T) == 8 ? 2 : 3) void condense_schur_kernel(CondenseWork<T> wk, int tiles, int ctiles) {
  typedef Tile<T, MM, 128, TN, false> TL;
  extern __shared__ __align__(16) unsigned char lds[];
  int it, tile;
  if (!condense_locate(wk, tiles, it, tile)) return;
  const Elem<T> el = condense_elem(wk, it);
  const int n = el.n, t = el.t, jl = el.F ? t + 1 : t;
  const int r0 = 128 * (tile / ctiles), j0 = TN * (tile % ctiles);
  if (j0 >= jl) return;
  unsigned short* sp = reinterpret_cast<unsigned short*>(lds + TL::STAGE);
  load_row_map<128>(el.perm, false, n, 0, n, -1, sp, nullptr);
  int lane = threadIdx.x & 63;
  const int li = lane & 15;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr0 = (wv % TL::WR) * TL::WM, wc0 = (wv / TL::WR) * TL::WN;
  typename TL::acc_t acc[TL::RB][TL::CB];
#pragma unroll
  for (int rb = 0; rb < TL::RB; ++rb) {
    input_step<T>(rb);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = r0 + wr0 + 16 * rb + Mfma<T>::row(lane, v);
#pragma unroll
      for (int cb = 0; cb < TL::CB; ++cb) {
        const int j = j0 + wc0 + 16 * cb + li;
        acc[rb][cb][v] = (row < t && j < t) ? (T)el.D[(size_t)row * t + j] : T(0);
      }
    }
  }
  typename TL::Ops o;
#pragma unroll
  for (int q = 0; q < TL::AL; ++q)
    o.a[q] = (typename TL::gptr)(el.L21 + (size_t)min(r0 + TL::a_row(q), t - 1) * n + TL::a_k());
  o.columns(el.U12, t, j0 + TL::b_col(), t, jl > t ? el.w : nullptr);
  TL::template product<true>(o, sp, n, lds, wr0, wc0, acc);
  lane = opaque(lane);
#pragma unroll
  for (int rb = 0; rb < TL::RB; ++rb)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = r0 + wr0 + 16 * rb + Mfma<T>::row(lane, v);
      if (row < t) {
#pragma unroll
        for (int cb = 0; cb < TL::CB; ++cb) {
          const int j = j0 + wc0 + 16 * cb + li;
          if (j < t) el.Ke[(size_t)row * t + j] = acc[rb][cb][v];
          else if (j < jl) el.r[row] = (double)acc[rb][cb][v];
        }
      }
    }
}

// ---- launches -----------------------------------------------------------------
inline hipError_t launch_lds(const void* kern, size_t smem) {
  if (smem <= 64 * 1024) return hipSuccess;
  return hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
}

template <typename T, int MM, int TN, int HALF>
hipError_t launch_col(const CondenseWork<T>& w, int c0, int c1, int kb, hipStream_t s) {
  typedef Tile<T, MM, 128, TN, false> TL;
  const int tiles = (w.n + w.t - c0 + 127) / 128;
  const size_t smem = TL::STAGE + sizeof(unsigned short) * (128 + (c0 - kb));
  auto k = condense_col_kernel<T, MM, TN, HALF>;
  hipError_t e = launch_lds(reinterpret_cast<const void*>(k), smem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, condense_grid(w, tiles), dim3(GT), smem, s, w, tiles, c0, c1, kb);
  return hipGetLastError();
}

template <typename T, int MM, int CT, int LW, bool SELF>
hipError_t launch_row(const CondenseWork<T>& w, int c0, int c1, hipStream_t s) {
  const int tiles0 = (w.n - c1 + 127) / 128, tiles = tiles0 + w.t / 128 + 1;  // t + 1 columns with w
  size_t smem = row_slab<T, MM, CT>() + sizeof(unsigned short) * ((CT + c0 + 7) & ~7);
  if (SELF) smem += sizeof(T) * (CT == 128 ? 3 * kInvBlock + LW * 64 + 64 * 65 : kInvBlock + 2 * LW * 64);
  auto k = condense_row_kernel<T, MM, CT, LW, SELF>;
  hipError_t e = launch_lds(reinterpret_cast<const void*>(k), smem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, condense_grid(w, tiles), dim3(GT), smem, s, w, tiles, tiles0, c0, c1);
  return hipGetLastError();
}

template <typename T, int MM, int TN>
hipError_t launch_schur(const CondenseWork<T>& w, hipStream_t s) {
  typedef Tile<T, MM, 128, TN, false> TL;
  const int ctiles = w.t / TN + 1, tiles = (w.t + 127) / 128 * ctiles;  // t + 1 columns with r
  const size_t smem = TL::STAGE + sizeof(unsigned short) * w.n;
  auto k = condense_schur_kernel<T, MM, TN>;
  hipError_t e = launch_lds(reinterpret_cast<const void*>(k), smem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, condense_grid(w, tiles), dim3(GT), smem, s, w, tiles, ctiles);
  return hipGetLastError();
}

template <typename T, int MM, int CT>
hipError_t condense_sequence(const CondenseWork<T>& w, int lw, hipStream_t s) {
#define IEDG_STEP(call)                  \
  do {                                   \
    hipError_t _e = (call);              \
    if (_e != hipSuccess) return _e;     \
  } while (0)
  const int n = w.n;
  for (int c0 = 0; c0 < n; c0 += CT) {
    const int c1 = std::min(c0 + CT, n), cm = std::min(c0 + 64, c1);
    IEDG_STEP((launch_col<T, MM, CT, 0>(w, c0, c1, 0, s)));
    IEDG_STEP((condense_panel<T>(w, lw, c0, c0, cm, c1 - cm, s)));
    if constexpr (CT == 128) {
      if (cm < c1) {
        IEDG_STEP((launch_col<T, 0, 64, 1>(w, cm, c1, c0, s)));
        IEDG_STEP((condense_panel<T>(w, lw, c0, cm, c1, 0, s)));
      }
    }
    if (!w.self) IEDG_STEP((launch_row<T, MM, CT, 16, false>(w, c0, c1, s)));
    else if (lw == 16) IEDG_STEP((launch_row<T, MM, CT, 16, true>(w, c0, c1, s)));
    else IEDG_STEP((launch_row<T, MM, CT, 8, true>(w, c0, c1, s)));
  }
  IEDG_STEP((launch_schur<T, MM, sizeof(T) == 8 ? 64 : 128>(w, s)));
#undef IEDG_STEP
  return hipSuccess;
}

template <typename T, int MM>
hipError_t condense_run(const CondenseWork<T>& w0, int lw, int ct, hipStream_t s) {
  CondenseWork<T> w = w0;
  w.self = !inverse_fits(w.n, w.t, ct);
  if (w.count == 0) return hipSuccess;
  if constexpr (sizeof(T) == 4) {
    if (ct == 128) return condense_sequence<T, MM, 128>(w, lw, s);
  }
  return condense_sequence<T, MM, 64>(w, lw, s);
}

}  // namespace iedg
