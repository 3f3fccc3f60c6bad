// Panel factorisation of the element condensation (section 2.2.1, eq. LS).
//
// One workgroup factors up to 64 columns [cb, ce) of one element's bordered
// matrix [A; C] below position cb with partial pivoting over the rows of A:
// the columns hold in - L U of every earlier panel.  Row interchanges change
// only the row map (perm); rows stay where they are.
//
// What bounds it: the chain of pivot columns.  A column costs one workgroup
// barrier, two round trips through LDS (each wave's candidate, then the pivot
// row) and the wave-wide search between them; its arithmetic is one rank-one
// update.  So the panel is a launch of its own, with few enough registers and
// little enough LDS that two workgroups share a CU and one column's waits are
// covered by another element's work.
//
// Sub-panels of LW (16 or 8) columns are held in registers, whole rows to
// lanes.  A row stays with its thread: an interchange swaps the two rows'
// position labels and moves no data.
//
// FP32 rows fit v_mfma_f32_4x4x1 as they lie: its B operand is a column of 64
// rows, its A operand four columns of one U row broadcast to all 16 blocks,
// its accumulator four columns of the lane's own row, and with k = 1 each
// entry takes exactly one fused multiply-add.  The rank-one updates therefore
// run on the matrix cores at twice the rate of
// vector FMAs with the same bits, and the pivot row is read as one vector per
// lane in place of LW broadcasts.  (v_mfma_f64_4x4x4 has no such form: FP64
// rows take vector FMAs.)
//
// Infinities and NaN (of an element without a pivot) stay where elimination
// entry by entry has them: rows before them keep their values.  Zeros of whole
// blocks would spread them, so products that come out not finite are formed
// again without those zeros, U rows that met an infinity in a rank-one update
// are put back, and the inverse grows entry by entry from the first missing
// pivot on.  None of it is on the chain of pivot columns (8 elements of
// n = 160, FP32 256 -> 261 us, FP64 335 -> 337 us; 256 of n = 1280, FP32 the
// same, FP64 25.4 -> 25.6 ms).
#include <climits>

#include "condense.h"

namespace iedg {

// Maximum over 16-lane rows, and over the wave, without a round trip through
// LDS: two quad permutations and two rotations (DPP) leave a row's maximum in
// every lane of the row; the four rows are then read as uniform values.
constexpr int kDppXor1 = 0xB1;   // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;   // quad_perm [2,3,0,1]
constexpr int kDppRor4 = 0x124;  // row_ror:4
constexpr int kDppRor8 = 0x128;  // row_ror:8

template <int CTRL>
__device__ __forceinline__ unsigned dpp_max(unsigned v) {
  return max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ unsigned row_max(unsigned v) {
  return dpp_max<kDppRor8>(dpp_max<kDppRor4>(dpp_max<kDppXor2>(dpp_max<kDppXor1>(v))));
}
__device__ __forceinline__ unsigned read_lane(unsigned v, int l) {
  return (unsigned)__builtin_amdgcn_readlane((int)v, l);
}
__device__ __forceinline__ unsigned wave_max(unsigned v) {
  v = row_max(v);
  return max(max(read_lane(v, 0), read_lane(v, 16)), max(read_lane(v, 32), read_lane(v, 48)));
}
__device__ __forceinline__ int read_lane(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ __forceinline__ float read_lane(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ double read_lane(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}

// Magnitudes are compared by a 32-bit key, 0 where there is none: all of an
// FP32 magnitude, the upper word of an FP64 one.
__device__ __forceinline__ unsigned mag_key(float a) { return a < 0.f ? 0u : __float_as_uint(a) + 1u; }
__device__ __forceinline__ unsigned mag_key(double a) { return a < 0.0 ? 0u : (unsigned)__double2hiint(a) + 1u; }

// Of the lanes in `mask` (not empty) the one with the largest a, ties to the
// smallest pos.  Mostly a single lane; FP64 lanes that share the key and equal
// magnitudes take the loop.
template <typename T>
__device__ __forceinline__ int best_lane(unsigned long long mask, T a, int pos) {
  int best = __ffsll(mask) - 1;
  mask &= mask - 1;
  if (mask) {
    T ba = read_lane(a, best);
    int bp = read_lane(pos, best);
    for (; mask; mask &= mask - 1) {
      const int l = __ffsll(mask) - 1, p = read_lane(pos, l);
      const T v = read_lane(a, l);
      if (v > ba || (v == ba && p < bp)) { ba = v; bp = p; best = l; }
    }
  }
  return best;
}

// 4 x 4 transpose of 16-lane groups over four registers: register r of lane
// group g takes what register g of lane group r held.
__device__ __forceinline__ void swap32(unsigned& a, unsigned& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0]; b = r[1];
}
__device__ __forceinline__ void swap16(unsigned& a, unsigned& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  a = r[0]; b = r[1];
}
__device__ __forceinline__ void transpose4(unsigned& a, unsigned& b, unsigned& c, unsigned& d) {
  swap32(a, c); swap32(b, d);
  swap16(a, b); swap16(c, d);
}

// A row of LW values in LDS is kept as four runs of LW / 4: entry j at
// (j % 4) (LW / 4) + j / 4, so that lane l finds columns l % 4, l % 4 + 4, ...
// (its share of the rank-one update's A operand) as one vector.
template <int LW>
__device__ __forceinline__ constexpr int row_slot(int j) {
  return (j & 3) * (LW / 4) + (j >> 2);
}

template <typename T, int LW, int R, int NT>
struct PanelSmem {
  static constexpr int NW = NT / 64, LIS = 65;
  T Li[64 * LIS];        // inverse of the panel's factored columns so far
  T Xu[64 * LW];         // rows above the sub-panel (input), then LW x 64 of scratch
  T Ut[64 * LW];         // U rows above the sub-panel, each in row_slot order
  T Lb[LW * 64];         // L rows of the sub-panel
  // each wave's best candidate row, by column (FP32) or its parity
  static constexpr int COLS = sizeof(T) == 4 ? LW : 2;
  T cand[COLS][NW][LW];
  T krow[LW];            // row at the pivot position where no pivot was found (FP64)
  T kval;                // and its entry
  T cval[2][NW];         // the candidates' pivot entries
  int cidx[2][NW];       // and positions
  int prow[64];          // physical rows of the panel's pivots
  T* rowp[NT * R];       // every row slot's row in LU or L21 (LU past the last)
  int phys[NT * R];      // and its physical row (rows of A)
  int odd;               // a pivot row was not finite (FP32)
};

// A row's columns in registers, in quads (the FP32 rank-one update's
// accumulators; FP64 values need no common registers).
struct DoubleQuad {
  double a[4];
  __device__ __forceinline__ double& operator[](int i) { return a[i]; }
  __device__ __forceinline__ const double& operator[](int i) const { return a[i]; }
};
template <typename T> struct Quad;
template <> struct Quad<float> { typedef f4 v; };
template <> struct Quad<double> { typedef DoubleQuad v; };

// Whether any entry of the wave's accumulator is not finite.
template <typename V>
__device__ __forceinline__ bool any_nonfinite(const V& a) {
  return __ballot(!(isfinite(a[0]) && isfinite(a[1]) && isfinite(a[2]) && isfinite(a[3]))) != 0;
}

// What the pivot columns of a sub-panel leave (uniform): none: a column had no
// pivot, so L may hold infinities or NaN; win: which wave's post is the pivot
// row, four bits a column.
struct Trail {
  bool none;
  unsigned long long win;
};

// x -= l u over a row's columns past KK (KK < 0: all), u in the lane's share
// layout with the columns up to KK zero.
template <int LW, int KK>
__device__ __forceinline__ void rank_one(f4 (&x)[LW / 4], float nl, const float (&u)[LW / 4]) {
#pragma unroll
  for (int c = KK < 0 ? 0 : (KK + 1) / 4; c < LW / 4; ++c) x[c] = __builtin_amdgcn_mfma_f32_4x4x1f32(u[c], nl, x[c], 4, 0, 0);
}

// Slot q's row to LDS (q uniform over the wave).  Each slot's branch ends in a
// statement of its own: branches that end alike are merged into one over a
// pointer to the row, and the rows would leave the registers.
template <int LW, int S, typename Q4, typename T, int R>
__device__ __forceinline__ void put_row(const Q4 (&x)[R][LW / 4], int q, int kk, T* row, T* val) {
  if constexpr (S < R) {
    if (q == S) {
#pragma unroll
      for (int j = 0; j < LW; ++j) row[row_slot<LW>(j)] = x[S][j / 4][j % 4];
#pragma unroll
      for (int j = 0; j < LW; ++j)
        if (j == kk) *val = x[S][j / 4][j % 4];
      asm volatile("; slot %0" ::"n"(S));
    }
    put_row<LW, S + 1>(x, q, kk, row, val);
  }
}

// One pivot column KK of a sub-panel in registers: k is its pivot position,
// pos[q] the position of slot q's row.
template <typename T, int LW, int R, int NT, int KK>
__device__ __forceinline__ void pivot_column(PanelSmem<T, LW, R, NT>& sm, typename Quad<T>::v (&x)[R][LW / 4], int (&pos)[R],
                                             int k, int n, DeviceStatus* status, int elem, Trail& tr) {
  constexpr int NW = NT / 64, par = KK & 1, col = KK % PanelSmem<T, LW, R, NT>::COLS;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the thread's candidate among the rows of A at positions >= k: largest
  // magnitude, ties to the smaller position (NaN is never taken)
  T best = T(-1);
  int bpos = INT_MAX, bq = 0;
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const T v = fabs(x[q][KK / 4][KK % 4]);
    const bool cand = (unsigned)(pos[q] - k) < (unsigned)(n - k);
    const bool take = cand & ((v > best) | ((v == best) & (pos[q] < bpos)));
    best = take ? v : best;
    bpos = take ? pos[q] : bpos;
    bq = take ? q : bq;
  }
  const unsigned key = mag_key(best), kmax = wave_max(key);
  if (kmax == 0) {
    if (lane == 0) sm.cidx[par][wv] = INT_MAX;
  } else {
    const int win = best_lane(__ballot(key == kmax), best, bpos);
    const int sq = read_lane(bq, win);
    if (lane == win) {
      put_row<LW, 0>(x, sq, KK, sm.cand[col][wv], &sm.cval[par][wv]);
      sm.cidx[par][wv] = bpos;
    }
  }
  __syncthreads();
  // the workgroup's pivot: lane w looks at wave w's candidate (and inverts
  // it, while the search goes on).  Buffers alternate by column parity: one
  // is rewritten only after every wave has passed the next column's barrier,
  // i.e. finished reading it.
  const int wl = lane & (NW - 1);
  const int ci = sm.cidx[par][wl];
  const T cv = sm.cval[par][wl], cinv = T(1) / cv;
  const T ca = ci == INT_MAX ? T(-1) : fabs(cv);
  const unsigned ckey = mag_key(ca), gkey = read_lane(row_max(ckey), 0);
  const int bw = best_lane(__ballot(ckey == gkey) & ((1ull << NW) - 1), ca, ci);
  int piv = read_lane(ci, bw), from = bw;
  T rinv = read_lane(cinv, bw);
  const T gbest = read_lane(ca, bw);
  const T* urow = sm.cand[col][bw];
  if (!(gbest > T(0)) || !isfinite(gbest)) {
    // no pivot: row k stays (the branch is uniform over the workgroup)
    if (tid == 0) latch_status(status, IEDG_ERR_SINGULAR, elem);
    tr.none = true;
    from = 0;  // (FP32: posted in place of a candidate, as its pivot row)
    T* row;
    if constexpr (sizeof(T) == 4) row = sm.cand[col][0];
    else row = sm.krow;
#pragma unroll
    for (int q = 0; q < R; ++q)
      if (pos[q] == k) put_row<LW, 0>(x, q, KK, row, &sm.kval);
    __syncthreads();
    piv = k;
    urow = row;
    rinv = T(1) / sm.kval;
    __syncthreads();  // read before another column posts its row k
  }
  if constexpr (sizeof(T) == 4) {
    urow = sm.cand[col][from];
    tr.win |= (unsigned long long)from << (4 * KK);
  }
#pragma unroll
  for (int q = 0; q < R; ++q) pos[q] = pos[q] == piv ? k : pos[q] == k ? piv : pos[q];
  // eliminate below the pivot; rows at positions <= k keep their values
  if constexpr (sizeof(T) == 4) {
    T u[LW / 4];
#pragma unroll
    for (int c = KK / 4; c < LW / 4; ++c) {
      u[c] = urow[(lane & 3) * (LW / 4) + c];
      if (c == KK / 4) u[c] = 4 * c + (lane & 3) > KK ? u[c] : T(0);
    }
    // (rows that stay take 0 times u: where u is not finite they are put back
    // after the sub-panel)
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const bool live = pos[q] > k;
      const T l = x[q][KK / 4][KK % 4] * rinv;
      x[q][KK / 4][KK % 4] = live ? l : x[q][KK / 4][KK % 4];
      rank_one<LW, KK>(x[q], live ? -l : T(0), u);
    }
  } else {
    T u[LW];
#pragma unroll
    for (int j = KK + 1; j < LW; ++j) u[j] = urow[row_slot<LW>(j)];
#pragma unroll
    for (int q = 0; q < R; ++q) {
      if (pos[q] > k) {
        const T l = x[q][KK / 4][KK % 4] * rinv;
        x[q][KK / 4][KK % 4] = l;
#pragma unroll
        for (int j = KK + 1; j < LW; ++j) x[q][j / 4][j % 4] = fma(-l, u[j], x[q][j / 4][j % 4]);
      }
    }
  }
}

template <typename T, int LW, int R, int NT, int KK>
__device__ __forceinline__ void pivot_columns(PanelSmem<T, LW, R, NT>& sm, typename Quad<T>::v (&x)[R][LW / 4], int (&pos)[R],
                                              int cs, int sw, int n, DeviceStatus* status, int elem, Trail& tr) {
  if constexpr (KK < LW) {
    if constexpr (KK % 4 == 0)  // sw is a multiple of 4, as n is
      if (KK >= sw) return;
    pivot_column<T, LW, R, NT, KK>(sm, x, pos, cs + KK, n, status, elem, tr);
    pivot_columns<T, LW, R, NT, KK + 1>(sm, x, pos, cs, sw, n, status, elem, tr);
  }
}

template <typename T, int LW, int R, int NT>
__global__ __launch_bounds__(NT, NT == 512 && R * LW * sizeof(T) <= 256 ? 4 : 1)
void condense_panel_kernel(CondenseWork<T> wk, int c0, int cb, int ce, int right) {
  typedef PanelSmem<T, LW, R, NT> SM;
  typedef Mfma<T> MF;
  constexpr int NW = NT / 64, LIS = SM::LIS;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  SM& sm = *reinterpret_cast<SM*>(smem_raw);
  const int* prow = sm.prow;

  const Elem<T> el = condense_elem(wk, blockIdx.x);
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lg = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = el.n, N = el.N, wp = ce - cb;

  int pos[R];  // positions (labels) of this thread's rows
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int p = cb + tid + NT * q;
    pos[q] = p;
    const int phys = p < n && cb > 0 ? el.perm[p] : p;
    sm.phys[tid + NT * q] = phys;
    sm.rowp[tid + NT * q] = p < N ? el.lrow(p, phys) : el.LU;
  }
  for (int i = tid; i < 64 * LIS; i += NT) sm.Li[i] = T(0);
  if (tid == 0) sm.odd = 0;
  __syncthreads();

  // Rows move between memory and lanes in 16-row groups: four lanes (one of
  // each 16-lane group) share a row's LW columns, so that a wave's access
  // covers whole segments of 16 rows and not 16 bytes of 64, and a transpose
  // over the lane groups gives each lane its own row.
  constexpr int CD = LW * (int)sizeof(T) / 16;  // dwords of a row per lane
  T* const* rowp = sm.rowp + 64 * wv + li;
  auto row_ptr = [&](int q, int g) __attribute__((always_inline)) -> T* { return rowp[NT * q + 16 * g]; };
  // columns [col, col + LW) of slot q's rows; those at and past col + w zero
  auto fetch = [&](int q, int col, int w, unsigned (&raw)[4][CD]) __attribute__((always_inline)) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const T* src = row_ptr(q, g) + col + lg * (LW / 4);
      const bool ok = lg * (LW / 4) < w;
      if constexpr (CD == 2) {
        const uint2 v = *reinterpret_cast<const uint2*>(ok ? src : src - lg * (LW / 4));
        raw[g][0] = ok ? v.x : 0u; raw[g][1] = ok ? v.y : 0u;
      } else {
#pragma unroll
        for (int d = 0; d < CD; d += 4) {
          // (w is a multiple of 4: FP64 in runs of two may end inside LW / 4)
          const bool okd = lg * (LW / 4) + d * 4 / (int)sizeof(T) < w;
          const uint4 v = *reinterpret_cast<const uint4*>(okd ? src + d * 4 / sizeof(T) : src - lg * (LW / 4));
          raw[g][d] = okd ? v.x : 0u; raw[g][d + 1] = okd ? v.y : 0u;
          raw[g][d + 2] = okd ? v.z : 0u; raw[g][d + 3] = okd ? v.w : 0u;
        }
      }
    }
  };
  typedef typename Quad<T>::v Q4;
  auto to_rows = [&](unsigned (&raw)[4][CD], Q4 (&xq)[LW / 4]) __attribute__((always_inline)) {
#pragma unroll
    for (int d = 0; d < CD; ++d) transpose4(raw[0][d], raw[1][d], raw[2][d], raw[3][d]);
#pragma unroll
    for (int j = 0; j < LW; ++j) {
      const int c = j / (LW / 4), e = j % (LW / 4);
      if constexpr (sizeof(T) == 4) xq[j / 4][j % 4] = __uint_as_float(raw[c][e]);
      else xq[j / 4][j % 4] = __hiloint2double((int)raw[c][2 * e + 1], (int)raw[c][2 * e]);
    }
  };

  unsigned raw[R][4][CD];
#pragma unroll
  for (int q = 0; q < R; ++q) fetch(q, cb, min(LW, wp), raw[q]);
  bool odd = false;  // a column so far had no pivot
  for (int cs = cb; cs < ce; cs += LW) {
    const int sw = min(LW, ce - cs), kp = cs - cb;
    Q4 x[R][LW / 4];
#pragma unroll
    for (int q = 0; q < R; ++q) to_rows(raw[q], x[q]);
    if (kp > 0) {
      // U rows [cb, cs) of the sub-panel's columns: L_pp^{-1} X
#pragma unroll
      for (int q = 0; q < R; ++q)
        if (pos[q] < cs) {
#pragma unroll
          for (int j = 0; j < LW; ++j) sm.Xu[(pos[q] - cb) * LW + j] = x[q][j / 4][j % 4];
        }
      __syncthreads();
      for (int ib = wv; ib < (kp + 15) / 16; ib += NW) {
        typename MF::acc_t acc = MF::zero();
        for (int m = 0; m < 16 * (ib + 1); m += 4) {
          const T bv = li < LW && m + lg < kp ? sm.Xu[(m + lg) * LW + (li & (LW - 1))] : T(0);
          acc = MF::mac(sm.Li[(16 * ib + li) * LIS + m + lg], bv, acc);
        }
        if (li < LW) {
#pragma unroll
          for (int v = 0; v < 4; ++v) sm.Ut[(16 * ib + MF::row(lane, v)) * LW + row_slot<LW>(li)] = acc[v];
        }
        if (__builtin_expect(any_nonfinite(acc), 0)) {  // (the zeros above the diagonal met an infinity)
          int ln = lane;
          asm volatile("" : "+v"(ln));  // (cold: nothing of it is computed ahead and kept)
          const int j = ln & 15;
#pragma unroll 1
          for (int v = 0; v < 4; ++v) {
            const int i = 16 * ib + MF::row(ln, v);
            T s = T(0);
#pragma unroll 1
            for (int m = 0; m <= min(i, kp - 1); ++m) s = fma(sm.Li[i * LIS + m], sm.Xu[m * LW + (j & (LW - 1))], s);
            if (j < LW) sm.Ut[i * LW + (j & 3) * (LW / 4) + (j >> 2)] = s;
          }
        }
      }
      __syncthreads();
      // the other rows: X -= L[:, cb:cs] U, LW columns of L at a time (from
      // this wave's own stores)
      for (int k0 = 0; k0 < kp; k0 += LW) {
#pragma unroll
        for (int q = 0; q < R; ++q) {
          unsigned lraw[4][CD];
          Q4 la[LW / 4];
          __builtin_amdgcn_sched_barrier(0);  // (one slot's loads at a time: more do not fit the registers)
          fetch(q, cb + k0, LW, lraw);
          to_rows(lraw, la);
#pragma unroll
          for (int kk = 0; kk < LW; ++kk) {
            const T* ur = sm.Ut + (k0 + kk) * LW;
            const T nl = -la[kk / 4][kk % 4];
            if constexpr (sizeof(T) == 4) {
              T u[LW / 4];
#pragma unroll
              for (int c = 0; c < LW / 4; ++c) u[c] = ur[(lane & 3) * (LW / 4) + c];
              rank_one<LW, -1>(x[q], nl, u);
            } else {
#pragma unroll
              for (int j = 0; j < LW; ++j) x[q][j / 4][j % 4] = fma(nl, ur[row_slot<LW>(j)], x[q][j / 4][j % 4]);
            }
          }
        }
      }
#pragma unroll
      for (int q = 0; q < R; ++q)
        if (pos[q] < cs) {
#pragma unroll
          for (int j = 0; j < LW; ++j) x[q][j / 4][j % 4] = sm.Ut[(pos[q] - cb) * LW + row_slot<LW>(j)];
        }
    }
    Trail tr = {false, 0};
    pivot_columns<T, LW, R, NT, 0>(sm, x, pos, cs, sw, n, el.status, el.id, tr);
    odd |= tr.none;
    const bool inverse = !wk.self || cs + LW < ce || right > 0;  // needed further
    // where the pivot rows are, and their own columns of L
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int i = pos[q] - cs;
      if (i >= 0 && i < sw) {
        sm.prow[kp + i] = sm.phys[tid + NT * q];
        T sum = T(0);
#pragma unroll
        for (int j = 0; j < LW; ++j) {
          if constexpr (sizeof(T) == 4) sum += fabs(x[q][j / 4][j % 4]);
          if (j < sw) sm.Lb[i * 64 + kp + j] = j < i ? x[q][j / 4][j % 4] : T(0);
        }
        if constexpr (sizeof(T) == 4)
          if (!isfinite(sum)) sm.odd = 1;
      }
    }
    // (nothing but earlier sub-panels' stores is in flight: the wait is short,
    // and the rows below are read by other waves than stored them)
    sync_global();
    if constexpr (sizeof(T) == 4) {
      if (__builtin_expect(__builtin_amdgcn_readfirstlane(sm.odd), 0)) {
        // a pivot row is not finite, and rows of U took 0 times its entries:
        // back as they were posted, or as they came
#pragma unroll
        for (int q = 0; q < R; ++q) {
          const int i = pos[q] - cs;
          if (i >= sw) continue;
          const T* row = i < 0 ? sm.Ut + (kp + i) * LW : sm.cand[i][(tr.win >> (4 * i)) & 15];
#pragma unroll
          for (int j = 0; j < LW; ++j) x[q][j / 4][j % 4] = row[row_slot<LW>(j)];
        }
      }
    }
    constexpr int LBV = (LW * 64 + NT - 1) / NT;
    T lb[LBV];
    if (inverse) {  // the panel's earlier columns of the pivot rows
#pragma unroll
      for (int v = 0; v < LBV; ++v) {
        const int o = tid + v * NT, i = o >> 6, k = o & 63;
        lb[v] = i < sw && k < kp ? el.LU[(size_t)sm.prow[kp + i] * n + cb + k] : T(0);
      }
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < LW; ++j) {
        const int c = j / (LW / 4), e = j % (LW / 4);
        if constexpr (sizeof(T) == 4) {
          raw[q][c][e] = __float_as_uint(x[q][j / 4][j % 4]);
        } else {
          raw[q][c][2 * e] = (unsigned)__double2loint(x[q][j / 4][j % 4]);
          raw[q][c][2 * e + 1] = (unsigned)__double2hiint(x[q][j / 4][j % 4]);
        }
      }
#pragma unroll
      for (int d = 0; d < CD; ++d) transpose4(raw[q][0][d], raw[q][1][d], raw[q][2][d], raw[q][3][d]);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        if (cb + NT * q + 64 * wv + 16 * g + li >= N) continue;
        T* dst = row_ptr(q, g) + cs + lg * (LW / 4);
        if constexpr (CD == 2) {
          if (lg * (LW / 4) < sw) *reinterpret_cast<uint2*>(dst) = make_uint2(raw[q][g][0], raw[q][g][1]);
        } else {
#pragma unroll
          for (int d = 0; d < CD; d += 4)
            if (lg * (LW / 4) + d * 4 / (int)sizeof(T) < sw)
              *reinterpret_cast<uint4*>(dst + d * 4 / sizeof(T)) =
                  make_uint4(raw[q][g][d], raw[q][g][d + 1], raw[q][g][d + 2], raw[q][g][d + 3]);
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (cs + LW < ce) {  // the next sub-panel's columns, while the inverse grows
#pragma unroll
      for (int q = 0; q < R; ++q) fetch(q, cs + LW, min(LW, ce - cs - LW), raw[q]);
    }
    if (inverse) {
#pragma unroll
      for (int v = 0; v < LBV; ++v) {
        const int o = tid + v * NT, i = o >> 6, k = o & 63;
        if (i < sw && k < kp) sm.Lb[i * 64 + k] = lb[v];
      }
      __syncthreads();
      grow_inverse<T, LW>(sm.Li, LIS, sm.Lb, sm.Xu, kp, sw, odd);
    }
  }
#pragma unroll
  for (int q = 0; q < R; ++q)
    if (cb + tid + NT * q < n) el.perm[pos[q]] = sm.phys[tid + NT * q];

  if constexpr (sizeof(T) == 4) {
    if (right > 0) {
      // left half of a 128-wide panel: U[cb:ce, ce:ce+right] = L11^{-1} X, a
      // wave 16 columns (wp = 64 rows)
      sync_global();
      for (int b = wv; b < (right + 15) / 16; b += NW) {
        const int col = ce + 16 * b + li;
        const bool ok = 16 * b + li < right;
        T xb[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) xb[q] = ok ? el.LU[(size_t)prow[4 * q + lg] * n + col] : T(0);
#pragma unroll
        for (int ib = 3; ib >= 0; --ib) {  // (from the last: X is overwritten, and read again below)
          typename MF::acc_t acc = MF::zero();
#pragma unroll
          for (int q = 0; q < 4 * (ib + 1); ++q)
            acc = MF::mac(sm.Li[(16 * ib + li) * LIS + 4 * q + lg], xb[q], acc);
          if (__builtin_expect(any_nonfinite(acc), 0)) {
#pragma unroll 1
            for (int v = 0; v < 4; ++v) {
              const int i = 16 * ib + MF::row(lane, v);
              T s = T(0);
#pragma unroll 1
              for (int m = 0; m <= i; ++m) s = fma(sm.Li[i * LIS + m], ok ? el.LU[(size_t)prow[m] * n + col] : T(0), s);
              acc[0] = v == 0 ? s : acc[0]; acc[1] = v == 1 ? s : acc[1];
              acc[2] = v == 2 ? s : acc[2]; acc[3] = v == 3 ? s : acc[3];
            }
          }
          if (ok) {
#pragma unroll
            for (int v = 0; v < 4; ++v) el.LU[(size_t)prow[16 * ib + MF::row(lane, v)] * n + col] = acc[v];
          }
        }
      }
    }
  }
  if (!wk.self) {
    if (cb == c0) {
      for (int i = tid; i < kInvBlock; i += NT) el.Ke[i] = sm.Li[(i >> 6) * LIS + (i & 63)];
    } else if constexpr (sizeof(T) == 4) {
      T* out = el.Ke;
      for (int i = tid; i < kInvBlock; i += NT) out[2 * kInvBlock + i] = sm.Li[(i >> 6) * LIS + (i & 63)];
      const int* sp = prow;
      const T* lu = el.LU;
      T* Y = reinterpret_cast<T*>(smem_raw + ((sizeof(SM) + 15) & ~size_t(15)));
      inverse_offdiag<T>(el.Ke, 64, sm.Li, LIS, wp,
                         [&](int i, int k) __attribute__((always_inline)) { return lu[(size_t)sp[i] * n + c0 + k]; }, Y,
                         el.Ke + kInvBlock, odd);
    }
  }
}

template <typename T, int LW, int R, int NT>
static hipError_t launch_panel(const CondenseWork<T>& w, int c0, int cb, int ce, int right, hipStream_t s) {
  size_t smem = (sizeof(PanelSmem<T, LW, R, NT>) + 15) & ~size_t(15);
  if (cb != c0 && !w.self) smem += sizeof(T) * 64 * 65;
  auto k = condense_panel_kernel<T, LW, R, NT>;
  if (smem > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)smem);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k, dim3(w.count), dim3(NT), smem, s, w, c0, cb, ce, right);
  return hipGetLastError();
}

template <typename T, int LW>
static hipError_t panel_rows(const CondenseWork<T>& w, int c0, int cb, int ce, int right, hipStream_t s) {
  const int rows = w.n + w.t - cb;
  if (rows <= 512) return launch_panel<T, LW, 1, 512>(w, c0, cb, ce, right, s);
  if (rows <= 1024) return launch_panel<T, LW, 2, 512>(w, c0, cb, ce, right, s);
  if constexpr (LW * sizeof(T) <= 64) {
    if (rows <= 1536) return launch_panel<T, LW, 3, 512>(w, c0, cb, ce, right, s);
    if (rows <= 2048) return launch_panel<T, LW, 4, 512>(w, c0, cb, ce, right, s);
  } else {
    if (rows <= 2048) return launch_panel<T, LW, 2, 1024>(w, c0, cb, ce, right, s);
  }
  if (rows <= 3072) return launch_panel<T, LW, 3, 1024>(w, c0, cb, ce, right, s);
  if (rows <= 4096) return launch_panel<T, LW, 4, 1024>(w, c0, cb, ce, right, s);
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t condense_panel(const CondenseWork<T>& w, int lw, int c0, int cb, int ce, int right, hipStream_t s) {
  if (lw == 16) return panel_rows<T, 16>(w, c0, cb, ce, right, s);
  return panel_rows<T, 8>(w, c0, cb, ce, right, s);
}
template hipError_t condense_panel<float>(const CondenseWork<float>&, int, int, int, int, int, hipStream_t);
template hipError_t condense_panel<double>(const CondenseWork<double>&, int, int, int, int, int, hipStream_t);

}  // namespace iedg
