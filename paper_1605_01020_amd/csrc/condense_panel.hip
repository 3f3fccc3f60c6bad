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
#include <climits>

#include "condense.h"

namespace iedg {

// Wave-wide maximum without a round trip through LDS: two quad permutations
// and two rotations inside each 16-lane row (DPP) leave the row's extremum in
// every lane of the row; the four rows are then read as uniform values.
constexpr int kDppXor1 = 0xB1;   // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;   // quad_perm [2,3,0,1]
constexpr int kDppRor4 = 0x124;  // row_ror:4
constexpr int kDppRor8 = 0x128;  // row_ror:8

template <int CTRL>
__device__ __forceinline__ int dpp_i32(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __int_as_float(dpp_i32<CTRL>(__float_as_int(v)));
}
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  return __hiloint2double(dpp_i32<CTRL>(__double2hiint(v)), dpp_i32<CTRL>(__double2loint(v)));
}
__device__ __forceinline__ int read_lane(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ __forceinline__ float read_lane(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ double read_lane(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}
// (values must not be NaN)
template <typename T>
__device__ __forceinline__ T row_max(T v) {
  v = fmax(v, dpp_move<kDppXor1>(v));
  v = fmax(v, dpp_move<kDppXor2>(v));
  v = fmax(v, dpp_move<kDppRor4>(v));
  return fmax(v, dpp_move<kDppRor8>(v));
}
template <typename T>
__device__ __forceinline__ T wave_max(T v) {
  v = row_max(v);
  return fmax(fmax(read_lane(v, 0), read_lane(v, 16)), fmax(read_lane(v, 32), read_lane(v, 48)));
}

// The lane of `mask` (not empty) with the smallest value of pos.
__device__ __forceinline__ int first_lane(unsigned long long mask, int pos) {
  int best = __ffsll(mask) - 1;
  mask &= mask - 1;
  if (mask) {  // several lanes hold the maximum
    int bp = read_lane(pos, best);
    for (; mask; mask &= mask - 1) {
      const int l = __ffsll(mask) - 1, p = read_lane(pos, l);
      if (p < bp) { bp = p; best = l; }
    }
  }
  return best;
}

// A row of LW values in LDS is kept as four runs of LW / 4: entry j at
// (j % 4) (LW / 4) + j / 4, so that lane l finds columns l % 4, l % 4 + 4, ...
// (its share of the rank-one update's A operand) as one vector.
template <int LW>
__device__ __forceinline__ constexpr int row_slot(int j) {
  return (j & 3) * (LW / 4) + (j >> 2);
}

template <typename T, int LW, int NT>
struct PanelSmem {
  static constexpr int NW = NT / 64, LIS = 65;
  T Li[64 * LIS];        // inverse of the panel's factored columns so far
  T Xu[64 * LW];         // rows above the sub-panel (input), then LW x 64 of scratch
  T Ut[64 * LW];         // U rows above the sub-panel, each in row_slot order
  T Lb[LW * 64];         // L rows of the sub-panel
  T cand[2][NW][LW];     // each wave's best candidate row, by column parity
  T krow[2][LW];         // row at the pivot position where no pivot was found, its entry
  T cval[2][NW];         // the candidates' pivot entries
  int cidx[2][NW];       // and positions
  int prow[64];          // physical rows of the panel's pivots
};

// A row's columns in registers, in quads (the rank-one update's accumulators).
template <typename T> struct Quad;
template <> struct Quad<float> { typedef f4 v; };
template <> struct Quad<double> { typedef d4 v; };

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
__device__ __forceinline__ void pivot_column(PanelSmem<T, LW, NT>& sm, typename Quad<T>::v (&x)[R][LW / 4], int (&pos)[R],
                                             int k, int n, DeviceStatus* status, int elem) {
  constexpr int NW = NT / 64, par = KK & 1;
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
  const T wbest = wave_max(best);
  if (wbest < T(0)) {
    if (lane == 0) sm.cidx[par][wv] = INT_MAX;
  } else {
    const int win = first_lane(__ballot(best == wbest), bpos);
    const int sq = read_lane(bq, win);
    if (lane == win) {
      put_row<LW, 0>(x, sq, KK, sm.cand[par][wv], &sm.cval[par][wv]);
      sm.cidx[par][wv] = bpos;
    }
  }
  __syncthreads();
  // the workgroup's pivot: lane w looks at wave w's candidate.  Buffers
  // alternate by column parity: one is rewritten only after every wave has
  // passed the next column's barrier, i.e. finished reading it.
  const int wl = lane & (NW - 1);
  const int ci = sm.cidx[par][wl];
  const T cv = sm.cval[par][wl];
  const T ca = ci == INT_MAX ? T(-1) : fabs(cv);
  const T gbest = read_lane(row_max(ca), 0);
  const int bw = first_lane(__ballot(ca == gbest) & ((1ull << NW) - 1), ci);
  int piv = read_lane(ci, bw);
  T u0 = read_lane(cv, bw);
  const T* urow = sm.cand[par][bw];
  if (!(gbest > T(0)) || !isfinite(gbest)) {
    // no pivot: row k stays (the branch is uniform over the workgroup)
    if (tid == 0) latch_status(status, IEDG_ERR_SINGULAR, elem);
#pragma unroll
    for (int q = 0; q < R; ++q)
      if (pos[q] == k) put_row<LW, 0>(x, q, KK, sm.krow[0], &sm.krow[1][0]);
    __syncthreads();
    piv = k;
    urow = sm.krow[0];
    u0 = sm.krow[1][0];
    __syncthreads();  // read before another column posts its row k
  }
  const T rinv = T(1) / u0;
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
    // (rows that stay take 0 times u: where u is not finite, which leaves the
    // element without a usable U in any case, their later entries turn NaN)
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
__device__ __forceinline__ void pivot_columns(PanelSmem<T, LW, NT>& sm, typename Quad<T>::v (&x)[R][LW / 4], int (&pos)[R],
                                              int cs, int sw, int n, DeviceStatus* status, int elem) {
  if constexpr (KK < LW) {
    if constexpr (KK % 4 == 0)  // sw is a multiple of 4, as n is
      if (KK >= sw) return;
    pivot_column<T, LW, R, NT, KK>(sm, x, pos, cs + KK, n, status, elem);
    pivot_columns<T, LW, R, NT, KK + 1>(sm, x, pos, cs, sw, n, status, elem);
  }
}

template <typename T, int LW, int R, int NT>
__global__ __launch_bounds__(NT, NT == 512 && R * LW * sizeof(T) <= 256 ? 4 : 1)
void condense_panel_kernel(CondenseWork<T> wk, int c0, int cb, int ce, int right) {
  typedef PanelSmem<T, LW, NT> SM;
  typedef Mfma<T> MF;
  constexpr int NW = NT / 64, LIS = SM::LIS, V = 16 / sizeof(T);  // values per 16-byte vector
  typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
  extern __shared__ __align__(16) unsigned char smem_raw[];
  SM& sm = *reinterpret_cast<SM*>(smem_raw);
  int* prow = sm.prow;

  const Elem<T> el = condense_elem(wk, blockIdx.x);
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lg = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = el.n, N = el.N, wp = ce - cb;

  int pos[R], phys[R];  // this thread's rows: position (a label), physical row
  T* rowp[R];
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int p = cb + tid + NT * q;
    pos[q] = p;
    phys[q] = p < n && cb > 0 ? el.perm[p] : p;
    rowp[q] = p < N ? el.lrow(p, phys[q]) : el.LU;  // slots past the last row: never stored
  }
  for (int i = tid; i < 64 * LIS; i += NT) sm.Li[i] = T(0);
  __syncthreads();

  for (int cs = cb; cs < ce; cs += LW) {
    const int sw = min(LW, ce - cs), kp = cs - cb;
    typename Quad<T>::v x[R][LW / 4];
#pragma unroll
    for (int q = 0; q < R; ++q)
#pragma unroll
      for (int j = 0; j < LW; j += V) {
        vec v = vec(T(0));
        if (j < sw) v = *reinterpret_cast<const vec*>(rowp[q] + cs + j);
#pragma unroll
        for (int i = 0; i < V; ++i) x[q][(j + i) / 4][(j + i) % 4] = v[i];
      }
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
      }
      __syncthreads();
      // the other rows: X -= L[:, cb:cs] U, 4 columns of L at a time
#pragma unroll 2
      for (int k0 = 0; k0 < kp; k0 += 4) {
        T la[R][4];
#pragma unroll
        for (int q = 0; q < R; ++q)
#pragma unroll
          for (int j = 0; j < 4; j += V) {
            const vec v = *reinterpret_cast<const vec*>(rowp[q] + cb + k0 + j);
#pragma unroll
            for (int i = 0; i < V; ++i) la[q][j + i] = v[i];
          }
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          const T* ur = sm.Ut + (k0 + kk) * LW;
          if constexpr (sizeof(T) == 4) {
            T u[LW / 4];
#pragma unroll
            for (int c = 0; c < LW / 4; ++c) u[c] = ur[(lane & 3) * (LW / 4) + c];
#pragma unroll
            for (int q = 0; q < R; ++q) rank_one<LW, -1>(x[q], -la[q][kk], u);
          } else {
#pragma unroll
            for (int j = 0; j < LW; ++j) {
              const T u = ur[row_slot<LW>(j)];
#pragma unroll
              for (int q = 0; q < R; ++q) x[q][j / 4][j % 4] = fma(-la[q][kk], u, x[q][j / 4][j % 4]);
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
    pivot_columns<T, LW, R, NT, 0>(sm, x, pos, cs, sw, n, el.status, el.id);
    // store; the pivot rows' own columns of L, and where they are
#pragma unroll
    for (int q = 0; q < R; ++q) {
      if (cb + tid + NT * q < N) {
#pragma unroll
        for (int j = 0; j < LW; j += V)
          if (j < sw) {
            vec v;
#pragma unroll
            for (int i = 0; i < V; ++i) v[i] = x[q][(j + i) / 4][(j + i) % 4];
            *reinterpret_cast<vec*>(rowp[q] + cs + j) = v;
          }
      }
      const int i = pos[q] - cs;
      if (i >= 0 && i < sw) {
        prow[kp + i] = phys[q];
#pragma unroll
        for (int j = 0; j < LW; ++j)
          if (j < sw) sm.Lb[i * 64 + kp + j] = j < i ? x[q][j / 4][j % 4] : T(0);
      }
    }
    if (!wk.self || cs + LW < ce || right > 0) {  // the inverse is needed further
      // the panel's earlier columns of them, from memory
      sync_global();
      for (int o = tid; o < sw * kp; o += NT) {
        const int i = o / kp, k = o % kp;
        sm.Lb[i * 64 + k] = el.LU[(size_t)prow[kp + i] * n + cb + k];
      }
      __syncthreads();
      grow_inverse<T, LW>(sm.Li, LIS, sm.Lb, sm.Xu, kp, sw);
    }
  }
#pragma unroll
  for (int q = 0; q < R; ++q)
    if (cb + tid + NT * q < n) el.perm[pos[q]] = phys[q];

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
        for (int ib = 0; ib < 4; ++ib) {
          typename MF::acc_t acc = MF::zero();
#pragma unroll
          for (int q = 0; q < 4 * (ib + 1); ++q)
            acc = MF::mac(sm.Li[(16 * ib + li) * LIS + 4 * q + lg], xb[q], acc);
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
                         el.Ke + kInvBlock);
    }
  }
}

template <typename T, int LW, int R, int NT>
static hipError_t launch_panel(const CondenseWork<T>& w, int c0, int cb, int ce, int right, hipStream_t s) {
  size_t smem = (sizeof(PanelSmem<T, LW, NT>) + 15) & ~size_t(15);
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
