// Element-local kernels on gfx950: recovery of the element unknowns
// (section 2.2.1) and the FP64 residual of the uncondensed Newton system.
#include <mutex>

#include "common.h"
#include "mesh.h"

namespace iedg {

constexpr int LTHR = 256;
constexpr int LWAVES = LTHR / 64;

// z_e = U^{-1} (w_e - U12_e uhat_e): one workgroup of THR threads per element.
// Position i of the factorisation lives in physical row perm[i] of LU, U12 and
// w.  Rows are processed four per wave at a time (wave_dot_rows) so each lane
// keeps 16 loads in flight; 64-row diagonal blocks of U (fetched ahead of the
// block's row sums by 1,024 threads) are staged in LDS in the storage precision and solved by
// one wave.  A step of that solve is a lane read and four fused multiply-adds:
// the quotient by the pivot is its reciprocal's product, corrected once.  That
// is a NaN where the reciprocal or the quotient is not finite (a zero, infinite
// or subnormal pivot, an overflow): a block whose solution is not finite is
// solved again with the quotients themselves, which keeps the test off the
// chain of steps.
template <typename T, int THR>
__global__ __launch_bounds__(THR) void backsolve_kernel(int n, int t, int b, int S, const int32_t* elem_faces, const T* LU,
                                                        const int32_t* perm, const T* U12, const double* w,
                                                        const double* uhat, double* z) {
  constexpr int WAVES = THR / 64, BV = 64 * 64 / THR;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* ue = reinterpret_cast<double*>(smem_raw);  // t
  double* y = ue + t;                                // n
  int* sp = reinterpret_cast<int*>(y + n);           // n
  T* blk = reinterpret_cast<T*>(sp + ((n + 3) & ~3));  // 64 x 65
  const int e = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  for (int i = tid; i < t; i += THR) {
    const int a = i / b, l = i % b;
    ue[i] = uhat[(size_t)elem_faces[S * e + a] * b + l];
  }
  for (int i = tid; i < n; i += THR) sp[i] = perm[(size_t)e * n + i];
  __syncthreads();
  const T* U12e = U12 + (size_t)e * n * t;
  for (int i = 4 * wv; i < n; i += 4 * WAVES) {
    const T* rows[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) rows[r] = U12e + (size_t)sp[min(i + r, n - 1)] * t;
    double s[4];
    wave_dot_rows<T, 4>(rows, ue, t, s);
    if (lane < 4 && i + lane < n) {
      double v = s[0];
#pragma unroll
      for (int r = 1; r < 4; ++r) v = lane == r ? s[r] : v;
      y[i + lane] = w[(size_t)e * n + sp[i + lane]] - v;
    }
  }
  __syncthreads();
  const T* U = LU + (size_t)e * n * n;
  const int nblk = (n + 63) / 64;
  for (int bi = nblk - 1; bi >= 0; --bi) {
    const int i0 = bi * 64, i1 = min(i0 + 64, n), bw = i1 - i0;
    // (256 threads would hold 16 values each, and occupancy matters there)
    constexpr bool AHEAD = BV <= 4;
    auto diagonal = [&](int q) __attribute__((always_inline)) -> T {
      const int rr = q / 64, cc = q % 64;
      return (rr < bw && cc < bw && cc >= rr) ? U[(size_t)sp[i0 + rr] * n + i0 + cc] : T(0);
    };
    T d[AHEAD ? BV : 1];
    if constexpr (AHEAD) {
#pragma unroll
      for (int v = 0; v < BV; ++v) d[v] = diagonal(tid + v * THR);
    }
    // y[i0:i1] -= U[i0:i1, i1:n] z[i1:n]   (z stored in y beyond i1)
    if (i1 < n) {
      for (int i = i0 + 4 * wv; i < i1; i += 4 * WAVES) {
        const T* rows[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) rows[r] = U + (size_t)sp[min(i + r, i1 - 1)] * n + i1;
        double s[4];
        wave_dot_rows<T, 4>(rows, y + i1, n - i1, s);
        if (lane < 4 && i + lane < i1) {
          double v = s[0];
#pragma unroll
          for (int r = 1; r < 4; ++r) v = lane == r ? s[r] : v;
          y[i + lane] -= v;
        }
      }
    }
    if constexpr (AHEAD) {
#pragma unroll
      for (int v = 0; v < BV; ++v) {
        const int q = tid + v * THR;
        blk[q / 64 * 65 + q % 64] = d[v];
      }
    } else {
      for (int q = tid; q < 64 * 64; q += THR) blk[q / 64 * 65 + q % 64] = diagonal(q);
    }
    __syncthreads();
    if (wv == 0) {
      const double y0 = lane < bw ? y[i0 + lane] : 0.0;
      const double dg = lane < bw ? (double)blk[lane * 65 + lane] : 1.0, rd = 1.0 / dg;
      double yl = y0;
#pragma unroll 4
      for (int k = bw - 1; k >= 0; --k) {
        const double u = (double)blk[lane * 65 + k];
        double zl = yl * rd;  // meant for lane k alone
        zl = fma(fma(-zl, dg, yl), rd, zl);
        const double zk = lane_value(zl, k);
        yl = lane == k ? zk : lane < k ? fma(-u, zk, yl) : yl;
      }
      if (__ballot(lane < bw && !isfinite(yl))) {
        yl = y0;
        for (int k = bw - 1; k >= 0; --k) {
          const double u = (double)blk[lane * 65 + k];
          const double zk = lane_value(yl, k) / lane_value(dg, k);
          yl = lane == k ? zk : lane < k ? fma(-u, zk, yl) : yl;
        }
      }
      if (lane < bw) y[i0 + lane] = yl;
    }
    __syncthreads();
  }
  for (int i = tid; i < n; i += THR) z[(size_t)e * n + i] = y[i];
}

// Rows of rF_e = F_e - A_e z_e - B_e u_e and of q_e = C_e z_e + D_e u_e: a
// workgroup takes `rows` consecutive rows of an element's [A B; C D], a wave
// four at a time with 16 loads in flight a lane.  Bound by HBM (every block is
// read once).  Split by rows, because one workgroup an element leaves CUs idle
// below 256 elements and in the last round above: 216 elements of n = 2500,
// t = 750 took 5.87 ms (3.1 TB/s) so, 3.00 ms (6.1 TB/s) split.  The element's
// first workgroup also sums F^2, before any row of it is written.
constexpr int RROWS = 64;

__global__ __launch_bounds__(LTHR) void residual_elem_kernel(int n, int t, int b, int S, int rows, int chunks,
                                                             const int32_t* elem_faces, const double* A,
                                                             const double* B, const double* C, const double* D,
                                                             const double* F, const double* z, const double* uhat,
                                                             double* rF, double* q, double* part_f) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* ue = reinterpret_cast<double*>(smem_raw);  // t
  double* ze = ue + t;                               // n
  double* red = ze + n;                              // LWAVES
  const int e = blockIdx.x / chunks, r0 = (blockIdx.x % chunks) * rows;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  for (int i = tid; i < t; i += LTHR) {
    const int a = i / b, l = i % b;
    ue[i] = uhat[(size_t)elem_faces[S * e + a] * b + l];
  }
  for (int i = tid; i < n; i += LTHR) ze[i] = z[(size_t)e * n + i];
  if (r0 == 0) {
    double f2 = 0.0;
    for (int i = tid; i < n; i += LTHR) f2 += F[(size_t)e * n + i] * F[(size_t)e * n + i];
    f2 = block_sum(f2, red);
    if (tid == 0) part_f[e] = f2;
  }
  __syncthreads();
  const size_t nn = (size_t)n * n, nt = (size_t)n * t, tt = (size_t)t * t;
  const double *Ae = A + e * nn, *Be = B + e * nt, *Ce = C + e * nt, *De = D + e * tt;
  const int r1 = min(r0 + rows, n + t);
  for (int i = r0 + 4 * wv; i < r1; i += 4 * LWAVES) {
    const double *left[4], *right[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = min(i + r, r1 - 1);
      left[r] = row < n ? Ae + (size_t)row * n : Ce + (size_t)(row - n) * n;
      right[r] = row < n ? Be + (size_t)row * t : De + (size_t)(row - n) * t;
    }
    double s[4], s2[4];
    wave_dot_rows<double, 4>(left, ze, n, s);
    wave_dot_rows<double, 4>(right, ue, t, s2);
    if (lane < 4 && i + lane < r1) {
      double v = s[0] + s2[0];
#pragma unroll
      for (int r = 1; r < 4; ++r) v = lane == r ? s[r] + s2[r] : v;
      const int row = i + lane;
      if (row < n) rF[(size_t)e * n + row] = F[(size_t)e * n + row] - v;
      else q[(size_t)e * t + row - n] = v;
    }
  }
}

// rG = G - sum_e P_e^T q_e (list order: ascending e, a) and per-unit sums of
// rG^2, G^2 (b <= 128 dofs a unit, one workgroup of 128 threads a unit); the
// workgroups past the units sum rF^2 of one element each.  Every sum
// has a fixed order.
__global__ __launch_bounds__(128) void residual_face_kernel(int NF, int n, int b, int t, int S, const int32_t* src_ptr,
                                                            const int32_t* src_list, const double* q,
                                                            const double* G, const double* rF, double* rG,
                                                            double* part_rg, double* part_g, double* part_rf) {
  __shared__ double red[2];
  const int f = blockIdx.x, l = threadIdx.x;
  double v = 0.0, g = 0.0;
  if (f >= NF) {
    const int e = f - NF;
    const double* re = rF + (size_t)e * n;
    for (int i = l; i < n; i += 128) v += re[i] * re[i];
    v = wave_sum(v);
    if (l == 64) red[0] = v;
    __syncthreads();
    if (l == 0) part_rf[e] = v + red[0];
    return;
  }
  if (l < b) {
    const size_t i = (size_t)f * b + l;
    g = G[i];
    v = g;
    for (int k = src_ptr[f]; k < src_ptr[f + 1]; ++k) {
      const int code = src_list[k], e = code / S, a = code - e * S;
      v -= q[(size_t)e * t + a * b + l];
    }
    rG[i] = v;
  }
  const double s1 = wave_sum(l < 64 ? v * v : 0.0) + 0.0;
  const double s2 = wave_sum(l < 64 ? g * g : 0.0);
  const double s3 = wave_sum(l >= 64 ? v * v : 0.0);
  const double s4 = wave_sum(l >= 64 ? g * g : 0.0);
  if (l == 64) { red[0] = s3; red[1] = s4; }
  __syncthreads();
  if (l == 0) {
    part_rg[f] = s1 + red[0];
    part_g[f] = s2 + red[1];
  }
}

// sums[k] = sum over i < len_k of part_k[i], fixed order, one wave each.
__global__ void sum4_kernel(const double* p0, int64_t n0, const double* p1, int64_t n1, const double* p2, int64_t n2,
                            const double* p3, int64_t n3, double* sums) {
  const int k = blockIdx.x, lane = threadIdx.x;
  const double* p = k == 0 ? p0 : k == 1 ? p1 : k == 2 ? p2 : p3;
  const int64_t n = k == 0 ? n0 : k == 1 ? n1 : k == 2 ? n2 : n3;
  double s = 0.0;
  for (int64_t i = lane; i < n; i += 64) s += p[i];
  s = wave_sum(s);
  if (lane == 0) sums[k] = s;
}

}  // namespace iedg

using namespace iedg;

extern "C" iedg_status iedg_backsolve_local(iedg_context ctx, iedg_mesh mesh, int32_t n_local, iedg_prec prec,
                                            const void* LU, const int32_t* perm, const void* U12, const double* w,
                                            const double* uhat, double* z, hipStream_t stream) {
  if (!ctx || !mesh || !LU || !perm || !U12 || !w || !uhat || !z || n_local <= 0) return IEDG_ERR_INVALID_ARG;
  const int n = n_local, t = mesh->t, b = mesh->b;
  const size_t smem_ints = sizeof(double) * (t + n) + sizeof(int) * ((n + 3) & ~3);
  const bool f64 = prec == IEDG_F64, wide = element_wide(mesh->n_elem);
  const size_t smem = smem_ints + (f64 ? sizeof(double) : sizeof(float)) * 64 * 65;
  const dim3 thr(wide ? kElementWide : kElementNarrow);
  if (f64) {
    auto k = wide ? backsolve_kernel<double, kElementWide> : backsolve_kernel<double, kElementNarrow>;
    IEDG_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
    hipLaunchKernelGGL(k, dim3(mesh->n_elem), thr, smem, stream, n, t, b, mesh->slots, mesh->d_elem_faces,
                       (const double*)LU, perm, (const double*)U12, w, uhat, z);
  } else {
    auto k = wide ? backsolve_kernel<float, kElementWide> : backsolve_kernel<float, kElementNarrow>;
    IEDG_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
    hipLaunchKernelGGL(k, dim3(mesh->n_elem), thr, smem, stream, n, t, b, mesh->slots, mesh->d_elem_faces,
                       (const float*)LU, perm, (const float*)U12, w, uhat, z);
  }
  IEDG_LAUNCH_CHECK(ctx, "backsolve launch");
  return IEDG_OK;
}

namespace iedg {

// Both residual entry points: `work` holds q [E][t] and the partial sums
// (2E + 2 n_face values); every entry is written before it is read.
static iedg_status residual_launch(iedg_context ctx, iedg_mesh mesh, int n, const double* A, const double* B,
                                   const double* C, const double* D, const double* F, const double* G,
                                   const double* z, const double* uhat, double* rF, double* rG, double* sums,
                                   double* work, hipStream_t stream) {
  const int t = mesh->t, b = mesh->b, E = mesh->n_elem, NF = mesh->n_face;
  double* q = work;
  double* prf = q + (size_t)E * t;
  double* pf = prf + E;
  double* prg = pf + E;
  double* pg = prg + NF;
  const size_t smem = sizeof(double) * (t + n + LWAVES);
  // rF written over F or z: the whole element in one workgroup, which reads
  // both before it writes (and where the split would be too many workgroups)
  const double* last = rF + (size_t)E * n;
  const bool over = (F < last && rF < F + (size_t)E * n) || (z < last && rF < z + (size_t)E * n);
  const int split = (n + t + RROWS - 1) / RROWS;
  const bool whole = over || (int64_t)E * split > launch_groups(LTHR);
  const int rows = whole ? n + t : RROWS, chunks = whole ? 1 : split;
  IEDG_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(residual_elem_kernel),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
  hipLaunchKernelGGL(residual_elem_kernel, dim3(E * chunks), dim3(LTHR), smem, stream, n, t, b, mesh->slots, rows, chunks,
                     mesh->d_elem_faces, A, B, C, D, F, z, uhat, rF, q, pf);
  // units and elements in one launch, or one launch each
  const bool one = (int64_t)NF + E <= launch_groups(128);
  hipLaunchKernelGGL(residual_face_kernel, dim3(one ? NF + E : NF), dim3(128), 0, stream, NF, n, b, t, mesh->slots,
                     mesh->d_src_ptr, mesh->d_src_list, q, G, rF, rG, prg, pg, prf);
  if (!one)
    hipLaunchKernelGGL(residual_face_kernel, dim3(E), dim3(128), 0, stream, 0, n, b, t, mesh->slots, mesh->d_src_ptr,
                       mesh->d_src_list, q, G, rF, rG, prg, pg, prf);
  hipLaunchKernelGGL(sum4_kernel, dim3(4), dim3(64), 0, stream, prf, (int64_t)E, prg, (int64_t)NF, pf, (int64_t)E, pg,
                     (int64_t)NF, sums);
  IEDG_LAUNCH_CHECK(ctx, "residual launch");
  return IEDG_OK;
}

static size_t residual_work_values(iedg_mesh mesh) {
  return (size_t)mesh->n_elem * mesh->t + 2 * (size_t)mesh->n_elem + 2 * (size_t)mesh->n_face;
}

// ---- the allocation-free residual ---------------------------------------
// File-scope device scratch of the allocation-free entry point.  In host
// code `residual_scratch` names a host-side stand-in, not device memory: the
// device address of each GPU's copy is looked up once per device (from
// iedg_create, with that device current) and only that address is used.
constexpr size_t kResidualScratchValues = size_t(2) << 20;   // 16 MiB of FP64
static __device__ __align__(256) double residual_scratch[kResidualScratchValues];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static double* g_scratch_ptr[kMaxDevices] = {};

iedg_status residual_scratch_init(iedg_context ctx) {
  const int dev = ctx->device;
  if (dev < 0 || dev >= kMaxDevices) return set_error(ctx, IEDG_ERR_UNSUPPORTED, "device %d >= %d", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev]) return IEDG_OK;
  void* p = nullptr;
  hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(residual_scratch));
  if (e != hipSuccess || !p) return hip_check(ctx, e != hipSuccess ? e : hipErrorInvalidSymbol, "hipGetSymbolAddress");
  g_scratch_ptr[dev] = static_cast<double*>(p);
  return IEDG_OK;
}

}  // namespace iedg

using namespace iedg;

extern "C" iedg_status iedg_residual_full(iedg_context ctx, iedg_mesh mesh, int32_t n_local, const double* A,
                                          const double* B, const double* C, const double* D, const double* F,
                                          const double* G, const double* z, const double* uhat, double* rF,
                                          double* rG, double* sums, hipStream_t stream) {
  if (!ctx || !mesh || !A || !B || !C || !D || !F || !G || !z || !uhat || !rF || !rG || !sums || n_local <= 0)
    return IEDG_ERR_INVALID_ARG;
  // mesh-owned scratch, allocated with the mesh
  return residual_launch(ctx, mesh, n_local, A, B, C, D, F, G, z, uhat, rF, rG, sums, mesh->d_rwork, stream);
}

extern "C" iedg_status iedg_residual_full_noalloc(iedg_context ctx, iedg_mesh mesh, int32_t n_local,
                                                  const double* A, const double* B, const double* C,
                                                  const double* D, const double* F, const double* G,
                                                  const double* z, const double* uhat, double* rF, double* rG,
                                                  double* sums, hipStream_t stream) {
  if (!ctx || !mesh || !A || !B || !C || !D || !F || !G || !z || !uhat || !rF || !rG || !sums || n_local <= 0)
    return set_error(ctx, IEDG_ERR_INVALID_ARG, "residual_full_noalloc: null argument or n <= 0");
  const size_t need = residual_work_values(mesh);
  if (need > kResidualScratchValues)
    return set_error(ctx, IEDG_ERR_UNSUPPORTED,
                     "residual_full_noalloc: needs %zu scratch values (E t + 2 E + 2 n_face), the static "
                     "scratch holds %zu", need, kResidualScratchValues);
  double* work = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (ctx->device >= 0 && ctx->device < kMaxDevices) work = g_scratch_ptr[ctx->device];
  }
  if (!work) return set_error(ctx, IEDG_ERR_HIP, "residual_full_noalloc: scratch address of device %d unknown",
                              ctx->device);
  return residual_launch(ctx, mesh, n_local, A, B, C, D, F, G, z, uhat, rF, rG, sums, work, stream);
}
