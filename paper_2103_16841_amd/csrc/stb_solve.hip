// stb_solve.hip -- the discrete indirect system (eq. df_ind): restarted
// GMRES over the assembled energetic single-layer matrix, on the device, and
// marching-on-in-time for slab-structured meshes.
//
// Every Krylov step is one FP64 product with the stored matrix plus
// classical Gram-Schmidt against the basis, done twice for orthogonality
// (CGS2): partial dot products of every basis vector per chunk of n, then one
// kernel that sums a vector's chunks in order and subtracts.  The small
// Hessenberg problem (Givens rotations, back substitution) stays on the host;
// a step's coefficients reach it through pinned memory while the next step's
// product is already running.  Every sum has a fixed order, so results do not
// depend on the schedule.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <vector>

#include "stb_internal.h"

namespace {

constexpr int kSolveThreads = 256;

// part[b * nch + c] = <V_b, w> over chunk c of kGsChunk elements, for b < k (V
// row-major, rows of n doubles): one wavefront per vector and chunk.  (One
// workgroup per vector took 37 us at n = 30,720: 120 dependent loads a lane,
// and one busy CU for the few vectors of the first steps.)
constexpr int64_t kGsChunk = 1024;
__global__ __launch_bounds__(kSolveThreads) void k_gs_dots(int64_t n, int k, const double* __restrict__ V,
                                                           const double* __restrict__ w,
                                                           double* __restrict__ part) {
  const int lane = threadIdx.x & 63;
  const int b = (int)blockIdx.y * (kSolveThreads / 64) + (int)(threadIdx.x >> 6);
  if (b >= k) return;
  const double* v = V + (int64_t)b * n;
  const int64_t i0 = (int64_t)blockIdx.x * kGsChunk, i1 = std::min<int64_t>(i0 + kGsChunk, n);
  double s = 0.0;
  if (i1 - i0 == kGsChunk) {
    double p[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int u = 0; u < (int)(kGsChunk / 64); ++u) p[u & 3] = fma(v[i0 + 64 * u + lane], w[i0 + 64 * u + lane], p[u & 3]);
    s = (p[0] + p[1]) + (p[2] + p[3]);
  } else {
    for (int64_t i = i0 + lane; i < i1; i += 64) s = fma(v[i], w[i], s);
  }
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if (lane == 0) part[(int64_t)b * gridDim.x + blockIdx.x] = s;
}

// h[b] = the sum of b's nch chunks (in order), w -= sum_{b < k} h[b] V_b; block 0
// writes h to hout.  npart (optional): per block the sum of its new w_i^2.
constexpr int kMaxBasis = 513;
__global__ __launch_bounds__(kSolveThreads) void k_gs_sub(int64_t n, int k, int64_t nch, const double* __restrict__ V,
                                                          const double* __restrict__ part, double* __restrict__ w,
                                                          double* __restrict__ hout, double* __restrict__ npart) {
  __shared__ double h[kMaxBasis];
  for (int b = threadIdx.x; b < k; b += kSolveThreads) {
    double s = 0.0;
    for (int64_t c = 0; c < nch; ++c) s += part[(int64_t)b * nch + c];
    h[b] = s;
    if (blockIdx.x == 0) hout[b] = s;
  }
  __syncthreads();
  const int64_t i = (int64_t)blockIdx.x * kSolveThreads + threadIdx.x;
  double s = 0.0;
  if (i < n) {
    s = w[i];
    int b = 0;
    for (; b + 8 <= k; b += 8) {
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = V[(int64_t)(b + u) * n + i];
#pragma unroll
      for (int u = 0; u < 8; ++u) s = fma(-h[b + u], v[u], s);
    }
    for (; b < k; ++b) s = fma(-h[b], V[(int64_t)b * n + i], s);
    w[i] = s;
  }
  if (!npart) return;
  double q = s * s;
  for (int off = 32; off > 0; off >>= 1) q += __shfl_down(q, off, 64);
  __shared__ double red[kSolveThreads / 64];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = q;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = red[0];
    for (int v = 1; v < kSolveThreads / 64; ++v) t += red[v];
    npart[blockIdx.x] = t;
  }
}

// Sum of m partial sums in a fixed order, by a whole block.
__device__ __forceinline__ double block_sum(const double* __restrict__ part, int64_t m) {
  __shared__ double red[kSolveThreads];
  double s = 0.0;
  for (int64_t c = threadIdx.x; c < m; c += kSolveThreads) s += part[c];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int off = kSolveThreads / 2; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  return red[0];
}

// out = w / |w| (0 for |w| = 0) from the m partial sums of |w|^2; block 0
// writes |w|^2 and, with k > 0, the k + k coefficients of the two Gram-Schmidt
// passes to `host` (pinned host memory): [0] |w|^2, [1 ...] first, then
// second pass.
__global__ __launch_bounds__(kSolveThreads) void k_gs_scale(int64_t n, int64_t m, const double* __restrict__ npart,
                                                            const double* w, double* out, int k,
                                                            const double* __restrict__ h1,
                                                            const double* __restrict__ h2, double* __restrict__ host) {
  const double q = block_sum(npart, m);
  const double f = q > 0.0 ? 1.0 / sqrt(q) : 0.0;
  const int64_t i = (int64_t)blockIdx.x * kSolveThreads + threadIdx.x;
  if (i < n) out[i] = f * w[i];
  if (blockIdx.x != 0) return;
  if (threadIdx.x == 0) host[0] = q;
  for (int b = threadIdx.x; b < k; b += kSolveThreads) {
    host[1 + b] = h1[b];
    host[1 + k + b] = h2[b];
  }
}

// Per block the sum of its a_i^2.
__global__ __launch_bounds__(kSolveThreads) void k_norm2(int64_t n, const double* __restrict__ a,
                                                         double* __restrict__ npart) {
  const int64_t i = (int64_t)blockIdx.x * kSolveThreads + threadIdx.x;
  double q = i < n ? a[i] * a[i] : 0.0;
  for (int off = 32; off > 0; off >>= 1) q += __shfl_down(q, off, 64);
  __shared__ double red[kSolveThreads / 64];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = q;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = red[0];
    for (int v = 1; v < kSolveThreads / 64; ++v) t += red[v];
    npart[blockIdx.x] = t;
  }
}

// x += sum_{b < k} y[b] V_b (b ascending).
__global__ __launch_bounds__(kSolveThreads) void k_combine(int64_t n, int k, const double* __restrict__ V,
                                                           const double* __restrict__ y, double* __restrict__ x) {
  const int64_t i = (int64_t)blockIdx.x * kSolveThreads + threadIdx.x;
  if (i >= n) return;
  double s = x[i];
  int b = 0;
  for (; b + 8 <= k; b += 8) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = V[(int64_t)(b + u) * n + i];
#pragma unroll
    for (int u = 0; u < 8; ++u) s = fma(y[b + u], v[u], s);
  }
  for (; b < k; ++b) s = fma(y[b], V[(int64_t)b * n + i], s);
  x[i] = s;
}

// r = b - r (r holds A x).
__global__ void k_residual(int64_t n, const double* __restrict__ b, double* __restrict__ r) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) r[i] = b[i] - r[i];
}

// b_i = sum_{q < n_i} w_iq g_iq, q ascending: the right-hand side of the
// indirect system from data g at panel i's outer points (eq. df_ind with the
// outer rule of eq. int_bform).
__global__ void k_outer_rhs(int64_t nt, int maxq, const double* __restrict__ w,
                            const int32_t* __restrict__ nq, const double* __restrict__ g,
                            double* __restrict__ b) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nt) return;
  double s = 0.0;
  for (int q = 0; q < nq[i]; ++q) s = fma(w[i * maxq + q], g[i * maxq + q], s);
  b[i] = s;
}


// ------------------------------------------------ marching-on-in-time
// Dense diagonal block D[k][l] = A[row_k][row_l] of the panels of slab 0
// (loc[j] = local index of panel j in its slab, slab[j] its slab).
__global__ void k_mot_block(int64_t K, const int32_t* __restrict__ rows0, const int64_t* __restrict__ rowptr,
                            const int32_t* __restrict__ cols, const double* __restrict__ vals,
                            const int32_t* __restrict__ slab, const int32_t* __restrict__ loc,
                            double* __restrict__ D) {
  const int64_t k = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;   // one wavefront per row
  if (k >= K) return;
  const int32_t i = rows0[k];
  for (int64_t e = rowptr[i] + (threadIdx.x & 63); e < rowptr[i + 1]; e += 64) {
    const int32_t j = cols[e];
    if (slab[j] == 0) D[k * K + loc[j]] = vals[e];
  }
}

// Every stored entry (i, j) has slab[j] <= slab[i] (block lower triangular
// in time); bad[0] counts the entries that do not.  One wavefront per row.
__global__ __launch_bounds__(256) void k_mot_lower(int64_t n, const int64_t* __restrict__ rowptr,
                                                   const int32_t* __restrict__ cols,
                                                   const int32_t* __restrict__ slab,
                                                   unsigned long long* __restrict__ bad) {
  const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  if (i >= n) return;
  const int lane = threadIdx.x & 63;
  const int32_t own = slab[i];
  const int64_t e = rowptr[i + 1];
  unsigned c = 0;
  int64_t k = rowptr[i] + lane;
  for (; k + 192 < e; k += 256) {
    const int32_t j0 = cols[k], j1 = cols[k + 64], j2 = cols[k + 128], j3 = cols[k + 192];
    c += (slab[j0] > own ? 1u : 0u) + (slab[j1] > own ? 1u : 0u) + (slab[j2] > own ? 1u : 0u) +
         (slab[j3] > own ? 1u : 0u);
  }
  for (; k < e; k += 64) c += slab[cols[k]] > own ? 1u : 0u;
  for (int off = 32; off > 0; off >>= 1) c += __shfl_down(c, off, 64);
  if (lane == 0 && c) atomicAdd(bad, (unsigned long long)c);
}

// Gauss-Jordan inversion of D (K x K, row-major) in place, NB columns at a
// time, with partial pivoting and no row interchanges: pivot k sits in a row
// p_k not used before, and the array ends as B[p_k][j] = (P D)^-1[k][j], so
// D^-1[k][p_j] = B[p_k][j] (k_gj_permute).
//
// Panel step (one workgroup): the NB columns from k0 on, the thread's RPT rows
// in registers; per column the pivot search over the unused rows and one
// elimination of the panel's columns, the pivot row passed through LDS.  Then
// the pivot rows' other columns, as they were, go to rbuf.  The step is a
// serial chain, so it runs on as few wavefronts as hold the rows (one per
// SIMD up to K = 1024), and pivots are compared by the upper halves of |D|
// (20 bits of mantissa) with one DPP maximum over the wave: a pivot within 1e-6 of
// the largest is as stable as the largest.  K = 960: eliminating the whole
// matrix column by column took two launches a column, 6.2 + 3.8 us; this
// panel with 16 waves and exact (value, row) shuffles 4.5 us a column, as it
// stands 2.5 us.  A pivot without a finite reciprocal (zero, NaN, infinity)
// makes the matrix singular: it is reported, not divided by.
//
// Maximum over the wavefront of a non-negative key (DPP row shifts, then the
// two row broadcasts; lane 63 holds it).
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  auto step = [](uint32_t x, uint32_t y) { return x > y ? x : y; };
  v = step(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));   // row_shr:1
  v = step(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));   // row_shr:2
  v = step(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));   // row_shr:4
  v = step(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));   // row_shr:8
  v = step(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));   // row_bcast:15
  v = step(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));   // row_bcast:31
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

template <int T, int RPT, int NB>
__global__ __launch_bounds__(T) void k_gj_panel(int64_t K, int64_t k0, double* __restrict__ D,
                                                int32_t* __restrict__ piv, uint8_t* __restrict__ used,
                                                double* __restrict__ rbuf, int* __restrict__ singular) {
  constexpr int kWaves = T / 64;
  const int nb = (int)(K - k0 < NB ? K - k0 : NB);
  const bool wide = nb == NB && (K & 1) == 0;   // whole panel, rows 16-byte aligned
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __shared__ uint32_t s_key[kWaves];
  __shared__ int32_t s_idx[kWaves], s_piv[NB];
  __shared__ double s_row[NB];
  double A[RPT][NB];
  bool free_row[RPT];
#pragma unroll
  for (int r = 0; r < RPT; ++r) {
    const int64_t i = threadIdx.x + (int64_t)r * T;
    free_row[r] = i < K && !used[i];
    if (i < K && wide) {
      const double2* d = reinterpret_cast<const double2*>(D + i * K + k0);
#pragma unroll
      for (int c = 0; c < NB; c += 2) {
        const double2 v = d[c / 2];
        A[r][c] = v.x;
        A[r][c + 1] = v.y;
      }
    } else {
#pragma unroll
      for (int c = 0; c < NB; ++c) A[r][c] = i < K && c < nb ? D[i * K + k0 + c] : 0.0;
    }
  }
#pragma unroll
  for (int c = 0; c < NB; ++c)
    if (c < nb) {
      // key of an unused row: 1 + the upper half of |entry| (1 for a NaN or an
      // infinity, so that there always is a pivot); 0 for the others
      uint32_t best = 0;
      int32_t bi = 0;
#pragma unroll
      for (int r = 0; r < RPT; ++r) {
        const uint32_t h = (uint32_t)__double2hiint(A[r][c]) & 0x7fffffffu;
        const uint32_t key = free_row[r] ? (h < 0x7ff00000u ? h : 0u) + 1u : 0u;
        bi = key > best ? (int32_t)(threadIdx.x + r * T) : bi;
        best = key > best ? key : best;
      }
      const uint32_t top = wave_max(best);
      const uint64_t at = __ballot(best == top);
      if (lane == __ffsll((long long)at) - 1) {
        s_key[wave] = top;
        s_idx[wave] = bi;
      }
      __syncthreads();
      best = s_key[0];
      bi = s_idx[0];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) {
        const uint32_t k = s_key[w];
        bi = k > best ? s_idx[w] : bi;
        best = k > best ? k : best;
      }
      // a pivot in frcp's range, by its key: 2^-1000 <= |pivot| < 2^1000
      const bool plain = best - 0x01700001u < 0x7d000000u;
      // the pivot row's owner scales it and passes it on
#pragma unroll
      for (int r = 0; r < RPT; ++r)
        if (threadIdx.x + r * T == (unsigned)bi) {
          double inv = stb::frcp(A[r][c]);
          if (!plain) {
            inv = 1.0 / A[r][c];
            if (!(fabs(A[r][c]) < HUGE_VAL && fabs(inv) < HUGE_VAL)) {
              *singular = 1;
              inv = 0.0;
            }
          }
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            A[r][j] = (j == c ? 1.0 : A[r][j]) * inv;
            s_row[j] = A[r][j];
          }
          free_row[r] = false;
          used[bi] = 1;
          s_piv[c] = bi;
          piv[k0 + c] = bi;
        }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < RPT; ++r)
        if (threadIdx.x + r * T != (unsigned)bi) {
          const double f = A[r][c];
#pragma unroll
          for (int j = 0; j < NB; ++j) A[r][j] = j == c ? -f * s_row[j] : fma(-f, s_row[j], A[r][j]);
        }
    }
  for (int64_t j = threadIdx.x; j < K; j += T) {
    double v[NB];
#pragma unroll
    for (int c = 0; c < NB; ++c) v[c] = c < nb ? D[(int64_t)s_piv[c] * K + j] : 0.0;
#pragma unroll
    for (int c = 0; c < NB; ++c)
      if (c < nb) rbuf[(int64_t)c * K + j] = v[c];
  }
  __syncthreads();   // (the panel's own columns of rbuf are not used)
#pragma unroll
  for (int r = 0; r < RPT; ++r) {
    const int64_t i = threadIdx.x + (int64_t)r * T;
    if (i < K && wide) {
      double2* d = reinterpret_cast<double2*>(D + i * K + k0);
#pragma unroll
      for (int c = 0; c < NB; c += 2) d[c / 2] = make_double2(A[r][c], A[r][c + 1]);
    } else if (i < K) {
#pragma unroll
      for (int c = 0; c < NB; ++c)
        if (c < nb) D[i * K + k0 + c] = A[r][c];
    }
  }
}

// The other columns: D[i][j] = D[i][j] + sum_c panel[i][c] rbuf[c][j], without
// the old D[i][j] in the panel's pivot rows.  Tiles of kGjRows rows by 256
// columns, the rows' panel entries in LDS.
constexpr int kGjRows = 8;
template <int NB>
__global__ __launch_bounds__(256) void k_gj_update(int64_t K, int64_t k0, double* __restrict__ D,
                                                   const double* __restrict__ rbuf, const int32_t* __restrict__ piv) {
  const int nb = (int)(K - k0 < NB ? K - k0 : NB);
  const int64_t i0 = (int64_t)blockIdx.y * kGjRows, j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  __shared__ double s_p[kGjRows][NB];
  __shared__ int s_piv[kGjRows];
  for (int g = threadIdx.x; g < kGjRows * NB; g += 256) {
    const int r = g / NB, c = g - r * NB;
    s_p[r][c] = i0 + r < K && c < nb ? D[(i0 + r) * K + k0 + c] : 0.0;
  }
  if (threadIdx.x < kGjRows) {
    int is = 0;
    for (int c = 0; c < nb; ++c) is |= piv[k0 + c] == (int32_t)(i0 + threadIdx.x) ? 1 : 0;
    s_piv[threadIdx.x] = is;
  }
  __syncthreads();
  if (j >= K || (j >= k0 && j < k0 + nb)) return;
  double b[NB];
#pragma unroll
  for (int c = 0; c < NB; ++c) b[c] = c < nb ? rbuf[(int64_t)c * K + j] : 0.0;
#pragma unroll 4
  for (int r = 0; r < kGjRows; ++r) {
    if (i0 + r >= K) break;
    double s = s_piv[r] ? 0.0 : D[(i0 + r) * K + j];
#pragma unroll
    for (int c = 0; c < NB; ++c) s = fma(s_p[r][c], b[c], s);
    D[(i0 + r) * K + j] = s;
  }
}

// out[k][p_j] = B[p_k][j].
__global__ __launch_bounds__(256) void k_gj_permute(int64_t K, const double* __restrict__ B,
                                                    const int32_t* __restrict__ piv, double* __restrict__ out) {
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x, k = blockIdx.y;
  if (j < K) out[k * K + piv[j]] = B[(int64_t)piv[k] * K + j];
}

template <int T, int RPT, int NB>
hipError_t gj_steps(int64_t K, double* D, int32_t* piv, uint8_t* used, double* rbuf, int* sing, hipStream_t st) {
  const dim3 gu((unsigned)((K + 255) / 256), (unsigned)((K + kGjRows - 1) / kGjRows));
  for (int64_t k0 = 0; k0 < K; k0 += NB) {
    hipLaunchKernelGGL((k_gj_panel<T, RPT, NB>), dim3(1), dim3(T), 0, st, K, k0, D, piv, used, rbuf, sing);
    if (K > NB) hipLaunchKernelGGL((k_gj_update<NB>), gu, dim3(256), 0, st, K, k0, D, rbuf, piv);
  }
  return hipGetLastError();
}

constexpr int64_t kMotMaxPanels = 16 * 1024;

// Time step n, part 1: r[k] = b[i] - sum_j A[i][j] x[j] for the rows i =
// rows[k] of the slab (x is zero on this and later slabs, so this is
// b_n - sum_{m<n} A_nm x_m); one workgroup per row (a slab has few rows, so
// one wavefront each left the chip idle: 26 us a step at K = 960), fixed-order
// reduction.
__global__ __launch_bounds__(256) void k_mot_rhs(int64_t K, const int32_t* __restrict__ rows,
                                                 const int64_t* __restrict__ rowptr,
                                                 const int32_t* __restrict__ cols,
                                                 const double* __restrict__ vals,
                                                 const double* __restrict__ x, const double* __restrict__ b,
                                                 double* __restrict__ r) {
  const int64_t k = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int32_t i = rows[k];
  const int64_t e = rowptr[i + 1];
  int64_t q = rowptr[i] + threadIdx.x;
  double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
  for (; q + 768 < e; q += 1024) {
    const int32_t c0 = cols[q], c1 = cols[q + 256], c2 = cols[q + 512], c3 = cols[q + 768];
    const double v0 = vals[q], v1 = vals[q + 256], v2 = vals[q + 512], v3 = vals[q + 768];
    s0 = fma(v0, x[c0], s0);
    s1 = fma(v1, x[c1], s1);
    s2 = fma(v2, x[c2], s2);
    s3 = fma(v3, x[c3], s3);
  }
  for (; q < e; q += 256) s0 = fma(vals[q], x[cols[q]], s0);
  double s = (s0 + s1) + (s2 + s3);
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  __shared__ double red[4];
  if (lane == 0) red[wave] = s;
  __syncthreads();
  if (threadIdx.x == 0) r[k] = b[i] - ((red[0] + red[1]) + (red[2] + red[3]));
}

// Part 2: x[rows[k]] = sum_l Dinv[k][l] r[l]; one wavefront per row.
__global__ __launch_bounds__(256) void k_mot_apply(int64_t K, const int32_t* __restrict__ rows,
                                                   const double* __restrict__ Dinv,
                                                   const double* __restrict__ r, double* __restrict__ x) {
  const int64_t k = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (k >= K) return;
  const double* d = Dinv + k * K;
  double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
  int64_t l = lane;
  for (; l + 192 < K; l += 256) {
    s0 = fma(d[l], r[l], s0);
    s1 = fma(d[l + 64], r[l + 64], s1);
    s2 = fma(d[l + 128], r[l + 128], s2);
    s3 = fma(d[l + 192], r[l + 192], s3);
  }
  for (; l < K; l += 64) s0 = fma(d[l], r[l], s0);
  double s = (s0 + s1) + (s2 + s3);
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if (lane == 0) x[rows[k]] = s;
}

}  // namespace

// A panel's rows stay in one workgroup's registers, so the panels narrow as K
// grows.
stb_status stb_gj_invert(stb_ctx* ctx, int64_t K, double* D, double* out) {
  if (K < 1 || K > kMotMaxPanels)
    return stb_fail(ctx, STB_E_INVALID_ARG, "inverse of order %lld (1 to %lld)", (long long)K, (long long)kMotMaxPanels);
  hipStream_t st = ctx->stream;
  // one block lent by the context: the pivot rows' columns, pivots, flag, used rows
  double* rbuf = nullptr;
  if (kalloc(ctx, &rbuf, (size_t)(16 * K + K + 1)) != hipSuccess)
    return stb_fail(ctx, STB_E_NO_MEMORY, "inverse of order %lld", (long long)K);
  int32_t* piv = reinterpret_cast<int32_t*>(rbuf + 16 * K);
  int* d_sing = piv + K;
  uint8_t* used = reinterpret_cast<uint8_t*>(d_sing + 1);
  hipError_t e = hipMemsetAsync(d_sing, 0, sizeof(int) + K, st);
  if (e == hipSuccess)
    e = K <= 1024   ? gj_steps<256, 4, 16>(K, D, piv, used, rbuf, d_sing, st)
        : K <= 2048 ? gj_steps<512, 4, 16>(K, D, piv, used, rbuf, d_sing, st)
        : K <= 4096 ? gj_steps<1024, 4, 8>(K, D, piv, used, rbuf, d_sing, st)
        : K <= 8192 ? gj_steps<1024, 8, 4>(K, D, piv, used, rbuf, d_sing, st)
                    : gj_steps<1024, 16, 2>(K, D, piv, used, rbuf, d_sing, st);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_gj_permute, dim3((unsigned)((K + 255) / 256), (unsigned)K), dim3(256), 0, st, K, D, piv, out);
    e = hipGetLastError();
  }
  int sing = 0;
  if (e == hipSuccess) e = hipMemcpyAsync(&sing, d_sing, sizeof(int), hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  else (void)hipStreamSynchronize(st);
  ctx_keep(ctx, rbuf);
  if (e != hipSuccess) return stb_fail(ctx, STB_E_DEVICE, "inverse: %s", hipGetErrorString(e));
  return sing ? stb_fail(ctx, STB_E_INTERNAL, "the diagonal block is singular") : STB_OK;
}

extern "C" {

stb_status stb_outer_rhs(stb_ctx* ctx, const stb_mesh* mesh_c, int32_t m_q, const double* g,
                         double* b) {
  if (!ctx || !mesh_c || !g || !b) return stb_fail(ctx, STB_E_INVALID_ARG, "NULL argument");
  if (m_q < 1 || m_q > 4) return stb_fail(ctx, STB_E_INVALID_ARG, "m_q must be in [1,4], got %d", m_q);
  stb_mesh* mesh = const_cast<stb_mesh*>(mesh_c);
  if (mesh->ctx != ctx) return stb_fail(ctx, STB_E_INVALID_ARG, "mesh belongs to another context");
  HIPCHK(ctx, hipSetDevice(ctx->device));
  stb_status s = stb_ensure_outer(ctx, mesh, m_q);
  if (s) return s;
  const int64_t nt = mesh->nt, maxq = mesh->maxq;
  if (nt == 0) return STB_OK;
  for (int64_t k = 0; k < nt * maxq; ++k)
    if (!std::isfinite(g[k])) return stb_fail(ctx, STB_E_INVALID_ARG, "non-finite data at outer point %lld", (long long)k);
  double *d_g = nullptr, *d_b = nullptr;
  if (dalloc(&d_g, (size_t)(nt * maxq)) != hipSuccess || dalloc(&d_b, (size_t)nt) != hipSuccess) {
    dfree(d_g); dfree(d_b);
    return stb_fail(ctx, STB_E_NO_MEMORY, "right-hand side buffers");
  }
  hipError_t e = hipMemcpyAsync(d_g, g, sizeof(double) * nt * maxq, hipMemcpyHostToDevice, ctx->stream);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_outer_rhs, dim3((unsigned)((nt + 255) / 256)), dim3(256), 0, ctx->stream, nt,
                       (int)maxq, mesh->d_ow, mesh->d_onq, d_g, d_b);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemcpyAsync(b, d_b, sizeof(double) * nt, hipMemcpyDeviceToHost, ctx->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
  dfree(d_g);
  dfree(d_b);
  if (e != hipSuccess) return stb_fail(ctx, STB_E_DEVICE, "right-hand side: %s", hipGetErrorString(e));
  return STB_OK;
}

stb_status stb_outer_points(stb_ctx* ctx, const stb_mesh* mesh_c, int32_t m_q, double* pts,
                            double* weights, int32_t* counts) {
  if (!ctx || !mesh_c || !pts || !weights || !counts)
    return stb_fail(ctx, STB_E_INVALID_ARG, "NULL argument");
  if (m_q < 1 || m_q > 4) return stb_fail(ctx, STB_E_INVALID_ARG, "m_q must be in [1,4], got %d", m_q);
  stb_mesh* mesh = const_cast<stb_mesh*>(mesh_c);
  if (mesh->ctx != ctx) return stb_fail(ctx, STB_E_INVALID_ARG, "mesh belongs to another context");
  HIPCHK(ctx, hipSetDevice(ctx->device));
  stb_status s = stb_ensure_outer(ctx, mesh, m_q);
  if (s) return s;
  const int64_t nt = mesh->nt, maxq = mesh->maxq;
  if (nt > 0) {
    HIPCHK(ctx, hipMemcpyAsync(pts, mesh->d_opts, sizeof(double) * nt * maxq * 4, hipMemcpyDeviceToHost,
                               ctx->stream));
    HIPCHK(ctx, hipMemcpyAsync(weights, mesh->d_ow, sizeof(double) * nt * maxq, hipMemcpyDeviceToHost,
                               ctx->stream));
    HIPCHK(ctx, hipMemcpyAsync(counts, mesh->d_onq, sizeof(int32_t) * nt, hipMemcpyDeviceToHost,
                               ctx->stream));
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
  }
  // entries past each panel's count are not part of the rule
  for (int64_t i = 0; i < nt; ++i)
    for (int64_t q = counts[i]; q < maxq; ++q) {
      weights[i * maxq + q] = 0.0;
      for (int c = 0; c < 4; ++c) pts[(i * maxq + q) * 4 + c] = 0.0;
    }
  return STB_OK;
}

stb_status stb_solve_gmres(stb_ctx* ctx, const stb_mat* A, const double* b_host, double* x_host,
                           int32_t restart, int32_t maxit, double rtol, int32_t* iters, double* relres) {
  if (!ctx || !A || !b_host || !x_host) return stb_fail(ctx, STB_E_INVALID_ARG, "NULL argument");
  if (A->ncols != 0 && A->ncols != A->n)
    return stb_fail(ctx, STB_E_INVALID_ARG, "GMRES needs the square matrix of a whole mesh");
  if (restart < 1 || restart > 512 || maxit < 1 || !(rtol > 0.0))
    return stb_fail(ctx, STB_E_INVALID_ARG, "restart in [1,512], maxit >= 1 and rtol > 0 required");
  HIPCHK(ctx, hipSetDevice(ctx->device));
  const int64_t n = A->n;
  const int m = restart;
  hipStream_t st = ctx->stream;
  if (iters) *iters = 0;
  if (relres) *relres = 0.0;
  if (n == 0) return STB_OK;
  // the basis is a block lent by the context; the rest is one allocation
  const unsigned g = (unsigned)((n + kSolveThreads - 1) / kSolveThreads);
  const int64_t nch = (n + kGsChunk - 1) / kGsChunk;
  const size_t need = (size_t)(3 * n + (m + 1) * nch + g + 3 * (m + 1));
  double *V = nullptr, *buf = nullptr;
  auto cleanup = [&]() { ctx_keep(ctx, V); ctx_keep(ctx, buf); };
  if (kalloc(ctx, &V, (size_t)(m + 1) * n) != hipSuccess || kalloc(ctx, &buf, need) != hipSuccess) {
    cleanup();
    return stb_fail(ctx, STB_E_NO_MEMORY, "GMRES basis of %d vectors of %lld", m + 1, (long long)n);
  }
  double *w = buf, *b = w + n, *x = b + n, *part = x + n, *npart = part + (m + 1) * nch, *h1 = npart + g,
         *h2 = h1 + (m + 1), *yd = h2 + (m + 1);
  stb_status s = STB_OK;
  hipError_t e = hipSuccess;
  if (!ctx->h_pin) e = hipHostMalloc((void**)&ctx->h_pin, sizeof(double) * kPinDoubles);
  double* host = ctx->h_pin;
  static_assert(kPinDoubles >= 1 + 2 * kMaxBasis, "a step's coefficients fit the pinned block");
  if (e == hipSuccess) e = hipMemcpyAsync(b, b_host, sizeof(double) * n, hipMemcpyHostToDevice, st);
  if (e == hipSuccess) e = hipMemcpyAsync(x, x_host, sizeof(double) * n, hipMemcpyHostToDevice, st);
  if (e != hipSuccess) { cleanup(); return stb_fail(ctx, STB_E_DEVICE, "GMRES copy: %s", hipGetErrorString(e)); }
  // |u|^2 to the host and u / |u| to `out`
  auto normalise = [&](const double* u, double* out, double* n2) -> stb_status {
    hipLaunchKernelGGL(k_norm2, dim3(g), dim3(kSolveThreads), 0, st, n, u, npart);
    hipLaunchKernelGGL(k_gs_scale, dim3(g), dim3(kSolveThreads), 0, st, n, (int64_t)g, npart, u, out, 0, h1, h2, host);
    hipError_t ee = hipGetLastError();
    if (ee == hipSuccess) ee = hipStreamSynchronize(st);
    *n2 = host[0];
    return ee == hipSuccess ? STB_OK : stb_fail(ctx, STB_E_DEVICE, "GMRES norm: %s", hipGetErrorString(ee));
  };
  double bnorm2 = 0.0;
  if ((s = normalise(b, V, &bnorm2))) { cleanup(); return s; }
  const double bnorm = std::sqrt(bnorm2);
  if (bnorm == 0.0) {
    for (int64_t i = 0; i < n; ++i) x_host[i] = 0.0;
    cleanup();
    return STB_OK;
  }
  std::vector<double> H((size_t)(m + 1) * m, 0.0), cs(m), sn(m), gv(m + 1), y(m);
  int total = 0;
  double res = 0.0;
  for (;;) {
    // r = b - A x, V_0 = r / |r|
    if ((s = stb_apply_dev(ctx, A, 1, x, w, st))) break;
    hipLaunchKernelGGL(k_residual, dim3(g), dim3(256), 0, st, n, b, w);
    double rn2 = 0.0;
    if ((s = normalise(w, V, &rn2))) break;
    const double rn = std::sqrt(rn2);
    res = rn / bnorm;
    if (res <= rtol || total >= maxit) break;
    std::fill(gv.begin(), gv.end(), 0.0);
    gv[0] = rn;
    int j = 0;
    bool ahead = false;   // the product A V_j is already enqueued
    for (; j < m && total < maxit; ++j, ++total) {
      double* vj1 = V + (int64_t)(j + 1) * n;
      if (!ahead && (s = stb_apply_dev(ctx, A, 1, V + (int64_t)j * n, vj1, st))) break;
      // classical Gram-Schmidt, twice, then the norm and V_{j+1}
      const int k = j + 1;
      const dim3 gd((unsigned)nch, (unsigned)((k + kSolveThreads / 64 - 1) / (kSolveThreads / 64)));
      for (int pass = 0; pass < 2; ++pass) {
        hipLaunchKernelGGL(k_gs_dots, gd, dim3(kSolveThreads), 0, st, n, k, V, vj1, part);
        hipLaunchKernelGGL(k_gs_sub, dim3(g), dim3(kSolveThreads), 0, st, n, k, nch, V, part, vj1,
                           pass == 0 ? h1 : h2, pass == 0 ? nullptr : npart);
      }
      hipLaunchKernelGGL(k_gs_scale, dim3(g), dim3(kSolveThreads), 0, st, n, (int64_t)g, npart, vj1, vj1, k, h1, h2,
                         host);
      if ((e = hipGetLastError()) == hipSuccess) e = hipEventRecord(ctx->ev[4], st);
      // the next product runs while the host waits for this step's
      // coefficients (unused if the step turns out to be the last)
      ahead = j + 1 < m && total + 1 < maxit;
      if (e == hipSuccess && ahead) s = stb_apply_dev(ctx, A, 1, vj1, vj1 + n, st);
      if (e == hipSuccess) e = hipEventSynchronize(ctx->ev[4]);
      if (e != hipSuccess) s = stb_fail(ctx, STB_E_DEVICE, "GMRES step: %s", hipGetErrorString(e));
      if (s) break;
      const double hn2 = host[0];
      for (int i = 0; i <= j; ++i) H[(size_t)i * m + j] = host[1 + i] + host[1 + k + i];
      const double hn = std::sqrt(hn2);
      H[(size_t)(j + 1) * m + j] = hn;
      // apply the previous rotations, then a new one for row j + 1
      for (int i = 0; i < j; ++i) {
        const double a = H[(size_t)i * m + j], c = H[(size_t)(i + 1) * m + j];
        H[(size_t)i * m + j] = cs[i] * a + sn[i] * c;
        H[(size_t)(i + 1) * m + j] = -sn[i] * a + cs[i] * c;
      }
      const double a = H[(size_t)j * m + j], c = H[(size_t)(j + 1) * m + j];
      const double r = std::hypot(a, c);
      cs[j] = r > 0.0 ? a / r : 1.0;
      sn[j] = r > 0.0 ? c / r : 0.0;
      H[(size_t)j * m + j] = r;
      H[(size_t)(j + 1) * m + j] = 0.0;
      gv[j + 1] = -sn[j] * gv[j];
      gv[j] = cs[j] * gv[j];
      if (std::fabs(gv[j + 1]) <= rtol * bnorm || hn == 0.0) { ++j; ++total; break; }
    }
    if (s) break;
    // x += V y with H y = g (upper triangular, j columns)
    for (int i = j - 1; i >= 0; --i) {
      double t = gv[i];
      for (int k = i + 1; k < j; ++k) t -= H[(size_t)i * m + k] * y[k];
      y[i] = H[(size_t)i * m + i] != 0.0 ? t / H[(size_t)i * m + i] : 0.0;
    }
    e = hipMemcpyAsync(yd, y.data(), sizeof(double) * j, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) {
      hipLaunchKernelGGL(k_combine, dim3(g), dim3(kSolveThreads), 0, st, n, j, V, yd, x);
      e = hipGetLastError();
    }
    if (e != hipSuccess) { s = stb_fail(ctx, STB_E_DEVICE, "GMRES: %s", hipGetErrorString(e)); break; }
  }
  if (s == STB_OK) {
    e = hipMemcpyAsync(x_host, x, sizeof(double) * n, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) s = stb_fail(ctx, STB_E_DEVICE, "GMRES copy: %s", hipGetErrorString(e));
  } else {
    (void)hipStreamSynchronize(st);   // nothing enqueued may outlive the buffers
  }
  cleanup();
  if (s) return s;
  if (iters) *iters = total;
  if (relres) *relres = res;
  return STB_OK;
}

stb_status stb_solve_mot(stb_ctx* ctx, const stb_mesh* mesh, const stb_mat* A, const double* b_host,
                         double* x_host, double* info4) {
  if (!ctx || !mesh || !A || !b_host || !x_host) return stb_fail(ctx, STB_E_INVALID_ARG, "NULL argument");
  if (mesh->ctx != ctx || A->ctx != ctx)
    return stb_fail(ctx, STB_E_INVALID_ARG, "mesh or matrix of another context");
  if ((A->ncols != 0 && A->ncols != A->n) || A->n != mesh->nt)
    return stb_fail(ctx, STB_E_INVALID_ARG, "marching-on-in-time needs the square matrix of this mesh");
  HIPCHK(ctx, hipSetDevice(ctx->device));
  const int64_t nt = mesh->nt, nv = mesh->nv;
  if (nt == 0) return STB_OK;
  hipStream_t st = ctx->stream;
  // ---- the slab structure, from the vertex times (host)
  std::vector<double> vtx((size_t)nv * 4);
  std::vector<int32_t> tet((size_t)nt * 4);
  HIPCHK(ctx, hipStreamSynchronize(st));
  HIPCHK(ctx, hipMemcpy(vtx.data(), mesh->d_vtx, sizeof(double) * 4 * nv, hipMemcpyDeviceToHost));
  HIPCHK(ctx, hipMemcpy(tet.data(), mesh->d_tet, sizeof(int32_t) * 4 * nt, hipMemcpyDeviceToHost));
  std::vector<double> tv((size_t)nv);
  double tscale = 0.0, xscale = 0.0;
  for (int64_t v = 0; v < nv; ++v) {
    tv[(size_t)v] = vtx[(size_t)v * 4];
    tscale = std::max(tscale, std::fabs(vtx[(size_t)v * 4]));
    for (int c = 1; c < 4; ++c) xscale = std::max(xscale, std::fabs(vtx[(size_t)v * 4 + c]));
  }
  const double ttol = 1e-12 * std::max(tscale, 1.0), xtol = 1e-12 * std::max(xscale, 1.0);
  std::sort(tv.begin(), tv.end());
  std::vector<double> lev;
  for (double t : tv)
    if (lev.empty() || t - lev.back() > ttol) lev.push_back(t);
  const int64_t S = (int64_t)lev.size() - 1;
  if (S < 1) return stb_fail(ctx, STB_E_INVALID_ARG, "no time slabs");
  const double dt = lev[1] - lev[0];
  for (int64_t n = 1; n < S; ++n)
    if (std::fabs((lev[(size_t)n + 1] - lev[(size_t)n]) - dt) > 1e-9 * dt)
      return stb_fail(ctx, STB_E_INVALID_ARG,
                      "time levels are not uniform (slab %lld): use GMRES", (long long)n);
  auto level_of = [&](double t) -> int64_t {
    const int64_t n = (int64_t)(std::lower_bound(lev.begin(), lev.end(), t - ttol) - lev.begin());
    return (n <= S && std::fabs(lev[(size_t)n] - t) <= ttol) ? n : -1;
  };
  std::vector<int32_t> slab((size_t)nt), loc((size_t)nt);
  std::vector<std::vector<int32_t>> rows((size_t)S);
  for (int64_t i = 0; i < nt; ++i) {
    int64_t lo = S + 1, hi = -1;
    for (int k = 0; k < 4; ++k) {
      const int64_t l = level_of(vtx[(size_t)tet[(size_t)i * 4 + k] * 4]);
      if (l < 0) return stb_fail(ctx, STB_E_INTERNAL, "vertex time off the levels");
      lo = std::min(lo, l);
      hi = std::max(hi, l);
    }
    if (hi != lo + 1)
      return stb_fail(ctx, STB_E_INVALID_ARG,
                      "panel %lld does not span exactly one slab between two time levels: use GMRES",
                      (long long)i);
    slab[(size_t)i] = (int32_t)lo;
    loc[(size_t)i] = (int32_t)rows[(size_t)lo].size();
    rows[(size_t)lo].push_back((int32_t)i);
  }
  const int64_t K = (int64_t)rows[0].size();
  for (int64_t n = 1; n < S; ++n)
    if ((int64_t)rows[(size_t)n].size() != K)
      return stb_fail(ctx, STB_E_INVALID_ARG, "slab %lld has %lld panels, slab 0 has %lld: use GMRES",
                      (long long)n, (long long)rows[(size_t)n].size(), (long long)K);
  static_assert(kMotMaxPanels == 16384, "the limit the interface states");
  if (K > kMotMaxPanels) return stb_fail(ctx, STB_E_INVALID_ARG, "%lld panels per slab (at most 16384)", (long long)K);
  // slab n must be slab 0 moved by (lev_n - lev_0) in time, panel by panel
  for (int64_t n = 1; n < S; ++n) {
    const double shift = lev[(size_t)n] - lev[0];
    for (int64_t k = 0; k < K; ++k) {
      const int32_t p = rows[(size_t)n][(size_t)k], q = rows[0][(size_t)k];
      for (int v = 0; v < 4; ++v) {
        const double* X = &vtx[(size_t)tet[(size_t)p * 4 + v] * 4];
        const double* Y = &vtx[(size_t)tet[(size_t)q * 4 + v] * 4];
        bool same = std::fabs(X[0] - Y[0] - shift) <= ttol;
        for (int c = 1; c < 4; ++c) same = same && std::fabs(X[c] - Y[c]) <= xtol;
        if (!same)
          return stb_fail(ctx, STB_E_INVALID_ARG,
                          "slab %lld is not slab 0 moved in time (panel %d vs %d): use GMRES",
                          (long long)n, p, q);
      }
    }
  }
  // ---- device: structure check, inverse of the diagonal block, time steps
  std::vector<int32_t> rflat((size_t)(S * K));
  for (int64_t n = 0; n < S; ++n)
    std::copy(rows[(size_t)n].begin(), rows[(size_t)n].end(), rflat.begin() + n * K);
  int32_t *d_slab = nullptr, *d_loc = nullptr, *d_rows = nullptr;
  double *D = nullptr, *Dinv = nullptr, *x = nullptr, *b = nullptr, *r = nullptr;
  unsigned long long* d_bad = nullptr;
  auto cleanup = [&]() {
    dfree(d_slab); dfree(d_loc); dfree(d_rows); ctx_keep(ctx, D); ctx_keep(ctx, Dinv);
    dfree(x); dfree(b); dfree(r); dfree(d_bad);
  };
  if (dalloc(&d_slab, (size_t)nt) != hipSuccess || dalloc(&d_loc, (size_t)nt) != hipSuccess ||
      dalloc(&d_rows, (size_t)(S * K)) != hipSuccess || kalloc(ctx, &D, (size_t)(K * K)) != hipSuccess ||
      kalloc(ctx, &Dinv, (size_t)(K * K)) != hipSuccess || dalloc(&x, (size_t)nt) != hipSuccess ||
      dalloc(&b, (size_t)nt) != hipSuccess || dalloc(&r, (size_t)K) != hipSuccess || dalloc(&d_bad, 1) != hipSuccess) {
    cleanup();
    return stb_fail(ctx, STB_E_NO_MEMORY, "marching-on-in-time buffers (%lld panels per slab)", (long long)K);
  }
  hipError_t e = hipMemcpyAsync(d_slab, slab.data(), 4 * nt, hipMemcpyHostToDevice, st);
  if (e == hipSuccess) e = hipMemcpyAsync(d_loc, loc.data(), 4 * nt, hipMemcpyHostToDevice, st);
  if (e == hipSuccess) e = hipMemcpyAsync(d_rows, rflat.data(), 4 * S * K, hipMemcpyHostToDevice, st);
  if (e == hipSuccess) e = hipMemcpyAsync(b, b_host, 8 * nt, hipMemcpyHostToDevice, st);
  if (e == hipSuccess) e = hipMemsetAsync(d_bad, 0, 8, st);
  if (e == hipSuccess) e = hipMemsetAsync(D, 0, 8 * K * K, st);
  if (e == hipSuccess) e = hipMemsetAsync(x, 0, 8 * nt, st);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_mot_lower, dim3((unsigned)((nt * 64 + 255) / 256)), dim3(256), 0, st, nt, A->d_rowptr,
                       A->d_cols, d_slab, d_bad);
    hipLaunchKernelGGL(k_mot_block, dim3((unsigned)((K * 64 + 255) / 256)), dim3(256), 0, st, K, d_rows,
                       A->d_rowptr, A->d_cols, A->d_vals, d_slab, d_loc, D);
    e = hipGetLastError();
  }
  unsigned long long bad = 0;
  if (e == hipSuccess) e = hipMemcpyAsync(&bad, d_bad, 8, hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) { cleanup(); return stb_fail(ctx, STB_E_DEVICE, "marching-on-in-time: %s", hipGetErrorString(e)); }
  if (bad) {
    cleanup();
    return stb_fail(ctx, STB_E_INVALID_ARG,
                    "%llu stored entries couple a slab to a later one (not lower triangular in time): use GMRES",
                    bad);
  }
  const auto c0 = std::chrono::steady_clock::now();
  const stb_status s = stb_gj_invert(ctx, K, D, Dinv);
  if (s) { cleanup(); return s; }
  const auto c1 = std::chrono::steady_clock::now();
  const unsigned gw = (unsigned)((K * 64 + 255) / 256);
  for (int64_t n = 0; n < S && e == hipSuccess; ++n) {
    hipLaunchKernelGGL(k_mot_rhs, dim3((unsigned)K), dim3(256), 0, st, K, d_rows + n * K, A->d_rowptr, A->d_cols,
                       A->d_vals, x, b, r);
    hipLaunchKernelGGL(k_mot_apply, dim3(gw), dim3(256), 0, st, K, d_rows + n * K, Dinv, r, x);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemcpyAsync(x_host, x, 8 * nt, hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  const auto c2 = std::chrono::steady_clock::now();
  cleanup();
  if (e != hipSuccess) return stb_fail(ctx, STB_E_DEVICE, "marching-on-in-time: %s", hipGetErrorString(e));
  if (info4) {
    info4[0] = (double)S;
    info4[1] = (double)K;
    info4[2] = std::chrono::duration<double, std::milli>(c1 - c0).count();
    info4[3] = std::chrono::duration<double, std::milli>(c2 - c1).count();
  }
  return STB_OK;
}

}  // extern "C"
