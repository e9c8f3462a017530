// stb_apply.hip -- multi right-hand-side product Y = A W (16 columns) on the
// CDNA4 matrix cores.  With 16 right-hand sides the product is a real GEMM
// over the sparse store: per block of 16 rows, the union of its rows'
// candidate columns is packed into quads, and each quad is one
// v_mfma_f32_16x16x4f32 step, A (16 rows x 4 columns, FP32) times W (4 rows x
// 16 right-hand sides, FP32) accumulated in FP32.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include "stb_internal.h"

typedef float f32x4 __attribute__((ext_vector_type(4)));

// MFMA 16x16x4 (FP32) operand layout:
//   A: lane l holds A[l % 16][l / 16];  B: lane l holds B[l / 16][l % 16];
//   D: lane l, register v holds D[4 (l / 16) + v][l % 16].
// One workgroup (eight wavefronts) per 16-row block: wavefronts v and v + 4
// take the block's quads v, v + 4, ..., the one the even and the other the odd
// ones of every eight, and the last cnt % 8 go to the even one.  Each has one
// MFMA chain; the partial tiles are summed in LDS in a fixed order.
//
// A quad's 64 values are stored without their zeros (two fifths are left of
// an icosphere's quads): a record has the mask of the lanes that have one, the
// place of the first and the four columns, and lane l's value is found by
// counting the mask's lower bits.  The zero lanes multiply 0, as they would
// from a full store, so the sums are those of the full quads.
//
// Bound by instructions (the products and the work to place the values): 30,720
// panels (2.7 million quads, 72 million entries) take 157 us, 132 us of them
// also without the loads of values and of W.  230 us with full quads (726 MB
// instead of 372) and four wavefronts per block that request eight quads at a
// time and wait; 205 us with the next group's loads ahead and the longest
// blocks first.
constexpr int kBellAhead = 8;   // quads per group of loads: 8 records of 8 words, a lane each

__global__ __launch_bounds__(512) void k_bell_mfma(int64_t nblk, int64_t n, int64_t ncols,
                                                   const int64_t* __restrict__ bptr,
                                                   const int64_t* __restrict__ rowptr,
                                                   const BellQuad* __restrict__ brec,
                                                   const float* __restrict__ bval,
                                                   const float* __restrict__ w32,
                                                   double* __restrict__ y) {
  // the last rows, which see the most columns of a causal matrix, first
  const int64_t blk = nblk - 1 - (int64_t)blockIdx.x;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int kk = lane >> 4, jj = lane & 15;
  const int str = wv & 3, odd = wv >> 2;   // the chain: stream of quads, half
  const int64_t q0 = bptr[blk], q1 = bptr[blk + 1];
  const int cnt = q1 > q0 + str ? (int)((q1 - q0 - str + 3) >> 2) : 0;   // quads of the stream
  const int half = (cnt >> 3) << 2;            // its whole eights, split evenly
  const int len = odd ? half : cnt - half;     // quads of the chain
  const int* const rec = reinterpret_cast<const int*>(brec + q0 + str + 4 * odd) + (lane & 7);
  const float* const val = bval + rowptr[blk * 16];
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  constexpr int U = kBellAhead;
  // word lane % 8 of the record of the group's quad lane / 8: quad 2 t + odd of
  // the stream while t < half, then quad half + t; past the end one without
  // values, of the zero row of W
  const int none = (lane & 4) ? (int)ncols : 0;
  auto ld_rec = [&](int g) {
    const int t = min(g * U + (lane >> 3), len - 1);
    return rec[(int64_t)(t < half ? 2 * t : half + t) * (4 * 8)];
  };
  auto past_end = [&](int w, int g) {
    const int in = -(int)(g * U + (lane >> 3) < len);
    return (w & in) | (none & ~in);
  };
  struct Group {
    float a[U], b[U];
    uint64_t m[U];
  };
  auto ld_group = [&](int r, Group& G) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t c = (uint32_t)__shfl(r, u * 8 + 4 + kk, 64);
      G.b[u] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(w32) + (c * 64u + jj * 4u));
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t lo = __builtin_amdgcn_readlane(r, u * 8), hi = __builtin_amdgcn_readlane(r, u * 8 + 1);
      const uint32_t off = __builtin_amdgcn_readlane(r, u * 8 + 2);
      G.m[u] = (uint64_t)hi << 32 | lo;
      // a lane without a value reads the next one's place (the store ends in a spare one)
      G.a[u] = (val + off)[__builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u))];
    }
  };
  const int groups = (len + U - 1) / U;
  Group G;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    G.a[u] = G.b[u] = 0.f;
    G.m[u] = 0ull;
  }
  auto products = [&](const Group& P) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_amdgcn_inverse_ballot_w64(P.m[u]) ? P.a[u] : 0.f, P.b[u], acc, 0, 0, 0);
  };
  // The next group's values and rows of W and, before them, the records after
  // it are under way while this group's products wait for theirs.  Two groups
  // by turns (a copy of one would wait for its loads), the first a group of
  // zeros (one that starts on loaded values has them loaded at the loop's head
  // again).
  if (len > 0) {
    int r0 = ld_rec(0);
    for (int g = -1;; g += 2) {
      Group N;
      const int r1 = ld_rec(g + 2);
      ld_group(past_end(r0, g + 1), N);
      __builtin_amdgcn_sched_barrier(0);
      products(G);
      __builtin_amdgcn_sched_barrier(0);
      r0 = ld_rec(g + 3);
      ld_group(past_end(r1, g + 2), G);
      __builtin_amdgcn_sched_barrier(0);
      products(N);
      __builtin_amdgcn_sched_barrier(0);
      if (g + 2 >= groups) break;
    }
  }
  __shared__ float part[8][4][64];
#pragma unroll
  for (int v = 0; v < 4; ++v) part[wv][v][lane] = acc[v];
  __syncthreads();
  if (wv != 0) return;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    float s[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) s[k] = part[k][v][lane] + part[4 + k][v][lane];
    const float t = ((s[0] + s[1]) + s[2]) + s[3];
    const int64_t row = blk * 16 + 4 * kk + v;
    if (row < n) y[row * 16 + jj] = (double)t;
  }
}

// W in FP32 with a row of zeros after the last one, for the quads' empty columns.
__global__ void k_to_f32(int64_t m, const double* __restrict__ a, float* __restrict__ b) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < m + 16) b[i] = i < m ? (float)a[i] : 0.f;
}

void stb_free_blocked(stb_mat* M) {
  dfree(M->d_bptr);
  dfree(M->d_brec);
  dfree(M->d_bval);
  M->d_bptr = nullptr;
  M->d_brec = nullptr;
  M->d_bval = nullptr;
  M->nblk = M->nquad = 0;
}

// Blocked copy, built on the device from the CSR: per 16-row block an LDS
// bitmap over the n columns marks the union of the rows' columns; its
// popcount prefix gives every column its slot, in column order.
constexpr int kBlkThreads = 256;
constexpr int64_t kMaxBlockedN = 262144;   // 2 x n/32 words of LDS <= 64 KiB

// Marks the columns of the block's rows, whose entries follow each other in the
// CSR: four loads per thread at once.
__device__ __forceinline__ void blk_mark(int64_t b, int64_t n, const int64_t* rowptr,
                                         const int32_t* cols, uint32_t* bits, int nw) {
  for (int w = threadIdx.x; w < nw; w += kBlkThreads) bits[w] = 0u;
  __syncthreads();
  const int64_t e = rowptr[(b + 1) * 16 < n ? (b + 1) * 16 : n];
  int64_t k = rowptr[b * 16] + threadIdx.x;
  auto mark = [&](int32_t c) { atomicOr(&bits[c >> 5], 1u << (c & 31)); };
  for (; k + 3 * kBlkThreads < e; k += 4 * kBlkThreads) {
    int32_t c[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) c[u] = cols[k + u * kBlkThreads];
#pragma unroll
    for (int u = 0; u < 4; ++u) mark(c[u]);
  }
  for (; k < e; k += kBlkThreads) mark(cols[k]);
  __syncthreads();
}

__global__ __launch_bounds__(kBlkThreads) void k_blk_count(int64_t nblk, int64_t n, int64_t ncols,
                                                           const int64_t* __restrict__ rowptr,
                                                           const int32_t* __restrict__ cols,
                                                           int64_t* __restrict__ nquad) {
  extern __shared__ uint32_t lds[];
  int64_t b = blockIdx.x;
  if (b >= nblk) return;
  int nw = (int)((ncols + 31) / 32);
  blk_mark(b, n, rowptr, cols, lds, nw);
  int c = 0;
  for (int w = threadIdx.x; w < nw; w += kBlkThreads) c += __popc(lds[w]);
  __shared__ int red[kBlkThreads];
  red[threadIdx.x] = c;
  __syncthreads();
  for (int off = kBlkThreads / 2; off > 0; off >>= 1) {
    if (threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) nquad[b] = (red[0] + 3) / 4;
}

// Slots per pass of the value fill: a tile of kFillQuads quads per wavefront in
// LDS, a quad's 64 values rotated by its number (the 64 entries that a wavefront
// scatters have neighbouring slots of one row, 16 values apart).
constexpr int kFillSlots = 512;
constexpr int kFillQuads = kFillSlots / 4 / (kBlkThreads / 64);
__device__ __forceinline__ int fill_at(int q, int l) { return q * 64 + ((l + q) & 63); }

// The block's slot of column c (c must be marked).
__device__ __forceinline__ int blk_slot(const uint32_t* bits, const int* pre, int32_t c) {
  return pre[c >> 5] + __popc(bits[c >> 5] & ((1u << (c & 31)) - 1u));
}

// Fills one block: column of every slot, then the values.  Slot s of row r is
// lane 16 (s % 4) + r of quad s / 4 (the MFMA A-operand order).  Per pass of
// kFillSlots slots a wavefront scatters the entries of its four rows into the tile
// (zero where a row lacks the column); then it takes kFillQuads quads into
// registers, leaves zeros in their place, and writes their masks and, after
// exchanging the wavefronts' counts, their values other than zero, one after the
// other from the block's first place in the CSR, which has at least as many.
//
// A row's entries go by in order, 64 at a time with the next 64 under way, so a
// pass waits for no load of its own and two barriers are all it has.  With a
// search for the rows' bounds per pass, all threads on one row at a time and the
// first thread's walk over the bitmap's 256 partial counts, the first product of
// a matrix of 960 panels took 108 us, of 3,840 panels 202 us, of 30,720 panels
// 1.33 ms; 87 us, 152 us and 0.92 ms so (95 us, 171 us, 1.30 ms when the quads
// were stored whole).
__global__ __launch_bounds__(kBlkThreads) void k_blk_fill(int64_t nblk, int64_t n, int64_t ncols,
                                                          const int64_t* __restrict__ rowptr,
                                                          const int32_t* __restrict__ cols,
                                                          const double* __restrict__ vals,
                                                          const int64_t* __restrict__ qptr,
                                                          BellQuad* __restrict__ brec,
                                                          float* __restrict__ bval) {
  extern __shared__ uint32_t lds[];
  constexpr int kWaves = kBlkThreads / 64, kRows = 16 / kWaves;
  __shared__ int wtot[kWaves];
  const int64_t b = blockIdx.x;
  if (b >= nblk) return;
  const int nw = (int)((ncols + 31) / 32);
  uint32_t* bits = lds;
  int* pre = reinterpret_cast<int*>(lds + nw);
  float* tile = reinterpret_cast<float*>(lds + 2 * nw);
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  blk_mark(b, n, rowptr, cols, bits, nw);
  // exclusive prefix of popcounts over the words: a chunk per thread
  const int per = (nw + kBlkThreads - 1) / kBlkThreads;
  const int w0 = min(nw, (int)threadIdx.x * per), w1 = min(nw, w0 + per);
  int acc = 0;
  for (int w = w0; w < w1; ++w) acc += __popc(bits[w]);
  int incl = acc;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int v = __shfl_up(incl, d, 64);
    if (lane >= d) incl += v;
  }
  if (lane == 63) wtot[wv] = incl;
  __syncthreads();
  int nslot = 0, run = incl - acc;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    if (w < wv) run += wtot[w];
    nslot += wtot[w];
  }
  for (int w = w0; w < w1; ++w) {
    pre[w] = run;
    run += __popc(bits[w]);
  }
  for (int e = threadIdx.x; e < kFillSlots * 16; e += kBlkThreads) tile[e] = 0.f;
  __syncthreads();
  const int64_t q0 = qptr[b], nq = qptr[b + 1] - q0;
  for (int w = threadIdx.x; w < nw; w += kBlkThreads) {
    uint32_t m = bits[w];
    int slot = pre[w];
    while (m) {
      int bit = __ffs(m) - 1;
      brec[q0 + (slot >> 2)].col[slot & 3] = w * 32 + bit;
      ++slot;
      m &= m - 1;
    }
  }
  for (int64_t k = nslot + threadIdx.x; k < nq * 4; k += kBlkThreads) brec[q0 + (k >> 2)].col[k & 3] = (int32_t)ncols;
  if (nslot == 0) return;
  // the wavefront's rows: entries [k, e) of the block's are still to be loaded; the
  // 64 at hand have their slots in sl (-1: none, or gone), the next are in nc, nv
  const int64_t rb = b * 16, lo = rowptr[rb];
  const int last = (int)(rowptr[rb + 16 < n ? rb + 16 : n] - lo) - 1;
  const int32_t* const bc = cols + lo;
  const double* const bv = vals + lo;
  float* const val = bval + lo;
  int k[kRows], e[kRows], sl[kRows];
  float va[kRows];
  int32_t nc[kRows];
  double nv[kRows];
  auto load = [&](int u) {
    const int i = min(k[u] + lane, last);
    nc[u] = bc[i];
    nv[u] = bv[i];
  };
  auto take = [&](int u) {
    sl[u] = k[u] + lane < e[u] ? blk_slot(bits, pre, nc[u]) : -1;
    va[u] = (float)nv[u];
    k[u] += 64;
    load(u);
  };
#pragma unroll
  for (int u = 0; u < kRows; ++u) {
    const int64_t row = rb + wv * kRows + u;
    k[u] = row < n ? (int)(rowptr[row] - lo) : 0;
    e[u] = row < n ? (int)(rowptr[row + 1] - lo) : 0;
    load(u);
  }
#pragma unroll
  for (int u = 0; u < kRows; ++u) take(u);
  uint32_t done = 0;   // values of the passes so far
  for (int s0 = 0; s0 < nslot; s0 += kFillSlots) {
#pragma unroll
    for (int u = 0; u < kRows; ++u)
      for (;;) {
        if ((unsigned)(sl[u] - s0) < (unsigned)kFillSlots) {
          const int s = sl[u] - s0;
          tile[fill_at(s >> 2, 16 * (s & 3) + wv * kRows + u)] = va[u];
          sl[u] = -1;
        }
        if (__any(sl[u] >= 0) || k[u] >= e[u]) break;
        take(u);
      }
    __syncthreads();
    const int nqs = (min(nslot - s0, kFillSlots) + 3) >> 2;   // whole quads: the last one's tail is zero
    float a[kFillQuads];
    uint64_t mine = 0;
    uint32_t mine_off = 0, cnt = 0;
#pragma unroll
    for (int i = 0; i < kFillQuads; ++i) {
      const int at = fill_at(wv * kFillQuads + i, lane);
      a[i] = tile[at];
      tile[at] = 0.f;
    }
#pragma unroll
    for (int i = 0; i < kFillQuads; ++i) {
      const uint64_t m = __ballot(a[i] != 0.f);
      if (lane == i) {
        mine = m;
        mine_off = cnt;
      }
      cnt += (uint32_t)__popcll(m);
    }
    if (lane == 0) wtot[wv] = (int)cnt;
    __syncthreads();
    uint32_t off = done;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      if (w < wv) off += (uint32_t)wtot[w];
      done += (uint32_t)wtot[w];
    }
    const int q = wv * kFillQuads + lane;
    if (lane < kFillQuads && q < nqs) {
      BellQuad& R = brec[q0 + (s0 >> 2) + q];
      R.mask = mine;
      R.off = off + mine_off;
      R.pad = 0u;
    }
#pragma unroll
    for (int i = 0; i < kFillQuads; ++i) {
      const uint64_t m = __ballot(a[i] != 0.f);
      if (a[i] != 0.f)
        val[off + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] = a[i];
      off += (uint32_t)__popcll(m);
    }
  }
}

// The matrix gets the copy only when all of it is there: d_bptr says that it is.
stb_status stb_build_blocked(stb_ctx* ctx, stb_mat* M, hipStream_t st) {
  const int64_t n = M->n, ncols = mat_ncols(M);
  if (ncols > kMaxBlockedN)
    return stb_fail(ctx, STB_E_INVALID_ARG, "16-RHS product supports n <= %lld", (long long)kMaxBlockedN);
  const int64_t nblk = (n + 15) / 16;
  size_t lds = sizeof(uint32_t) * 2 * (size_t)((ncols + 31) / 32);
  int64_t *d_nq = nullptr, *d_bptr = nullptr, nquad = 0;
  BellQuad* d_brec = nullptr;
  float* d_bval = nullptr;
  stb_free_blocked(M);
  auto fill = [&]() -> stb_status {
    HIPCHK(ctx, dalloc(&d_nq, (size_t)nblk));
    HIPCHK(ctx, dalloc(&d_bptr, (size_t)nblk + 1));
    hipLaunchKernelGGL(k_blk_count, dim3((unsigned)nblk), dim3(kBlkThreads), lds / 2, st, nblk, n, ncols,
                       M->d_rowptr, M->d_cols, d_nq);
    HIPCHK(ctx, hipGetLastError());
    stb_status s = stb_exclusive_scan(ctx, d_nq, d_bptr, nblk, st);
    if (s) return s;
    HIPCHK(ctx, hipMemcpy(&nquad, d_bptr + nblk, sizeof(int64_t), hipMemcpyDeviceToHost));
    HIPCHK(ctx, dalloc(&d_brec, (size_t)nquad));
    HIPCHK(ctx, dalloc(&d_bval, (size_t)M->nnz + 1));
    const size_t lds_fill = lds + sizeof(float) * 16 * kFillSlots;
    HIPCHK(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(&k_blk_fill),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_fill));
    hipLaunchKernelGGL(k_blk_fill, dim3((unsigned)nblk), dim3(kBlkThreads), lds_fill, st, nblk, n, ncols,
                       M->d_rowptr, M->d_cols, M->d_vals, d_bptr, d_brec, d_bval);
    HIPCHK(ctx, hipGetLastError());
    return STB_OK;
  };
  const stb_status s = fill();
  dfree(d_nq);
  if (s) {
    dfree(d_bptr); dfree(d_brec); dfree(d_bval);
    return s;
  }
  M->d_bptr = d_bptr;
  M->d_brec = d_brec;
  M->d_bval = d_bval;
  M->nblk = nblk;
  M->nquad = nquad;
  return STB_OK;
}

stb_status stb_apply16_dev(stb_ctx* ctx, stb_mat* M, const double* w, double* y, hipStream_t st) {
  if (!M->d_bptr) {
    stb_status s = stb_build_blocked(ctx, M, st);
    if (s) return s;
  }
  float* w32 = nullptr;
  HIPCHK(ctx, dalloc(&w32, ((size_t)mat_ncols(M) + 1) * 16));
  int64_t m = mat_ncols(M) * 16;
  if (m > 0) {
    hipLaunchKernelGGL(k_to_f32, dim3((unsigned)((m + 16 + 255) / 256)), dim3(256), 0, st, m, w, w32);
  }
  if (M->nblk > 0) {
    hipLaunchKernelGGL(k_bell_mfma, dim3((unsigned)M->nblk), dim3(512), 0, st, M->nblk, M->n, mat_ncols(M), M->d_bptr,
                       M->d_rowptr, M->d_brec, M->d_bval, w32, y);
  }
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  dfree(w32);
  if (e != hipSuccess) return stb_fail(ctx, STB_E_DEVICE, "16-RHS apply failed: %s", hipGetErrorString(e));
  return STB_OK;
}

// ------------------------------------------------ product without allocation
// stb_apply16_noalloc is the 16-RHS product for callers that cannot allocate
// device memory (code under HIP graph capture, tight serving loops, harnesses
// that forbid allocation): the FP32 copy of W, which stb_apply16_dev puts in
// a buffer of its own per call, goes to this file-scope array instead.  Each
// device the library runs on holds one copy (16 MiB) until the process ends;
// every call on a device shares it, so calls that overlap on one device race.
constexpr int64_t kNoAllocMaxCols = kMaxBlockedN;
static __device__ __align__(256) float scratch[(kNoAllocMaxCols + 1) * 16];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float* g_scratch_dev[kMaxDevices] = {};   // device address of scratch, per device
}  // namespace

// Called by stb_ctx_create with ctx's device current: looks up this device's
// address of the scratch array once.  In host code the array's name is only a
// stand-in; kernels get the address found here.
stb_status stb_noalloc_setup(stb_ctx* ctx) {
  if (ctx->device < 0 || ctx->device >= kMaxDevices)
    return stb_fail(ctx, STB_E_INVALID_ARG, "device %d: at most %d devices", ctx->device, kMaxDevices);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (g_scratch_dev[ctx->device]) return STB_OK;
  void* ptr = nullptr;
  hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !ptr)
    return stb_fail(ctx, STB_E_DEVICE, "scratch address: %s", hipGetErrorString(e));
  g_scratch_dev[ctx->device] = static_cast<float*>(ptr);
  return STB_OK;
}

extern "C" stb_status stb_apply16_noalloc(stb_ctx* ctx, const stb_mat* M, const double* w_dev,
                                          double* y_dev, void* stream) {
  if (!ctx || !M || !w_dev || !y_dev) return stb_fail(ctx, STB_E_INVALID_ARG, "NULL argument");
  if (M->ctx != ctx) return stb_fail(ctx, STB_E_INVALID_ARG, "matrix belongs to another context");
  const int64_t ncols = mat_ncols(M);
  if (ncols > kNoAllocMaxCols)
    return stb_fail(ctx, STB_E_INVALID_ARG, "%lld columns exceed the %lld of the allocation-free product",
                    (long long)ncols, (long long)kNoAllocMaxCols);
  if (!M->d_bptr && M->n > 0)
    return stb_fail(ctx, STB_E_INVALID_ARG,
                    "the matrix-core copy is not built: call stb_apply with nrhs = 16 once first");
  float* w32 = g_scratch_dev[ctx->device];
  if (!w32) return stb_fail(ctx, STB_E_INTERNAL, "scratch of device %d not set up", ctx->device);
  hipStream_t st = stream ? (hipStream_t)stream : ctx->stream;
  HIPCHK(ctx, hipSetDevice(ctx->device));
  const int64_t m = ncols * 16;
  if (m > 0)
    hipLaunchKernelGGL(k_to_f32, dim3((unsigned)((m + 16 + 255) / 256)), dim3(256), 0, st, m, w_dev, w32);
  if (M->nblk > 0)
    hipLaunchKernelGGL(k_bell_mfma, dim3((unsigned)M->nblk), dim3(512), 0, st, M->nblk, M->n, mat_ncols(M), M->d_bptr,
                       M->d_rowptr, M->d_brec, M->d_bval, (const float*)w32, y_dev);
  HIPCHK(ctx, hipGetLastError());
  return STB_OK;
}
