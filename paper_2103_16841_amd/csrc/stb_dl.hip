// stb_dl.hip -- retarded double-layer potential (eq. dlp, kernels k2 and k3
// of eq. kfunc) of a density in V_h^1 (continuous, linear on every panel;
// def. st_be), at points off or on the surface.
//
// The candidates (point, panel) come from the single layer's cull and go
// through its pair pipeline (stb_pairs.hip) with the double layer's node
// kernels; here are the densities' coefficients per panel before it and the sums
// per point after it, in a fixed order.  stb_inner_values_D keeps one lane per
// pair (inner_dl_serial) for checks.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "stb_internal.h"
#include "stb_pairs.h"

using namespace stb;

namespace {

// nsign[j] = +1 where the given outward normal has a positive component along
// the frame normal n of panel j, -1 where negative; status 1 where the given
// normal is not finite or is within 60 degrees of the panel's plane.
__global__ void k_normal_sign(int64_t nt, const TrialRec* __restrict__ trial,
                              const double* __restrict__ nrm, double* __restrict__ nsign,
                              int32_t* __restrict__ status) {
  int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= nt) return;
  const double* g = nrm + 3 * j;
  const TrialRec& T = trial[j];
  double l = sqrt(g[0] * g[0] + g[1] * g[1] + g[2] * g[2]);
  double c = g[0] * T.n[0] + g[1] * T.n[1] + g[2] * T.n[2];
  bool ok = l > 0.0 && isfinite(l) && fabs(c) >= 0.5 * l;
  nsign[j] = c > 0.0 ? 1.0 : -1.0;
  status[j] = ok ? 0 : 1;
}

// The panels' linear densities from the vertex values v (kDlCoef doubles each,
// see PairJob::dl_coef).  The hat of vertex m is lambda_m = (h_m - a_m tau - b_m u -
// c_m v) / D_m over face m (opposite vertex m), D_m its value at vertex m.
__global__ void k_dl_coef(int64_t nt, const TrialRec* __restrict__ trial, const int32_t* __restrict__ tet,
                          const double* __restrict__ v, const double* __restrict__ nsign,
                          double* __restrict__ coef) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= nt) return;
  const TrialRec& T = trial[j];
  double* o = coef + kDlCoef * j;
  double gu = 0.0, gv = 0.0;
  for (int m = 0; m < 4; ++m) {
    const double Dm = T.fh[m] - T.fa[m] * T.V[m][0] - T.fb[m] * T.V[m][1] - T.fc[m] * T.V[m][2];
    const double a = v[tet[4 * j + m]] / Dm;
    o[m] = a;
    gu -= a * T.fb[m];
    gv -= a * T.fc[m];
  }
  o[4] = gu;
  o[5] = gv;
  o[6] = nsign[j];
  o[7] = 0.0;
}

// u(p) = sum over p's candidates: one wavefront per point, lane-strided partial
// sums and a fixed-order shuffle reduction.
__global__ __launch_bounds__(256) void k_dl_point_sum(int64_t np, const int64_t* __restrict__ rowptr,
                                                      const double* __restrict__ I, double* __restrict__ out) {
  const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (i >= np) return;
  double s = 0.0;
  for (int64_t c = rowptr[i] + lane; c < rowptr[i + 1]; c += 64) s += I[c];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if (lane == 0) out[i] = s;
}

__global__ void k_dl_pairs(int64_t k, const TrialRec* __restrict__ trial,
                           const FaceAng* __restrict__ fang, const double* __restrict__ nsign,
                           const double* __restrict__ pts, const int32_t* __restrict__ panel,
                           const double* __restrict__ gl, int ng, double* __restrict__ out4) {
  int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= k) return;
  const int32_t j = panel[m];
  double x4[4] = {pts[4 * m], pts[4 * m + 1], pts[4 * m + 2], pts[4 * m + 3]};
  double h[4];
  inner_dl_serial(trial[j], fang[j], x4, nsign[j], ng, gl, gl + kMaxNg, h);
  for (int q = 0; q < 4; ++q) out4[4 * m + q] = h[q];
}

// The points of entities [r0, r0 + nr) (faces), maxq slots each, packed
// without padding: point q of entity i goes to off[i] - off[r0] + q (off:
// exclusive prefix of the counts).
__global__ void k_pack_outer(int64_t r0, int64_t nr, int maxq, const double* __restrict__ opts,
                             const int64_t* __restrict__ off, double* __restrict__ pts) {
  int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= nr * maxq) return;
  const int64_t i = r0 + g / maxq;
  const int q = (int)(g % maxq);
  if (q >= off[i + 1] - off[i]) return;
  const double* src = opts + (i * maxq + q) * 4;
  double* dst = pts + (off[i] - off[r0] + q) * 4;
  for (int c = 0; c < 4; ++c) dst[c] = src[c];
}

// Sum of K v over each face's points: kf[f] = sum_q kv[off[f] - off[f0] + q]
// for faces [f0, f0 + nf) (off: exclusive prefix of the faces' counts).
__global__ void k_face_ksum(int64_t f0, int64_t nf, const int64_t* __restrict__ off,
                            const double* __restrict__ kv, double* __restrict__ kf) {
  int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= nf) return;
  const int64_t f = f0 + g;
  double s = 0.0;
  for (int64_t k = off[f]; k < off[f + 1]; ++k) s += kv[k - off[f0]];
  kf[f] = s;
}

// out[i] = sum_q w_iq (c_id v_h(x_iq) + (K v)(x_iq)): the energetic forms of
// eq. int_bform with A = I and A = K.  v_h at an outer point of panel i is
// panel i's own linear function: its hats are (h_m - a_m tau - b_m u -
// c_m v) / D_m in the local frame.  The K part comes per slot (face) of the
// panel: its per-point weight times the face's sum kf (the outer points of a
// face are the same for both panels that share it).
__global__ void k_dl_outer_sum(int64_t nt, int maxq, const TrialRec* __restrict__ trial,
                               const int32_t* __restrict__ tet, const double* __restrict__ v,
                               const double* __restrict__ opts, const double* __restrict__ ow,
                               const int32_t* __restrict__ onq, const int32_t* __restrict__ pf,
                               const double* __restrict__ pw, const double* __restrict__ kf,
                               double c_id, double* __restrict__ out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nt) return;
  const TrialRec& T = trial[i];
  double coef[4];
  for (int m = 0; m < 4; ++m) {
    const double Dm = T.fh[m] - T.fa[m] * T.V[m][0] - T.fb[m] * T.V[m][1] - T.fc[m] * T.V[m][2];
    coef[m] = v[tet[4 * i + m]] / Dm;
  }
  double id = 0.0;
  for (int q = 0; q < onq[i]; ++q) {
    const double* x = opts + (i * maxq + q) * 4;
    const double dx = x[1] - T.o[0], dy = x[2] - T.o[1], dz = x[3] - T.o[2];
    const double u = dx * T.e1[0] + dy * T.e1[1] + dz * T.e1[2];
    const double w = dx * T.e2[0] + dy * T.e2[1] + dz * T.e2[2];
    double vq = 0.0;
    for (int m = 0; m < 4; ++m) vq += coef[m] * (T.fh[m] - T.fa[m] * x[0] - T.fb[m] * u - T.fc[m] * w);
    id += ow[i * maxq + q] * vq;
  }
  double kk = 0.0;
  for (int k = 0; k < 4; ++k) {
    const int32_t f = pf[4 * i + k];
    if (f >= 0) kk += pw[4 * i + k] * kf[f];
  }
  out[i] = c_id * id + kk;
}

unsigned grid_for(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

}  // namespace

// Double-layer potential with device inputs and output on the context stream.
// coef: kDlCoef doubles per panel (k_dl_coef).
static stb_status dl_core(stb_ctx* ctx, stb_mesh* mesh, const stb_quad_params& p, const double* d_coef,
                          int64_t np, const double* d_pts, double* d_out) {
  stb_status s;
  if ((s = stb_ensure_gl(ctx, p.n_g))) return s;
  double* d_I = nullptr;
  int64_t* d_rowptr = nullptr;
  int32_t *d_cols = nullptr, *d_rowof = nullptr;
  auto cleanup = [&]() {
    ctx_keep(ctx, d_I); dfree(d_rowptr); ctx_keep(ctx, d_cols); ctx_keep(ctx, d_rowof);
  };
  int64_t nnz = 0;
  s = stb_cull_points(ctx, mesh, p, np, d_pts, &d_rowptr, &d_cols, &d_rowof, &nnz);
  if (s) { cleanup(); return s; }
  if (kalloc(ctx, &d_I, (size_t)nnz) != hipSuccess) {
    cleanup();
    return stb_fail(ctx, STB_E_NO_MEMORY, "double-layer candidates");
  }
  // the kernel times and path counts describe single-layer runs: kept as they are
  double ms[8];
  int64_t n[8], units[8], path[4];
  std::copy(ctx->kern_ms, ctx->kern_ms + 8, ms);
  std::copy(ctx->kern_n, ctx->kern_n + 8, n);
  std::copy(ctx->kern_units, ctx->kern_units + 8, units);
  std::copy(ctx->path_counts, ctx->path_counts + 4, path);
  PairJob J;
  J.nnz = nnz;
  J.rows = d_rowof;
  J.cols = d_cols;
  J.trial = mesh->d_trial;
  J.fang = mesh->d_fang;
  J.apex = d_pts;
  J.maxq = 1;
  J.gl = ctx->d_gl;
  J.ng = p.n_g;
  J.out = d_I;
  J.dl_coef = d_coef;
  unsigned long long work[4];
  s = stb_run_pairs(ctx, J, work);
  std::copy(ms, ms + 8, ctx->kern_ms);
  std::copy(n, n + 8, ctx->kern_n);
  std::copy(units, units + 8, ctx->kern_units);
  std::copy(path, path + 4, ctx->path_counts);
  if (s) { cleanup(); return s; }
  hipLaunchKernelGGL(k_dl_point_sum, dim3(grid_for(np * 64, 256)), dim3(256), 0, ctx->stream, np, d_rowptr, d_I,
                     d_out);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
  cleanup();
  ctx->work[0] = 0;
  ctx->work[1] = 0;
  ctx->work[2] = nnz;
  ctx->work[3] = 0;
  if (e != hipSuccess) return stb_fail(ctx, STB_E_DEVICE, "double layer failed: %s", hipGetErrorString(e));
  return STB_OK;
}

// The panels' densities for vertex values d_v, then f(coef).
template <class F>
static stb_status with_coef(stb_ctx* ctx, stb_mesh* mesh, const double* d_v, F f) {
  double* d_coef = nullptr;
  if (kalloc(ctx, &d_coef, (size_t)mesh->nt * kDlCoef) != hipSuccess)
    return stb_fail(ctx, STB_E_NO_MEMORY, "double-layer density");
  hipLaunchKernelGGL(k_dl_coef, dim3(grid_for(mesh->nt, 256)), dim3(256), 0, ctx->stream, mesh->nt, mesh->d_trial,
                     mesh->d_tet, d_v, mesh->d_nsign, d_coef);
  const hipError_t e = hipGetLastError();
  const stb_status s = e == hipSuccess ? f((const double*)d_coef)
                                       : stb_fail(ctx, STB_E_DEVICE, "double-layer density: %s", hipGetErrorString(e));
  (void)hipStreamSynchronize(ctx->stream);
  ctx_keep(ctx, d_coef);
  return s;
}

static stb_status dl_check(stb_ctx* ctx, const stb_mesh* mesh, const stb_quad_params* params,
                           stb_quad_params* p) {
  if (mesh->ctx != ctx) return stb_fail(ctx, STB_E_INVALID_ARG, "mesh belongs to another context");
  if (!mesh->d_nsign)
    return stb_fail(ctx, STB_E_INVALID_ARG, "the mesh has no outward normals (stb_mesh_set_normals)");
  *p = params ? *params : stb_default_params();
  return stb_check_params(ctx, p);
}

extern "C" {

stb_status stb_mesh_set_normals(stb_ctx* ctx, stb_mesh* mesh, const double* nrm) {
  if (!ctx || !mesh || !nrm) return stb_fail(ctx, STB_E_INVALID_ARG, "bad arguments");
  if (mesh->ctx != ctx) return stb_fail(ctx, STB_E_INVALID_ARG, "mesh belongs to another context");
  const int64_t nt = mesh->nt;
  if (nt == 0) return STB_OK;
  HIPCHK(ctx, hipSetDevice(ctx->device));
  double* d_n = nullptr;
  int32_t* d_st = nullptr;
  if (!mesh->d_nsign && dalloc(&mesh->d_nsign, (size_t)nt) != hipSuccess)
    return stb_fail(ctx, STB_E_NO_MEMORY, "normal signs");
  if (dalloc(&d_n, (size_t)nt * 3) != hipSuccess || dalloc(&d_st, (size_t)nt) != hipSuccess) {
    dfree(d_n); dfree(d_st);
    return stb_fail(ctx, STB_E_NO_MEMORY, "normals");
  }
  std::vector<int32_t> st((size_t)nt);
  hipError_t e = hipMemcpyAsync(d_n, nrm, sizeof(double) * 3 * nt, hipMemcpyHostToDevice, ctx->stream);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_normal_sign, dim3(grid_for(nt, 256)), dim3(256), 0, ctx->stream, nt,
                       mesh->d_trial, d_n, mesh->d_nsign, d_st);
    e = hipGetLastError();
  }
  if (e == hipSuccess)
    e = hipMemcpyAsync(st.data(), d_st, sizeof(int32_t) * nt, hipMemcpyDeviceToHost, ctx->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
  dfree(d_n);
  dfree(d_st);
  if (e != hipSuccess) return stb_fail(ctx, STB_E_DEVICE, "normals failed: %s", hipGetErrorString(e));
  for (int64_t j = 0; j < nt; ++j)
    if (st[j]) {
      dfree(mesh->d_nsign);
      mesh->d_nsign = nullptr;
      return stb_fail(ctx, STB_E_INVALID_ARG,
                      "normal of panel %lld is not finite or not transversal to the panel's plane",
                      (long long)j);
    }
  return STB_OK;
}

stb_status stb_potential_D(stb_ctx* ctx, const stb_mesh* mesh_c, const stb_quad_params* params,
                           const double* v, int64_t np, const double* pts, double* out) {
  if (!ctx || !mesh_c || !v || (np > 0 && (!pts || !out)) || np < 0)
    return stb_fail(ctx, STB_E_INVALID_ARG, "bad arguments");
  stb_mesh* mesh = const_cast<stb_mesh*>(mesh_c);
  stb_quad_params p;
  stb_status s = dl_check(ctx, mesh, params, &p);
  if (s) return s;
  if (np == 0) return STB_OK;
  for (int64_t i = 0; i < 4 * np; ++i)
    if (!std::isfinite(pts[i]))
      return stb_fail(ctx, STB_E_INVALID_ARG, "non-finite point %lld", (long long)(i / 4));
  HIPCHK(ctx, hipSetDevice(ctx->device));
  double *d_pts = nullptr, *d_v = nullptr, *d_out = nullptr;
  if (dalloc(&d_pts, (size_t)np * 4) != hipSuccess || dalloc(&d_v, (size_t)mesh->nv) != hipSuccess ||
      dalloc(&d_out, (size_t)np) != hipSuccess) {
    dfree(d_pts); dfree(d_v); dfree(d_out);
    return stb_fail(ctx, STB_E_NO_MEMORY, "double-layer buffers");
  }
  hipError_t e = hipMemcpyAsync(d_pts, pts, sizeof(double) * 4 * np, hipMemcpyHostToDevice, ctx->stream);
  if (e == hipSuccess) e = hipMemcpyAsync(d_v, v, sizeof(double) * mesh->nv, hipMemcpyHostToDevice, ctx->stream);
  s = e == hipSuccess ? with_coef(ctx, mesh, d_v,
                                  [&](const double* c) { return dl_core(ctx, mesh, p, c, np, d_pts, d_out); })
                      : stb_fail(ctx, STB_E_DEVICE, "copy failed");
  if (s == STB_OK) {
    e = hipMemcpy(out, d_out, sizeof(double) * np, hipMemcpyDeviceToHost);
    if (e != hipSuccess) s = stb_fail(ctx, STB_E_DEVICE, "copy back failed: %s", hipGetErrorString(e));
  }
  dfree(d_pts); dfree(d_v); dfree(d_out);
  return s;
}

stb_status stb_potential_D_dev(stb_ctx* ctx, const stb_mesh* mesh_c, const stb_quad_params* params,
                               const double* v_dev, int64_t np, const double* pts_dev, double* out_dev,
                               void* stream) {
  if (!ctx || !mesh_c || !v_dev || (np > 0 && (!pts_dev || !out_dev)) || np < 0)
    return stb_fail(ctx, STB_E_INVALID_ARG, "bad arguments");
  stb_mesh* mesh = const_cast<stb_mesh*>(mesh_c);
  stb_quad_params p;
  stb_status s = dl_check(ctx, mesh, params, &p);
  if (s) return s;
  if (np == 0) return STB_OK;
  HIPCHK(ctx, hipSetDevice(ctx->device));
  if (stream) HIPCHK(ctx, hipStreamSynchronize((hipStream_t)stream));
  return with_coef(ctx, mesh, v_dev,
                   [&](const double* c) { return dl_core(ctx, mesh, p, c, np, pts_dev, out_dev); });
}

// Face points per chunk of the energetic form (candidates are about 1e3-1e4
// per point: a chunk's candidate lists stay within a few GB).
constexpr int64_t kDlChunkPoints = 32768;

stb_status stb_dl_energetic(stb_ctx* ctx, const stb_mesh* mesh_c, const stb_quad_params* params,
                            const double* v, double c_id, double* out) {
  if (!ctx || !mesh_c || !v || !out || !std::isfinite(c_id))
    return stb_fail(ctx, STB_E_INVALID_ARG, "bad arguments");
  stb_mesh* mesh = const_cast<stb_mesh*>(mesh_c);
  stb_quad_params p;
  stb_status s = dl_check(ctx, mesh, params, &p);
  if (s) return s;
  const int64_t nt = mesh->nt;
  if (nt == 0) return STB_OK;
  HIPCHK(ctx, hipSetDevice(ctx->device));
  if ((s = stb_ensure_outer(ctx, mesh, p.m_q))) return s;
  if ((s = stb_ensure_faces(ctx, mesh, p.m_q))) return s;
  const int maxq = mesh->maxq, fq = p.m_q * p.m_q;
  const int64_t nf = mesh->nf;
  std::vector<int32_t> nq((size_t)std::max<int64_t>(nf, 1));
  std::vector<int64_t> off((size_t)nf + 1, 0);
  if (nf > 0) {
    HIPCHK(ctx, hipMemcpyAsync(nq.data(), mesh->d_fnq, sizeof(int32_t) * nf, hipMemcpyDeviceToHost,
                               ctx->stream));
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
  }
  for (int64_t f = 0; f < nf; ++f) off[f + 1] = off[f] + nq[f];
  double *d_v = nullptr, *d_out = nullptr, *d_pts = nullptr, *d_kv = nullptr, *d_kf = nullptr;
  int64_t* d_off = nullptr;
  const int64_t cap = std::max<int64_t>(kDlChunkPoints, fq);
  auto cleanup = [&]() { dfree(d_v); dfree(d_out); dfree(d_pts); dfree(d_kv); dfree(d_kf); dfree(d_off); };
  if (dalloc(&d_v, (size_t)mesh->nv) != hipSuccess || dalloc(&d_out, (size_t)nt) != hipSuccess ||
      dalloc(&d_pts, (size_t)cap * 4) != hipSuccess || dalloc(&d_kv, (size_t)cap) != hipSuccess ||
      dalloc(&d_kf, (size_t)std::max<int64_t>(nf, 1)) != hipSuccess ||
      dalloc(&d_off, (size_t)nf + 1) != hipSuccess) {
    cleanup();
    return stb_fail(ctx, STB_E_NO_MEMORY, "double-layer energetic buffers");
  }
  hipError_t e = hipMemcpyAsync(d_v, v, sizeof(double) * mesh->nv, hipMemcpyHostToDevice, ctx->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(d_off, off.data(), sizeof(int64_t) * (nf + 1), hipMemcpyHostToDevice, ctx->stream);
  if (e != hipSuccess) { cleanup(); return stb_fail(ctx, STB_E_DEVICE, "copy failed"); }
  // K v at every distinct face point, in chunks of faces
  int64_t cand = 0;
  s = with_coef(ctx, mesh, d_v, [&](const double* d_coef) -> stb_status {
    for (int64_t f0 = 0; f0 < nf;) {
      int64_t f1 = f0 + 1;
      while (f1 < nf && off[f1 + 1] - off[f0] <= cap) ++f1;
      const int64_t nfc = f1 - f0, np = off[f1] - off[f0];
      hipLaunchKernelGGL(k_pack_outer, dim3(grid_for(nfc * fq, 256)), dim3(256), 0, ctx->stream, f0, nfc, fq,
                         mesh->d_fpts, d_off, d_pts);
      HIPCHK(ctx, hipGetLastError());
      if (np > 0) {
        const stb_status q = dl_core(ctx, mesh, p, d_coef, np, d_pts, d_kv);
        if (q) return q;
        cand += ctx->work[2];
      }
      hipLaunchKernelGGL(k_face_ksum, dim3(grid_for(nfc, 256)), dim3(256), 0, ctx->stream, f0, nfc, d_off, d_kv,
                         d_kf);
      HIPCHK(ctx, hipGetLastError());
      f0 = f1;
    }
    return STB_OK;
  });
  if (s) { cleanup(); return s; }
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_dl_outer_sum, dim3(grid_for(nt, 128)), dim3(128), 0, ctx->stream, nt, maxq,
                       mesh->d_trial, mesh->d_tet, d_v, mesh->d_opts, mesh->d_ow, mesh->d_onq, mesh->d_pf,
                       mesh->d_pw, d_kf, c_id, d_out);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemcpyAsync(out, d_out, sizeof(double) * nt, hipMemcpyDeviceToHost, ctx->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
  cleanup();
  ctx->work[2] = cand;
  if (e != hipSuccess) return stb_fail(ctx, STB_E_DEVICE, "double-layer energetic form failed: %s",
                                       hipGetErrorString(e));
  return STB_OK;
}

stb_status stb_inner_values_D(stb_ctx* ctx, const stb_mesh* mesh, const stb_quad_params* params,
                              int64_t k, const double* pts, const int32_t* panel, double* out) {
  if (!ctx || !mesh || k < 0 || (k > 0 && (!pts || !panel || !out)))
    return stb_fail(ctx, STB_E_INVALID_ARG, "bad arguments");
  stb_quad_params p;
  stb_status s = dl_check(ctx, mesh, params, &p);
  if (s) return s;
  for (int64_t m = 0; m < k; ++m)
    if (panel[m] < 0 || panel[m] >= mesh->nt)
      return stb_fail(ctx, STB_E_INVALID_ARG, "panel index %d out of range", panel[m]);
  if (k == 0) return STB_OK;
  HIPCHK(ctx, hipSetDevice(ctx->device));
  if ((s = stb_ensure_gl(ctx, p.n_g))) return s;
  double *d_pts = nullptr, *d_out = nullptr;
  int32_t* d_pan = nullptr;
  if (dalloc(&d_pts, (size_t)k * 4) != hipSuccess || dalloc(&d_out, (size_t)k * 4) != hipSuccess ||
      dalloc(&d_pan, (size_t)k) != hipSuccess) {
    dfree(d_pts); dfree(d_out); dfree(d_pan);
    return stb_fail(ctx, STB_E_NO_MEMORY, "buffers");
  }
  hipError_t e = hipMemcpyAsync(d_pts, pts, 32 * k, hipMemcpyHostToDevice, ctx->stream);
  if (e == hipSuccess) e = hipMemcpyAsync(d_pan, panel, 4 * k, hipMemcpyHostToDevice, ctx->stream);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_dl_pairs, dim3(grid_for(k, 128)), dim3(128), 0, ctx->stream, k, mesh->d_trial,
                       mesh->d_fang, mesh->d_nsign, d_pts, d_pan, ctx->d_gl, p.n_g, d_out);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemcpyAsync(out, d_out, 32 * k, hipMemcpyDeviceToHost, ctx->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
  dfree(d_pts); dfree(d_out); dfree(d_pan);
  if (e != hipSuccess)
    return stb_fail(ctx, STB_E_DEVICE, "double-layer values failed: %s", hipGetErrorString(e));
  return STB_OK;
}

}  // extern "C"
