// Host side of the steps around the altGDmin loop (include/altgdmin.h):
// the mean image and the residual measurements of Algorithm 1, the automatic
// rank of Algorithm 2's parameter setting, and the modelling-error
// corrections of Algorithm 3 (MEC-1 by per-frame CGLS, MEC-2 by ISTA on the
// temporal DFT).  Every step is a launch sequence on the context's stream
// over a caller-provided auxiliary workspace.
#include <math.h>

#include <algorithm>
#include <mutex>
#include <vector>

#include "ctx.hpp"
#include "kernels_mri.hpp"

using ag_host::map_hip;

// The scratch of altgdmin_mean_noalloc (the CG vectors, the normal operator's
// coil images, the reduction partials and the CG scalars): one copy per GPU,
// held until the process ends.  Host code uses only the device address that
// hipGetSymbolAddress returns for the current device, never this name.
constexpr size_t kMeanScratchBytes = size_t(16) << 20;
static __device__ __align__(256) char scratch[kMeanScratchBytes];

namespace {

size_t al256(size_t v) { return (v + 255) & ~(size_t)255; }

// workgroups per system of the CG vector updates: about a thousand in all
int cg_nb(const altgdmin_ctx* c, int images) {
  return (int)std::max(1L, std::min({256L, ((long)c->n + 255) / 256, 1024L / images}));
}

// coil groups of the normal operator over `images` images: as many as bring
// the launch to about three workgroups per compute unit, each group's sum
// being one more part of the result to write and to add
int normal_groups(const altgdmin_ctx* c, int images, int* cgs) {
  const long tiles = (c->p.nx + op_tile(c->p.ny) - 1) / op_tile(c->p.ny);
  const int want = (int)std::max(1L, std::min<long>(c->p.nc, (768 + tiles * images - 1) / (tiles * images)));
  const int per = (c->p.nc + want - 1) / want;
  *cgs = per;
  return (c->p.nc + per - 1) / per;
}

// shares of ||A p||^2 per image that one application of the normal operator writes
int normal_ndot(const altgdmin_ctx* c, int groups) {
  const altgdmin_params& p = c->p;
  if (c->lines) return (p.nx + op_tile(p.ny) - 1) / op_tile(p.ny) * groups;
  return (p.nc * p.ny + op_tile(p.nx) - 1) / op_tile(p.nx);
}

// the auxiliary workspace, carved from its base
struct Aux {
  float2 *v0, *v1, *v2;  // n x q each
  float2* w;             // parts of an operator's result, one per coil group (v0 when there is one group)
  float2 *y0, *y1;       // q x nc x m_max each
  float2* ci;            // nc x n: coil images of the mean's normal operator
  double *part, *dot;    // reduction partials
  FrameCg* fc;           // two slots of q
  IstaState* is;         // two slots
  double* ipart[2];      // ISTA's partial sums, two buffers
  double* lam;           // 16
};

size_t aux_layout(const altgdmin_ctx* c, char* base, Aux* a) {
  const altgdmin_params& p = c->p;
  const size_t nq = sizeof(float2) * (size_t)c->n * p.q;
  const size_t ys = sizeof(float2) * (size_t)p.q * p.nc * p.m_max;
  const size_t tiles = (p.nx + op_tile(p.ny) - 1) / op_tile(p.ny);
  int cgs;
  const int g1 = normal_groups(c, 1, &cgs), gq = normal_groups(c, p.q, &cgs);
  const size_t nparts = std::max<size_t>({(size_t)cg_nb(c, 1), (size_t)p.q * cg_nb(c, p.q), (size_t)p.q * tiles});
  const size_t ndots = std::max<size_t>(normal_ndot(c, g1), (size_t)p.q * normal_ndot(c, gq));
  size_t off = 0;
  auto take = [&](size_t b) {
    size_t o = off;
    off = al256(off + b);
    return base ? base + o : nullptr;
  };
  Aux t{};
  t.v0 = reinterpret_cast<float2*>(take(nq));
  t.v1 = reinterpret_cast<float2*>(take(nq));
  t.v2 = reinterpret_cast<float2*>(take(nq));
  t.w = gq > 1 ? reinterpret_cast<float2*>(take(nq * gq)) : t.v0;
  t.y0 = reinterpret_cast<float2*>(take(ys));
  t.y1 = reinterpret_cast<float2*>(take(ys));
  t.ci = reinterpret_cast<float2*>(take(sizeof(float2) * (size_t)p.nc * c->n));
  t.part = reinterpret_cast<double*>(take(sizeof(double) * nparts));
  t.dot = reinterpret_cast<double*>(take(sizeof(double) * ndots));
  t.fc = reinterpret_cast<FrameCg*>(take(sizeof(FrameCg) * 2 * p.q));
  t.is = reinterpret_cast<IstaState*>(take(sizeof(IstaState) * 2));
  t.ipart[0] = reinterpret_cast<double*>(take(sizeof(double) * 2 * (size_t)(c->n / 64)));
  t.ipart[1] = reinterpret_cast<double*>(take(sizeof(double) * 2 * (size_t)(c->n / 64)));
  t.lam = reinterpret_cast<double*>(take(sizeof(double) * 16));
  if (a) *a = t;
  return off;
}

bool overlap(const float2* a, size_t an, const float2* b, size_t bn) { return a && b && a < b + bn && b < a + an; }

bool aux_ok(const void* d_aux) { return d_aux && (reinterpret_cast<uintptr_t>(d_aux) & 255) == 0; }


#define AGCHK(x)                     \
  do {                               \
    hipError_t _e = (x);             \
    if (_e != hipSuccess) return _e; \
  } while (0)

NormalArgs normal_args(altgdmin_ctx* c) {
  const altgdmin_params& p = c->p;
  NormalArgs a{};
  a.coils = c->coils;
  a.n = c->n;
  a.nx = p.nx;
  a.ny = p.ny;
  a.nc = p.nc;
  a.tw = c->at<float2>(c->o_twy);
  a.tw_x = c->at<float2>(c->o_twx);
  a.rows = c->mask;
  a.rows_img_stride = c->width;
  a.m_k = c->m_k;
  a.m_max = p.m_max;
  a.scale = (float)(1.0 / sqrt((double)p.ny));
  a.st = c->st();
  return a;
}

// the adjoint columns of one image's full k-space rows T, coil by coil, in place
hipError_t adj_cols_in_place(altgdmin_ctx* c, float2* T) {
  ColAdjArgs d = ag_host::col_adj_args(c, T, T);
  d.src_c_stride = c->n;
  d.src_img_stride = 0;
  d.rows = nullptr;
  d.cgs = 1;  // each workgroup writes the columns of the one coil image that it has read
  d.dst_part_stride = c->n;
  return launch_cols_adj(c->p.ny, d, false, 1, c->stream);
}

// The mean image by CG: s_0 = A^H y from the frames' sum per k-space location (FP64,
// in the workspace's temporary), then two launches per iteration (four for
// general masks).  Vectors: s in v0, the directions in v1 and v2, the coil
// groups' parts of A^H A p in ci.
hipError_t mean_seq(altgdmin_ctx* c, double tol, int maxit, float2* x, const Aux& a, int* it_slot) {
  const altgdmin_params& p = c->p;
  hipStream_t s = c->stream;
  const long n = c->n;
  DevState* st = c->st();
  double2* const T = c->at<double2>(c->o_T);  // nc coil images
  int per = 1;
  if (c->lines) {
    hipLaunchKernelGGL(k_line_sum, dim3(p.ny, p.nc), dim3(256), 0, s, c->at<float2>(c->o_yh),
                       c->at<int32_t>(c->o_locptr), p.nc, p.nx, T, st);
  } else {
    hipLaunchKernelGGL(k_loc_sum, dim3((unsigned)((n + 255) / 256), p.nc), dim3(256), 0, s, c->y,
                       c->at<int2>(c->o_pairs), c->at<int32_t>(c->o_locptr), n, p.nc, p.m_max, T, st);
    AGCHK(launch_rhs_rows(T, p.nx, p.nc * p.ny, st, s));
  }
  AGCHK(hipGetLastError());
  AGCHK(launch_rhs_cols(T, c->coils, p.nx, p.ny, p.nc, &per, st, s));
  const int nb = cg_nb(c, 1);
  hipLaunchKernelGGL(k_cg_begin, dim3(nb), dim3(256), 0, s, T, (p.nc + per - 1) / per, per * n, a.v0, x, n, a.part, st);
  AGCHK(hipGetLastError());
  int cgs = 1;
  const int groups = c->lines ? normal_groups(c, 1, &cgs) : p.nc;
  NormalArgs na = normal_args(c);
  na.s = a.v0;
  na.loc_ptr = c->at<int32_t>(c->o_locptr);
  na.cgs = cgs;
  na.w = na.T = a.ci;
  na.part_stride = n;
  na.dot = a.dot;
  CgArgs cg{};
  cg.nrm = a.part;
  cg.nnrm = nb;
  cg.tol = tol;
  CgStepArgs sa{};
  sa.w = a.ci;
  sa.x = x;
  sa.s = a.v0;
  sa.nsum = groups;
  sa.part_stride = n;
  sa.n = n;
  sa.dot = a.dot;
  sa.ndot = normal_ndot(c, groups);
  sa.nrm = a.part;
  sa.st = st;
  float2* const pv[2] = {a.v1, a.v2};
  for (int it = 0; it <= maxit; ++it) {
    cg.it = it;
    cg.in = a.fc + ((it + 1) & 1);
    cg.out = a.fc + (it & 1);
    if (it == maxit) {  // the last iteration's stop test, for the count
      if (it_slot) {
        hipLaunchKernelGGL(k_cg_end, dim3(1), dim3(64), 0, s, cg, st);
        *it_slot = it & 1;
      }
      break;
    }
    na.cg = cg;
    na.p_old = pv[(it + 1) & 1];
    na.p_new = pv[it & 1];
    if (c->lines) {
      AGCHK(launch_normal_lines(na, NORMAL_MEAN, 1, groups, s));
    } else {
      ColFwdArgs f = ag_host::col_fwd_args(c, a.v0, a.ci);
      f.p_old = na.p_old;
      f.p_new = na.p_new;
      f.cg = cg;
      AGCHK(launch_cols_fwd(p.ny, f, true, 1, s));
      AGCHK(launch_normal_rows(na, s));
      AGCHK(adj_cols_in_place(c, a.ci));
    }
    sa.p = na.p_new;
    sa.cg = cg.out;
    hipLaunchKernelGGL(k_cg_step, dim3(nb), dim3(256), 0, s, sa);
  }
  return hipGetLastError();
}

// MEC-1: CGLS for every frame, from e = 0.  Vectors: s in v0, the directions in
// v1 and v2, the residual r in y0 and A p in y1 (line masks: both after the
// inverse x transform, which is unitary on full-readout lines, so that the
// iterations need the y transforms alone).  An iteration is the forward
// columns (p = s + beta p, A p, its norm) and the adjoint columns (x += alpha p,
// r -= alpha A p, s = A^H r, its norm), with a row pass after and before them for
// general masks and a sum over coil groups where few frames leave the chip
// idle.
hipError_t cgls_frames(altgdmin_ctx* c, const float2* yres, int iters, double tol, float2* E, const Aux& a) {
  const altgdmin_params& p = c->p;
  hipStream_t s = c->stream;
  DevState* st = c->st();
  const long n = c->n;
  int cgs;
  const int groups = normal_groups(c, p.q, &cgs), nb = cg_nb(c, p.q);
  const int tiles = (p.nx + op_tile(p.ny) - 1) / op_tile(p.ny);
  float2* const T = c->at<float2>(c->o_T) + (size_t)n * p.q;  // general masks: kc frames of coil images
  if (c->lines) AGCHK(launch_rows(p.nx, ag_host::row_args(c, yres, a.y0), true, s));
  ColAdjArgs d = ag_host::col_adj_args(c, c->lines ? a.y0 : T, a.w);
  d.cgs = cgs;
  d.dst_part_stride = n * p.q;
  d.x = E;
  d.dot = a.dot;
  d.ndot = normal_ndot(c, groups);
  d.nrm = groups == 1 ? a.part : nullptr;
  if (c->lines) d.r = a.y0;
  ColFwdArgs f = ag_host::col_fwd_args(c, a.v0, c->lines ? a.y1 : T);
  f.pad_rows = 0;
  f.cgs = cgs;
  f.dot = c->lines ? a.dot : nullptr;
  f.cg.nrm = a.part;
  f.cg.nnrm = groups == 1 ? tiles : nb;
  f.cg.tol = tol;
  IndexRowArgs fr = ag_host::index_row_args(c, T), ar = fr;
  fr.y = a.y1;
  fr.dot = a.dot;
  ar.r = a.y0;
  ar.dot = a.dot;
  ar.ndot = d.ndot;
  const int kc = c->lines ? p.q : c->kc;
  float2* const pv[2] = {a.v1, a.v2};
  for (int it = -1; it < iters; ++it) {  // -1: the start, s = A^H yres and x = 0
    FrameCg* const slot = a.fc + (it & 1) * p.q;
    if (it >= 0) {
      f.cg.it = it;
      f.cg.in = a.fc + ((it + 1) & 1) * p.q;
      f.cg.out = slot;
      f.p_old = pv[(it + 1) & 1];
      f.p_new = pv[it & 1];
      fr.cg = slot;
      for (int k0 = 0; k0 < p.q; k0 += kc) {
        const int kn = std::min(kc, p.q - k0);
        f.img0 = fr.img0 = k0;
        AGCHK(launch_cols_fwd(p.ny, f, true, kn, s));
        if (!c->lines) AGCHK(launch_index_rows(p.nx, fr, IDX_FWD, true, kn, s));
      }
      d.p = f.p_new;
      d.q = c->lines ? a.y1 : nullptr;
      d.cg = ar.cg = slot;
      ar.q = a.y1;
    }
    d.first = it < 0;
    ar.yin = it <= 0 ? yres : a.y0;
    for (int k0 = 0; k0 < p.q; k0 += kc) {
      const int kn = std::min(kc, p.q - k0);
      d.img0 = ar.img0 = k0;
      if (!c->lines) AGCHK(launch_index_rows(p.nx, ar, IDX_ADJ, true, kn, s));
      AGCHK(launch_cols_adj(p.ny, d, true, kn, s));
    }
    if (groups > 1) {
      hipLaunchKernelGGL(k_cgls_sum, dim3(nb, p.q), dim3(256), 0, s, a.w, groups, n * p.q, a.v0, n, a.part,
                         it >= 0 ? slot : nullptr, st);
      AGCHK(hipGetLastError());
    }
  }
  return hipSuccess;
}

// MEC-2: ISTA on the temporal DFT, two launches per update (four for general
// masks).  Line masks: the hybrid data (after the inverse x transform) in y0.
hipError_t ista_frames(altgdmin_ctx* c, const float2* yres, int max_iter, double frac, double tol, float2* E,
                       const Aux& a, int* it_slot) {
  const altgdmin_params& p = c->p;
  hipStream_t s = c->stream;
  DevState* st = c->st();
  const long n = c->n;
  int cgs;
  const int groups = normal_groups(c, p.q, &cgs);
  hipLaunchKernelGGL(k_ista_begin, dim3(1024), dim3(256), 0, s, E, n * p.q, a.is);
  AGCHK(hipGetLastError());
  if (c->lines && max_iter > 0) AGCHK(launch_rows(p.nx, ag_host::row_args(c, yres, a.y0), true, s));
  NormalArgs na = normal_args(c);
  na.s = E;
  na.y = a.y0;
  na.w = a.w;
  na.part_stride = n * p.q;
  na.cgs = cgs;
  float2* const T = c->at<float2>(c->o_T) + (size_t)n * p.q;
  ColFwdArgs f = ag_host::col_fwd_args(c, E, T);
  IndexRowArgs ir = ag_host::index_row_args(c, T);
  ir.yin = yres;
  ColAdjArgs d = ag_host::col_adj_args(c, T, a.w);
  d.cgs = cgs;
  d.dst_part_stride = n * p.q;
  IstaArgs ia{};
  ia.E = E;
  ia.w = a.w;
  ia.nsum = groups;
  ia.part_stride = n * p.q;
  ia.M = a.v1;
  ia.n = n;
  ia.q = p.q;
  ia.scale = (float)(1.0 / sqrt((double)p.q));
  ia.frac = frac;
  ia.tol = tol;
  ia.st = st;
  for (int t = 0; t < max_iter; ++t) {
    ia.t = t;
    ia.in = a.is + ((t + 1) & 1);
    ia.out = a.is + (t & 1);
    // the newest scalars that are known: a stop found from update t - 1's
    // change only skips the launches after this operator
    na.ista = f.ista = ir.ista = d.ista = ia.in;
    if (c->lines) {
      AGCHK(launch_normal_lines(na, NORMAL_ISTA, p.q, groups, s));
    } else {
      for (int k0 = 0; k0 < p.q; k0 += c->kc) {
        const int kn = std::min(c->kc, p.q - k0);
        f.img0 = ir.img0 = d.img0 = k0;
        AGCHK(launch_cols_fwd(p.ny, f, false, kn, s));
        AGCHK(launch_index_rows(p.nx, ir, IDX_RES, false, kn, s));
        AGCHK(launch_cols_adj(p.ny, d, false, kn, s));
      }
    }
    if (t == 0) {
      ia.pout = a.ipart[0];
      AGCHK(launch_ista_dft(ia, ISTA_FIRST, s));
      ia.pin = a.ipart[0];
      AGCHK(launch_ista_dft(ia, ISTA_THRESH, s));
    } else {
      ia.pin = a.ipart[(t + 1) & 1];
      ia.pout = a.ipart[t & 1];
      AGCHK(launch_ista_dft(ia, ISTA_STEP, s));
    }
  }
  if (it_slot && max_iter > 0) {
    const int t = max_iter;
    hipLaunchKernelGGL(k_ista_end, dim3(1), dim3(64), 0, s, a.is + ((t + 1) & 1), a.is + (t & 1),
                       a.ipart[(t + 1) & 1], (int)(n / 64), t, tol, st);
    *it_slot = t & 1;
  }
  return hipGetLastError();
}

// ---- the no-allocation variant of the mean image ---------------------------
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// the scratch's device address on the current device (looked up once per device)
altgdmin_status scratch_address(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return ALTGDMIN_EHIP;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return ALTGDMIN_EHIP;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return ALTGDMIN_OK;
}

// the mean image's buffers carved from a base: three n-vectors, the coil
// images, the partials and the scalars; returns the bytes used
size_t mean_layout(const altgdmin_ctx* c, char* base, Aux* a) {
  size_t off = 0;
  auto take = [&](size_t b) {
    size_t o = off;
    off = al256(off + b);
    return base ? base + o : nullptr;
  };
  Aux t{};
  t.v0 = reinterpret_cast<float2*>(take(sizeof(float2) * (size_t)c->n));
  t.v1 = reinterpret_cast<float2*>(take(sizeof(float2) * (size_t)c->n));
  t.v2 = reinterpret_cast<float2*>(take(sizeof(float2) * (size_t)c->n));
  t.ci = reinterpret_cast<float2*>(take(sizeof(float2) * (size_t)c->p.nc * c->n));
  t.part = reinterpret_cast<double*>(take(sizeof(double) * cg_nb(c, 1)));
  int cgs;
  t.dot = reinterpret_cast<double*>(take(sizeof(double) * normal_ndot(c, normal_groups(c, 1, &cgs))));
  t.fc = reinterpret_cast<FrameCg*>(take(sizeof(FrameCg) * 2));
  if (a) *a = t;
  return off;
}

// the device error, if any, after a synchronisation
altgdmin_status sync_status(altgdmin_ctx* c) {
  if (hipStreamSynchronize(c->stream) != hipSuccess) return ALTGDMIN_EHIP;
  int32_t err = 0;
  if (hipMemcpy(&err, &c->st()->err, sizeof(int32_t), hipMemcpyDeviceToHost) != hipSuccess) return ALTGDMIN_EHIP;
  return (altgdmin_status)err;
}

}  // namespace

extern "C" {

altgdmin_status altgdmin_aux_bytes(const altgdmin_ctx* c, size_t* bytes) {
  if (!c || !bytes) return ALTGDMIN_EINVAL;
  *bytes = aux_layout(c, nullptr, nullptr);
  return ALTGDMIN_OK;
}

altgdmin_status altgdmin_mean(altgdmin_ctx* c, double tol, int32_t maxit, void* d_zbar, void* d_aux,
                              int32_t* h_iters) {
  if (!c || !d_zbar || !aux_ok(d_aux) || maxit < 0 || !(tol >= 0.0) || !isfinite(tol)) return ALTGDMIN_EINVAL;
  if (!c->bound || !c->y) return ALTGDMIN_ESTATE;
  Aux a;
  aux_layout(c, static_cast<char*>(d_aux), &a);
  int slot = 0;
  HIPCHK(mean_seq(c, tol, maxit, static_cast<float2*>(d_zbar), a, h_iters ? &slot : nullptr));
  if (h_iters) {
    const altgdmin_status e = sync_status(c);
    HIPCHK(hipMemcpy(h_iters, &a.fc[slot].iters, sizeof(int32_t), hipMemcpyDeviceToHost));
    if (e != ALTGDMIN_OK) return e;
  }
  return ALTGDMIN_OK;
}

altgdmin_status altgdmin_mean_noalloc(altgdmin_ctx* c, double tol, int32_t maxit, void* d_zbar, int32_t* h_iters) {
  if (!c || !d_zbar || maxit < 0 || !(tol >= 0.0) || !isfinite(tol)) return ALTGDMIN_EINVAL;
  if (mean_layout(c, nullptr, nullptr) > kMeanScratchBytes) return ALTGDMIN_ESCRATCH;
  if (!c->bound || !c->y) return ALTGDMIN_ESTATE;
  void* base = nullptr;
  const altgdmin_status s = scratch_address(&base);
  if (s != ALTGDMIN_OK) return s;
  Aux a;
  mean_layout(c, static_cast<char*>(base), &a);
  int slot = 0;
  HIPCHK(mean_seq(c, tol, maxit, static_cast<float2*>(d_zbar), a, h_iters ? &slot : nullptr));
  if (h_iters) {
    const altgdmin_status e = sync_status(c);
    HIPCHK(hipMemcpy(h_iters, &a.fc[slot].iters, sizeof(int32_t), hipMemcpyDeviceToHost));
    if (e != ALTGDMIN_OK) return e;
  }
  return ALTGDMIN_OK;
}

altgdmin_status altgdmin_residual(altgdmin_ctx* c, const void* d_zbar, const void* d_X, void* d_yres, void* d_aux) {
  if (!c || !d_yres || !aux_ok(d_aux)) return ALTGDMIN_EINVAL;
  if (!c->bound || !c->y) return ALTGDMIN_ESTATE;
  const altgdmin_params& p = c->p;
  const float2* X = static_cast<const float2*>(d_X);
  const float2* zbar = static_cast<const float2*>(d_zbar);
  float2* Y = static_cast<float2*>(d_yres);
  const size_t yn = (size_t)p.q * p.nc * p.m_max;
  if (overlap(Y, yn, X, (size_t)c->n * p.q) || overlap(Y, yn, zbar, c->n)) {
    // the images share memory with the output, which the passes write before
    // every image is read: z = X + zbar goes through the auxiliary workspace
    Aux a;
    aux_layout(c, static_cast<char*>(d_aux), &a);
    HIPCHK(launch_expand(nullptr, nullptr, zbar, X, (long)c->n, p.q, p.r, a.v0, c->st(), c->stream));
    X = a.v0;
    zbar = nullptr;
  }
  return map_hip(ag_host::forward_op(c, X, Y, zbar, c->y));
}

altgdmin_status altgdmin_mec_cgls(altgdmin_ctx* c, const void* d_yres, int32_t iters, double tol, void* d_E,
                                  void* d_aux) {
  if (!c || !d_yres || !d_E || !aux_ok(d_aux) || iters < 0 || !(tol >= 0.0)) return ALTGDMIN_EINVAL;
  if (!c->bound) return ALTGDMIN_ESTATE;
  Aux a;
  aux_layout(c, static_cast<char*>(d_aux), &a);
  return map_hip(cgls_frames(c, static_cast<const float2*>(d_yres), iters, tol, static_cast<float2*>(d_E), a));
}

altgdmin_status altgdmin_mec_ista(altgdmin_ctx* c, const void* d_yres, int32_t max_iter, double omega_frac,
                                  double tol, void* d_E, void* d_aux, int32_t* h_iters) {
  if (!c || !d_yres || !d_E || !aux_ok(d_aux) || max_iter < 0 || !(omega_frac >= 0.0) || !(tol >= 0.0))
    return ALTGDMIN_EINVAL;
  if (!c->bound) return ALTGDMIN_ESTATE;
  Aux a;
  aux_layout(c, static_cast<char*>(d_aux), &a);
  int slot = 0;
  HIPCHK(ista_frames(c, static_cast<const float2*>(d_yres), max_iter, omega_frac, tol, static_cast<float2*>(d_E), a,
                     h_iters ? &slot : nullptr));
  if (h_iters) {
    const altgdmin_status e = sync_status(c);
    HIPCHK(hipMemcpy(h_iters, &a.is[slot].iters, sizeof(int32_t), hipMemcpyDeviceToHost));
    if (e != ALTGDMIN_OK) return e;
  }
  return ALTGDMIN_OK;
}

altgdmin_status altgdmin_expand(altgdmin_ctx* c, const void* d_U, const void* d_B, const void* d_zbar,
                                const void* d_E, void* d_Z) {
  if (!c || !d_Z || (!d_U) != (!d_B)) return ALTGDMIN_EINVAL;
  if (!c->bound) return ALTGDMIN_ESTATE;
  return map_hip(launch_expand(static_cast<const float2*>(d_U), static_cast<const float2*>(d_B),
                               static_cast<const float2*>(d_zbar), static_cast<const float2*>(d_E), (long)c->n, c->p.q,
                               c->p.r, static_cast<float2*>(d_Z), c->st(), c->stream));
}

altgdmin_status altgdmin_rank_energy(altgdmin_ctx* c, int32_t r_cap, double* h_sigma2, void* d_aux) {
  if (!c || !h_sigma2 || !aux_ok(d_aux) || r_cap < 1 || r_cap > 16) return ALTGDMIN_EINVAL;
  if (!c->bound || !c->y) return ALTGDMIN_ESTATE;
  if (r_cap > c->p.q) return ALTGDMIN_EINVAL;
  Aux a;
  aux_layout(c, static_cast<char*>(d_aux), &a);
  HIPCHK(ag_host::spectral_eig(c, r_cap, a.lam));
  const altgdmin_status e = sync_status(c);
  if (e != ALTGDMIN_OK) return e;
  HIPCHK(hipMemcpy(h_sigma2, a.lam, sizeof(double) * r_cap, hipMemcpyDeviceToHost));
  return ALTGDMIN_OK;
}

altgdmin_status altgdmin_auto_rank(altgdmin_ctx* c, double b_percent, int32_t* h_rank, int32_t* h_rcap,
                                   void* d_aux) {
  if (!c || !h_rank || !aux_ok(d_aux) || !(b_percent > 0.0) || !(b_percent <= 100.0)) return ALTGDMIN_EINVAL;
  if (!c->bound || !c->y) return ALTGDMIN_ESTATE;
  const altgdmin_params& p = c->p;
  std::vector<int32_t> mk(p.q);
  HIPCHK(hipStreamSynchronize(c->stream));
  HIPCHK(hipMemcpy(mk.data(), c->m_k, sizeof(int32_t) * p.q, hipMemcpyDeviceToHost));
  const long mmin = *std::min_element(mk.begin(), mk.end());
  const long lim = std::min<long>(std::min<long>(c->n, p.q), (long)p.nc * mmin);
  const int r_cap = (int)std::max(1L, std::min(16L, lim / 10));
  double e2[16];
  const altgdmin_status st = altgdmin_rank_energy(c, r_cap, e2, d_aux);
  if (st != ALTGDMIN_OK) return st;
  double tot = 0.0;
  for (int j = 0; j < r_cap; ++j) tot += e2[j];
  const double target = b_percent / 100.0 * tot;
  int r = r_cap;
  double acc = 0.0;
  for (int j = 0; j < r_cap; ++j) {
    acc += e2[j];
    if (acc >= target) {
      r = j + 1;
      break;
    }
  }
  *h_rank = r;
  if (h_rcap) *h_rcap = r_cap;
  return ALTGDMIN_OK;
}

}  // extern "C"
