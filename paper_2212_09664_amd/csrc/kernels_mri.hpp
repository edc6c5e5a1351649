// Device state and kernels of the steps around the altGDmin loop (the mean
// image, the modelling-error corrections, the output); see kernels_normal.hip
// and kernels_mri.hip.
#pragma once

#include "kernels_core.hpp"

namespace ag {

// the normal operator over image columns (line masks) or k-space rows
// (general masks, the mean image)
struct NormalArgs {
  const float2* s;        // the image of each system (the mean: the residual s; ISTA: E)
  const float2* p_old;    // the mean: the last direction
  float2* p_new;          // the mean: this iteration's direction
  const float2* coils;
  long n;
  int nx, ny, nc;
  const float2 *tw, *tw_x;
  const int32_t* loc_ptr; // the mean: counts of frames per row or location
  const int32_t* rows;    // ISTA: a frame's sampled rows and hybrid data [frame][c][line][x]
  long rows_img_stride;
  const int32_t* m_k;
  const float2* y;
  int m_max;
  float2* w;              // line masks: out, one part per coil group
  long part_stride;
  int cgs;                // coils per group
  float2* T;              // general masks: k-space rows [c][ky][x]
  float scale;            // ISTA: 1 / sqrt(ny)
  double* dot;            // the mean: shares of <p, A^H A p>
  CgArgs cg;
  const IstaState* ista;  // non-null: nothing to do once its done is set
  const DevState* st;
};

struct CgStepArgs {
  const float2 *w, *p;
  float2 *x, *s;
  int nsum;               // parts of w
  long part_stride, n;
  FrameCg* cg;            // this iteration's slot
  const double* dot;
  int ndot;
  double* nrm;
  const DevState* st;
};

// sum of part[0..nb) by one wave (every lane active), in a fixed order
__device__ __forceinline__ double wave_sum_parts(const double* part, int nb, int lane) {
  double s = 0.0;
  for (int i = lane; i < nb; i += 64) s += part[i];
  return wave_sum(s);
}

// The start of CG iteration a.it for system `img`: the stop test of the
// iteration before, beta, and the new scalars (written by the one workgroup
// with `writer`).  Every wave computes the same values.  False: stopped.
__device__ __forceinline__ bool cg_open(const CgArgs& a, int img, bool writer, float& beta) {
  const int lane = threadIdx.x & 63;
  const double g = wave_sum_parts(a.nrm + (long)img * a.nnrm, a.nnrm, lane);
  FrameCg o;
  beta = 0.f;
  if (a.it == 0) {
    o.gamma = o.gamma0 = g;
    o.iters = 0;
    o.done = !(g > 0.0);
  } else {
    const FrameCg i = a.in[img];
    o = i;
    o.done = i.done | i.brk;
    if (!o.done) {
      o.iters = i.iters + 1;
      o.done = sqrt(g) <= a.tol * sqrt(i.gamma0);
      beta = (float)(g / i.gamma);
      o.gamma = g;
    }
  }
  o.brk = 0;
  if (writer && threadIdx.x == 0) a.out[img] = o;
  return !o.done;
}

// consecutive workgroups go to the eight XCDs in turn: tile b of a row of
// nt tiles is dealt so that an XCD's tiles are neighbours, which share the
// cache lines that a tile narrower than a line splits
__device__ __forceinline__ int xcd_tile(int b, int nt) { return nt % 8 == 0 ? (b % 8) * (nt / 8) + b / 8 : b; }

enum { NORMAL_MEAN = 0, NORMAL_ISTA = 1 };
hipError_t launch_normal_lines(const NormalArgs& a, int mode, int images, int groups, hipStream_t s);
hipError_t launch_normal_rows(const NormalArgs& a, hipStream_t s);  // the mean
__global__ void k_cg_begin(const double2* src, int nsum, long part_stride, float2* s, float2* x, long n, double* nrm,
                           const DevState* st);
__global__ void k_cg_step(CgStepArgs a);
__global__ void k_cgls_sum(const float2* src, int nsum, long part_stride, float2* s, long n, double* nrm,
                           const FrameCg* cg, const DevState* st);
__global__ void k_cg_end(CgArgs a, const DevState* st);
// the mean's right-hand side in FP64: the frames' sums T[c][ky][x], then the adjoint in
// place (cgs: coils per group, whose first plane receives the group's part)
__global__ void k_line_sum(const float2* yu, const int32_t* loc_ptr, int nc, int nx, double2* T, const DevState* st);
__global__ void k_loc_sum(const float2* y, const int2* pairs, const int32_t* loc_ptr, long n, int nc, int m_max,
                          double2* T, const DevState* st);
hipError_t launch_rhs_rows(double2* T, int nx, int nrows, const DevState* st, hipStream_t s);
hipError_t launch_rhs_cols(double2* T, const float2* coils, int nx, int ny, int nc, int* cgs, const DevState* st,
                           hipStream_t s);
hipError_t launch_expand(const float2* U, const float2* B, const float2* zbar, const float2* E, long n, int q, int r,
                         float2* Z, const DevState* st, hipStream_t s);

// ISTA's temporal step (kernels_mri.hip); partial sums: one pair per 64 pixels
struct IstaArgs {
  float2* E;              // n x q
  const float2* w;        // parts of A^H(yres - A(E))
  int nsum;
  long part_stride;
  float2* M;              // n x q: M_{t-1} in, M_t out
  long n;
  int q, t;
  float scale;            // 1 / sqrt(q)
  double frac, tol;
  const IstaState* in;    // the scalars of update t - 1 / t
  IstaState* out;
  const double* pin;      // partial sums of update t - 1 / t
  double* pout;
  const DevState* st;
};
enum { ISTA_FIRST = 0, ISTA_THRESH = 1, ISTA_STEP = 2 };
hipError_t launch_ista_dft(const IstaArgs& a, int phase, hipStream_t s);
__global__ void k_ista_begin(float2* E, long total, IstaState* is);
__global__ void k_ista_end(const IstaState* in, IstaState* out, const double* pin, int np, int t, double tol,
                           const DevState* st);

}  // namespace ag
