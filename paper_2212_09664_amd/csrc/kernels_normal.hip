// The normal operator A^H A applied in one pass, and the vector updates of
// the conjugate gradients (the mean image of Algorithm 1, step 1; the
// per-frame CGLS of Algorithm 3's model 1, whose operator passes are in
// kernels_fft.hip) and of ISTA's residual step (Algorithm 3's model 2).
//
// Line masks: the kx transform of a full-readout line is unitary, so
//   sum_k A_k^H A_k p = sum_c conj(s_c) F_y^H (cnt o F_y (s_c p)),
// cnt the number of frames sampling each row; ISTA's A_k^H (y_k - A_k e) takes
// the frame's own rows and its hybrid data in the middle.  A tile of image
// columns goes through both transforms without leaving the workgroup: the
// forward transform's outputs stay in registers and are the reversed plan's
// inputs, and the coil values used on the way in serve the combine on the
// way out.  General masks need the x transforms in between: forward columns,
// one pass over the k-space rows (transform, weight, transform back), adjoint
// columns.
//
// The mean's CG runs on the normal equations (s is updated by -alpha A^H A p)
// with <p, A^H A p> summed where F(s_c p) is in registers; MEC-1 keeps CGLS's
// residual r, because a frame that converges early leaves rounding noise in
// s, which only A^H r keeps in the range of A^H.  Scalars are FP64 and every sum
// runs in a fixed order.  The scalars of an iteration live in one of two
// slots: the operator's launch of iteration t reads slot t - 1 and writes slot
// t, so that no workgroup reads what another one of its launch writes.
#include <algorithm>

#include "kernels_mri.hpp"

namespace ag {

// ---------------------------------------------------------------------------
// line masks: a tile of CT image columns (grid: column tiles, images, coil
// groups; each group's sum over its coils goes to its own part of w).
//   NORMAL_MEAN  w = sum_k A_k^H A_k p, p = s + beta p_old formed here (and
//                stored by the first group); the tile's share of
//                <p, w> goes to dot
//   NORMAL_ISTA  w = A_k^H (y_k - A_k s) for image k = s
// Bound by the transforms' arithmetic and their LDS exchanges.  Mean image,
// 256 x 256, 12 coils: 900 -> 167 us with its ten iterations (a CG iteration
// from eight launches, 90 us, to two).  ISTA, 48 frames of 128 x 128, 8 coils:
// 26 us (27.7 with the data requested where it is used, under a branch, and the
// next coil after its transform; the image values in LDS leave the registers
// for both).
// ---------------------------------------------------------------------------
template <int N, int CT, int NT, int MODE>
__global__ __launch_bounds__(NT) void k_normal_lines(NormalArgs a) {
  using GM = FftGeom<N, CT, NT>;
  constexpr int IT0 = GM::IT0, R0 = GM::R0, ITL = GM::ITL, RL = GM::RL;
  constexpr bool MEAN = MODE == NORMAL_MEAN;
  __shared__ float2 s[GM::LDS];
  __shared__ float2 s_p[IT0 * R0 * NT];  // each thread's image values, used once a coil
  __shared__ float2 s_tw[N];
  __shared__ float s_wt[MEAN ? N : 1];
  __shared__ int s_li[MEAN ? 1 : N];
  __shared__ double s_red[NT / 64];
  const int tid = threadIdx.x;
  const int x0 = xcd_tile(blockIdx.x, gridDim.x) * CT, img = blockIdx.y, grp = blockIdx.z;
  if (halted(a.st, 0)) return;  // (a mask that failed its checks at bind sets err)
  if (!MEAN && a.ista->done) return;
  const int cb = grp * a.cgs, ce = min(a.nc, cb + a.cgs);
  // the tile's image values and the first coil's, from valid addresses
  // (columns past a narrow image and idle threads are zeroed below)
  int off[IT0];
  bool ok[IT0];
#pragma unroll
  for (int it = 0; it < IT0; ++it) {
    const int g = tid + it * NT, col = GM::in_col(g);
    ok[it] = GM::in_ok(g) && x0 + col < a.nx;
    off[it] = ok[it] ? GM::in_row(g, 0) * a.nx + x0 + col : 0;
  }
  const int rs = (N / R0) * a.nx;  // from one of a thread's input rows to its next
  auto load = [&](const float2* p, float2 (&v)[IT0][R0]) {
#pragma unroll
    for (int it = 0; it < IT0; ++it)
#pragma unroll
      for (int q = 0; q < R0; ++q) v[it][q] = p[off[it] + (ok[it] ? q * rs : 0)];
  };
  float2 pv[IT0][R0], cv[IT0][R0];
  load(a.s + (long)img * a.n, pv);
  load(a.coils + (long)min(cb, a.nc - 1) * a.n, cv);
  const float inv = 1.f / N;  // both transforms' 1 / sqrt(N)
  for (int e = tid; e < N; e += NT) {
    s_tw[e] = a.tw[e];
    if constexpr (MEAN) s_wt[e] = (float)(a.loc_ptr[e + 1] - a.loc_ptr[e]) * inv;
    else s_li[e] = -1;
  }
  if constexpr (MEAN) {
    float beta;
    if (!cg_open(a.cg, img, blockIdx.x == 0 && grp == 0, beta)) return;
    if (a.cg.it > 0) {
      float2 po[IT0][R0];
      load(a.p_old + (long)img * a.n, po);
#pragma unroll
      for (int it = 0; it < IT0; ++it)
#pragma unroll
        for (int q = 0; q < R0; ++q)
          pv[it][q] = make_float2(pv[it][q].x + beta * po[it][q].x, pv[it][q].y + beta * po[it][q].y);
    }
    if (grp == 0) {
      float2* const pn = a.p_new + (long)img * a.n;
#pragma unroll
      for (int it = 0; it < IT0; ++it)
        if (ok[it]) {
#pragma unroll
          for (int q = 0; q < R0; ++q) pn[off[it] + q * rs] = pv[it][q];
        }
    }
  }
  __syncthreads();
  if constexpr (!MEAN) {  // the frame's sampled rows (distinct)
    const int n_rows = a.m_k[img] / a.nx;
    const int32_t* rows = a.rows + (long)img * a.rows_img_stride;
    for (int l = tid; l < n_rows; l += NT) s_li[min(max(rows[l], 0), N - 1)] = l;
    __syncthreads();
  }
  float2 acc[IT0][R0];
#pragma unroll
  for (int it = 0; it < IT0; ++it)
#pragma unroll
    for (int q = 0; q < R0; ++q) {
      acc[it][q] = make_float2(0.f, 0.f);
      s_p[(it * R0 + q) * NT + tid] = ok[it] ? pv[it][q] : make_float2(0.f, 0.f);
    }
  double dot = 0.0;
  for (int c = cb; c < ce; ++c) {
    float2 v0[IT0][R0], vo[ITL][RL];
#pragma unroll
    for (int it = 0; it < IT0; ++it)
#pragma unroll
      for (int q = 0; q < R0; ++q) v0[it][q] = cmul(cv[it][q], s_p[(it * R0 + q) * NT + tid]);
    // the frame's data at the transform's outputs, in flight during it (the
    // rows that are not sampled request the frame's first)
    float2 yv[MEAN ? 1 : ITL][MEAN ? 1 : RL];
    if constexpr (!MEAN) {
      const float2* yc = a.y + ((long)img * a.nc + c) * a.m_max;
#pragma unroll
      for (int it = 0; it < ITL; ++it) {
        const int g = tid + it * NT, x = min(x0 + GM::out_col(g), a.nx - 1);
#pragma unroll
        for (int q = 0; q < RL; ++q) yv[it][q] = yc[max(GM::out_ok(g) ? s_li[GM::out_row(g, q)] : 0, 0) * a.nx + x];
      }
    }
    fft_regs<N, CT, NT, false>(v0, vo, s, s_tw);
#pragma unroll
    for (int it = 0; it < ITL; ++it) {
      const int g = tid + it * NT, x = x0 + GM::out_col(g);
      const bool in = GM::out_ok(g) && x < a.nx;
#pragma unroll
      for (int q = 0; q < RL; ++q) {
        const float2 v = vo[it][q];
        if constexpr (MEAN) {
          const float w = in ? s_wt[GM::out_row(g, q)] : 0.f;
          vo[it][q] = cscale(v, w);
          dot += (double)w * ((double)v.x * v.x + (double)v.y * v.y);
        } else {
          const float w = in && s_li[GM::out_row(g, q)] >= 0 ? a.scale : 0.f;
          const float2 r = csub(yv[it][q], cscale(v, a.scale));
          vo[it][q] = w != 0.f ? cscale(r, w) : make_float2(0.f, 0.f);
        }
      }
    }
    float2 cn[IT0][R0];
    load(a.coils + (long)min(c + 1, ce - 1) * a.n, cn);  // the next coil's, in flight during the transform
    fft_regs<N, CT, NT, true, true, true>(vo, v0, s, s_tw);
#pragma unroll
    for (int it = 0; it < IT0; ++it)
#pragma unroll
      for (int q = 0; q < R0; ++q) {
        acc[it][q] = cjfma(acc[it][q], cv[it][q], v0[it][q]);
        cv[it][q] = cn[it][q];
      }
  }
  float2* const out = a.w + (long)grp * a.part_stride + (long)img * a.n;
#pragma unroll
  for (int it = 0; it < IT0; ++it)
    if (ok[it]) {
#pragma unroll
      for (int q = 0; q < R0; ++q) out[off[it] + q * rs] = acc[it][q];
    }
  if constexpr (MEAN) {
    dot = wave_sum(dot);
    if ((tid & 63) == 0) s_red[tid >> 6] = dot;
    __syncthreads();
    if (tid == 0) {
      double t = 0.0;
      for (int w = 0; w < NT / 64; ++w) t += s_red[w];
      a.dot[((long)img * gridDim.x + blockIdx.x) * gridDim.z + grp] = t;
    }
  }
}

// general masks, the mean image: F_x^H (count o F_x row) in place on the
// k-space rows of the coil images in T, TR rows per workgroup, with the
// tile's share of <p, A^H A p>
template <int N, int TR, int NT>
__global__ __launch_bounds__(NT) void k_normal_rows(NormalArgs a) {
  using GM = FftGeom<N, TR, NT, false, true>;
  constexpr int IT0 = GM::IT0, R0 = GM::R0, ITL = GM::ITL, RL = GM::RL;
  __shared__ float2 s[GM::LDS];
  __shared__ float2 s_tw[N];
  __shared__ double s_red[NT / 64];
  const int tid = threadIdx.x;
  const int nrows = a.nc * a.ny, row0 = blockIdx.x * TR;
  if (halted(a.st, 0) || a.cg.out[0].done) return;  // (the columns' launch wrote this iteration's slot)
  float2 v0[IT0][R0], vo[ITL][RL];
#pragma unroll
  for (int it = 0; it < IT0; ++it) {
    const int g = tid + it * NT, row = row0 + GM::in_col(g);
    const bool ok = GM::in_ok(g) && row < nrows;
    const float2* src = a.T + (ok ? (long)row * N + GM::in_row(g, 0) : 0);
#pragma unroll
    for (int q = 0; q < R0; ++q) {
      const float2 v = src[ok ? q * (N / R0) : 0];
      v0[it][q] = ok ? v : make_float2(0.f, 0.f);
    }
  }
  const float inv = 1.f / N;  // both transforms' 1 / sqrt(N)
  float wt[ITL][RL];
#pragma unroll
  for (int it = 0; it < ITL; ++it) {
    const int g = tid + it * NT, row = row0 + GM::out_col(g);
    const bool ok = GM::out_ok(g) && row < nrows;
    const int ky = ok ? row % a.ny : 0;
#pragma unroll
    for (int q = 0; q < RL; ++q) {
      const int loc = ky * N + (ok ? GM::out_row(g, q) : 0);
      const float w = (float)(a.loc_ptr[loc + 1] - a.loc_ptr[loc]);
      wt[it][q] = ok ? w * inv : 0.f;
    }
  }
  for (int e = tid; e < N; e += NT) s_tw[e] = a.tw_x[e];
  __syncthreads();
  fft_regs<N, TR, NT, false, false, false, true>(v0, vo, s, s_tw);
  double dot = 0.0;
#pragma unroll
  for (int it = 0; it < ITL; ++it)
#pragma unroll
    for (int q = 0; q < RL; ++q) {
      const float2 v = vo[it][q];
      dot += (double)wt[it][q] * ((double)v.x * v.x + (double)v.y * v.y);
      vo[it][q] = cscale(v, wt[it][q]);
    }
  fft_regs<N, TR, NT, true, true, true, true>(vo, v0, s, s_tw);
#pragma unroll
  for (int it = 0; it < IT0; ++it) {
    const int g = tid + it * NT, row = row0 + GM::in_col(g);
    if (GM::in_ok(g) && row < nrows) {
#pragma unroll
      for (int q = 0; q < R0; ++q) a.T[(long)row * N + GM::in_row(g, q)] = v0[it][q];
    }
  }
  dot = wave_sum(dot);
  if ((tid & 63) == 0) s_red[tid >> 6] = dot;
  __syncthreads();
  if (tid == 0) {
    double t = 0.0;
    for (int w = 0; w < NT / 64; ++w) t += s_red[w];
    a.dot[blockIdx.x] = t;
  }
}

// CGLS over several coil groups: s = the sum of the groups' parts, and each
// workgroup's share of ||s||^2.  Grid (NB, images).
__global__ __launch_bounds__(256) void k_cgls_sum(const float2* src, int nsum, long part_stride, float2* s, long n,
                                                  double* nrm, const FrameCg* cg, const DevState* st) {
  __shared__ double sh[4];
  const int img = blockIdx.y, tid = threadIdx.x;
  if (st->err || (cg && (cg[img].done | cg[img].brk))) return;
  double acc = 0.0;
  for (long i = (long)blockIdx.x * 256 + tid; i < n; i += (long)gridDim.x * 256) {
    const long e = (long)img * n + i;
    float2 v = src[e];
    for (int g = 1; g < nsum; ++g) v = cadd(v, src[g * part_stride + e]);
    s[e] = v;
    acc += (double)v.x * v.x + (double)v.y * v.y;
  }
  acc = wave_sum(acc);
  if ((tid & 63) == 0) sh[tid >> 6] = acc;
  __syncthreads();
  if (tid == 0) nrm[(long)img * gridDim.x + blockIdx.x] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// ---------------------------------------------------------------------------
// x = 0, s = the sum of nsum FP64 parts of the right-hand side (rounded to FP32
// once, here), and each workgroup's share of ||s||^2.  One image.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_cg_begin(const double2* src, int nsum, long part_stride, float2* s, float2* x,
                                                  long n, double* nrm, const DevState* st) {
  __shared__ double sh[4];
  const int tid = threadIdx.x;
  const bool bad = st->err != 0;
  double acc = 0.0;
  for (long i = (long)blockIdx.x * 256 + tid; i < n; i += (long)gridDim.x * 256) {
    x[i] = make_float2(0.f, 0.f);
    if (bad) continue;
    double2 d = src[i];
#pragma unroll 4
    for (int g = 1; g < nsum; ++g) d = dadd(d, src[g * part_stride + i]);
    const float2 v = d2f(d);
    s[i] = v;
    acc += (double)v.x * v.x + (double)v.y * v.y;
  }
  acc = wave_sum(acc);
  if ((tid & 63) == 0) sh[tid >> 6] = acc;
  __syncthreads();
  if (tid == 0) nrm[blockIdx.x] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// alpha = gamma / ||A p||^2; x += alpha p; s -= alpha w; the workgroup's share of
// ||s||^2.  Grid (NB, images).  A system whose ||A p|| is zero stops (brk).
__global__ __launch_bounds__(256) void k_cg_step(CgStepArgs a) {
  __shared__ double sh[4];
  const int img = blockIdx.y, tid = threadIdx.x;
  if (a.st->err) return;
  if (a.cg[img].done) return;
  const double d = wave_sum_parts(a.dot + (long)img * a.ndot, a.ndot, tid & 63);
  if (!(d > 0.0)) {
    if (blockIdx.x == 0 && tid == 0) a.cg[img].brk = 1;
    return;
  }
  const float al = (float)(a.cg[img].gamma / d);
  double acc = 0.0;
  for (long i = (long)blockIdx.x * 256 + tid; i < a.n; i += (long)gridDim.x * 256) {
    const long e = (long)img * a.n + i;
    float2 w = a.w[e];
    for (int g = 1; g < a.nsum; ++g) w = cadd(w, a.w[g * a.part_stride + e]);
    const float2 pv = a.p[e], xv = a.x[e];
    float2 sv = a.s[e];
    a.x[e] = make_float2(xv.x + al * pv.x, xv.y + al * pv.y);
    sv = make_float2(sv.x - al * w.x, sv.y - al * w.y);
    a.s[e] = sv;
    acc += (double)sv.x * sv.x + (double)sv.y * sv.y;
  }
  acc = wave_sum(acc);
  if ((tid & 63) == 0) sh[tid >> 6] = acc;
  __syncthreads();
  if (tid == 0) a.nrm[(long)img * gridDim.x + blockIdx.x] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// the stop test after the last iteration: the iteration count of system 0
__global__ void k_cg_end(CgArgs a, const DevState* st) {
  if (st->err) return;
  float beta;
  (void)cg_open(a, 0, true, beta);
}

// ---------------------------------------------------------------------------
// the mean image's right-hand side A^H y = sum_c conj(s_c) F^H sum_k y_{k,c}: the
// frames are summed in k-space and one adjoint carries the sum, in FP64 until
// the image is rounded to FP32 (k_cg_begin).  An FP32 adjoint of every frame
// averages its roundings out over the frames; an FP32 adjoint of their sum would
// not, and the image would be 1.3 times as far from the 64-bit one (256 x 256,
// 12 coils, 40 frames: 9.0e-7 against 6.8e-7, and 7.0e-7 with a frame at a time).
// That size: sums 15 us, columns 13 us, 6 us more than an FP32 adjoint.
// ---------------------------------------------------------------------------
// k-space sums over the frames, per (row or location, coil), zero where no frame
// samples.  Line masks: the hybrid data's lines, yu as built at setup; grid (ny, nc)
__global__ __launch_bounds__(256) void k_line_sum(const float2* yu, const int32_t* loc_ptr, int nc, int nx, double2* T,
                                                  const DevState* st) {
  if (st->err) return;
  const int ky = blockIdx.x, c = blockIdx.y;
  const int first = loc_ptr[ky], np = loc_ptr[ky + 1] - first;
  const float2* src = yu + (long)nc * nx * first + (long)c * np * nx;
  double2* dst = T + ((long)c * gridDim.x + ky) * nx;
  for (int x = threadIdx.x; x < nx; x += 256) {
    double2 s = make_double2(0.0, 0.0);
    for (int p0 = 0; p0 < np; p0 += 8) {  // eight loads in flight, the last batch's too
      float2 v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = src[(long)min(p0 + i, np - 1) * nx + x];
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (p0 + i < np) s = dadd(s, f2d(v[i]));
    }
    dst[x] = s;
  }
}

// general masks: the (frame, sample) pairs of each location; grid (locations / 256, nc)
__global__ __launch_bounds__(256) void k_loc_sum(const float2* y, const int2* pairs, const int32_t* loc_ptr, long n,
                                                 int nc, int m_max, double2* T, const DevState* st) {
  if (st->err) return;
  const long loc = (long)blockIdx.x * 256 + threadIdx.x;
  const int c = blockIdx.y;
  if (loc >= n) return;
  const int p0 = loc_ptr[loc], p1 = loc_ptr[loc + 1];
  const float2* yc = y + (long)c * m_max;
  const long ks = (long)nc * m_max;
  double2 s = make_double2(0.0, 0.0);
#pragma unroll 4
  for (int p = p0; p < p1; ++p) {
    const int2 ke = pairs[p];
    s = dadd(s, f2d(yc[ke.x * ks + ke.y]));
  }
  T[(long)c * n + loc] = s;
}

// the FP64 adjoint's tile: CT columns (or rows) of N points in 32 KB of LDS
template <int N>
constexpr int RHS_CT = N == 512 ? 4 : N == 256 ? 8 : 16;

template <int N>
__device__ __forceinline__ void rhs_twiddles(double2* tw) {
  for (int e = threadIdx.x; e < N; e += 256) {
    double sv, cv;
    sincospi(2.0 * (double)e / (double)N, &sv, &cv);
    tw[e] = make_double2(cv, -sv);
  }
}

// general masks: F_x^H of T's nrows rows in place, CT rows per workgroup
template <int N>
__global__ __launch_bounds__(256) void k_rhs_rows(double2* T, int nrows, const DevState* st) {
  constexpr int CT = RHS_CT<N>;
  __shared__ double2 s[N * CT], tw[N];
  if (st->err) return;
  const int row0 = blockIdx.x * CT;
  for (int e = threadIdx.x; e < N * CT; e += 256) {
    const int row = row0 + e / N;
    s[(e % N) * CT + e / N] = row < nrows ? T[(long)row * N + e % N] : make_double2(0.0, 0.0);
  }
  rhs_twiddles<N>(tw);
  __syncthreads();
  fft_lds<N, CT, 256, true>(s, tw);
  const double sc = 1.0 / sqrt((double)N);
  for (int e = threadIdx.x; e < N * CT; e += 256) {
    const int row = row0 + e / N;
    const double2 v = s[(e % N) * CT + e / N];
    if (row < nrows) T[(long)row * N + e % N] = make_double2(v.x * sc, v.y * sc);
  }
}

// F_y^H of a tile of columns and the combine over a group's coils, in place: the
// group's first coil plane receives its sum.  Grid (column tiles, coil groups).
template <int N>
__global__ __launch_bounds__(256) void k_rhs_cols(double2* T, const float2* coils, long n, int nx, int nc, int cgs,
                                                  const DevState* st) {
  constexpr int CT = RHS_CT<N>, EM = (N * CT + 255) / 256;
  __shared__ double2 s[N * CT], tw[N];
  if (st->err) return;
  const int tid = threadIdx.x, x0 = blockIdx.x * CT, cb = blockIdx.y * cgs, ce = min(nc, cb + cgs);
  // this thread's entries of the tile: offset in an image, -1 past its columns
  int off[EM];
  double2 v[EM], acc[EM];
  float2 cv[EM];
#pragma unroll
  for (int i = 0; i < EM; ++i) {
    const int e = tid + 256 * i, x = x0 + e % CT;
    off[i] = e < N * CT && x < nx ? (e / CT) * nx + x : -1;
    acc[i] = make_double2(0.0, 0.0);
  }
  auto load = [&](int c) {
#pragma unroll
    for (int i = 0; i < EM; ++i) v[i] = T[(long)c * n + max(off[i], 0)];
  };
  load(cb);
  rhs_twiddles<N>(tw);
  for (int c = cb; c < ce; ++c) {
#pragma unroll
    for (int i = 0; i < EM; ++i)
      if (tid + 256 * i < N * CT) s[tid + 256 * i] = v[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < EM; ++i) cv[i] = coils[(long)c * n + max(off[i], 0)];
    if (c + 1 < ce) load(c + 1);
    fft_lds<N, CT, 256, true>(s, tw);
#pragma unroll
    for (int i = 0; i < EM; ++i)
      if (off[i] >= 0) acc[i] = dadd(acc[i], djmul(f2d(cv[i]), s[tid + 256 * i]));
    // (the next coil's values go where this thread has just read)
  }
  const double sc = 1.0 / sqrt((double)N);
#pragma unroll
  for (int i = 0; i < EM; ++i)
    if (off[i] >= 0) T[(long)cb * n + off[i]] = make_double2(acc[i].x * sc, acc[i].y * sc);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
namespace {
template <int N>
hipError_t lines_n(const NormalArgs& a, int mode, int images, int groups, hipStream_t s) {
  constexpr int CT = OpTile<N>::CT, NT = OpTile<N>::NT;
  const dim3 g((a.nx + CT - 1) / CT, images, groups);
  if (mode == NORMAL_MEAN) hipLaunchKernelGGL((k_normal_lines<N, CT, NT, NORMAL_MEAN>), g, dim3(NT), 0, s, a);
  else hipLaunchKernelGGL((k_normal_lines<N, CT, NT, NORMAL_ISTA>), g, dim3(NT), 0, s, a);
  return hipGetLastError();
}

template <int N>
hipError_t normal_rows_n(const NormalArgs& a, hipStream_t s) {
  constexpr int TR = OpTile<N>::CT, NT = OpTile<N>::NT;
  hipLaunchKernelGGL((k_normal_rows<N, TR, NT>), dim3((a.nc * a.ny + TR - 1) / TR), dim3(NT), 0, s, a);
  return hipGetLastError();
}

template <int N>
hipError_t rhs_rows_n(double2* T, int nrows, const DevState* st, hipStream_t s) {
  constexpr int CT = RHS_CT<N>;
  hipLaunchKernelGGL((k_rhs_rows<N>), dim3((nrows + CT - 1) / CT), dim3(256), 0, s, T, nrows, st);
  return hipGetLastError();
}

template <int N>
hipError_t rhs_cols_n(double2* T, const float2* coils, long n, int nx, int nc, int* cgs, const DevState* st,
                      hipStream_t s) {
  // coil groups for about two workgroups per compute unit
  const int tiles = (nx + RHS_CT<N> - 1) / RHS_CT<N>, want = std::max(1, std::min(nc, 512 / tiles));
  *cgs = (nc + want - 1) / want;
  hipLaunchKernelGGL((k_rhs_cols<N>), dim3(tiles, (nc + *cgs - 1) / *cgs), dim3(256), 0, s, T, coils, n, nx, nc, *cgs, st);
  return hipGetLastError();
}
}  // namespace

#define NORMAL_DISPATCH(fn, N, ...)          \
  switch (N) {                               \
    case 8: return fn<8>(__VA_ARGS__);       \
    case 16: return fn<16>(__VA_ARGS__);     \
    case 32: return fn<32>(__VA_ARGS__);     \
    case 64: return fn<64>(__VA_ARGS__);     \
    case 128: return fn<128>(__VA_ARGS__);   \
    case 256: return fn<256>(__VA_ARGS__);   \
    case 512: return fn<512>(__VA_ARGS__);   \
  }                                          \
  return hipErrorInvalidValue

hipError_t launch_normal_lines(const NormalArgs& a, int mode, int images, int groups, hipStream_t s) {
  NORMAL_DISPATCH(lines_n, a.ny, a, mode, images, groups, s);
}
hipError_t launch_normal_rows(const NormalArgs& a, hipStream_t s) { NORMAL_DISPATCH(normal_rows_n, a.nx, a, s); }
hipError_t launch_rhs_rows(double2* T, int nx, int nrows, const DevState* st, hipStream_t s) {
  NORMAL_DISPATCH(rhs_rows_n, nx, T, nrows, st, s);
}
hipError_t launch_rhs_cols(double2* T, const float2* coils, int nx, int ny, int nc, int* cgs, const DevState* st,
                           hipStream_t s) {
  NORMAL_DISPATCH(rhs_cols_n, ny, T, coils, (long)nx * ny, nx, nc, cgs, st, s);
}

}  // namespace ag
