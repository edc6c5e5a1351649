// Transform kernels of the measurement operators: batched 1D DFTs along x
// (contiguous rows) and along y (image columns), with the coil weighting, the
// sampling selection, the conjugate-coil combine and the CG vector updates
// fused into their loads and stores.
//
// The 2D DFT of the measurement model (Sec. II-A) is separable, F = F_y F_x.
// For 1D Cartesian masks every sampled line is complete along kx, so the
// kx half moves to a one-time pass over the data and each iteration needs
// only the y half, restricted on output to the sampled lines.  For general
// masks both halves run.
//
// Every transform is register-fed (fft_regs): its inputs come from memory
// straight into the first radix pass and its last pass is stored from
// registers, so that only the exchanges between passes go through LDS.
#include <algorithm>

#include "kernels_mri.hpp"

namespace ag {

// ---------------------------------------------------------------------------
// rows: FFT along x of TR rows of length N per workgroup.
// Row rho of the batch lives at src + rho*N.  With m_k != null the rows are
// the padded measurement lines rho = (k*nc + c)*lmax + l, valid when
// l < m_k[k]/N; invalid rows are written as zeros.  trunc: zero every input
// sample with |v|^2 > gamma (state) before the transform.  Consecutive lanes
// hold consecutive elements of a row (whole segments of the row per load);
// bound by memory.
// ---------------------------------------------------------------------------
template <int N, int TR, int NT, bool INV>
__global__ __launch_bounds__(NT) void k_rows(RowArgs a) {
  using GM = FftGeom<N, TR, NT, false, true>;
  constexpr int IT0 = GM::IT0, R0 = GM::R0, ITL = GM::ITL, RL = GM::RL;
  __shared__ float2 s[GM::LDS];
  __shared__ float2 s_tw[N];
  const int tid = threadIdx.x;
  const long rho0 = (long)blockIdx.x * TR;
  if (halted(a.st, 0)) return;
  float2 v0[IT0][R0];
  bool okr[IT0];
#pragma unroll
  for (int it = 0; it < IT0; ++it) {
    const int g = tid + it * NT;
    const long rho = rho0 + GM::in_col(g);
    okr[it] = GM::in_ok(g) && rho < a.nrows && row_valid(a, rho, N);
    const float2* src = a.src + (okr[it] ? rho * N + GM::in_row(g, 0) : 0);
#pragma unroll
    for (int q = 0; q < R0; ++q) v0[it][q] = src[okr[it] ? q * (N / R0) : 0];
  }
  for (int e = tid; e < N; e += NT) s_tw[e] = a.tw[e];
  const double gamma = a.trunc ? a.st->gamma : 0.0;
  int n_cut = 0;
#pragma unroll
  for (int it = 0; it < IT0; ++it)
#pragma unroll
    for (int q = 0; q < R0; ++q) {
      const float2 v = v0[it][q];
      const bool cut = a.trunc && okr[it] && ((double)v.x * v.x + (double)v.y * v.y > gamma);
      n_cut += cut;
      if (!okr[it] || cut) v0[it][q] = make_float2(0.f, 0.f);
    }
  if (n_cut && a.trunc_count) atomicAdd(a.trunc_count, n_cut);
  __syncthreads();
  float2 vo[ITL][RL];
  fft_regs<N, TR, NT, INV, INV, false, true>(v0, vo, s, s_tw);
#pragma unroll
  for (int it = 0; it < ITL; ++it) {
    const int g = tid + it * NT;
    const long rho = rho0 + GM::out_col(g);
    if (GM::out_ok(g) && rho < a.nrows) {
      const bool valid = row_valid(a, rho, N);
#pragma unroll
      for (int q = 0; q < RL; ++q) {
        const long o = rho * N + GM::out_row(g, q);
        float2 v = valid ? cscale(vo[it][q], a.scale) : make_float2(0.f, 0.f);
        if (a.sub && valid) v = csub(a.sub[o], v);
        a.dst[o] = v;
      }
    }
  }
}

// an image's sampled rows (distinct): their number and this thread's first are
// requested when the list is made, before anything waits
struct RowList {
  const int32_t* rows;
  int mk = 0, r0 = 0;
  __device__ RowList(const int32_t* list, long stride, const int32_t* m_k, int img, int tid)
      : rows(list ? list + img * stride : nullptr) {
    if (!rows) return;
    mk = m_k[img];
    r0 = rows[min(tid, (int)stride - 1)];
  }
  // li[k-space row] = the line that holds it
  template <int N, int NT>
  __device__ void invert(int* li, int n_rows, int tid) const {
    for (int l = tid; l < n_rows; l += NT) li[min(max(l == tid ? r0 : rows[l], 0), N - 1)] = l;
  }
};

// ---------------------------------------------------------------------------
// image columns -> k-space rows: F_y (s_c o image) for the coils of a group,
// restricted to the image's sampled rows (or all rows).  Grid: column tiles,
// images, coil groups.  The image tile stays in registers over the group's
// coils; the inverse row map (k-space row -> the image's line, -1) is in LDS.
// CG: the image is p = s + beta p_old, formed here and stored by group 0, and
// the tile's share of ||A p||^2 over the sampled rows goes to dot.
// ---------------------------------------------------------------------------
template <int N, int CT, int NT, bool CG>
__global__ __launch_bounds__(NT) void k_cols_fwd(ColFwdArgs a) {
  using GM = FftGeom<N, CT, NT>;
  constexpr int IT0 = GM::IT0, R0 = GM::R0, ITL = GM::ITL, RL = GM::RL;
  __shared__ float2 s[GM::LDS];
  __shared__ float2 s_tw[N];
  __shared__ int s_li[N];
  __shared__ double s_red[NT / 64];
  const int tid = threadIdx.x;
  const int x0 = xcd_tile(blockIdx.x, gridDim.x) * CT, im = blockIdx.y, img = a.img0 + im, grp = blockIdx.z;
  const int cb = grp * a.cgs, ce = min(a.nc, cb + a.cgs);
  const RowList rl(a.rows, a.rows_img_stride, a.m_k, img, tid);
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
  if (a.src) {
    load(a.src + (long)img * a.n, pv);
  } else {
#pragma unroll
    for (int it = 0; it < IT0; ++it)
#pragma unroll
      for (int q = 0; q < R0; ++q) pv[it][q] = make_float2(0.f, 0.f);
  }
  load(a.coils + (long)min(cb, a.nc - 1) * a.n, cv);
  // the state is read once the first loads are in flight (their addresses are valid either way)
  if (halted(a.st, 0)) return;  // (a mask that failed its checks at bind sets err)
  if (a.ista && a.ista->done) return;
  if (a.add) {
    float2 zv[IT0][R0];
    load(a.add, zv);
#pragma unroll
    for (int it = 0; it < IT0; ++it)
#pragma unroll
      for (int q = 0; q < R0; ++q) pv[it][q] = cadd(pv[it][q], zv[it][q]);
  }
  for (int e = tid; e < N; e += NT) {
    s_tw[e] = a.tw[e];
    s_li[e] = a.rows ? -1 : e;
  }
  if constexpr (CG) {
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
  int n_rows = N;
  if (a.rows) {
    n_rows = rl.mk / a.nx;
    rl.invert<N, NT>(s_li, n_rows, tid);
    __syncthreads();
  }
#pragma unroll
  for (int it = 0; it < IT0; ++it)
#pragma unroll
    for (int q = 0; q < R0; ++q)
      if (!ok[it]) pv[it][q] = make_float2(0.f, 0.f);
  double dot = 0.0;
  for (int c = cb; c < ce; ++c) {
    float2 v0[IT0][R0], vo[ITL][RL];
#pragma unroll
    for (int it = 0; it < IT0; ++it)
#pragma unroll
      for (int q = 0; q < R0; ++q) v0[it][q] = cmul(cv[it][q], pv[it][q]);
    if (c + 1 < ce) load(a.coils + (long)(c + 1) * a.n, cv);  // in flight during this coil's transform
    fft_regs<N, CT, NT, false>(v0, vo, s, s_tw);
    float2* const dst = a.dst + (long)c * a.dst_c_stride + (long)im * a.dst_img_stride;
#pragma unroll
    for (int it = 0; it < ITL; ++it) {
      const int g = tid + it * NT, x = x0 + GM::out_col(g);
      if (GM::out_ok(g) && x < a.nx) {
        int u[RL];  // looked up together: a lookup before each store would wait on its own
#pragma unroll
        for (int q = 0; q < RL; ++q) u[q] = s_li[GM::out_row(g, q)];
#pragma unroll
        for (int q = 0; q < RL; ++q) {
          if (u[q] >= 0) {
            const float2 v = cscale(vo[it][q], a.scale);
            dst[(long)u[q] * a.nx + x] = v;
            if constexpr (CG) dot += (double)v.x * v.x + (double)v.y * v.y;
          }
        }
      }
    }
    if (a.rows) {  // padding lines of the measurement layout
      for (int g = tid; g < (a.pad_rows - n_rows) * CT; g += NT) {
        const int u = n_rows + g / CT, x = x0 + g % CT;
        if (x < a.nx) dst[(long)u * a.nx + x] = make_float2(0.f, 0.f);
      }
    }
  }
  if constexpr (CG) {
    if (!a.dot) return;
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

// ---------------------------------------------------------------------------
// k-space rows -> image columns with the coil combine:
//   dst_img = scale_img * sum_c conj(s_c) o F_y^H (rows of src_{c,img} at their
//             ky, zeros elsewhere)
// over the coils of a group.  Grid: column tiles, images, coil groups.  The
// sampled rows enter the first radix pass straight from registers through
// the inverse row map in LDS, the coil-weighted sum is taken on the last
// pass's registers, and the next coil's rows are loaded during the current
// transform.  512 x 512, 16 coils, 24 frames: 219 us and the forward columns
// 185 us (578 and 301 us with every radix pass through LDS), bound by the
// radix arithmetic.  Each workgroup runs NG groups of NT threads on alternate coils,
// whose sums meet in LDS: the waves that one tile of columns can keep busy.  A
// coil in turn costs a round trip to memory, 2.5 us, so the short columns (one or
// two waves a tile) take up to eight coils at once.  32 frames of 16 x 16, 8
// coils: 7.5 us for the adjoint with its row pass; 26.6 us with one group and 16
// rows in a thread's registers, 12.4 us with every pass through LDS.
// CGLS: see ColAdjArgs (alpha from the shares of ||A p||^2, every wave the same).
// ---------------------------------------------------------------------------
template <int N, int CT, int NT, int NG, bool CGLS>
__global__ __launch_bounds__(NT * NG) void k_cols_adj(ColAdjArgs a) {
  using GM = FftGeom<N, CT, NT>;
  constexpr int IT0 = GM::IT0, R0 = GM::R0, ITL = GM::ITL, RL = GM::RL;
  constexpr int SUM = NG > 1 ? ITL * RL * NT : 1;  // a group's sums
  constexpr int LW = GM::LDS > SUM ? GM::LDS : SUM;
  __shared__ float2 s[NG][LW];
  __shared__ float2 s_tw[N];
  __shared__ int s_li[N];
  __shared__ double s_red[NT / 64];
  const int tid = threadIdx.x, ng = tid / NT, lt = tid % NT;
  const int x0 = xcd_tile(blockIdx.x, gridDim.x) * CT, im = blockIdx.y, img = a.img0 + im, grp = blockIdx.z;
  // a system starts from x = 0, also where an error keeps it from running
  if (CGLS && a.first && grp == 0) {
    float2* const xp = a.x + (long)img * a.n;
    for (int e = tid; e < N * CT; e += NT * NG) {
      const int x = x0 + e % CT;
      if (x < a.nx) xp[(e / CT) * a.nx + x] = make_float2(0.f, 0.f);
    }
  }
  const RowList rl(a.rows, a.rows_img_stride, a.m_k, img, tid);
  if (halted(a.st, 0)) return;  // (a mask that failed its checks at bind sets err)
  if (a.ista && a.ista->done) return;
  float al = 0.f;
  if constexpr (CGLS) {
    if (!a.first) {
      if (a.cg[img].done) return;
      const double d = wave_sum_parts(a.dot + (long)img * a.ndot, a.ndot, tid & 63);
      if (!(d > 0.0)) {  // A p = 0: the system stops
        if (blockIdx.x == 0 && grp == 0 && tid == 0) a.cg[img].brk = 1;
        return;
      }
      al = (float)(a.cg[img].gamma / d);
    }
    if (!a.first && grp == 0) {  // x over this tile
      float2* const xp = a.x + (long)img * a.n;
      const float2* const pp = a.p + (long)img * a.n;
      for (int e = tid; e < N * CT; e += NT * NG) {
        const int x = x0 + e % CT;
        if (x < a.nx) {
          const int o = (e / CT) * a.nx + x;
          const float2 xv = xp[o], pv = pp[o];
          xp[o] = make_float2(xv.x + al * pv.x, xv.y + al * pv.y);
        }
      }
    }
  }
  for (int e = tid; e < N; e += NT * NG) {
    s_tw[e] = a.tw[e];
    s_li[e] = a.rows ? -1 : e;
  }
  __syncthreads();
  if (a.rows) {
    rl.invert<N, NT * NG>(s_li, rl.mk / a.nx, tid);
    __syncthreads();
  }
  float2 acc[ITL][RL];
#pragma unroll
  for (int it = 0; it < ITL; ++it)
#pragma unroll
    for (int q = 0; q < RL; ++q) acc[it][q] = make_float2(0.f, 0.f);
  const int cb = grp * a.cgs, ce = min(a.nc, cb + a.cgs);
  // this thread's input rows: the line holding each, -1 for a zero row
  int li[IT0][R0];
#pragma unroll
  for (int it = 0; it < IT0; ++it) {
    const int g = lt + it * NT;
    const bool ok = GM::in_ok(g) && x0 + GM::in_col(g) < a.nx;
#pragma unroll
    for (int q = 0; q < R0; ++q) li[it][q] = ok ? s_li[GM::in_row(g, q)] : -1;
  }
  const long ioff = (long)im * a.src_img_stride + x0;
  float2 kv[IT0][R0];
  auto fetch = [&](int c) {  // valid addresses for every lane; zero rows selected afterwards
    const long o0 = ioff + (long)c * a.src_c_stride;
#pragma unroll
    for (int it = 0; it < IT0; ++it) {
      const int g = lt + it * NT, col = GM::in_col(g);
#pragma unroll
      for (int q = 0; q < R0; ++q) {
        const long o = o0 + (li[it][q] >= 0 ? (long)li[it][q] * a.nx + col : 0);
        float2 v = a.src[o];
        if constexpr (CGLS) {
          if (a.q) {
            const float2 qv = a.q[o];
            v = make_float2(v.x - al * qv.x, v.y - al * qv.y);
            if (li[it][q] >= 0) a.r[o] = v;
          }
        }
        kv[it][q] = li[it][q] >= 0 ? v : make_float2(0.f, 0.f);
      }
    }
  };
  // (with a whole column in its registers a thread has none for the next coil's)
  constexpr bool AHEAD = FftPlan<N>::P > 1;
  if (AHEAD && cb + ng < ce) fetch(cb + ng);
  // every group of threads runs the same number of rounds (the transforms'
  // barriers are the workgroup's); one past the last coil adds nothing
  for (int c0 = cb; c0 < ce; c0 += NG) {
    const int c = c0 + ng;
    float2 v0[IT0][R0], vo[ITL][RL];
    if (!AHEAD) {
      if (c >= ce) break;  // (one pass: no barriers to reach)
      fetch(c);
    }
#pragma unroll
    for (int it = 0; it < IT0; ++it)
#pragma unroll
      for (int q = 0; q < R0; ++q) v0[it][q] = c < ce ? kv[it][q] : make_float2(0.f, 0.f);
    if (AHEAD && c + NG < ce) fetch(c + NG);
    fft_regs<N, CT, NT, true, true>(v0, vo, s[ng], s_tw);
    // the coil values at the output rows come from the cache (every image
    // reads the same maps); loading them one coil ahead cost more in
    // registers than it saved
    if (c < ce) {
      const float2* coil = a.coils + (long)c * a.n + x0;
#pragma unroll
      for (int it = 0; it < ITL; ++it) {
        const int g = lt + it * NT, col = GM::out_col(g);
        if (GM::out_ok(g) && x0 + col < a.nx) {
#pragma unroll
          for (int q = 0; q < RL; ++q)
            acc[it][q] = cjfma(acc[it][q], coil[GM::out_row(g, q) * a.nx + col], vo[it][q]);
        }
      }
    }
  }
  if constexpr (NG > 1) {  // groups 1.. leave their sums in their (now free) LDS tiles
    if (ng > 0 && ng < ce - cb) {
#pragma unroll
      for (int it = 0; it < ITL; ++it)
#pragma unroll
        for (int q = 0; q < RL; ++q) s[ng][(it * RL + q) * NT + lt] = acc[it][q];
    }
    __syncthreads();
    if (ng == 0) {
#pragma unroll 1  // (one group's sums in registers at a time)
      for (int g2 = 1; g2 < min(NG, ce - cb); ++g2)
#pragma unroll
        for (int it = 0; it < ITL; ++it)
#pragma unroll
          for (int q = 0; q < RL; ++q) acc[it][q] = cadd(acc[it][q], s[g2][(it * RL + q) * NT + lt]);
    }
  }
  double nrm = 0.0;
  if (ng == 0) {
    float sc = a.scale;
    if (a.m_k_scale) sc *= (float)(1.0 / sqrt((double)a.m_k_scale[img] * a.st->mbar));
    float2* const dst = a.dst + (long)img * a.dst_img_stride + (long)grp * a.dst_part_stride + x0;
#pragma unroll
    for (int it = 0; it < ITL; ++it) {
      const int g = lt + it * NT, col = GM::out_col(g);
      if (GM::out_ok(g) && x0 + col < a.nx) {
#pragma unroll
        for (int q = 0; q < RL; ++q) {
          const float2 v = cscale(acc[it][q], sc);
          dst[GM::out_row(g, q) * a.nx + col] = v;
          if constexpr (CGLS) nrm += (double)v.x * v.x + (double)v.y * v.y;
        }
      }
    }
  }
  if constexpr (CGLS) {
    if (!a.nrm) return;
    nrm = wave_sum(nrm);
    if (tid < NT && (tid & 63) == 0) s_red[tid >> 6] = nrm;
    __syncthreads();
    if (tid == 0) {
      double t = 0.0;
      for (int w = 0; w < NT / 64; ++w) t += s_red[w];
      a.nrm[(long)img * gridDim.x + blockIdx.x] = t;
    }
  }
}

// ---------------------------------------------------------------------------
// general masks: the x transform of the k-space rows of an image together
// with the frame's sampling, TR rows of (coil, ky) per workgroup (grid: row
// tiles of an image, images):
//   IDX_FWD  y = the samples of F_x T        (stored as yin - y when yin is set)
//   IDX_ADJ  T = F_x^H of the samples on the grid, zero elsewhere
//   IDX_RES  T = F_x^H (yin - F_x T at the samples, zero elsewhere), in place
// The frame's map of locations to samples (imap) is read per row: the k-space
// grid itself is never filled, zeroed or gathered in memory.  CGLS: FWD adds
// its share of ||q||^2 to dot, ADJ takes r - alpha q and stores it as r.
// Bound by the rows' traffic; 64 frames of 8 coils, 128 x 128: 19 us forward
// and 28 us back (with r - alpha q), against 50 and 58 us for passes that gather
// from, zero and scatter to the k-space grid on their own.
// ---------------------------------------------------------------------------
template <int N, int TR, int NT, int MODE, bool CGLS>
__global__ __launch_bounds__(NT) void k_index_rows(IndexRowArgs a) {
  using GF = FftGeom<N, TR, NT, false, true>;
  constexpr int IT0 = GF::IT0, R0 = GF::R0, ITL = GF::ITL, RL = GF::RL;
  __shared__ float2 s[GF::LDS];
  __shared__ float2 s_tw[N];
  __shared__ double s_red[NT / 64];
  const int tid = threadIdx.x, im = blockIdx.y, img = a.img0 + im;
  const int nrows = a.nc * a.ny, row0 = blockIdx.x * TR;
  if (halted(a.st, 0)) return;
  if (a.ista && a.ista->done) return;
  float al = 0.f;
  if constexpr (CGLS) {
    if (a.cg && a.cg[img].done) return;
    if (MODE == IDX_ADJ && a.q) {
      const double d = wave_sum_parts(a.dot + (long)img * a.ndot, a.ndot, tid & 63);
      if (!(d > 0.0)) return;  // the columns' launch records the stop
      al = (float)(a.cg[img].gamma / d);
    }
  }
  float2* const T = a.T + (long)im * a.nc * a.n;
  const int32_t* const map = a.imap + (long)img * a.n;
  const long y0 = (long)img * a.nc * a.m_max;
  float2 v0[IT0][R0], vo[ITL][RL];
  // T's rows, from valid addresses; rows past the image are zeroed
  if constexpr (MODE != IDX_ADJ) {
#pragma unroll
    for (int it = 0; it < IT0; ++it) {
      const int g = tid + it * NT, row = row0 + GF::in_col(g);
      const bool ok = GF::in_ok(g) && row < nrows;
      const float2* src = T + (ok ? (long)row * N + GF::in_row(g, 0) : 0);
#pragma unroll
      for (int q = 0; q < R0; ++q) {
        const float2 v = src[ok ? q * (N / R0) : 0];
        v0[it][q] = ok ? v : make_float2(0.f, 0.f);
      }
    }
  }
  for (int e = tid; e < N; e += NT) s_tw[e] = a.tw[e];
  // the samples of this thread's k-space positions, in the forward
  // transform's output layout (= the reversed plan's input layout)
  int sm[ITL][RL];
  int yc[ITL];  // offset of the row's coil in the frame's measurements
#pragma unroll
  for (int it = 0; it < ITL; ++it) {
    const int g = tid + it * NT, row = row0 + GF::out_col(g);
    const bool ok = GF::out_ok(g) && row < nrows;
    const int c = ok ? row / a.ny : 0, ky = ok ? row - c * a.ny : 0;
    yc[it] = c * a.m_max;
#pragma unroll
    for (int q = 0; q < RL; ++q) {
      const int e = map[ky * N + (ok ? GF::out_row(g, q) : 0)];
      sm[it][q] = ok ? e : -1;
    }
  }
  __syncthreads();
  if constexpr (MODE != IDX_ADJ) fft_regs<N, TR, NT, false, false, false, true>(v0, vo, s, s_tw);
  double dot = 0.0;
  int n_cut = 0;
  const double gamma = a.trunc ? a.st->gamma : 0.0;
#pragma unroll
  for (int it = 0; it < ITL; ++it)
#pragma unroll
    for (int q = 0; q < RL; ++q) {
      const int e = sm[it][q];
      if constexpr (MODE == IDX_FWD) {
        if (e >= 0) {
          float2 v = cscale(vo[it][q], a.scale);
          if constexpr (CGLS) dot += (double)v.x * v.x + (double)v.y * v.y;
          const long o = y0 + yc[it] + e;
          if (a.yin) v = csub(a.yin[o], v);
          a.y[o] = v;
        }
      } else {
        float2 v = make_float2(0.f, 0.f);
        if (e >= 0) {
          const long o = y0 + yc[it] + e;
          v = a.yin[o];
          if constexpr (MODE == IDX_RES) v = csub(v, cscale(vo[it][q], a.scale));
          if (CGLS && a.q) {
            const float2 qv = a.q[o];
            v = make_float2(v.x - al * qv.x, v.y - al * qv.y);
            a.r[o] = v;
          }
          if (a.trunc && (double)v.x * v.x + (double)v.y * v.y > gamma) {
            v = make_float2(0.f, 0.f);
            ++n_cut;
          }
        }
        vo[it][q] = v;
      }
    }
  if constexpr (MODE == IDX_FWD) {
    // the padding of the frame's measurements
    const int mk = a.m_k[img];
    for (int c = blockIdx.x; c < a.nc; c += gridDim.x)
      for (int e = mk + tid; e < a.m_max; e += NT) a.y[y0 + (long)c * a.m_max + e] = make_float2(0.f, 0.f);
    if constexpr (CGLS) {
      dot = wave_sum(dot);
      if ((tid & 63) == 0) s_red[tid >> 6] = dot;
      __syncthreads();
      if (tid == 0) {
        double t = 0.0;
        for (int w = 0; w < NT / 64; ++w) t += s_red[w];
        a.dot[(long)img * gridDim.x + blockIdx.x] = t;
      }
    }
  } else {
    if (n_cut && a.trunc_count) atomicAdd(a.trunc_count, n_cut);
    fft_regs<N, TR, NT, true, true, true, true>(vo, v0, s, s_tw);
#pragma unroll
    for (int it = 0; it < IT0; ++it) {
      const int g = tid + it * NT, row = row0 + GF::in_col(g);
      if (GF::in_ok(g) && row < nrows) {
#pragma unroll
        for (int q = 0; q < R0; ++q) T[(long)row * N + GF::in_row(g, q)] = cscale(v0[it][q], a.scale);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// host-side dispatch over the transform length
// ---------------------------------------------------------------------------
int op_tile(int N) {
  switch (N) {
    case 8: return OpTile<8>::CT;
    case 16: return OpTile<16>::CT;
    case 32: return OpTile<32>::CT;
    case 64: return OpTile<64>::CT;
    case 128: return OpTile<128>::CT;
    case 256: return OpTile<256>::CT;
    default: return OpTile<512>::CT;
  }
}

namespace {

template <int N>
hipError_t rows_n(const RowArgs& a, bool inv, hipStream_t st) {
  constexpr int TR = OpTile<N>::CT, NT = OpTile<N>::NT;
  const dim3 grid((unsigned)((a.nrows + TR - 1) / TR));
  if (inv) hipLaunchKernelGGL((k_rows<N, TR, NT, true>), grid, dim3(NT), 0, st, a);
  else hipLaunchKernelGGL((k_rows<N, TR, NT, false>), grid, dim3(NT), 0, st, a);
  return hipGetLastError();
}

template <int N>
hipError_t fwd_n(const ColFwdArgs& a, bool cg, int images, hipStream_t st) {
  constexpr int CT = OpTile<N>::CT, NT = OpTile<N>::NT;
  const dim3 grid((a.nx + CT - 1) / CT, images, (a.nc + a.cgs - 1) / a.cgs);
  if (cg) hipLaunchKernelGGL((k_cols_fwd<N, CT, NT, true>), grid, dim3(NT), 0, st, a);
  else hipLaunchKernelGGL((k_cols_fwd<N, CT, NT, false>), grid, dim3(NT), 0, st, a);
  return hipGetLastError();
}

template <int N>
hipError_t adj_n(const ColAdjArgs& a, bool cgls, int images, hipStream_t st) {
  constexpr int CT = OpTile<N>::CT, NT = OpTile<N>::NT;
  constexpr int NG = N >= 64 ? 2 : N == 32 ? 4 : 8;
  const dim3 grid((a.nx + CT - 1) / CT, images, (a.nc + a.cgs - 1) / a.cgs);
  if (a.cgs == 1) {  // one coil per workgroup: one group of threads
    if (cgls) hipLaunchKernelGGL((k_cols_adj<N, CT, NT, 1, true>), grid, dim3(NT), 0, st, a);
    else hipLaunchKernelGGL((k_cols_adj<N, CT, NT, 1, false>), grid, dim3(NT), 0, st, a);
  } else {
    if (cgls) hipLaunchKernelGGL((k_cols_adj<N, CT, NT, NG, true>), grid, dim3(NT * NG), 0, st, a);
    else hipLaunchKernelGGL((k_cols_adj<N, CT, NT, NG, false>), grid, dim3(NT * NG), 0, st, a);
  }
  return hipGetLastError();
}

template <int N>
hipError_t idx_n(const IndexRowArgs& a, int mode, bool cgls, int images, hipStream_t st) {
  constexpr int TR = OpTile<N>::CT, NT = OpTile<N>::NT;
  const dim3 g((a.nc * a.ny + TR - 1) / TR, images);
  if (mode == IDX_FWD && cgls) hipLaunchKernelGGL((k_index_rows<N, TR, NT, IDX_FWD, true>), g, dim3(NT), 0, st, a);
  else if (mode == IDX_FWD) hipLaunchKernelGGL((k_index_rows<N, TR, NT, IDX_FWD, false>), g, dim3(NT), 0, st, a);
  else if (mode == IDX_ADJ && cgls) hipLaunchKernelGGL((k_index_rows<N, TR, NT, IDX_ADJ, true>), g, dim3(NT), 0, st, a);
  else if (mode == IDX_ADJ) hipLaunchKernelGGL((k_index_rows<N, TR, NT, IDX_ADJ, false>), g, dim3(NT), 0, st, a);
  else hipLaunchKernelGGL((k_index_rows<N, TR, NT, IDX_RES, false>), g, dim3(NT), 0, st, a);
  return hipGetLastError();
}

}  // namespace

#define OP_DISPATCH(fn, N, ...)              \
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

hipError_t launch_rows(int N, const RowArgs& a, bool inv, hipStream_t st) {
  if (a.nrows <= 0) return hipSuccess;
  OP_DISPATCH(rows_n, N, a, inv, st);
}

hipError_t launch_cols_fwd(int N, const ColFwdArgs& args, bool cg, int images, hipStream_t st) {
  if (images <= 0) return hipSuccess;
  ColFwdArgs a = args;
  if (a.cgs <= 0) {  // enough coil groups for about four workgroups per compute unit (no sum to pay for)
    const long tiles = (long)((a.nx + op_tile(N) - 1) / op_tile(N)) * images;
    const int want = (int)std::max(1L, std::min<long>(a.nc, (1024 + tiles - 1) / tiles));
    a.cgs = (a.nc + want - 1) / want;
  }
  OP_DISPATCH(fwd_n, N, a, cg, images, st);
}

hipError_t launch_cols_adj(int N, const ColAdjArgs& args, bool cgls, int images, hipStream_t st) {
  if (images <= 0) return hipSuccess;
  ColAdjArgs a = args;
  if (a.cgs <= 0) a.cgs = a.nc;
  OP_DISPATCH(adj_n, N, a, cgls, images, st);
}

hipError_t launch_index_rows(int N, const IndexRowArgs& a, int mode, bool cgls, int images, hipStream_t st) {
  if (images <= 0) return hipSuccess;
  OP_DISPATCH(idx_n, N, a, mode, cgls, images, st);
}

}  // namespace ag
