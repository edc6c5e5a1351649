// The index tables of a bound problem, the QR step fused with the update, and
// the spectral initialisation's q x q eigenproblem with the helpers around it.
#include "kernels_core.hpp"

namespace ag {


// ===========================================================================
// setup: inverse sampling map
// A "location" is a phase-encode line ky (LINES) or a flat k-space index
// (INDEX).  For every location the list of (frame k, position e) samples
// that hit it is stored contiguously, in increasing k (deterministic).
// ===========================================================================
__device__ __forceinline__ void state_reset(DevState* st, int full) {
  if (full) {
    st->err = 0;
    st->err_frame = -1;
    st->n_units = 0;
    st->n_gwork = 0;
  }
  st->halt = 0;
  st->step_ok = 0;
  st->t = 0;
  st->exited = 0;
  st->converged = 0;
  st->eta = -1.0;
  st->step_flags = 0;
  st->eta_next = -1.0;
  st->f = 0.0;
  st->sd = 0.0;
  st->grad_norm = 0.0;
  st->stats_pending = 0;
  st->n_trunc = 0;
  st->exit_run = 0;
}

// What needs nothing but the arguments, in one launch: the state, the twiddle
// tables tw[t] = exp(-2 pi i t / N) (from a double-precision sincospi), the coil
// maps in the layout the basis transforms read ([c][x / txx][y][x % txx], so that a
// workgroup's txx columns are one contiguous block per coil), the zeroed
// bitmap and (general masks) the map of locations to samples set to -1.
__global__ __launch_bounds__(256) void k_bind_begin(BindArgs a) {
  const long t0 = (long)blockIdx.x * 256 + threadIdx.x, nt = (long)gridDim.x * 256;
  if (t0 == 0) state_reset(a.st, 1);
  if (t0 < a.nx + a.ny) {
    const int N = t0 < a.nx ? a.nx : a.ny, t = t0 < a.nx ? (int)t0 : (int)t0 - a.nx;
    double s, c;
    sincospi(2.0 * (double)t / (double)N, &s, &c);
    (t0 < a.nx ? a.twx : a.twy)[t] = make_float2((float)c, (float)(-s));
  }
  for (long e = t0; e < (long)a.n_loc * a.nw; e += nt) a.bitmap[e] = 0;
  if (a.imap)
    for (long e = t0; e < (long)a.q * a.n; e += nt) a.imap[e] = -1;
  for (long e = t0; e < a.n * a.nc; e += nt) {
    const long c = e / a.n, rem = e - c * a.n;
    const long xg = rem / ((long)a.ny * a.txx), rem2 = rem - xg * a.ny * a.txx;
    const int y = (int)(rem2 / a.txx), xl = (int)(rem2 - (long)y * a.txx);
    a.coilb[e] = a.coils[c * a.n + (long)y * a.nx + xg * a.txx + xl];
  }
}

// the masks' bits (a workgroup per 256 entries of a frame: blocks 0 ..
// nb q - 1), and with measurements ||y_{k,c}||^2 in FP64 (the next q nc blocks)
__global__ __launch_bounds__(256) void k_bind_mask(BindArgs a) {
  __shared__ double red[4];
  const int nb = (a.width + 255) / 256, tid = threadIdx.x;
  if ((int)blockIdx.x >= nb * a.q) {
    const int kc = blockIdx.x - nb * a.q, k = kc / a.nc;
    const int mk = min(max(a.m_k[k], 0), a.m_max);
    const float2* yk = a.y + (long)kc * a.m_max;
    double s = 0.0;
#pragma unroll 8
    for (int i = tid; i < mk; i += 256) {
      const float2 v = yk[i];
      s += (double)v.x * v.x + (double)v.y * v.y;
    }
    s = wave_sum(s);
    if ((tid & 63) == 0) red[tid >> 6] = s;
    __syncthreads();
    if (tid == 0) a.ysqp[kc] = (red[0] + red[1]) + (red[2] + red[3]);
    return;
  }
  const int e = (blockIdx.x % nb) * 256 + tid, k = blockIdx.x / nb;
  const int mk = a.m_k[k];
  if (mk < 0 || mk > a.width * a.per || (mk % a.per) != 0) {
    if (e == 0) set_error(a.st, 1 /*EINVAL: bad m_k*/, k);
    return;
  }
  if (e >= mk / a.per) return;
  const int loc = a.mask[(long)k * a.width + e];
  if (loc < 0 || loc >= a.n_loc) {
    set_error(a.st, 1 /*EINVAL*/, k);
    return;
  }
  const uint32_t bit = 1u << (k & 31);
  const uint32_t old = atomicOr(&a.bitmap[(long)loc * a.nw + (k >> 5)], bit);
  if (old & bit) set_error(a.st, 1 /*EINVAL: repeated location in a frame*/, k);
}

// ||y_k||^2 (its coils' parts in order), gamma = trunc_c * sum |y|^2 / (m q) with
// m = max_k m_k, and mbar = sum_k m_k / q, by one workgroup (q <= 128 <= threads)
__device__ __forceinline__ void bind_stats(const BindArgs& a) {
  __shared__ double s_ys[128];
  __shared__ int s_mk[128];
  const int tid = threadIdx.x;
  if (!a.y) return;
  if (tid < a.q) {
    double s = 0.0;
    for (int c = 0; c < a.nc; ++c) s += a.ysqp[(long)tid * a.nc + c];
    a.ysq_k[tid] = s;
    s_ys[tid] = s;
    s_mk[tid] = a.m_k[tid];
  }
  __syncthreads();
  if (tid != 0) return;
  double ys = 0.0, msum = 0.0;
  int mmax = 0;
  for (int k = 0; k < a.q; ++k) {
    ys += s_ys[k];
    msum += s_mk[k];
    mmax = max(mmax, s_mk[k]);
  }
  a.st->ysq = ys;
  a.st->mbar = msum / a.q;
  a.st->gamma = a.trunc_c > 0 ? a.trunc_c * ys / ((double)mmax * a.q) : INFINITY;
}

// inclusive scan of v over the 1024 threads of the workgroup (s_w: 16 ints)
__device__ __forceinline__ int block_scan(int v, int* s_w) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int off = 1; off < 64; off <<= 1) {
    const int u = __shfl_up(v, off);
    if (lane >= off) v += u;
  }
  __syncthreads();
  if (lane == 63) s_w[wv] = v;
  __syncthreads();
  for (int w = 0; w < wv; ++w) v += s_w[w];
  return v;
}

// rank of frame k among the frames that sample location loc
__device__ __forceinline__ int frame_rank(const uint32_t* bm, int k) {
  int rank = 0;
  for (int w = 0; w < (k >> 5); ++w) rank += __popc(bm[w]);
  return rank + __popc(bm[k >> 5] & ((1u << (k & 31)) - 1u));
}

// Line masks, the rest of the index tables by one workgroup (n_loc = ny <=
// 512 lines, one per thread): the lines' pair counts and offsets, the sampled
// lines (units) in order, the Gram kernel's work items (unit u, tile t of 8 of
// its pairs), the fold's dispatch order (units by pair count, the largest
// first, ties by index, then the unsampled rows, so that the longest fold
// workgroups start first instead of ending the launch), every frame's pairs,
// and the data's statistics.  15 launches of a bind became 5.
__global__ __launch_bounds__(1024) void k_bind_lines(BindArgs a) {
  __shared__ int s_w[16], s_ptr[512], s_unit[512], s_np[512], s_p0[512], s_nu;
  const int tid = threadIdx.x;
  int c = 0;
  if (tid < a.n_loc)
    for (int w = 0; w < a.nw; ++w) c += __popc(a.bitmap[(long)tid * a.nw + w]);
  const int pc = block_scan(c, s_w) - c, pu = block_scan(c > 0, s_w) - (c > 0);
  if (tid < a.n_loc) {
    a.loc_ptr[tid] = pc;
    a.loc2unit[tid] = c > 0 ? pu : -1;
    s_ptr[tid] = pc;
    s_unit[tid] = c > 0 ? pu : -1;
    if (c > 0) {
      s_np[pu] = c;
      s_p0[pu] = pc;
    }
    if (tid == a.n_loc - 1) {
      a.loc_ptr[a.n_loc] = pc + c;
      s_nu = pu + (c > 0);
      a.st->n_units = s_nu;
    }
  }
  __syncthreads();
  const int nu = s_nu, np = tid < nu ? s_np[tid] : 0, nt = (np + 7) / 8;
  const int o1 = block_scan(nt, s_w);
  for (int t = 0; t < nt; ++t) a.items[o1 - nt + t] = make_int4(tid, t, s_p0[tid], np);
  if (tid == 1023) a.st->n_gwork = o1;
  if (tid < nu) {
    int rk = 0;
    for (int v = 0; v < nu; ++v) rk += (s_np[v] > np) || (s_np[v] == np && v < tid);
    a.line_order[rk] = make_int4(tid, s_p0[tid], np, 0);
  } else if (tid < a.n_loc) {
    a.line_order[tid] = make_int4(tid, 0, 0, 0);
  }
  if (!a.st->err) {  // (a mask that failed its checks has no valid pairs)
    for (int i = tid; i < a.q * a.width; i += 1024) {
      const int k = i / a.width, e = i - k * a.width;
      if (e >= a.m_k[k] / a.per) continue;
      const int loc = a.mask[i], pos = s_ptr[loc] + frame_rank(a.bitmap + (long)loc * a.nw, k);
      a.pairs[pos] = make_int2(k, e);
      a.pair_of[i] = pos;
      a.unit_of[i] = s_unit[loc];
    }
  }
  bind_stats(a);
}

// General masks: the locations' sample counts and their exclusive prefix sums (pairs per
// location), and the sampled locations (units) numbered in order; one block
// of 1024 threads over tiles of 1024 locations, scans within waves by
// shuffles, a running total across tiles
__global__ __launch_bounds__(1024) void k_bind_index(BindArgs a) {
  const uint32_t* const bitmap = a.bitmap;
  const int nw = a.nw, n_loc = a.n_loc;
  int32_t* const loc_ptr = a.loc_ptr;
  int32_t* const loc2unit = a.loc2unit;
  constexpr int LPT = 1;  // locations per thread and tile (4: slower, the loads less coalesced)
  __shared__ int s_wc[16], s_wu[16];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  int carry_c = 0, carry_u = 0;  // totals of the tiles before this one
  for (int base = 0; base < n_loc; base += 1024 * LPT) {
    const int l0 = base + LPT * tid;
    int cs[LPT], tc = 0, tu = 0;
#pragma unroll
    for (int s2 = 0; s2 < LPT; ++s2) {
      const int l = l0 + s2, lc = min(l, n_loc - 1);
      int c = 0;
      for (int w = 0; w < nw; ++w) c += __popc(bitmap[(long)lc * nw + w]);
      cs[s2] = l < n_loc ? c : 0;
      tc += cs[s2];
      tu += cs[s2] > 0;
    }
    int sc = tc, su = tu;  // inclusive scans over the wave
    for (int off = 1; off < 64; off <<= 1) {
      const int vc = __shfl_up(sc, off), vu = __shfl_up(su, off);
      if (lane >= off) {
        sc += vc;
        su += vu;
      }
    }
    if (lane == 63) {
      s_wc[wv] = sc;
      s_wu[wv] = su;
    }
    __syncthreads();
    int pc = carry_c + sc - tc, pu = carry_u + su - tu;  // exclusive prefixes of this thread's first location
    for (int w2 = 0; w2 < 16; ++w2) {
      const int vc = s_wc[w2], vu = s_wu[w2];
      if (w2 < wv) {
        pc += vc;
        pu += vu;
      }
      carry_c += vc;
      carry_u += vu;
    }
#pragma unroll
    for (int s2 = 0; s2 < LPT; ++s2) {
      const int l = l0 + s2, c = cs[s2];
      if (l < n_loc) {
        loc_ptr[l] = pc;
        if (c > 0) {
          loc2unit[l] = pu;
          ++pu;
        } else {
          loc2unit[l] = -1;
        }
      }
      pc += c;
    }
    __syncthreads();  // the wave totals are read before the next tile writes them
  }
  if (tid == 0) {
    loc_ptr[n_loc] = carry_c;
    a.st->n_units = carry_u;
  }
  bind_stats(a);
}

// general masks: every frame's pairs and its map of locations to samples
__global__ __launch_bounds__(256) void k_bind_fill(BindArgs a) {
  const int e = blockIdx.x * 256 + threadIdx.x, k = blockIdx.y;
  if (a.st->err) return;
  if (e >= a.m_k[k] / a.per) return;
  const int loc = a.mask[(long)k * a.width + e];
  const int pos = a.loc_ptr[loc] + frame_rank(a.bitmap + (long)loc * a.nw, k);
  a.pairs[pos] = make_int2(k, e);
  a.pair_of[(long)k * a.width + e] = pos;
  a.unit_of[(long)k * a.width + e] = a.loc2unit[loc];
  a.imap[(long)k * a.n_loc + loc] = e;
}

__global__ void k_state_reset(DevState* st, int full) {
  if (threadIdx.x == 0) state_reset(st, full);
}

__global__ void k_state_set_eta(DevState* st, double eta) {
  if (threadIdx.x == 0) st->eta = eta;
}

// reciprocal in FP64 from the hardware estimate (v_rcp_f64) refined by two
// Newton steps, to about one ulp: a shorter dependent chain than the
// IEEE-exact division
__device__ __forceinline__ double rcp_nr(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(y, fma(-x, y, 1.0), y);
  y = fma(y, fma(-x, y, 1.0), y);
  return y;
}
// The largest eigenvalue of the Hermitian positive semidefinite r x r matrix M
// (LDS, rows of 16, destroyed; S is scratch of the same shape) by the whole
// workgroup (256 threads or more): M is scaled to unit trace and squared until
// it is rank one to rounding, or 30 times, by when eigenvalues closer to the
// largest than 1e-8 of it are all that is left beside it; the result is the
// weighted mean tr(M^p A) / tr(M^p) of A = M's eigenvalues.  Each squaring is one
// short product in LDS, where a cyclic Jacobi takes r rotation rounds a sweep.
// A matrix whose trace is not finite gives its largest diagonal entry: an
// overflow stays infinite, and the factor of the step it leads to fails and is
// reported (zero would pass for a stationary start).
__device__ __forceinline__ double spectral_norm2(double2* M, double2* S, double2* A, int r) {
  const int tid = threadIdx.x, i = (tid >> 4) & 15, j = tid & 15;
  const bool in = tid < 256 && i < r && j < r;
  auto trace = [&](const double2* X) {
    double t = 0.0;
#pragma unroll 8
    for (int k = 0; k < r; ++k) t += X[k * 16 + k].x;
    return t;
  };
  if (in) A[i * 16 + j] = M[i * 16 + j];
  double t = trace(M);
  if (!(t > 0.0) || !isfinite(t)) {  // the same in every thread
    double m = 0.0;
    for (int k = 0; k < r; ++k) m = fmax(m, M[k * 16 + k].x);
    return m;
  }
  for (int it = 0; it < 30; ++it) {
    double2 v = make_double2(0.0, 0.0);
    if (in) {
#pragma unroll 8
      for (int k = 0; k < r; ++k) v = dadd(v, dmul(M[i * 16 + k], M[k * 16 + j]));
    }
    if (in) S[i * 16 + j] = make_double2(v.x / t / t, v.y / t / t);
    __syncthreads();
    double2* const w = M;
    M = S;
    S = w;
    t = trace(M);  // sum of squared eigenvalue weights: 1 when one weight holds all
    if (!(t < 1.0 - 1e-14)) break;
  }
  // every wave the same sum: lane l's entries in order, then over the lanes
  double num = 0.0;
  for (int e = tid & 63; e < r * 16; e += 64)
    if ((e & 15) < r) num += M[e].x * A[e].x + M[e].y * A[e].y;
  return wave_sum(num) / t;
}

// entry e = (i, j) of R = L^H with the reciprocal on the diagonal, from the
// lower Cholesky factor L (LDS, row pitch CHOL_LD): the form the update solves with
__device__ __forceinline__ float2 rfac_entry(const double2* L, int r, int e) {
  const int i = e / r, j = e - (e / r) * r;
  if (i < j) return make_float2((float)L[j * CHOL_LD + i].x, -(float)L[j * CHOL_LD + i].y);
  if (i == j) return make_float2((float)(1.0 / L[i * CHOL_LD + i].x), 0.f);
  return make_float2(0.f, 0.f);
}

// ||U^H U+||_F^2 = ||(U^H U - eta U^H G) R^{-1}||_F^2, lanes l < r taking
// row l by forward substitution with R = L^H (L in Gh, row pitch CHOL_LD;
// x is a row scratch of stride 16); the caller sums over the wave.  The
// fused step and the deferred statistics both use it, so that SD is the
// same number either way.
__device__ __forceinline__ double sd_row_sum(const double2* UU, const double2* UG, const double2* Gh, double2* Tm,
                                             double eta, int r, int l) {
  double fro = 0.0;
  if (l < r) {
    double2* x = Tm + l * 16;
    for (int j = 0; j < r; ++j) {
      double2 acc = make_double2(UU[l * 16 + j].x - eta * UG[l * 16 + j].x, UU[l * 16 + j].y - eta * UG[l * 16 + j].y);
      for (int k = 0; k < j; ++k) acc = dsub(acc, dmul(x[k], dconj(Gh[j * CHOL_LD + k])));
      const double rd = 1.0 / Gh[j * CHOL_LD + j].x;
      const double2 xj = make_double2(acc.x * rd, acc.y * rd);
      x[j] = xj;
      fro += xj.x * xj.x + xj.y * xj.y;
    }
  }
  return fro;
}

// ---------------------------------------------------------------------------
// tot[o] = sum over the nblk QR Gram partials (FP32 pairs when f32, else
// FP64) of nout complex entries, in FP64; workgroup wg of nwg takes a range
// of the 16-byte units (one or two entries).  Thread = (unit, slice): slice
// sl sums partials sl, sl + NS, sl + 2 NS, ... in that order, with PL loads
// in flight (issued from clamped, valid addresses before any is used), and
// the slices are then added in order.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void unit_add(double2& a0, double2&, const double2 w) { a0 = dadd(a0, w); }
__device__ __forceinline__ void unit_add(double2& a0, double2&, const float2 w) { a0 = dadd(a0, f2d(w)); }
__device__ __forceinline__ void unit_add(double2& a0, double2& a1, const float4 w) {
  a0 = dadd(a0, make_double2(w.x, w.y));
  a1 = dadd(a1, make_double2(w.z, w.w));
}

template <int PL, typename L>
__device__ __forceinline__ void slice_sum(const L* src, int nblk, int nunit, int u, int sl, int NS, double2& a0,
                                          double2& a1) {
  for (int b0 = sl; b0 < nblk; b0 += NS * PL) {
    L w[PL];
#pragma unroll
    for (int k = 0; k < PL; ++k) w[k] = src[(long)min(b0 + k * NS, nblk - 1) * nunit + u];
#pragma unroll
    for (int k = 0; k < PL; ++k)
      if (b0 + k * NS < nblk) unit_add(a0, a1, w[k]);
  }
}

template <int NT>
__device__ __forceinline__ void partials_sum(const double2* part, int f32, int nblk, int nout, double2* tot, int wg,
                                             int nwg) {
  constexpr int PL = 16;
  static_assert(NT <= 256, "16 loads of 16 bytes in flight per thread need more than 1024-thread workgroups allow");
  __shared__ double2 s_sum[2][NT];
  const int tid = threadIdx.x;
  const int per = (f32 && (nout & 1) == 0) ? 2 : 1;  // outputs per load
  const int nunit = nout / per, cu = (nunit + nwg - 1) / nwg, ub = wg * cu, ue = min(nunit, ub + cu);
  const int nu = max(0, ue - ub);
  const int NS = max(1, min(32, NT / max(nu, 1))), OW = NT / NS;  // (at most 32 slices: their sum is serial)
  for (int u0 = 0; u0 < nu; u0 += OW) {
    const int u = ub + u0 + tid % OW, sl = tid / OW, uc = min(u, ue - 1);
    double2 a0 = make_double2(0.0, 0.0), a1 = a0;
    if (sl < NS) {
      if (!f32) slice_sum<PL>(part, nblk, nunit, uc, sl, NS, a0, a1);
      else if (per == 2) slice_sum<PL>(reinterpret_cast<const float4*>(part), nblk, nunit, uc, sl, NS, a0, a1);
      else slice_sum<PL>(reinterpret_cast<const float2*>(part), nblk, nunit, uc, sl, NS, a0, a1);
    }
    s_sum[0][tid] = a0;
    s_sum[1][tid] = a1;
    __syncthreads();
    if (sl == 0 && u < ue) {
      for (int q = 1; q < NS; ++q) {
        a0 = dadd(a0, s_sum[0][tid + q * OW]);
        a1 = dadd(a1, s_sum[1][tid + q * OW]);
      }
      tot[u * per] = a0;
      if (per == 2) tot[u * per + 1] = a1;
    }
    __syncthreads();
  }
}

// ===========================================================================
// the QR step fused with the update: every workgroup takes the summed Gram of
// [U G] and the step size (Algorithm 2's rule at t = 1, then the stored one),
// factors Uhat^H Uhat = L L^H in one wave, and solves U+ R = U - eta grad for its
// 256 pixels, R = L^H.  Every workgroup computes the same factor from the same
// sum in the same order.  With the exit rule on, workgroup 0 also forms
// SD(U, U+) and the cost, and the outcome (applied, exit rule, stationary
// start) and the step size go to step_flags / eta_next and are committed by
// k_step_commit, because a halt written during the launch would stop
// workgroups that have not yet updated their pixels.  With it off
// (commit_direct), workgroup 0 commits t and eta itself: t is read by no
// workgroup, and a workgroup that reads the new eta instead of the unset one
// gets the value it would have computed (the same rule on the same sum,
// bitwise); the stationary start halts every workgroup alike.  SD, the cost
// and ||grad|| are then only reported: their inputs (r x r matrices and the
// frames' costs, which a later solve overwrites) are stored and k_stats_finish
// forms them on request.
//
// STEP_MODE_QR: U+ = CholeskyQR of src (the sum is the Gram of src alone, a
// small ridge is added if it is numerically singular; U+ = src where an error
// is pending or the factor fails all the same).  STEP_MODE_ETA (one
// workgroup): only the step size is set.
//
// The factor's wave takes its entries straight from the sum (a lane's four
// rows of loads in flight at once); the other waves' pixels wait for it at one
// barrier.  Bound by the latency of that chain.  Rank 16, 256 x 256: 25 us with
// the partials' sum, against 61 us for a one-workgroup factor and a separate
// update; rank 8: 11.3 us, 12.2 us with the Gram staged in LDS by the workgroup.
// ===========================================================================
template <int RT, bool SUM>
__global__ __launch_bounds__(256) void k_step_apply(QrSmallArgs a, ApplyArgs ap) {
  __shared__ double2 L[16 * CHOL_LD], W0[256], W1[256], W2[256];
  __shared__ float2 Rf[RT * RT];
  __shared__ int s_ok;
  __shared__ double s_eta;
  const int tid = threadIdx.x, r = a.r, l = tid & 63, ri = l & 15, rg = l >> 4;
  DevState* st = a.st;
  const long n = ap.n, p = (long)blockIdx.x * 256 + tid, pc = min(p, n - 1);
  const bool step = a.mode != STEP_MODE_QR;
  const int m = step ? 2 * r : r;
  // the state, this pixel's basis row and gradient and the factor's entries
  // are requested first (clamped, valid addresses); the state's loads are in
  // every thread, so that no branch waits on them
  const int err0 = st->err;
  const int halt0 = __hip_atomic_load(&st->halt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const double eta0 = __hip_atomic_load(&st->eta, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // ... and, for the deferred statistics, a frame's cost per thread of workgroup 0's last two waves
  const bool keep_cost = blockIdx.x == 0 && step && a.commit_direct && tid >= 128 && tid - 128 < a.q;
  double cost = 0.0;
  if (keep_cost) cost = a.cost_k[tid - 128];
  float2 u0[RT], g0[RT];
  if (a.mode != STEP_MODE_ETA) {
#pragma unroll
    for (int i = 0; i < RT; ++i) u0[i] = (i < r) ? ap.src[(long)i * n + pc] : make_float2(0.f, 0.f);
    if (!step) {
#pragma unroll
      for (int i = 0; i < RT; ++i) g0[i] = make_float2(0.f, 0.f);
    } else if ((r & 1) == 0) {  // the pixel-major gradient row as 16-byte loads
      const float4* gs = reinterpret_cast<const float4*>(ap.G + pc * r);
#pragma unroll
      for (int h = 0; h < RT / 2; ++h) {
        const float4 w = 2 * h < r ? gs[h] : make_float4(0.f, 0.f, 0.f, 0.f);
        g0[2 * h] = make_float2(w.x, w.y);
        g0[2 * h + 1] = make_float2(w.z, w.w);
      }
    } else {
#pragma unroll
      for (int i = 0; i < RT; ++i) g0[i] = (i < r) ? ap.G[pc * r + i] : make_float2(0.f, 0.f);
    }
  }
  __shared__ double2 s_tot[SUM ? 16 * 33 : 1];
  if constexpr (SUM) partials_sum<256>(a.part, a.part_f32, a.nblk, m * (m + 1) / 2, s_tot, 0, 1);
  // entry (x, y) of the Hermitian Gram, from its upper triangle in tri order
  auto gram = [&](int x, int y) -> double2 {
    const int lo = min(x, y), hi = max(x, y), e = lo * m - lo * (lo - 1) / 2 + (hi - lo);
    const double2 v = SUM ? s_tot[e] : a.part[e];
    return make_double2(v.x, x <= y ? v.y : -v.y);
  };
  // this lane's entries (ri, 4 t + rg) of U^H U, U^H G, G^H U and G^H G
  double2 uu[4], ug[4], gu[4], gg[4];
  if (tid < 64) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int x = min(ri, r - 1), y = min(4 * t + rg, r - 1);
      uu[t] = gram(x, y);
      if (step) {
        ug[t] = gram(x, r + y);
        gu[t] = gram(r + x, y);
        gg[t] = gram(r + x, r + y);
      }
    }
  }
  // err is written during this launch only when a factor fails, which then
  // fails in every workgroup alike; halt and eta only by workgroup 0, with
  // the values every workgroup derives itself (see above)
  if (tid == 0) {
    s_ok = !(err0 || (step && a.check_halt && halt0));
    s_eta = step ? eta0 : 0.0;
  }
  __syncthreads();
  auto keep_src = [&] {
    if (step || ap.src == ap.U || p >= n) return;
#pragma unroll
    for (int i = 0; i < RT; ++i)
      if (i < r) ap.U[(long)i * n + p] = u0[i];
  };
  if (!s_ok) {
    keep_src();
    return;
  }
  if (step && !(s_eta > 0.0)) {  // first iteration: eta = eta_c / ||grad||_2 (with the guard and the cap)
    const int x = tid >> 4, y = tid & 15;
    if (x < r && y < r) W0[tid] = gram(r + x, r + y);
    __syncthreads();
    const double smax = sqrt(spectral_norm2(W0, W1, W2, r));
    const bool go = smax > a.guard * st->ysq;
    __syncthreads();
    if (tid == 0) {
      if (!go) {
        s_ok = 0;  // stationary start
        if (blockIdx.x == 0) {
          st->grad_norm = smax;
          if (a.commit_direct) {
            st->converged = 1;
            __hip_atomic_store(&st->halt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          } else {
            st->step_flags = STEP_CONVERGED;
          }
        }
      } else {
        s_eta = a.eta_c / smax;
      }
    }
    __syncthreads();
    if (!s_ok) return;
    if (a.eta_cap_c > 0.0) {  // cap: eta <= c n / (mbar ||B_0||_2^2)
      if (x < r && y < r) {
        double2 sum = make_double2(0.0, 0.0);
        for (int k = 0; k < a.q; ++k)
          sum = dadd(sum, dmul(f2d(a.B[(long)k * r + x]), dconj(f2d(a.B[(long)k * r + y]))));
        W0[tid] = sum;
      }
      __syncthreads();
      const double lam = spectral_norm2(W0, W1, W2, r);
      const double cap = a.eta_cap_c * (double)a.n / (st->mbar * lam);
      __syncthreads();
      if (tid == 0 && cap < s_eta) s_eta = cap;
      __syncthreads();
    }
    if (a.mode == STEP_MODE_ETA) {
      if (tid == 0) {
        st->grad_norm = smax;
        st->eta = s_eta;
      }
      return;
    }
  }
  if (a.mode == STEP_MODE_ETA) return;
  const double eta = s_eta;
  if (tid < 64) {  // one wave: the Cholesky factor of Uhat^H Uhat
    double2 h[4], dummy = make_double2(0.0, 0.0);
    double tr = 0.0, dmax = 0.0, inv_own;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int y = 4 * t + rg;
      h[t] = uu[t];
      if (step)
        h[t] = make_double2(uu[t].x - eta * (ug[t].x + gu[t].x) + eta * eta * gg[t].x,
                            uu[t].y - eta * (ug[t].y + gu[t].y) + eta * eta * gg[t].y);
      if (ri >= r || y >= r) h[t] = make_double2(0.0, 0.0);
      if (ri == y && y < r) {
        dmax = h[t].x;
        tr = step ? gg[t].x : h[t].x;
      }
    }
    dmax = wave_max(dmax);
    tr = wave_sum(tr);  // of G^H G, or of the Gram of src
    double2 h0[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) h0[t] = h[t];
    bool ok = wave_chol<double, double2, false>(h, L, r, 1e-14 * dmax, dummy, inv_own);
    if (!ok && !step && tr > 0.0 && isfinite(tr)) {  // numerically rank-deficient basis: retry with a small ridge
      const double ridge = 1e-6 * tr / r;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        h[t] = h0[t];
        if (ri == 4 * t + rg && ri < r) h[t].x += ridge;
      }
      ok = wave_chol<double, double2, false>(h, L, r, 1e-14 * (dmax + ridge), dummy, inv_own);
    }
    if (!ok) {
      if (l == 0) {
        s_ok = 0;
        set_error(st, 4, -1);
      }
    } else {
      wave_sync();
      for (int e = l; e < r * r; e += 64) Rf[(e / r) * RT + (e % r)] = rfac_entry(L, r, e);
      if (blockIdx.x == 0 && step) {
        if (a.commit_direct) {
          // exit rule off: SD, f and ||grad|| are only reported; their r x r
          // inputs are stored and k_stats_finish forms them when asked
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const int e = ri * 16 + 4 * t + rg;
            a.stats_src[e] = uu[t];
            a.stats_src[256 + e] = ug[t];
            a.stats_src[512 + e] = (ri < r && 4 * t + rg <= ri) ? L[ri * CHOL_LD + 4 * t + rg] : make_double2(0.0, 0.0);
          }
          if (l == 0) {
            a.stats_src[768] = make_double2(eta, tr);
            st->stats_pending = 1;
            __hip_atomic_store(&st->eta, eta, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            st->t += 1;
            st->step_ok = 1;
          }
        } else {
          // SD^2 = r - ||U^H U+||_F^2 decides the exit rule
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            W0[ri * 16 + 4 * t + rg] = uu[t];
            W1[ri * 16 + 4 * t + rg] = ug[t];
          }
          wave_sync();
          const double fro = wave_sum(sd_row_sum(W0, W1, L, W2, eta, r, l));
          double fv = 0.0;  // f = sum_k cost_k
          for (int k = l; k < a.q; k += 64) fv += a.cost_k[k];
          fv = wave_sum(fv);
          if (l == 0) {
            const double sd2 = fmax(0.0, (double)r - fro);
            st->sd = sqrt(sd2);
            st->grad_norm = sqrt(tr);
            st->f = fv;
            st->stats_pending = 0;
            st->eta_next = eta;
            st->step_flags = STEP_APPLIED | ((a.eps_exit > 0.0 && sqrt(sd2 / r) < a.eps_exit) ? STEP_EXIT : 0);
          }
        }
      }
    }
  }
  __syncthreads();
  if (!s_ok) {
    keep_src();
    return;
  }
  if (keep_cost) reinterpret_cast<double*>(a.stats_src + 769)[tid - 128] = cost;
  if (p >= n) return;
  // U+ R = U - eta grad for this pixel (forward substitution, 1 / R_jj on the diagonal)
  const float etaf = (float)eta;
  float2 un[RT];
#pragma unroll
  for (int j = 0; j < RT; ++j) {
    un[j] = make_float2(0.f, 0.f);
    if (j < r) {
      if (ap.U_prev) ap.U_prev[(long)j * n + p] = u0[j];
      float2 sv = make_float2(u0[j].x - etaf * g0[j].x, u0[j].y - etaf * g0[j].y);
#pragma unroll
      for (int i = 0; i < j; ++i) sv = csub(sv, cmul(un[i], Rf[i * RT + j]));
      un[j] = cscale(sv, Rf[j * RT + j].x);
      ap.U[(long)j * n + p] = un[j];
      if (ap.Ui && (r & 1)) ap.Ui[p * r + j] = un[j];
    }
  }
  if (ap.Ui && (r & 1) == 0) {  // the pixel-major row as 16-byte stores
    float4* dst = reinterpret_cast<float4*>(ap.Ui + p * r);
#pragma unroll
    for (int h = 0; h < RT / 2; ++h)
      if (2 * h < r) dst[h] = make_float4(un[2 * h].x, un[2 * h].y, un[2 * h + 1].x, un[2 * h + 1].y);
  }
}

// the fused step's outcome into the state (one thread, after it)
__global__ void k_step_commit(DevState* st, int exit_consec) {
  if (threadIdx.x != 0) return;
  const int f = st->step_flags;
  st->step_flags = 0;
  st->step_ok = 0;
  if (st->err) return;
  if (f & STEP_CONVERGED) {
    st->converged = 1;
    st->halt = 1;
  } else if (f & STEP_APPLIED) {
    st->eta = st->eta_next;
    st->t += 1;
    st->step_ok = 1;
    if (f & STEP_EXIT) {
      st->exit_run += 1;
      if (st->exit_run >= exit_consec) {
        st->exited = 1;
        st->halt = 1;
      }
    } else {
      st->exit_run = 0;
    }
  }
}

// the statistics the fused step left pending (exit rule off): SD, f and
// ||grad||_F of the last applied step, from its stored inputs, with the fused
// step's own code
__global__ __launch_bounds__(64) void k_stats_finish(DevState* st, const double2* src, int q, int r) {
  __shared__ double2 UU[256], UG[256], Gh[16 * CHOL_LD], Tm[256];
  const int l = threadIdx.x;
  if (!st->stats_pending) return;
  for (int e = l; e < 256; e += 64) {
    UU[e] = src[e];
    UG[e] = src[256 + e];
    Gh[(e >> 4) * CHOL_LD + (e & 15)] = src[512 + e];
  }
  const double2 et = src[768];
  wave_sync();
  const double fro = wave_sum(sd_row_sum(UU, UG, Gh, Tm, et.x, r, l));
  const double* const cost_k = reinterpret_cast<const double*>(src + 769);
  double fv = 0.0;
  for (int k = l; k < q; k += 64) fv += cost_k[k];
  fv = wave_sum(fv);
  if (l == 0) {
    st->sd = sqrt(fmax(0.0, (double)r - fro));
    st->grad_norm = sqrt(et.y);
    st->f = fv;
    st->stats_pending = 0;
  }
}

hipError_t launch_stats_finish(DevState* st, const double2* src, int q, int r, hipStream_t s) {
  hipLaunchKernelGGL(k_stats_finish, dim3(1), dim3(64), 0, s, st, src, q, r);
  return hipGetLastError();
}

// the QR Gram partials summed once for the fused step: workgroups of 256
// threads, each over a few 16-byte units, so that one round of loads covers
// its partials
__global__ __launch_bounds__(256) void k_partials_total(const double2* part, int f32, int nblk, int nout,
                                                        double2* total) {
  partials_sum<256>(part, f32, nblk, nout, total, blockIdx.x, gridDim.x);
}

hipError_t launch_partials_total(const double2* part, int f32, int nblk, int nout, double2* total, hipStream_t s) {
  const int per = (f32 && (nout & 1) == 0) ? 2 : 1, nunit = nout / per;
  // 8 units per workgroup: 32 slices of 16 loads in flight cover 512 partials
  const int nwg = (nunit + 7) / 8;
  hipLaunchKernelGGL(k_partials_total, dim3(nwg), dim3(256), 0, s, part, f32, nblk, nout, total);
  return hipGetLastError();
}

hipError_t launch_step_apply(const QrSmallArgs& a, const ApplyArgs& ap, hipStream_t s) {
  if (a.r < 1 || a.r > 16) return hipErrorInvalidValue;
  // 256 pixels per workgroup: the update's stores spread over every compute
  // unit; register rows of 4, 8, 12 or 16
  const dim3 g(a.mode == STEP_MODE_ETA ? 1u : (unsigned)((ap.n + 255) / 256));
  switch (2 * ((a.r + 3) / 4) + !a.summed) {
    case 2: hipLaunchKernelGGL((k_step_apply<4, false>), g, dim3(256), 0, s, a, ap); break;
    case 3: hipLaunchKernelGGL((k_step_apply<4, true>), g, dim3(256), 0, s, a, ap); break;
    case 4: hipLaunchKernelGGL((k_step_apply<8, false>), g, dim3(256), 0, s, a, ap); break;
    case 5: hipLaunchKernelGGL((k_step_apply<8, true>), g, dim3(256), 0, s, a, ap); break;
    case 6: hipLaunchKernelGGL((k_step_apply<12, false>), g, dim3(256), 0, s, a, ap); break;
    case 7: hipLaunchKernelGGL((k_step_apply<12, true>), g, dim3(256), 0, s, a, ap); break;
    case 8: hipLaunchKernelGGL((k_step_apply<16, false>), g, dim3(256), 0, s, a, ap); break;
    default: hipLaunchKernelGGL((k_step_apply<16, true>), g, dim3(256), 0, s, a, ap); break;
  }
  if (a.mode == STEP_MODE_STEP && !a.commit_direct)
    hipLaunchKernelGGL(k_step_commit, dim3(1), dim3(64), 0, s, a.st, a.exit_consec);
  return hipGetLastError();
}

// Number of eigenvalues below each of E points of the real symmetric
// tridiagonal (d, e), scaled so that |d|, |e| <= 1 and padded to a multiple of
// eight rows by d = 4, e = 0.  The sign changes of the leading minors' sequence
// p_i = (d_i - x) p_{i-1} - e_{i-1}^2 p_{i-2}, whose pair of values is scaled by a
// power of two every eight rows: four instructions a row and one dependent
// multiply-add, where the pivots' quotients need a division.  A single minor of
// zero changes no count (its neighbours' signs differ); two in a row, also by
// underflow within eight rows, are reported in `zero` and left to sturm_pivots.
template <int E>
__device__ __forceinline__ bool sturm_minors(const double* d, const double* e2, int n, const double (&x)[E],
                                             int (&cnt)[E]) {
  double p[E], pp[E], eb = 0.0;  // eb: the squared off-diagonal before the row
  bool zero = false;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    p[e] = 1.0;
    pp[e] = 0.0;
    cnt[e] = 0;
  }
#pragma unroll 1
  for (int i0 = 0; i0 < n; i0 += 8) {
    unsigned sg[E];  // the signs of the minor before the block and of its eight
#pragma unroll
    for (int e = 0; e < E; ++e) sg[e] = (unsigned)__double2hiint(p[e]) >> 31;
#pragma unroll
    for (int i = i0; i < i0 + 8; ++i) {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const double q = fma(d[i] - x[e], p[e], -(eb * pp[e]));
        sg[e] = __builtin_amdgcn_alignbit(sg[e], (unsigned)__double2hiint(q), 31);
        pp[e] = p[e];
        p[e] = q;
      }
      eb = e2[i];
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
      cnt[e] += __popc((sg[e] ^ (sg[e] >> 1)) & 0xffu);
      zero = zero || (p[e] == 0.0 && pp[e] == 0.0);
      const int ex = -__builtin_amdgcn_frexp_exp(fabs(p[e]) > fabs(pp[e]) ? p[e] : pp[e]);
      p[e] = __builtin_amdgcn_ldexp(p[e], ex);
      pp[e] = __builtin_amdgcn_ldexp(pp[e], ex);
    }
  }
  return zero;
}

// the same count from the LDL^T pivots, tiny ones replaced by -pivmin
__device__ __noinline__ int sturm_pivots(const double* d, const double* e2, int n, double x) {
  const double pivmin = 1e-300;
  double q = d[0] - x;
  if (fabs(q) < pivmin) q = -pivmin;
  int cnt = q < 0.0;
#pragma unroll 1
  for (int i = 1; i < n; ++i) {
    q = d[i] - x - e2[i - 1] * rcp_nr(q);
    if (fabs(q) < pivmin) q = -pivmin;
    cnt += q < 0.0;
  }
  return cnt;
}

// multisection by one wave: E eigenvalues at once, of ascending indices idx[e],
// 64 lanes with one count each per round (a 65-section of the interval), to an
// isolating interval of relative width 1e-10, whose middle goes to lam[e * step]
template <int E>
__device__ __forceinline__ void multisect(const double* d, const double* e2, int n, double lo0, double hi0, int l,
                                          const int (&idx)[E], double* lam, int step) {
  double lo[E], hi[E], x[E];
  int cnt[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    lo[e] = lo0;
    hi[e] = hi0;
  }
#pragma unroll 1
  for (int rnd = 0; rnd < 80; ++rnd) {
#pragma unroll
    for (int e = 0; e < E; ++e) x[e] = lo[e] + (hi[e] - lo[e]) * (double)(l + 1) * (1.0 / 65.0);
    if (__any(sturm_minors<E>(d, e2, n, x, cnt))) {
#pragma unroll
      for (int e = 0; e < E; ++e) cnt[e] = sturm_pivots(d, e2, n, x[e]);
    }
    bool done = true;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      // the counts rise with the lane: the last point at or below the eigenvalue, the first above it
      const unsigned long long above = __ballot(cnt[e] > idx[e]);
      const int f = above ? __builtin_ctzll(above) : 64;
      const double nlo = lane_get(x[e], f > 0 ? f - 1 : 0), nhi = lane_get(x[e], f < 64 ? f : 63);
      if (f > 0) lo[e] = nlo;
      if (f < 64) hi[e] = nhi;
      done = done && hi[e] - lo[e] <= 1e-10 * fmax(fabs(lo[e]), fabs(hi[e])) + 1e-300;
    }
    if (done) break;  // the same in every lane
  }
  if (l == 0) {
#pragma unroll
    for (int e = 0; e < E; ++e) lam[e * step] = 0.5 * (lo[e] + hi[e]);
  }
}

// c ? v : 0, part by part (a selected struct would go through memory)
__device__ __forceinline__ double2 dkeep(bool c, double2 v) { return make_double2(c ? v.x : 0.0, c ? v.y : 0.0); }

// inclusive product over the lanes 0 .. l
__device__ __forceinline__ double2 wave_scan_mul(double2 v, int l) {
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const double2 u = make_double2(__shfl_up(v.x, off), __shfl_up(v.y, off));
    if (l >= off) v = dmul(u, v);
  }
  return v;
}

__host__ __device__ constexpr int eig_vh_off(int n, int k) { return k * (n - 1) - k * (k - 1) / 2; }
// waves: 16 columns each.  What every wave computes for itself is issued once per
// wave, so one wave per SIMD where the columns fit (q <= 64), else two.
template <int NH>
constexpr int EIG_W = 4 * NH;
// LDS of the reduction beside the reflectors, in double2: partial products, column, w and two v
template <int NH>
constexpr int EIG_WORK = EIG_W<NH> * 64 * NH + 64 * NH + 3 * (64 * NH + 1);

// back-transformation by one wave: Y = Q D Z with Q = H_0 ... H_{n-3}, then V_r
// Sigma_r^{-1} = Y diag(1 / sqrt(lambda_j)) into Vs, for the columns 4 wv .. 4 wv + 3.
// Sixteen lanes per column keep its rows g, g + 16, ... in registers for the
// whole product, a reflector's column sums are DPP moves, and there is no
// barrier; the next reflector's rows are read during this one's arithmetic.
template <int NH>
__device__ __forceinline__ void backtransform(const double2* Vh, const double* s_beta, const double2* s_ph,
                                              const double* sy, const double* s_lam, double unit, int n, int r, int wv,
                                              int l, float2* Vs) {
  constexpr int NT = 4 * NH;
  const int g = l & 15, j = 4 * wv + (l >> 4), jc = min(j, r - 1);
  const int zr = n * (n - 1) / 2 - 1;  // a row of zero: the last column has no reflector
  double2 y[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int i = min(g + 16 * t, n - 1);
    const double z = sy[i * r + jc];
    y[t] = dkeep(g + 16 * t < n, make_double2(s_ph[i].x * z, s_ph[i].y * z));
  }
  auto reflector = [&](int k, double2 (&dst)[NT]) {  // rows outside it are zero
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int i = g + 16 * t, kc = max(k, 0);
      dst[t] = Vh[i > kc && i < n ? eig_vh_off(n, kc) + i - kc - 1 : zr];
    }
  };
  if (n > 2) {
    double2 vc[NT], vx[NT];
    reflector(n - 3, vc);
#pragma unroll 1
    for (int k = n - 3; k >= 0; --k) {
      const double bk = s_beta[k];
      reflector(k - 1, vx);
      double2 s = make_double2(0.0, 0.0);
#pragma unroll
      for (int t = 0; t < NT; ++t) {  // conj(v) y
        s.x = fma(vc[t].x, y[t].x, fma(vc[t].y, y[t].y, s.x));
        s.y = fma(vc[t].x, y[t].y, fma(-vc[t].y, y[t].x, s.y));
      }
      s = make_double2(s.x + dpp_get<DPP_XOR1>(s.x), s.y + dpp_get<DPP_XOR1>(s.y));
      s = make_double2(s.x + dpp_get<DPP_XOR2>(s.x), s.y + dpp_get<DPP_XOR2>(s.y));
      s = make_double2(s.x + dpp_get<DPP_ROR4>(s.x), s.y + dpp_get<DPP_ROR4>(s.y));
      s = make_double2(bk * (s.x + dpp_get<DPP_ROR8>(s.x)), bk * (s.y + dpp_get<DPP_ROR8>(s.y)));
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        y[t].x = fma(-vc[t].x, s.x, fma(vc[t].y, s.y, y[t].x));
        y[t].y = fma(-vc[t].x, s.y, fma(-vc[t].y, s.x, y[t].y));
        vc[t] = vx[t];
      }
    }
  }
  const double sc = 1.0 / sqrt(s_lam[jc] * unit);
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int i = g + 16 * t;
    if (i < n && j < r) Vs[i * r + j] = make_float2((float)(y[t].x * sc), (float)(y[t].y * sc));
  }
}

// ===========================================================================
// spectral initialisation, the q x q eigenproblem: the r largest eigenpairs
// of the Hermitian X_0^H X_0 (q <= 64 NH) by one workgroup, then V_r Sigma_r^{-1}:
//  1. Householder reduction M = Q T Q^H, T tridiagonal with complex
//     off-diagonals e_k; reflectors H_k = I - beta_k v_k v_k^H kept in LDS,
//     packed (column k from eig_vh_off(n, k), its rows k + 1 .. n - 1);
//  2. a diagonal unitary D makes T real: T = D T_r D^H, off-diagonals |e_k|;
//  3. the r largest eigenvalues of T_r by multisection on Sturm counts;
//  4. their eigenvectors by inverse iteration (one lane each, LDL^T without
//     pivoting, tiny pivots replaced), orthogonalised within clusters;
//  5. back-transformation Y = Q D Z.
//
// The reduction's q - 2 dependent steps bound it, not its arithmetic, and a
// lone wave issues an instruction every four cycles at best: a step is as long
// as its longest wave's instructions.  The matrix stays in registers: lane l
// holds rows l and l + 64, wave w of W the columns w, w + W, ..., and a wave
// drops its first column as the step passes it, so the column a step needs is
// always its owner's register 0.  The rank-2 update of one step and the product
// with the next step's reflector are one pass over the registers; the values a
// column needs (v, w and the new v at its index) are loaded by lane t for
// column t and read with v_readlane.  Wave 0 alone forms w, the next column
// and its reflector in between: two barriers a step.  (A version with the matrix
// in LDS and four barriers took 580 us at 100 frames and rank 10, 140 us at 40
// and rank 8, 53 us at 16 and rank 4; this one 363, 95 and 35 us.)
// ===========================================================================
template <int NH>
__global__ __launch_bounds__(64 * EIG_W<NH>) void k_init_eig(InitEigArgs a) {
  constexpr int NR = 64 * NH, W = EIG_W<NH>, CT = NR / W, PP = NR;
  extern __shared__ double2 lds_m[];  // the packed reflectors, then the work region
  __shared__ double s_d[NR], s_ea[NR], s_e2[NR], s_beta[NR];
  __shared__ double2 s_ec[NR], s_ph[NR];
  __shared__ double s_lam[16];
  __shared__ double s_gs[4];  // Gershgorin interval (lo, hi) and scale of the scaled T_r, its unit in the matrix's terms
  const int tid = threadIdx.x, l = tid & 63, n = a.q, r = a.r;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  double2* const Vh = lds_m;
  double2* const work = lds_m + n * (n - 1) / 2;
  double2* const s_pp = work;            // [wave][row] partial products
  double2* const s_c = work + W * PP;    // [row] the next column, before its update
  double2* const s_w = s_c + NR;         // [row] w, and a row of zero
  double2* const s_v = s_w + NR + 1;     // [2][row] v and the new v, and a row of zero each
  const double2 zero2 = make_double2(0.0, 0.0);

  // ---- 1. Householder tridiagonalisation
  double2 A[NH][CT];
#pragma unroll
  for (int h = 0; h < NH; ++h)
#pragma unroll
    for (int t = 0; t < CT; ++t) {
      const int i = min(l + 64 * h, n - 1), j = min(wv + W * t, n - 1), lo = min(i, j), hi = max(i, j);
      A[h][t] = a.part[lo * n - lo * (lo - 1) / 2 + (hi - lo)];  // entry (lo, hi) of the upper triangle
    }
  double dg[NH];
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    const int i = min(l + 64 * h, n - 1);
    dg[h] = a.part[i * n - i * (i - 1) / 2].x;
  }
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    asm volatile("" : "+v"(dg[h]));  // loaded, all at once, before anything is selected
#pragma unroll
    for (int t = 0; t < CT; ++t) asm volatile("" : "+v"(A[h][t].x), "+v"(A[h][t].y));
  }
  // scaled by a power of two to a largest entry of 0.5 to 1 (the diagonal's: the
  // matrix is positive semidefinite)
  const int ex0 = __builtin_amdgcn_frexp_exp(wave_max(NH == 2 ? fmax(dg[0], dg[NH - 1]) : dg[0]));
#pragma unroll
  for (int h = 0; h < NH; ++h)
#pragma unroll
    for (int t = 0; t < CT; ++t) {
      const int i = l + 64 * h, j = wv + W * t;
      const double re = __builtin_amdgcn_ldexp(A[h][t].x, -ex0), im = __builtin_amdgcn_ldexp(A[h][t].y, -ex0);
      A[h][t] = dkeep(i < n && j < n, make_double2(re, i == j ? 0.0 : i < j ? im : -im));
    }
  int jb = wv;  // the column in register 0
  if (wv == 0) {
#pragma unroll
    for (int h = 0; h < NH; ++h) s_c[l + 64 * h] = A[h][0];
  }
  for (int i = tid; i < 3 * (NR + 1); i += 64 * W) s_w[i] = zero2;
  // wave 0's state of the last step: v, its first entry, beta
  double2 v[NH], v0 = zero2;
  double beta = 0.0;
#pragma unroll
  for (int h = 0; h < NH; ++h) v[h] = zero2;
  __syncthreads();
#pragma unroll 1
  for (int k = 0; k + 1 < n; ++k) {
    const int k1 = k + 1;
    double2* const s_vn = s_v + (k & 1) * (NR + 1);
    const double2* const s_vo = s_v + (k1 & 1) * (NR + 1);
    if (wv == 0) {
      // step k - 1's product p = beta B v, K = (beta / 2) v^H p, w = p - K v
      double2 w[NH], x[NH];
      double kp = 0.0;
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        const int i = l + 64 * h;
        x[h] = s_c[i];
        w[h] = zero2;
        if (k > 0) {
          double2 q[W];
#pragma unroll
          for (int e = 0; e < W; ++e) q[e] = s_pp[e * PP + i];
#pragma unroll
          for (int d = W / 2; d > 0; d >>= 1)
#pragma unroll
            for (int e = 0; e < d; ++e) q[e] = dadd(q[e], q[e + d]);
          w[h] = dkeep(i >= k && i < n, q[0]);
        }
        kp = fma(v[h].x, w[h].x, fma(v[h].y, w[h].y, kp));
      }
      const double K = 0.5 * beta * beta * wave_sum(kp);  // v^H B v is real
#pragma unroll
      for (int h = 0; h < NH; ++h)
        w[h] = make_double2(fma(beta, w[h].x, -K * v[h].x), fma(beta, w[h].y, -K * v[h].y));
      auto row = [&](const double2 (&z)[NH], int i) {  // entry i (uniform)
        if constexpr (NH == 2)
          return lane_get(make_double2(i >= 64 ? z[1].x : z[0].x, i >= 64 ? z[1].y : z[0].y), i & 63);
        else
          return lane_get(z[0], i);
      };
      // column k after its update; rows before k hold values of earlier steps, never read again
      const double2 wk = row(w, k);
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        x[h].x = fma(-v[h].x, wk.x, fma(-v[h].y, wk.y, fma(-w[h].x, v0.x, fma(-w[h].y, v0.y, x[h].x))));
        x[h].y = fma(-v[h].y, wk.x, fma(v[h].x, wk.y, fma(-w[h].y, v0.x, fma(w[h].x, v0.y, x[h].y))));
        if (l + 64 * h == k) s_d[k] = x[h].x;
        s_w[l + 64 * h] = w[h];
      }
      // the reflector of its rows k1 .. n - 1 (none for the last column)
      const double2 x0 = row(x, k1);
      double sig = 0.0;
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        const int i = l + 64 * h;
        const double2 z = dkeep(i > k1 && i < n, x[h]);
        sig = fma(z.x, z.x, fma(z.y, z.y, sig));
      }
      sig = wave_sum(sig);
      double2 alpha = x0;
      v0 = zero2;
      beta = 0.0;
      // none either where the column has vanished beside the matrix: rounding
      // errors of a rank-deficient one shrink by 1e-16 a step, and their squares
      // would underflow (no reflector: the column's rest, below 1e-60, is dropped)
      const double t = x0.x * x0.x + x0.y * x0.y, s = t + sig;
      const bool refl = k + 2 < n && s > 1e-120 && !(sig == 0.0 && x0.y == 0.0);  // the same in every lane
      if (refl) {
        const double nrm = s * cx_rsqrt(s);
        const bool big = t > 1e-290;
        const double rt = cx_rsqrt(big ? t : 1.0), ax0 = big ? t * rt : 0.0;
        const double2 ph = make_double2(big ? x0.x * rt : 1.0, big ? x0.y * rt : 0.0);
        alpha = make_double2(-ph.x * nrm, -ph.y * nrm);
        v0 = make_double2(ph.x * (ax0 + nrm), ph.y * (ax0 + nrm));
        beta = rcp_nr(fma(nrm, ax0, s));  // 2 / |v|^2
      }
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        const int i = l + 64 * h;
        v[h] = dkeep(refl && i >= k1 && i < n, make_double2(i == k1 ? v0.x : x[h].x, i == k1 ? v0.y : x[h].y));
        s_vn[i] = v[h];
        if (i >= k1 && i < n) Vh[eig_vh_off(n, k) + i - k1] = v[h];
      }
      if (l == 0) {
        s_beta[k] = beta;
        s_ec[k] = alpha;
      }
    }
    __syncthreads();
    if (wv == (k & (W - 1))) {  // column k is past: the wave's columns move down
#pragma unroll
      for (int h = 0; h < NH; ++h) {
#pragma unroll
        for (int t = 0; t + 1 < CT; ++t) A[h][t] = A[h][t + 1];
        A[h][CT - 1] = zero2;
      }
      jb += W;
    }
    // B -= v w^H + w v^H, and the product with the new reflector
    const int jc = min(jb + W * (l & (CT - 1)), NR);  // lane t: column t of this wave
    const double2 vj = s_vo[jc], wj = s_w[jc], nj = s_vn[jc];
    double2 vr[NH], wr[NH], pp[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      vr[h] = s_vo[l + 64 * h];
      wr[h] = s_w[l + 64 * h];
      pp[h] = zero2;
    }
    const int nact = (n - jb + W - 1) / W;
#pragma unroll
    for (int t0 = 0; t0 < CT; t0 += 2) {
      if (t0 < nact) {
#pragma unroll
        for (int t = t0; t < t0 + 2; ++t) {
          const double2 cv = lane_get(vj, t), cw = lane_get(wj, t), cn = lane_get(nj, t);
#pragma unroll
          for (int h = 0; h < NH; ++h) {
            if (NH == 2 && h == 0 && k1 >= 64) continue;  // rows that are done
            double2 b = A[h][t];
            b.x = fma(-vr[h].x, cw.x, fma(-vr[h].y, cw.y, fma(-wr[h].x, cv.x, fma(-wr[h].y, cv.y, b.x))));
            b.y = fma(-vr[h].y, cw.x, fma(vr[h].x, cw.y, fma(-wr[h].y, cv.x, fma(wr[h].x, cv.y, b.y))));
            A[h][t] = b;
            pp[h].x = fma(b.x, cn.x, fma(-b.y, cn.y, pp[h].x));
            pp[h].y = fma(b.x, cn.y, fma(b.y, cn.x, pp[h].y));
          }
        }
      }
    }
#pragma unroll
    for (int h = 0; h < NH; ++h) s_pp[wv * PP + l + 64 * h] = pp[h];
    if (wv == (k1 & (W - 1))) {
#pragma unroll
      for (int h = 0; h < NH; ++h) s_c[l + 64 * h] = A[h][0];
    }
    __syncthreads();
  }
  // the last diagonal entry: column n - 1 before any update of the last step (there is none: its v is zero)
  if (wv == ((n - 1) & (W - 1))) {
#pragma unroll
    for (int h = 0; h < NH; ++h)
      if (l + 64 * h == n - 1) s_d[n - 1] = A[h][0].x;
  }
  __syncthreads();
  if (wv == 0) {  // one wave: the tridiagonal eigenproblem
    // ---- 2. T_r: diagonal, |e_k|, and the phases of D (a running product)
    double2 u[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      const int i = NH * l + h;
      u[h] = make_double2(1.0, 0.0);
      if (i + 1 < n) {
        const double2 e = s_ec[i];
        const double ae = sqrt(e.x * e.x + e.y * e.y);
        s_ea[i] = ae;
        s_e2[i] = ae * ae;
        if (ae > 0.0) u[h] = make_double2(e.x / ae, e.y / ae);
      }
      if (h > 0) u[h] = dmul(u[h - 1], u[h]);
    }
    const double2 inc = wave_scan_mul(u[NH - 1], l);
    double2 exc = make_double2(__shfl_up(inc.x, 1), __shfl_up(inc.y, 1));
    if (l == 0) {
      exc = make_double2(1.0, 0.0);
      s_ph[0] = exc;
    }
#pragma unroll
    for (int h = 0; h < NH; ++h)
      if (NH * l + h + 1 < n) s_ph[NH * l + h + 1] = dmul(exc, u[h]);
    wave_sync();
    // Gershgorin interval and scale; T_r is scaled in place by a power of two
    double glo = INFINITY, ghi = -INFINITY, scale = 0.0;
    for (int i = l; i < n; i += 64) {
      const double rad = (i > 0 ? s_ea[i - 1] : 0.0) + (i + 1 < n ? s_ea[i] : 0.0);
      glo = fmin(glo, s_d[i] - rad);
      ghi = fmax(ghi, s_d[i] + rad);
      scale = fmax(scale, fabs(s_d[i]) + rad);
    }
    glo = wave_min(glo);
    ghi = wave_max(ghi);
    scale = fmax(wave_max(scale), 1e-300);
    const int ex = __builtin_amdgcn_frexp_exp(scale);
    for (int i = l; i < NR; i += 64) {  // rows past n: no sign changes, no part in any vector
      const double d = i < n ? __builtin_amdgcn_ldexp(s_d[i], -ex) : 4.0;
      const double e = i + 1 < n ? __builtin_amdgcn_ldexp(s_ea[i], -ex) : 0.0;
      s_d[i] = d;
      s_ea[i] = e;
      s_e2[i] = e * e;
    }
    if (l == 0) {
      const double wdt = ghi - glo;
      s_gs[0] = __builtin_amdgcn_ldexp(glo - (1e-3 * wdt + 1e-300), -ex);
      s_gs[1] = __builtin_amdgcn_ldexp(ghi + (1e-3 * wdt + 1e-300), -ex);
      s_gs[2] = __builtin_amdgcn_ldexp(scale, -ex);
      s_gs[3] = __builtin_amdgcn_ldexp(1.0, ex + ex0);
    }
  }
  __syncthreads();
  // ---- 3. wave w takes the eigenvalues w, w + W, ... (descending; ascending
  // index n - 1 - w), two at a time; inverse iteration converges from the
  // interval's middle and the Rayleigh quotient refines the value
  const double scale = s_gs[2], unit = s_gs[3];
#pragma unroll 1
  for (int j = wv; j < r; j += 2 * W) {
    if (j + W < r) {
      const int idx[2] = {n - 1 - j, n - 1 - j - W};
      multisect<2>(s_d, s_e2, n, s_gs[0], s_gs[1], l, idx, s_lam + j, W);
    } else {
      const int idx[1] = {n - 1 - j};
      multisect<1>(s_d, s_e2, n, s_gs[0], s_gs[1], l, idx, s_lam + j, W);
    }
  }
  __syncthreads();
  double* const sy = reinterpret_cast<double*>(work);  // right-hand side / solution [i * r + j]
  if (wv == 0) {
    // ---- 4. inverse iteration, one lane per eigenvalue, a.gw of them at a
    // time (all r, unless the reciprocal pivots' room is short); values in
    // LDS are read sixteen rows at a time ahead of the serial chains that use
    // them, over the padded rows, whose entries are zero in every vector
    const int gw = a.gw, n16 = (n + 15) & ~15;
    double* const su = sy + n16 * r;  // 1 / u pivots [i * gw + j]
#pragma unroll 1
    for (int j0 = 0; j0 < r; j0 += gw) {
      const int j = j0 + l;
      if (l < gw && j < r) {
        const double lam = s_lam[j], tiny = 1e-14 * scale;
        {  // the reciprocal pivots, and a start vector of its own per eigenvalue (golden-ratio sequence)
          double u = s_d[0] - lam;
#pragma unroll 1
          for (int i0 = 0; i0 < n16; i0 += 8) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const int i = i0 + e;
              if (fabs(u) <= tiny) u = tiny;
              const double ru = rcp_nr(u);
              u = s_d[min(i + 1, NR - 1)] - lam - s_e2[i] * ru;
              const double t = (double)(i + 1) * (double)(2 * j + 3) * 0.6180339887498949;
              su[i * gw + l] = ru;
              sy[i * r + j] = i < n ? 0.5 + (t - floor(t)) : 0.0;
            }
          }
        }
        double inv = 1.0, nrm2 = 0.0;
#pragma unroll 1
        for (int it = 0; it < 3; ++it) {
          double y = 0.0, lmp = 0.0;  // the row before's value and its multiplier
#pragma unroll 1
          for (int i0 = 0; i0 < n16; i0 += 16) {
            double lm[16], yn[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) {
              lm[e] = s_ea[i0 + e] * su[(i0 + e) * gw + l];
              yn[e] = sy[(i0 + e) * r + j] * inv;
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) {
              y = fma(-lmp, y, yn[e]);
              lmp = lm[e];
              sy[(i0 + e) * r + j] = y;
            }
          }
          double xn = 0.0;
          nrm2 = 0.0;
#pragma unroll 1
          for (int i0 = n16 - 16; i0 >= 0; i0 -= 16) {
            double ys[16], es[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) {
              const double ru = su[(i0 + e) * gw + l];
              ys[e] = sy[(i0 + e) * r + j] * ru;
              es[e] = s_ea[i0 + e] * ru;
            }
#pragma unroll
            for (int e = 15; e >= 0; --e) {
              xn = fma(-es[e], xn, ys[e]);
              sy[(i0 + e) * r + j] = xn;
              nrm2 = fma(xn, xn, nrm2);
            }
          }
          inv = 1.0 / sqrt(nrm2);
        }
        // normalised, and its Rayleigh quotient z^T T_r z
        double rq = 0.0, ez = 0.0;  // ez: off-diagonal times the value before
#pragma unroll 1
        for (int i0 = 0; i0 < n16; i0 += 8) {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int i = i0 + e;
            const double z = sy[i * r + j] * inv;
            sy[i * r + j] = z;
            rq = fma(z, fma(s_d[i], z, 2.0 * ez), rq);
            ez = s_ea[i] * z;
          }
        }
        s_lam[j] = rq;
      }
      wave_sync();
    }
    // orthogonalise within clusters of close eigenvalues, twice, in descending order
    for (int j = 1; j < r; ++j) {
      bool any = false;
      for (int jp = 0; jp < j; ++jp) any = any || fabs(s_lam[jp] - s_lam[j]) <= 1e-3 * scale;
      if (!any) continue;
      for (int rep = 0; rep < 2; ++rep) {
        for (int jp = 0; jp < j; ++jp) {
          if (!(fabs(s_lam[jp] - s_lam[j]) <= 1e-3 * scale)) continue;
          double dot = 0.0;
          for (int i = l; i < n; i += 64) dot += sy[i * r + jp] * sy[i * r + j];
          dot = wave_sum(dot);
          for (int i = l; i < n; i += 64) sy[i * r + j] -= dot * sy[i * r + jp];
          wave_sync();
        }
      }
      double nn = 0.0;
      for (int i = l; i < n; i += 64) nn += sy[i * r + j] * sy[i * r + j];
      const double inv = 1.0 / sqrt(wave_sum(nn));
      for (int i = l; i < n; i += 64) sy[i * r + j] *= inv;
      wave_sync();
    }
  }
  __syncthreads();
  if (a.lam_out) {  // only the spectrum was asked for
    if (tid < r) a.lam_out[tid] = s_lam[tid] * unit;
    return;
  }
  const double lam0 = s_lam[0], lamr = s_lam[r - 1];
  if (!(lamr > 1e-14 * lam0) || !(lam0 > 0.0)) {
    if (tid == 0) set_error(a.st, 4, -1);
    return;
  }
  // ---- 5. wave w the columns 4 w .. 4 w + 3
  if (4 * wv < r) backtransform<NH>(Vh, s_beta, s_ph, sy, s_lam, unit, n, r, wv, l, a.Vs);
}

// U0[:, j] = sum_k X0[:, k] Vs[k][j]: a workgroup takes 64 pixels, its four
// waves the same pixels and a quarter of the r <= RT columns each (the
// frames' values, loaded by each wave, come from the cache for three of
// them); the frames' values KB at a time in flight, every LDS read of Vs
// unconditional (a read under a branch would be waited on alone)
template <int RT>
__global__ __launch_bounds__(AG_NT) void k_x_times_v(const float2* X, const float2* Vs, int n, int q, int r,
                                                     float2* U, const DevState* st) {
  static_assert(AG_NT == 256, "four waves per workgroup");
  constexpr int CPT = RT / 4;  // columns per thread
  __shared__ float2 V[128 * 16];
  const int tid = threadIdx.x, pl = tid & 63, jg = tid >> 6;
  const long p = (long)blockIdx.x * 64 + pl, pc = min(p, (long)n - 1);
  // the first frames' values requested before the state and the table (valid, clamped addresses)
  constexpr int KB = 16;
  float2 xv[KB];
#pragma unroll
  for (int i = 0; i < KB; ++i) xv[i] = X[(long)min(i, q - 1) * n + pc];
  if (st->err) return;
  for (int e = tid; e < q * r; e += AG_NT) V[e] = Vs[e];
  __syncthreads();
  int jc[CPT];
#pragma unroll
  for (int c = 0; c < CPT; ++c) jc[c] = min(jg * CPT + c, r - 1);
  float2 acc[CPT];
#pragma unroll
  for (int c = 0; c < CPT; ++c) acc[c] = make_float2(0.f, 0.f);
  for (int k0 = 0; k0 < q; k0 += KB) {
    float2 xn[KB];
    const bool more = k0 + KB < q;
#pragma unroll
    for (int i = 0; i < KB; ++i) xn[i] = X[(long)min(k0 + KB + i, q - 1) * n + pc];  // the next batch
#pragma unroll
    for (int i = 0; i < KB; ++i) {
      const int k = min(k0 + i, q - 1);
      const float2 x = (k0 + i < q) ? xv[i] : make_float2(0.f, 0.f);
      const float2* vk = V + k * r;
#pragma unroll
      for (int c = 0; c < CPT; ++c) acc[c] = cadd(acc[c], cmul(x, vk[jc[c]]));
    }
    if (!more) break;
#pragma unroll
    for (int i = 0; i < KB; ++i) xv[i] = xn[i];
  }
  if (p >= n) return;
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int j = jg * CPT + c;
    if (j < r) U[(long)j * n + p] = acc[c];
  }
}

hipError_t launch_x_times_v(const float2* X, const float2* Vs, int n, int q, int r, float2* U, const DevState* st,
                            hipStream_t s) {
  const dim3 g((n + 63) / 64), b(AG_NT);
  if (r <= 8) hipLaunchKernelGGL(k_x_times_v<8>, g, b, 0, s, X, Vs, n, q, r, U, st);
  else hipLaunchKernelGGL(k_x_times_v<16>, g, b, 0, s, X, Vs, n, q, r, U, st);
  return hipGetLastError();
}

// keep the learned U (src) only if its cost f[1] is strictly below the
// spectral one f[0]; a non-finite learned cost keeps the spectral U
// The error and halt flags as they stood before the learned guess was scored
// (raising an error also halts the loop).
__global__ void k_err_snapshot(const DevState* st, int32_t* snap) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    snap[0] = st->err;
    snap[1] = st->halt;
  }
}

// Keep the learned basis (src) only if its cost f[1] is strictly below the
// fallback's f[0].  A guess whose scoring raised an error (a Gram of the
// guess or of A_k U that is not positive definite, a non-finite value) counts
// as infinitely costly: the fallback stays.  An error that was already set
// before the guess was scored (snap) is left for the caller.
__global__ void k_pick_init(const double* f, const int32_t* snap, const float2* src, float2* dst, long n,
                            int32_t* choice, const DevState* st) {
  if (*snap) return;
  const bool take = st->err == 0 && f[1] < f[0];
  if (choice && blockIdx.x == 0 && threadIdx.x == 0) *choice = take ? 1 : 0;
  if (!take) return;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) dst[i] = src[i];
}

// After k_pick_init: an error raised only by the rejected guess is cleared,
// with the halt it raised.
__global__ void k_err_restore(const int32_t* snap, DevState* st) {
  if (threadIdx.x != 0 || snap[0]) return;
  if (st->err) {
    st->err = 0;
    st->err_frame = -1;
    st->halt = snap[1];
  }
}

__global__ void k_copy(const float2* src, float2* dst, long n) {
  long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  long stride = (long)gridDim.x * blockDim.x;
  for (; i < n; i += stride) dst[i] = src[i];
}

__global__ void k_cost_total(const double* cost_k, int q, double* out, DevState* st) {
  if (threadIdx.x != 0) return;
  double f = 0.0;
  for (int k = 0; k < q; ++k) f += cost_k[k];
  st->cost_out = f;
  if (out) *out = f;
}

// ---------------------------------------------------------------------------
// launchers (explicit instantiations behind plain functions)
// ---------------------------------------------------------------------------
template <int NH>
static hipError_t launch_init_eig_nh(InitEigArgs a, hipStream_t s) {
  constexpr int NR = 64 * NH;
  // room for all r pivot columns of the inverse iteration, or for eight at a time
  const size_t vh = (size_t)a.q * (a.q - 1) / 2 * sizeof(double2), fixed = NR * 64 + 512, room = 160 * 1024 - fixed - vh;
  const size_t q16 = (a.q + 15) / 16 * 16;
  a.gw = q16 * a.r * 16 <= room ? a.r : std::min(a.r, 8);
  const size_t reduce = (size_t)EIG_WORK<NH> * sizeof(double2), iterate = q16 * (a.r + a.gw) * 8;
  const size_t lds = vh + std::max(reduce, iterate);
  if (lds > 48 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)k_init_eig<NH>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_init_eig<NH>, dim3(1), dim3(64 * EIG_W<NH>), lds, s, a);
  return hipGetLastError();
}

hipError_t launch_init_eig(const InitEigArgs& a, hipStream_t s) {
  if (a.q < 1 || a.q > 128 || a.r < 1 || a.r > 16 || a.r > a.q) return hipErrorInvalidValue;
  return a.q <= 64 ? launch_init_eig_nh<1>(a, s) : launch_init_eig_nh<2>(a, s);
}

}  // namespace ag
