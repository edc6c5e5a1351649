// Kernels of the steps around the altGDmin loop: the output assembly of
// Algorithm 1 and ISTA's temporal step (Algorithm 3, model 2).  The normal
// operator and the conjugate gradients are in kernels_normal.hip, the
// operator passes in kernels_fft.hip.
#include <algorithm>

#include "kernels_mri.hpp"
#include "mma.hpp"

namespace ag {

// Z[:, k] = (zbar or 0) + U b_k (when U) + (E[:, k] or 0): the output
// assembly of Algorithm 1 (z_k = zbar + x_k + e_k), U n x r column-major,
// B r x q column-major.  A thread keeps its pixel's r values of U for the
// workgroup's frames (blockIdx.y: fb of them), whose b_k are the same in every
// lane: U is read once per fb frames.  Bound by Z's stores:
// 256 x 256, 40 frames, rank 8: 12.1 us (24.6 with U read again for every
// frame).
template <int RT>
__global__ __launch_bounds__(256) void k_expand(const float2* U, const float2* B, const float2* zbar, const float2* E,
                                                long n, int q, int r, int fb, float2* Z, const DevState* st) {
  __shared__ float2 s_b[128 * RT];  // the frames' b_k (q <= 128)
  const long p = (long)blockIdx.x * 256 + threadIdx.x, pc = p < n ? p : n - 1;
  const int k0 = blockIdx.y * fb, k1 = min(q, k0 + fb);
  float2 u[RT];
  if (U) {
#pragma unroll
    for (int j = 0; j < RT; ++j) u[j] = U[(long)min(j, r - 1) * n + pc];
    for (int i = threadIdx.x; i < (k1 - k0) * RT; i += 256) {
      const int k = i / RT, j = i % RT;
      s_b[i] = B[(long)(k0 + k) * r + min(j, r - 1)];
    }
  }
  if (st->err) return;
  __syncthreads();
  const float2 z0 = zbar ? zbar[pc] : make_float2(0.f, 0.f);
#pragma unroll 2
  for (int k = k0; k < k1; ++k) {
    const float2 e = E ? E[(long)k * n + pc] : make_float2(0.f, 0.f);
    float re = 0.f, im = 0.f;
    if (U) {
#pragma unroll
      for (int j = 0; j < RT; ++j)
        if (j < r) {
          const float2 b = s_b[(k - k0) * RT + j];
          re += u[j].x * b.x - u[j].y * b.y;
          im += u[j].x * b.y + u[j].y * b.x;
        }
    }
    if (zbar) {
      re += z0.x;
      im += z0.y;
    }
    if (E) {
      re += e.x;
      im += e.y;
    }
    if (p < n) Z[(long)k * n + p] = make_float2(re, im);
  }
}

hipError_t launch_expand(const float2* U, const float2* B, const float2* zbar, const float2* E, long n, int q, int r,
                         float2* Z, const DevState* st, hipStream_t s) {
  // frames per workgroup: about 1,024 workgroups where there is that much work
  const long nx = (n + 255) / 256;
  const int fb = (int)std::max(1L, std::min<long>(q, nx * q / 1024));
  const dim3 g((unsigned)nx, (unsigned)((q + fb - 1) / fb));
  if (r <= 4) hipLaunchKernelGGL(k_expand<4>, g, dim3(256), 0, s, U, B, zbar, E, n, q, r, fb, Z, st);
  else if (r <= 8) hipLaunchKernelGGL(k_expand<8>, g, dim3(256), 0, s, U, B, zbar, E, n, q, r, fb, Z, st);
  else hipLaunchKernelGGL(k_expand<16>, g, dim3(256), 0, s, U, B, zbar, E, n, q, r, fb, Z, st);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// ISTA (MEC-2)
// ---------------------------------------------------------------------------
// The unitary DFT along the frames of 16 pixels by one wave on the matrix
// cores (v_mfma_f32_16x16x4f32: rows = frequencies, columns = pixels,
// contraction = frames).  Frames t and q - t share a twiddle up to conjugation,
// and so do frequencies k and q - k; with H = q/2 + 1 and
//   P_t = v_t + v_{q-t}, D_t = v_t - v_{q-t}   (v_{q-t} = 0 for t = 0, q/2)
//   A = sum_t Re P_t c_kt, B = sum_t Im D_t s_kt, C = sum_t Re D_t s_kt,
//   G = sum_t Im P_t c_kt,   c, s = cos, sin(2 pi k t / q), t < H,
// the forward transform is X_k = (A + B) + i (G - C), X_{q-k} = (A - B) + i (G + C)
// and the inverse the same with s negated: a quarter of the direct sum's
// products.  Contraction slot (ft, v) of lane group kk takes frame
// 16 ft + 4 kk + v, the order in which an accumulator holds its rows, so that
// one transform's results are the next one's operands without leaving their
// registers, and memory is read and written in 128-byte segments.
// f holds the lane's frames 16 ft + 4 kk + v of pixel l % 16, b their mirrors.
template <int FT, bool INV>
__device__ __forceinline__ void tdft_wave(float2 (&f)[FT][4], float2 (&b)[FT][4], const float2* s_tw, int q,
                                          float scale) {
  using Mf = Mma<float>;
  const int lane = threadIdx.x & 63, col = lane & 15, kk = lane >> 4;
  typename Mf::V A[FT], B[FT], C[FT], G[FT];
  int k1[FT], k13[FT], m[FT];  // the frequency, 13 times it (from frame 16 ft + 4 kk + 3 to the next tile's first), k t: mod q
#pragma unroll
  for (int o = 0; o < FT; ++o) {
    A[o] = B[o] = C[o] = G[o] = Mf::zero();
    k1[o] = (16 * o + col) % q;
    k13[o] = (13 * k1[o]) % q;
    m[o] = (4 * kk * k1[o]) % q;
  }
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float2 P = cadd(f[ft][v], b[ft][v]), D = csub(f[ft][v], b[ft][v]);
#pragma unroll
      for (int o = 0; o < FT; ++o) {
        const float2 w = s_tw[m[o]];
        m[o] += v < 3 ? k1[o] : k13[o];
        if (m[o] >= q) m[o] -= q;
        A[o] = Mf::mma(w.x, P.x, A[o]);
        B[o] = Mf::mma(w.y, D.y, B[o]);
        C[o] = Mf::mma(w.y, D.x, C[o]);
        G[o] = Mf::mma(w.x, P.y, G[o]);
      }
    }
  }
#pragma unroll
  for (int o = 0; o < FT; ++o)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float sb = INV ? -B[o][v] : B[o][v], sc = INV ? -C[o][v] : C[o][v];
      const int k = 16 * o + 4 * kk + v;
      const bool in = 2 * k <= q, mir = k > 0 && 2 * k < q;
      const float2 x = make_float2((A[o][v] + sb) * scale, (G[o][v] - sc) * scale);
      const float2 y = make_float2((A[o][v] - sb) * scale, (G[o][v] + sc) * scale);
      f[o][v] = in ? x : make_float2(0.f, 0.f);
      b[o][v] = mir ? y : make_float2(0.f, 0.f);
    }
}

__device__ __forceinline__ double wave_max_parts(const double* p, int nb, int lane) {
  double m = 0.0;
  for (int i = lane; i < nb; i += 64) m = fmax(m, p[i]);
  return wave_max(m);
}

// the scalars before update t >= 1: the stop test of update t - 1 (its change
// is defined from t - 1 >= 1 on), the same in every wave
__device__ __forceinline__ IstaState ista_open(const IstaState* in, const double* pin, int np, int t, double tol) {
  IstaState o = *in;
  if (o.done || t < 1) return o;
  const int lane = threadIdx.x & 63;
  if (t >= 2) {
    double d = 0.0, r = 0.0;
    for (int i = lane; i < np; i += 64) {
      d += pin[2 * i];
      r += pin[2 * i + 1];
    }
    d = wave_sum(d);
    r = wave_sum(r);
    o.last_change = r > 0.0 ? sqrt(d / r) : 0.0;
    o.done = o.last_change < tol;
  }
  o.iters = t;
  return o;
}

// One wave per 16 pixels:
//   ISTA_FIRST   M_0 = F_t(sum of w's parts) (E_0 = 0); partial max |M_0|
//   ISTA_THRESH  omega = frac max |M_0|; E_1 = F_t^-1(SThr_omega(M_0))
//   ISTA_STEP    M_t = F_t(E_t + sum of w's parts), its distance to M_{t-1}
//                (replaced in memory), E_{t+1} = F_t^-1(SThr_omega(M_t))
// SThr: s/|s| (|s| - omega) where |s| > omega, else 0.  Bound by memory
// latency at 128 x 128 (one wave per SIMD) and by memory above.  q = 48,
// 128 x 128: 14 us an update, against 95 us for a direct-summation DFT each
// way (54) and separate kernels for the sum, the change and the scalars.
template <int FT, int PHASE>
__global__ __launch_bounds__(256) void k_ista_dft(IstaArgs a) {
  __shared__ float2 s_tw[128];
  __shared__ double s_red[2][4];
  if (a.st->err) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 15, kk = lane >> 4;
  const int q = a.q, np = gridDim.x;
  const bool w0 = blockIdx.x == 0 && tid == 0;
  const long p = (long)blockIdx.x * 64 + 16 * wave + col;  // n is a multiple of 64
  // requested first: every frame of the pixel, valid (clamped) addresses
  float2 f[FT][4], b[FT][4], mf[FT][4], mb[FT][4];
  auto load = [&](const float2* src, float2 (&x)[FT][4], float2 (&y)[FT][4]) {
#pragma unroll
    for (int o = 0; o < FT; ++o)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int t = 16 * o + 4 * kk + v, t0 = 2 * t <= q ? t : 0, t1 = t > 0 && 2 * t < q ? q - t : 0;
        x[o][v] = src[(long)t0 * a.n + p];
        y[o][v] = src[(long)t1 * a.n + p];
      }
  };
  if (PHASE == ISTA_THRESH) {
    load(a.M, f, b);
  } else {
    load(a.w, f, b);
    if (PHASE == ISTA_STEP) {
      load(a.E, mf, mb);
#pragma unroll
      for (int o = 0; o < FT; ++o)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          f[o][v] = cadd(mf[o][v], f[o][v]);
          b[o][v] = cadd(mb[o][v], b[o][v]);
        }
      load(a.M, mf, mb);
    }
    for (int g = 1; g < a.nsum; ++g) {
      float2 x[FT][4], y[FT][4];
      load(a.w + g * a.part_stride, x, y);
#pragma unroll
      for (int o = 0; o < FT; ++o)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          f[o][v] = cadd(f[o][v], x[o][v]);
          b[o][v] = cadd(b[o][v], y[o][v]);
        }
    }
  }
  for (int e = tid; e < q; e += 256) {
    double sv, cv;
    sincospi(2.0 * (double)e / (double)q, &sv, &cv);
    s_tw[e] = make_float2((float)cv, (float)sv);
  }
  double om = 0.0;
  if (PHASE == ISTA_THRESH) {
    om = a.frac * wave_max_parts(a.pin, np, lane);
    if (w0) {
      IstaState o{};
      o.omega = om;
      *a.out = o;
    }
  } else if (PHASE == ISTA_STEP) {
    const IstaState o = ista_open(a.in, a.pin, np, a.t, a.tol);
    if (w0) *a.out = o;
    if (o.done) return;
    om = o.omega;
  }
  __syncthreads();
  // values at no frame (t past q/2, mirrors of 0 and q/2) are zero
  auto mask = [&](float2 (&x)[FT][4], float2 (&y)[FT][4]) {
#pragma unroll
    for (int o = 0; o < FT; ++o)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int t = 16 * o + 4 * kk + v;
        if (!(2 * t <= q)) x[o][v] = make_float2(0.f, 0.f);
        if (!(t > 0 && 2 * t < q)) y[o][v] = make_float2(0.f, 0.f);
      }
  };
  mask(f, b);
  auto store = [&](float2* dst) {
#pragma unroll
    for (int o = 0; o < FT; ++o)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int t = 16 * o + 4 * kk + v;
        if (2 * t <= q) dst[(long)t * a.n + p] = f[o][v];
        if (t > 0 && 2 * t < q) dst[(long)(q - t) * a.n + p] = b[o][v];
      }
  };
  double r0 = 0.0, r1 = 0.0;
  if (PHASE != ISTA_THRESH) {
    tdft_wave<FT, false>(f, b, s_tw, q, a.scale);
    store(a.M);
    if (PHASE == ISTA_STEP) mask(mf, mb);
#pragma unroll
    for (int o = 0; o < FT; ++o)
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const float2 u = h ? b[o][v] : f[o][v];
          if (PHASE == ISTA_FIRST) {
            r0 = fmax(r0, (double)u.x * u.x + (double)u.y * u.y);
          } else {
            const float2 m = h ? mb[o][v] : mf[o][v];
            const double dx = (double)u.x - m.x, dy = (double)u.y - m.y;
            r0 += dx * dx + dy * dy;
            r1 += (double)m.x * m.x + (double)m.y * m.y;
          }
        }
  }
  if (PHASE != ISTA_FIRST) {
    const float omf = (float)om;
    auto thr = [&](float2 v) {
      const float m = sqrtf(v.x * v.x + v.y * v.y);
      return cscale(v, m > omf ? (m - omf) / m : 0.f);
    };
#pragma unroll
    for (int o = 0; o < FT; ++o)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        f[o][v] = thr(f[o][v]);
        b[o][v] = thr(b[o][v]);
      }
    tdft_wave<FT, true>(f, b, s_tw, q, a.scale);
    store(a.E);
  }
  if (PHASE == ISTA_THRESH) return;
  if (PHASE == ISTA_FIRST) {
    r0 = wave_max(sqrt(r0));
  } else {
    r0 = wave_sum(r0);
    r1 = wave_sum(r1);
  }
  if (lane == 0) {
    s_red[0][wave] = r0;
    s_red[1][wave] = r1;
  }
  __syncthreads();
  if (tid == 0) {
    if (PHASE == ISTA_FIRST) {
      a.pout[blockIdx.x] = fmax(fmax(s_red[0][0], s_red[0][1]), fmax(s_red[0][2], s_red[0][3]));
    } else {
      a.pout[2 * blockIdx.x] = (s_red[0][0] + s_red[0][1]) + (s_red[0][2] + s_red[0][3]);
      a.pout[2 * blockIdx.x + 1] = (s_red[1][0] + s_red[1][1]) + (s_red[1][2] + s_red[1][3]);
    }
  }
}

// E_0 = 0, and the scalars' first slots
__global__ void k_ista_begin(float2* E, long total, IstaState* is) {
  if (blockIdx.x == 0 && threadIdx.x < 2) is[threadIdx.x] = IstaState{};
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (long)gridDim.x * blockDim.x)
    E[i] = make_float2(0.f, 0.f);
}

// the stop test after the last update, for the count
__global__ void k_ista_end(const IstaState* in, IstaState* out, const double* pin, int np, int t, double tol,
                           const DevState* st) {
  if (st->err) return;
  const IstaState o = ista_open(in, pin, np, t, tol);
  if (threadIdx.x == 0) *out = o;
}

// FT: tiles of 16 frequencies that hold 0 .. q/2
template <int PHASE>
static void ista_launch(const IstaArgs& a, hipStream_t s) {
  const dim3 g((unsigned)(a.n / 64));
  switch ((a.q / 2 + 16) / 16) {
    case 1: hipLaunchKernelGGL((k_ista_dft<1, PHASE>), g, dim3(256), 0, s, a); break;
    case 2: hipLaunchKernelGGL((k_ista_dft<2, PHASE>), g, dim3(256), 0, s, a); break;
    case 3: hipLaunchKernelGGL((k_ista_dft<3, PHASE>), g, dim3(256), 0, s, a); break;
    case 4: hipLaunchKernelGGL((k_ista_dft<4, PHASE>), g, dim3(256), 0, s, a); break;
    default: hipLaunchKernelGGL((k_ista_dft<5, PHASE>), g, dim3(256), 0, s, a); break;
  }
}

hipError_t launch_ista_dft(const IstaArgs& a, int phase, hipStream_t s) {
  if (a.n % 64 != 0 || a.q < 1 || a.q > 128) return hipErrorInvalidValue;
  if (phase == ISTA_FIRST) ista_launch<ISTA_FIRST>(a, s);
  else if (phase == ISTA_THRESH) ista_launch<ISTA_THRESH>(a, s);
  else ista_launch<ISTA_STEP>(a, s);
  return hipGetLastError();
}

}  // namespace ag
