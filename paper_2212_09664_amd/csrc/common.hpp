// Shared device helpers for the altGDmin kernels (gfx950): complex
// arithmetic, the device-side state block and an LDS-staged Stockham FFT.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#define AG_NT 256  // threads per workgroup for the streaming kernels

// ---------------------------------------------------------------------------
// complex helpers (interleaved float2 / double2)
// ---------------------------------------------------------------------------
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// conj(a) * b
__device__ __forceinline__ float2 cjmul(float2 a, float2 b) {
  return make_float2(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);
}
__device__ __forceinline__ float2 cscale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }
// acc + a * b and acc + a * conj(b) as two fused multiply-adds per part
// (cadd(acc, cmul(a, b)) costs six instructions: the sum is rounded apart)
__device__ __forceinline__ float2 cfma(float2 acc, float2 a, float2 b) {
  return make_float2(fmaf(-a.y, b.y, fmaf(a.x, b.x, acc.x)), fmaf(a.y, b.x, fmaf(a.x, b.y, acc.y)));
}
__device__ __forceinline__ float2 cfmaj(float2 acc, float2 a, float2 b) {
  return make_float2(fmaf(a.y, b.y, fmaf(a.x, b.x, acc.x)), fmaf(-a.x, b.y, fmaf(a.y, b.x, acc.y)));
}
// acc + conj(a) * b
__device__ __forceinline__ float2 cjfma(float2 acc, float2 a, float2 b) {
  return make_float2(fmaf(a.y, b.y, fmaf(a.x, b.x, acc.x)), fmaf(-a.y, b.x, fmaf(a.x, b.y, acc.y)));
}

__device__ __forceinline__ double2 dadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 dsub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 dmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 djmul(double2 a, double2 b) {  // conj(a) * b
  return make_double2(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);
}
__device__ __forceinline__ double2 dconj(double2 a) { return make_double2(a.x, -a.y); }
// the names the transforms use in either precision
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return dadd(a, b); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return dsub(a, b); }
__device__ __forceinline__ double2 cmul(double2 a, double2 b) { return dmul(a, b); }
__device__ __forceinline__ double2 f2d(float2 a) { return make_double2((double)a.x, (double)a.y); }
__device__ __forceinline__ float2 d2f(double2 a) { return make_float2((float)a.x, (float)a.y); }

// ---------------------------------------------------------------------------
// device state (one block at the start of the workspace)
// ---------------------------------------------------------------------------
struct DevState {
  int32_t err;        // 0 or an altgdmin_status
  int32_t err_frame;  // frame of a non-positive-definite Gram, -1 otherwise
  int32_t halt;       // 1: every later kernel of the loop returns at once
  int32_t step_ok;    // 1: the current iteration's GD + QR step is applied
  int32_t t;          // iterations completed
  int32_t exited;     // exit rule fired
  int32_t converged;  // stationary start (grad_0 = 0)
  int32_t n_units;    // distinct sampled lines (LINES) / locations (INDEX)
  double eta;         // step size (<= 0: not yet set)
  double gamma;       // truncation threshold
  double ysq;         // sum_k ||y_k||^2
  double mbar;        // mean samples per coil
  double f;           // cost of the last iteration
  double sd;          // SD(U_{t-1}, U_t)
  double grad_norm;   // ||grad||_F of the last iteration
  double cost_out;    // scratch for altgdmin_cost
  int32_t n_gwork;    // LINES: (line, sample tile) work items of the Gram kernel
  int32_t step_flags; // the fused QR step's outcome, committed after it (STEP_*)
  double eta_next;    // the step size it used (committed after it)
  int32_t stats_pending;  // 1: f, sd and grad_norm of the last step wait in the statistics inputs
  int32_t n_trunc;    // samples zeroed by the truncation of the last initialisation
  int32_t exit_run;   // consecutive iterations that met the exit test
  int32_t pad_e;
  double pad[2];
};
// the loop's stop test: err and halt both requested before either is tested
// (a short-circuit test waits for one load before issuing the other)
__device__ __forceinline__ bool halted(const DevState* st, int check_halt) {
  const int e = st->err, h = st->halt;
  return (e | (h & -(check_halt != 0))) != 0;
}
#define STEP_APPLIED 1
#define STEP_EXIT 2
#define STEP_CONVERGED 4

// ---------------------------------------------------------------------------
// in-register DFTs of radix 2, 4, 8, 16 (C: float2 or double2)
// Output k of the radix-R DFT ends up in register out_pos<R>(k).
// ---------------------------------------------------------------------------
template <bool INV, typename C>
__device__ __forceinline__ C mul_mi(C v) {  // * (-i) forward, * (+i) inverse
  return INV ? C{-v.y, v.x} : C{v.y, -v.x};
}

template <bool INV, typename C>
__device__ __forceinline__ void dft2(C& a, C& b) {
  C t = a;
  a = cadd(t, b);
  b = csub(t, b);
}

template <bool INV, typename C>
__device__ __forceinline__ void dft4(C& a0, C& a1, C& a2, C& a3) {
  C s02 = cadd(a0, a2), d02 = csub(a0, a2), s13 = cadd(a1, a3), d13 = csub(a1, a3);
  C t = mul_mi<INV>(d13);
  a0 = cadd(s02, s13);
  a2 = csub(s02, s13);
  a1 = cadd(d02, t);
  a3 = csub(d02, t);
}

// v * exp(-+ 2 pi i k / 16), k a compile-time constant after unrolling
template <bool INV, typename C>
__device__ __forceinline__ C tw16(C v, int k) {
  using F = decltype(v.x + v.x);
  const F C1 = (F)0.92387953251128674, C2 = (F)0.70710678118654752, C3 = (F)0.38268343236508977;
  F c, s;
  switch (k & 15) {
    case 0: return v;
    case 1: c = C1; s = C3; break;
    case 2: c = C2; s = C2; break;
    case 3: c = C3; s = C1; break;
    case 4: return mul_mi<INV>(v);
    case 5: c = -C3; s = C1; break;
    case 6: c = -C2; s = C2; break;
    case 7: c = -C1; s = C3; break;
    case 8: return C{-v.x, -v.y};
    case 9: c = -C1; s = -C3; break;
    default: c = (F)1; s = (F)0; break;
  }
  // forward: (c - i s); inverse: (c + i s)
  return cmul(v, INV ? C{c, s} : C{c, -s});
}

template <int R>
__device__ __forceinline__ constexpr int out_pos(int k) {
  return R == 16 ? 4 * (k % 4) + k / 4 : (R == 8 ? 4 * (k % 2) + k / 2 : k);
}

template <int R, bool INV, typename C>
__device__ __forceinline__ void dft_reg(C* v) {
  if constexpr (R == 2) {
    dft2<INV>(v[0], v[1]);
  } else if constexpr (R == 4) {
    dft4<INV>(v[0], v[1], v[2], v[3]);
  } else if constexpr (R == 8) {
    // n = 4a + b, k = c + 2d
#pragma unroll
    for (int b = 0; b < 4; ++b) dft2<INV>(v[b], v[4 + b]);
#pragma unroll
    for (int b = 1; b < 4; ++b) v[4 + b] = tw16<INV>(v[4 + b], 2 * b);
#pragma unroll
    for (int c = 0; c < 2; ++c) dft4<INV>(v[4 * c], v[4 * c + 1], v[4 * c + 2], v[4 * c + 3]);
  } else if constexpr (R == 16) {
    // n = 4a + b, k = c + 4d
#pragma unroll
    for (int b = 0; b < 4; ++b) dft4<INV>(v[b], v[4 + b], v[8 + b], v[12 + b]);
#pragma unroll
    for (int c = 1; c < 4; ++c)
#pragma unroll
      for (int b = 1; b < 4; ++b) v[4 * c + b] = tw16<INV>(v[4 * c + b], b * c);
#pragma unroll
    for (int c = 0; c < 4; ++c) dft4<INV>(v[4 * c], v[4 * c + 1], v[4 * c + 2], v[4 * c + 3]);
  }
}

// ---------------------------------------------------------------------------
// Stockham autosort FFT of TX columns of length N (a power of two in [8, 512])
// held in LDS as s[e*TX+col] (column index fastest), by a workgroup of NT
// threads.  Each pass of radix R reads R points at stride N/R, applies the
// twiddles exp(-+2 pi i (j mod Ns) r / (Ns R)), does an in-register radix-R DFT
// and writes them at stride Ns.  tw[t] holds exp(-2 pi i t / N).
// Unnormalised.  The double-precision transforms of the mean's right-hand
// side run once a call through this form; the others are register-fed.
// ---------------------------------------------------------------------------
template <int N, int R, int TX, int NT, bool INV, typename C>
__device__ __forceinline__ void stockham_pass(C* s, const C* tw, int Ns) {
  constexpr int G = TX * (N / R), IT = (G + NT - 1) / NT;
  C v[IT][R];
  const int tid = threadIdx.x;
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int g = tid + it * NT;
    if (g < G) {
      const int col = g % TX, j = g / TX, step = (j % Ns) * (N / (Ns * R));
#pragma unroll
      for (int r = 0; r < R; ++r) {
        v[it][r] = s[(j + r * (N / R)) * TX + col];
        if (Ns > 1 && r > 0) {
          const C w = tw[step * r];
          v[it][r] = cmul(v[it][r], INV ? C{w.x, -w.y} : w);
        }
      }
      dft_reg<R, INV>(v[it]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int g = tid + it * NT;
    if (g < G) {
      const int col = g % TX, j = g / TX, d = (j / Ns) * Ns * R + (j % Ns);
#pragma unroll
      for (int r = 0; r < R; ++r) s[(d + r * Ns) * TX + col] = v[it][out_pos<R>(r)];
    }
  }
  __syncthreads();
}

template <int N, int TX, int NT, bool INV, typename C>
__device__ __forceinline__ void fft_lds(C* s, const C* tw) {
  constexpr int R0 = N == 16 ? 4 : 8, N1 = N / R0;                  // 8: one pass of radix 8
  constexpr int R1 = N1 == 1 ? 1 : (N1 % 8 == 0 ? 8 : 4), N2 = N1 / R1;
  stockham_pass<N, R0, TX, NT, INV>(s, tw, 1);
  if constexpr (R1 > 1) stockham_pass<N, R1, TX, NT, INV>(s, tw, R0);
  if constexpr (N2 > 1) stockham_pass<N, N2, TX, NT, INV>(s, tw, R0 * R1);
}

// ---------------------------------------------------------------------------
// The transform with its first pass fed from registers and its last pass
// left in registers: only the passes in between go through LDS.
//   input  item (it, r) of thread t, g = t + it*NT: row g/TX + r*(N/R0),
//          column g%TX;
//   output item (it, r): row out_row(g, r), column g%TX.
// tw[t] = exp(-+2 pi i t / N) in the transform's own direction (the caller
// passes the conjugated table for the inverse).  For N = 8 (one pass) no
// LDS is touched.  The function returns with the LDS tile free for reuse
// (its last LDS read is followed by a barrier).
// ---------------------------------------------------------------------------
// (16 as 4 x 4: one pass of radix 16 keeps a whole column in a thread, 160 to
// 240 registers in the operators' kernels, and leaves most of a small tile's
// threads idle: 3.3 us against 6.3 for the columns of 16 x 16)
template <int N> struct FftPlan;
template <> struct FftPlan<8>   { static constexpr int P = 1, R0 = 8,  RL = 8;  };
template <> struct FftPlan<16>  { static constexpr int P = 2, R0 = 4,  RL = 4;  };
template <> struct FftPlan<32>  { static constexpr int P = 2, R0 = 8,  RL = 4;  };
template <> struct FftPlan<64>  { static constexpr int P = 2, R0 = 8,  RL = 8;  };
template <> struct FftPlan<128> { static constexpr int P = 2, R0 = 16, RL = 8;  };
template <> struct FftPlan<256> { static constexpr int P = 2, R0 = 16, RL = 16; };
template <> struct FftPlan<512> { static constexpr int P = 3, R0 = 8,  RL = 8;  };

// REV swaps the radices of the first and the last pass (the input layout of
// the reversed plan is the output layout of the plain one and the other way
// round, so that a transform can feed an inverse one without leaving its
// registers).  ROWS transforms TX contiguous rows instead of TX interleaved
// columns: consecutive threads take consecutive elements of a row, so that
// memory rows are read and written in whole segments, and the LDS tile holds
// row after row, one element of padding after every 16 (the first pass's
// strided writes then fall in different banks).
template <int N, int TX, int NT, bool REV = false, bool ROWS = false>
struct FftGeom {
  using PL = FftPlan<N>;
  static constexpr int R0 = REV ? PL::RL : PL::R0, RL = REV ? PL::R0 : PL::RL;
  static constexpr int G0 = TX * (N / R0), IT0 = (G0 + NT - 1) / NT;
  static constexpr int GL = TX * (N / RL), ITL = (GL + NT - 1) / NT;
  static constexpr int PITCH = N + N / 16;                      // ROWS: LDS row pitch
  static constexpr int LDS = PL::P == 1 ? 1 : (ROWS ? PITCH * TX : N * TX);  // float2 entries of the tile
  __device__ static bool in_ok(int g) { return (G0 % NT == 0) || g < G0; }
  __device__ static bool out_ok(int g) { return (GL % NT == 0) || g < GL; }
  // column (ROWS: row of the batch) and sub-index of group g of a pass of radix R
  template <int R> __device__ static int colr(int g) { return ROWS ? g / (N / R) : g % TX; }
  template <int R> __device__ static int jr(int g) { return ROWS ? g % (N / R) : g / TX; }
  __device__ static int in_col(int g) { return colr<R0>(g); }
  __device__ static int out_col(int g) { return colr<RL>(g); }
  __device__ static int in_row(int g, int r) { return jr<R0>(g) + r * (N / R0); }
  __device__ static int out_row(int g, int r) {
    return PL::P == 1 ? jr<RL>(g) * R0 + r : jr<RL>(g) + r * (N / RL);
  }
  __device__ static int at(int e, int col) { return ROWS ? col * PITCH + e + e / 16 : e * TX + col; }
};

// CONJ: tw is the forward table and the transform wants its conjugate
template <int N, int TX, int NT, bool INV, bool CONJ = false, bool REV = false, bool ROWS = false, int IT0_, int R0_,
          int ITL_, int RL_>
__device__ __forceinline__ void fft_regs(float2 (&v0)[IT0_][R0_], float2 (&vo)[ITL_][RL_], float2* s,
                                         const float2* __restrict__ tw) {
  using GM = FftGeom<N, TX, NT, REV, ROWS>;
  static_assert(IT0_ == GM::IT0 && R0_ == GM::R0 && ITL_ == GM::ITL && RL_ == GM::RL,
                "register tiles do not match the plan");
  constexpr int R0 = GM::R0, RL = GM::RL, P = FftPlan<N>::P;
  const int tid = threadIdx.x % NT;
  auto twd = [&](int t) {
    const float2 w = tw[t];
    return CONJ ? make_float2(w.x, -w.y) : w;
  };
#pragma unroll
  for (int it = 0; it < GM::IT0; ++it)
    if (GM::in_ok(tid + it * NT)) dft_reg<R0, INV>(v0[it]);
  if constexpr (P == 1) {
#pragma unroll
    for (int it = 0; it < GM::IT0; ++it)
#pragma unroll
      for (int r = 0; r < R0; ++r) vo[it][r] = v0[it][out_pos<R0>(r)];
    return;
  } else {
    // first pass: Ns = 1, outputs to rows j*R0 + r
#pragma unroll
    for (int it = 0; it < GM::IT0; ++it) {
      const int g = tid + it * NT;
      if (GM::in_ok(g)) {
        const int col = GM::in_col(g), j = GM::template jr<R0>(g);
#pragma unroll
        for (int r = 0; r < R0; ++r) s[GM::at(j * R0 + r, col)] = v0[it][out_pos<R0>(r)];
      }
    }
    __syncthreads();
    if constexpr (P == 3) {  // the middle pass, radix 8 at Ns = R0, in place
      constexpr int G = TX * (N / 8), IT = (G + NT - 1) / NT;
      float2 v[IT][8];
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int g = tid + it * NT;
        if ((G % NT == 0) || g < G) {
          const int col = GM::template colr<8>(g), j = GM::template jr<8>(g);
#pragma unroll
          for (int r = 0; r < 8; ++r) v[it][r] = s[GM::at(j + r * (N / 8), col)];
          const int step = (j % R0) * (N / (R0 * 8));
#pragma unroll
          for (int r = 1; r < 8; ++r) v[it][r] = cmul(v[it][r], twd(step * r));
          dft_reg<8, INV>(v[it]);
        }
      }
      __syncthreads();
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int g = tid + it * NT;
        if ((G % NT == 0) || g < G) {
          const int col = GM::template colr<8>(g), j = GM::template jr<8>(g);
          const int d = (j / R0) * R0 * 8 + (j % R0);
#pragma unroll
          for (int r = 0; r < 8; ++r) s[GM::at(d + r * R0, col)] = v[it][out_pos<8>(r)];
        }
      }
      __syncthreads();
    }
    // last pass: Ns = N/RL, reads rows j + r*Ns, outputs rows j + r*Ns
#pragma unroll
    for (int it = 0; it < GM::ITL; ++it) {
      const int g = tid + it * NT;
      if (GM::out_ok(g)) {
        const int col = GM::out_col(g), j = GM::template jr<RL>(g);
#pragma unroll
        for (int r = 0; r < RL; ++r) vo[it][r] = s[GM::at(j + r * (N / RL), col)];
      }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < GM::ITL; ++it) {
      const int g = tid + it * NT;
      if (GM::out_ok(g)) {
        const int j = GM::template jr<RL>(g);
#pragma unroll
        for (int r = 1; r < RL; ++r) vo[it][r] = cmul(vo[it][r], twd(j * r));
        dft_reg<RL, INV>(vo[it]);
        float2 t[RL];
#pragma unroll
        for (int r = 0; r < RL; ++r) t[r] = vo[it][out_pos<RL>(r)];
#pragma unroll
        for (int r = 0; r < RL; ++r) vo[it][r] = t[r];
      }
    }
  }
}
