// The learned warm start: a 4-layer 3x3 CNN mapping the 2q back-projected
// planes of a sequence to an n x r complex matrix M (channel 2j = Re M[:, j],
// 2j + 1 = Im M[:, j]), its projection loss L = r - tr(G^-1 C C^H)
// (G = M^H M, C = M^H U_tgt), the backward pass and Adam.
//
// Convolutions are implicit GEMMs on the matrix cores with BF16 operands and
// FP32 accumulation (v_mfma_f32_16x16x32_bf16; activations, gradients and
// the parameters stay FP32 in memory; activations are rounded to BF16 as they
// are staged in LDS, weights when they are packed):
//   forward      D[co][px] = sum over (channel chunk, tap) of W[co][ci] X'[ci][px],
//                plus the bias in FP32;
//   input grad   the same kernel on dY with the flipped, transposed weights,
//                times the ReLU mask of the layer below;
//   weight grad  D[co][ci] = sum_px dY'[co][px] X[ci][px] per tap (dY' the
//                shifted dY), per band of image rows, then a deterministic
//                reduction.
// X'[kappa][px] is the input channel ci shifted by the tap (zero outside the
// image).  Activations are [b][c][H][W] FP32.  MFMA lane layout (16x16x32):
// lane l holds A[l%16][8(l/16)+e] and B[8(l/16)+e][l%16], e = 0..7; result
// register v holds D[4(l/16)+v][l%16].
#include <algorithm>

#include "kernels_core.hpp"
#include "mma.hpp"

namespace ag {

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f4v mfma_bf16(const bf8& a, const bf8& b, f4v c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// loads of four consecutive floats at any float's address
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
typedef __bf16 bf4 __attribute__((ext_vector_type(4)));

constexpr int CV_CH = 32;   // input channels per chunk (one matrix-core contraction)
constexpr int CV_CHP = 40;  // BF16 pitch of a staged pixel's channels (80 bytes: 16-byte aligned, banks spread)

// ---------------------------------------------------------------------------
// every layer's weights in BF16, in the order the matrix cores take them:
// [chunk of 32 input channels][tap][output tile of 16][lane][8], so that a
// wave loads an operand as 1 KB in one piece.  Forward: the layer's weights;
// input gradient: the flipped, transposed ones.  Rounded once per pass, not
// once per tile.  Grid (blocks, 2 * layers).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_cnn_pack(CnnLayers a) {
  const int l = blockIdx.y >> 1, back = blockIdx.y & 1;
  __bf16* out = reinterpret_cast<__bf16*>(back ? a.Wb[l] : a.Wf[l]);
  if (!out) return;
  const int cin = a.cin[l], cout = a.cout[l];
  const int ki = back ? cout : cin, ko = back ? cin : cout;  // contraction and output channels
  const float* W = a.W[l];
  const int total = (ki + CV_CH - 1) / CV_CH * 9 * 2 * 512;
  for (int e = blockIdx.x * 256 + threadIdx.x; e < total; e += gridDim.x * 256) {
    const int q = e & 7, lane = (e >> 3) & 63, ot = (e >> 9) & 1, tap = (e >> 10) % 9, ch = (e >> 10) / 9;
    const int o = 16 * ot + (lane & 15), i = ch * CV_CH + 8 * (lane >> 4) + q;
    float v = 0.f;
    if (o < ko && i < ki) v = back ? W[((long)i * cin + o) * 9 + (8 - tap)] : W[((long)o * cin + i) * 9 + tap];
    out[e] = (__bf16)v;
  }
}

// ---------------------------------------------------------------------------
// convolution as implicit GEMM: grid (tiles of TW x TH = 256 or 64 pixels, batch),
// 256 threads; a wave computes TH / 4 tile rows, 16 pixels of a row per
// matrix-core product, for all output channels (<= 32).  Per chunk of 32
// input channels the tile's inputs (with the halo) are staged once as BF16
// [pixel][channel], the chunk's weights come packed straight to registers,
// and a staged row serves the output rows it belongs to.  Products of an
// output are added in the order chunk, tap.  Bound by the latency of the
// staging loads.  16 sequences of 128 x 128: 96 -> 32 channels 54 us, 32 -> 32
// 28 us; 8 x 8 tiles that staged and rounded the weights each time took 59 us
// a layer on average.
// ---------------------------------------------------------------------------
template <int TW, int TH>
__global__ __launch_bounds__(256) void k_conv(ConvArgs a) {
  constexpr int HW = TW + 2, NPX = HW * (TH + 2), RW = TH / 4, NX = TW / 16;
  __shared__ __attribute__((aligned(16))) __bf16 xs[NPX * CV_CHP];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tiles_x = (a.W + TW - 1) / TW;
  const int ty0 = (blockIdx.x / tiles_x) * TH, tx0 = (blockIdx.x % tiles_x) * TW;
  const int b = blockIdx.y;
  const long plane = (long)a.H * a.W;
  const float* Xb = a.X + (long)b * a.cin * plane;
  const int pl = lane & 15, kq = lane >> 4;
  f4v acc[RW][NX][2];
#pragma unroll
  for (int y = 0; y < RW; ++y)
#pragma unroll
    for (int x = 0; x < NX; ++x) acc[y][x][0] = acc[y][x][1] = f4v{0.f, 0.f, 0.f, 0.f};
  for (int c0 = 0; c0 < a.cin; c0 += CV_CH) {
    const int nch = min(CV_CH, a.cin - c0);
    __syncthreads();
    // (pixel, channel octet); every load comes from a valid address and
    // values outside the image or past cin are selected to zero
    for (int e = tid; e < NPX * 4; e += 256) {
      const int pix = e % NPX, j = e / NPX;
      const int gy = ty0 + pix / HW - 1, gx = tx0 + pix % HW - 1;
      const bool in = gy >= 0 && gy < a.H && gx >= 0 && gx < a.W;
      const long off = in ? (long)gy * a.W + gx : 0;
      float f[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) f[q] = Xb[(long)(c0 + min(8 * j + q, nch - 1)) * plane + off];
      bf8 v;
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = (__bf16)((in && 8 * j + q < nch) ? f[q] : 0.f);
      *reinterpret_cast<bf8*>(&xs[pix * CV_CHP + 8 * j]) = v;
    }
    const bf8* wq = reinterpret_cast<const bf8*>(a.Wq) + (long)(c0 / CV_CH) * 18 * 64 + lane;
    bf8 w[9][2];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      w[t][0] = wq[(2 * t) * 64];
      w[t][1] = wq[(2 * t + 1) * 64];
    }
    __syncthreads();
    // output row y takes staged row y + dy for tap row dy; rows in order, so
    // that each output's taps are added in order
#pragma unroll
    for (int y = 0; y < RW + 2; ++y) {
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) {
#pragma unroll
        for (int x = 0; x < NX; ++x) {
          const bf8 bv =
              *reinterpret_cast<const bf8*>(&xs[((RW * wave + y) * HW + 16 * x + pl + dx) * CV_CHP + 8 * kq]);
#pragma unroll
          for (int dy = 0; dy < 3; ++dy) {
            const int o = y - dy;
            if (o >= 0 && o < RW) {
              acc[o][x][0] = mfma_bf16(w[3 * dy + dx][0], bv, acc[o][x][0]);
              acc[o][x][1] = mfma_bf16(w[3 * dy + dx][1], bv, acc[o][x][1]);
            }
          }
        }
      }
    }
  }
  float* Yb = a.Y + (long)b * a.cout * plane;
  // one output tile of 16 channels at a time; its mask values are requested
  // together (valid, clamped addresses) before any is used
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    if (16 * t >= a.cout) break;
    float mk[4][RW][NX];
    if (a.mask) {
      const float* Mb = a.mask + (long)b * a.cout * plane;
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int y = 0; y < RW; ++y)
#pragma unroll
          for (int x = 0; x < NX; ++x)
            mk[v][y][x] = Mb[(long)min(16 * t + 4 * kq + v, a.cout - 1) * plane +
                             (long)min(ty0 + RW * wave + y, a.H - 1) * a.W + min(tx0 + 16 * x + pl, a.W - 1)];
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int co = 16 * t + 4 * kq + v;
      if (co < a.cout) {
        const float bias = a.bias ? a.bias[co] : 0.f;
#pragma unroll
        for (int y = 0; y < RW; ++y) {
#pragma unroll
          for (int x = 0; x < NX; ++x) {
            const int oy = ty0 + RW * wave + y, ox = tx0 + 16 * x + pl;
            if (oy < a.H && ox < a.W) {
              float o = acc[y][x][t][v];
              if (a.bias) o += bias;
              if (a.relu) o = fmaxf(o, 0.f);
              if (a.mask && !(mk[v][y][x] > 0.f)) o = 0.f;
              Yb[(long)co * plane + (long)oy * a.W + ox] = o;
            }
          }
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// weight gradient: dW[co][ci][dy][dx] = sum over pixels (y, x) of
// dY[co][y - dy + 1][x - dx + 1] X[ci][y][x], one 16 x 16 x 32 product per tap for 32
// pixels of a row.  The shift is put on dY, whose 32 channels are staged in
// three copies (one per dx), so that every operand of the matrix cores is
// one aligned 16-byte LDS read; a staged row of dY serves the three rows of X
// that its dy reach.  Grid (bands of CNN_BAND image rows, batch, groups of
// 32 CIT input channels), 256 threads: wave w takes output tile w % 2 and
// input tiles (w / 2) CIT .. + CIT - 1, all nine taps.  The next block of rows
// is loaded while the current one feeds the matrix cores.  Partials
// part[kappa = tap*cin + ci][co], kappa = 9 cin the bias.  16 sequences of
// 128 x 128: 96 channels 55 us and 32 channels 31 us, 150 us over the four
// layers; with the shift on X (eight 2-byte LDS reads per operand) 764 us.
// ---------------------------------------------------------------------------
constexpr int WG_R = 4;                      // rows of X per block
constexpr int WG_X = 32;                     // pixels of a row per block
constexpr int WG_XP = WG_R * WG_X + 8;       // BF16 pitch of a staged input channel
constexpr int WG_DP = (WG_R + 2) * WG_X + 8; // and of an output channel's copy
template <int CIT>
__global__ __launch_bounds__(256) void k_conv_wgrad(WgradArgs a) {
  constexpr int NCI = 32 * CIT;
  constexpr int XI = NCI * WG_R * (WG_X / 4) / 256;        // groups of 4 pixels of X per thread
  constexpr int DI = 32 * (WG_R + 2) * (WG_X / 4) / 256;   // and of dY
  __shared__ __attribute__((aligned(16))) __bf16 xs[NCI * WG_XP];
  __shared__ __attribute__((aligned(16))) __bf16 ds[3 * 32 * WG_DP];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int pl = lane & 15, kq = lane >> 4, cot = wave & 1, half = wave >> 1;
  const int b = blockIdx.y, ci0 = blockIdx.z * NCI;
  const long plane = (long)a.H * a.W;
  const float* Xb = a.X + (long)b * a.cin * plane;
  const float* Db = a.dY + (long)b * a.cout * plane;
  const int row0 = blockIdx.x * CNN_BAND;
  const int nbx = (a.W + WG_X - 1) / WG_X, nblk = (CNN_BAND / WG_R) * nbx;
  f4v acc[9][CIT], accb = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int c = 0; c < CIT; ++c) acc[t][c] = f4v{0.f, 0.f, 0.f, 0.f};
  const bool bias = blockIdx.z == 0 && half == 0;
  bf8 ones;
#pragma unroll
  for (int q = 0; q < 8; ++q) ones[q] = (__bf16)1.f;
  f4u xv[XI];
  float dv[DI][6];
  auto load = [&](int blk) {
    const int y0 = row0 + (blk / nbx) * WG_R, x0 = (blk % nbx) * WG_X;
#pragma unroll
    for (int i = 0; i < XI; ++i) {  // 8 threads per row of 32 pixels (W is a multiple of 8)
      const int e = tid + 256 * i, x = x0 + 4 * (e & 7), r = (e >> 3) % WG_R, c = ci0 + (e >> 3) / WG_R;
      const bool ok = x < a.W && c < a.cin;
      xv[i] = *reinterpret_cast<const f4u*>(Xb + (ok ? (long)c * plane + (long)(y0 + r) * a.W + x : 0));
      if (!ok) xv[i] = f4u{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int i = 0; i < DI; ++i) {  // pixels x - 1 .. x + 4 of rows y0 - 1 .. y0 + WG_R
      const int e = tid + 256 * i, x = x0 + 4 * (e & 7), r = (e >> 3) % (WG_R + 2), co = (e >> 3) / (WG_R + 2);
      const int y = y0 + r - 1;
      const bool oky = y >= 0 && y < a.H && co < a.cout;
      const float* src = Db + (oky ? (long)co * plane + (long)y * a.W : 0);
#pragma unroll
      for (int q = 0; q < 6; ++q) {
        const int xq = x + q - 1;
        const bool ok = oky && xq >= 0 && xq < a.W;
        const float v = src[ok ? xq : 0];
        dv[i][q] = ok ? v : 0.f;
      }
    }
  };
  load(0);
  for (int blk = 0; blk < nblk; ++blk) {
    __syncthreads();  // the previous block's operand reads are done
#pragma unroll
    for (int i = 0; i < XI; ++i) {
      const int e = tid + 256 * i, xg = e & 7, r = (e >> 3) % WG_R, c = (e >> 3) / WG_R;
      bf4 v;
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = (__bf16)xv[i][q];
      *reinterpret_cast<bf4*>(&xs[c * WG_XP + r * WG_X + 4 * xg]) = v;
    }
#pragma unroll
    for (int i = 0; i < DI; ++i) {
      const int e = tid + 256 * i, xg = e & 7, r = (e >> 3) % (WG_R + 2), co = (e >> 3) / (WG_R + 2);
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) {  // copy dx holds dY at x - dx + 1
        bf4 v;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = (__bf16)dv[i][q - dx + 2];
        *reinterpret_cast<bf4*>(&ds[(dx * 32 + co) * WG_DP + r * WG_X + 4 * xg]) = v;
      }
    }
    __syncthreads();
    if (blk + 1 < nblk) load(blk + 1);
    bf8 xb[WG_R][CIT];
#pragma unroll
    for (int r = 0; r < WG_R; ++r)
#pragma unroll
      for (int c = 0; c < CIT; ++c)
        xb[r][c] = *reinterpret_cast<const bf8*>(&xs[(16 * (half * CIT + c) + pl) * WG_XP + r * WG_X + 8 * kq]);
    // staged row ry of dY meets X's row ry + dy - 2 at tap row dy
#pragma unroll
    for (int ry = 0; ry < WG_R + 2; ++ry) {
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) {
        const bf8 av = *reinterpret_cast<const bf8*>(&ds[(dx * 32 + 16 * cot + pl) * WG_DP + ry * WG_X + 8 * kq]);
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) {
          const int r = ry + dy - 2;
          if (r >= 0 && r < WG_R) {
#pragma unroll
            for (int c = 0; c < CIT; ++c) acc[3 * dy + dx][c] = mfma_bf16(av, xb[r][c], acc[3 * dy + dx][c]);
            if (dy == 1 && dx == 1 && bias) accb = mfma_bf16(av, ones, accb);
          }
        }
      }
    }
  }
  float* out = a.part + (long)(blockIdx.y * gridDim.x + blockIdx.x) * a.kp * 32 + 16 * cot + 4 * kq;
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int c = 0; c < CIT; ++c) {
      const int ci = ci0 + 16 * (half * CIT + c) + pl;
      if (ci < a.cin) *reinterpret_cast<f4v*>(out + ((long)t * a.cin + ci) * 32) = acc[t][c];
    }
  if (bias && pl == 0) *reinterpret_cast<f4v*>(out + 9L * a.cin * 32) = accb;
}

// sum the weight-gradient partials into the flat parameter gradient (W then
// b of every layer): one workgroup per row kappa of 32 entries, eight slices
// of the partials, FP64, a fixed order.  Grid (largest kappa count, layers).
// 256 partials of 96 channels: 4 layers in 12 us, against 348 us for one
// thread per entry.
__global__ __launch_bounds__(256) void k_wgrad_reduce(CnnLayers a) {
  __shared__ double red[256];
  const int l = blockIdx.y, kap = blockIdx.x, cin = a.cin[l], cout = a.cout[l], kp = a.kp[l];
  if (kap > 9 * cin) return;
  const int co = threadIdx.x & 31, sl = threadIdx.x >> 5;
  const float* p = a.part[l] + (long)kap * 32 + co;
  double s = 0.0;
#pragma unroll 8
  for (int q = sl; q < a.nparts; q += 8) s += p[(long)q * kp * 32];
  red[threadIdx.x] = s;
  __syncthreads();
  if (sl != 0 || co >= cout) return;
#pragma unroll
  for (int w = 1; w < 8; ++w) s += red[32 * w + co];
  const long o = kap < 9 * cin ? ((long)co * cin + kap % cin) * 9 + kap / cin : (long)cout * cin * 9 + co;
  a.g[l][o] = (float)s;
}

// ---------------------------------------------------------------------------
// loss: Gram of [M U_tgt] per sequence (FP64 partials over pixel chunks),
// the r x r algebra, then the output-channel gradient
// ---------------------------------------------------------------------------
// The Gram on the FP64 matrix cores: the 4r real columns [Re m_0, Im m_0, ..,
// Re u_0, Im u_0, ..] in TR tiles of 16, upper tiles; a lane's column over four
// consecutive pixels is one load and feeds four products.  One wave per
// workgroup slice of the chunk (4), summed in order.  16 sequences of 128 x 128,
// rank 6: 21 us, against 70 us for FP64 multiply-adds by 78 of 256 threads.
template <int TR>
__global__ __launch_bounds__(256) void k_loss_gram(LossArgs a) {
  using M = Mma<double>;
  constexpr int NT = TR * (TR + 1) / 2;
  __shared__ double red[NT * 256];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 15, kk = lane >> 4;
  const int b = blockIdx.y, r = a.r, m = 2 * r;
  const float* Yb = a.Y4 + (long)b * 2 * r * a.n;
  const float* Ub = reinterpret_cast<const float*>(a.Ut + (long)b * r * a.n);
  // column i < 2r: plane i of the output; then component i % 2 of target (i - 2r) / 2
  const float* src[TR];
  int st[TR];
  bool ok[TR];
#pragma unroll
  for (int t = 0; t < TR; ++t) {
    const int i = 16 * t + col;
    ok[t] = i < 4 * r;
    const bool u = i >= 2 * r && ok[t];
    src[t] = u ? Ub + 2L * ((i - 2 * r) >> 1) * a.n + (i & 1) : Yb + (long)(ok[t] ? i : 0) * a.n;
    st[t] = u ? 2 : 1;
  }
  typename M::V acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = M::zero();
  const long p0 = (long)blockIdx.x * a.chunk, p1 = min(a.n, p0 + a.chunk);  // n is a multiple of 64
  for (long pb = p0 + 16 * wave; pb < p1; pb += 64) {
    float v[TR][4];
#pragma unroll
    for (int t = 0; t < TR; ++t) {
      const float* s = src[t] + (pb + 4 * kk) * st[t];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float x = s[e * st[t]];
        v[t][e] = ok[t] ? x : 0.f;
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int ti = 0; ti < TR; ++ti)
#pragma unroll
        for (int tj = ti; tj < TR; ++tj) {
          const int o = ti * TR - ti * (ti - 1) / 2 + (tj - ti);
          acc[o] = M::mma((double)v[ti][e], (double)v[tj][e], acc[o]);
        }
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) tile_reduce_n<double, 4>(red + t * 256, acc[t], wave, lane);
  auto C = [&](int i, int j) -> double {
    if (i > j) {
      const int t = i;
      i = j;
      j = t;
    }
    const int ti = i / 16, tj = j / 16;
    return red[(ti * TR - ti * (ti - 1) / 2 + (tj - ti)) * 256 + (i % 16) * 16 + (j % 16)];
  };
  const int nout = m * (m + 1) / 2;
  for (int o = tid; o < nout; o += 256) {
    int i, j;
    tri_index(o, m, i, j);
    a.part[((long)b * gridDim.x + blockIdx.x) * nout + o] =
        make_double2(C(2 * i, 2 * j) + C(2 * i + 1, 2 * j + 1), C(2 * i, 2 * j + 1) - C(2 * i + 1, 2 * j));
  }
}

// one workgroup per sequence does the r x r work (r <= 16), thread (i, j) on
// entry (i, j), the matrices in LDS: 12 us at rank 6 (265 us by one thread)
__global__ __launch_bounds__(256) void k_loss_small(LossArgs a) {
  __shared__ double2 L[16][17], Li[16][17], Gi[16][17], Cm[16][17], X[16][17];
  __shared__ double2 tri[528];
  __shared__ double s_tr[16];
  const int b = blockIdx.x, tid = threadIdx.x, i = tid >> 4, j = tid & 15;
  const int r = a.r, m = 2 * r, nout = m * (m + 1) / 2;
  const bool in = i < r && j < r;
  for (int o = tid; o < nout; o += 256) {  // the Gram of [M U], chunks in order
    double2 s = make_double2(0.0, 0.0);
#pragma unroll 4
    for (int q = 0; q < a.nchunks; ++q) s = dadd(s, a.part[((long)b * a.nchunks + q) * nout + o]);
    tri[o] = s;
  }
  __syncthreads();
  auto entry = [&](int p, int q) { return tri[p * m - p * (p - 1) / 2 + (q - p)]; };  // p <= q
  if (in) {
    Cm[i][j] = entry(i, r + j);  // M^H U
    if (i == j) s_tr[i] = entry(i, i).x;
  }
  __syncthreads();
  double tr = 0.0;
  for (int k = 0; k < r; ++k) tr += s_tr[k];
  // G_ij (i >= j) = conj(entry(j, i)); a tiny ridge keeps a rank-deficient M finite
  if (in && i >= j) {
    L[i][j] = i == j ? make_double2(entry(i, i).x + 1e-12 * tr / r, 0.0) : dconj(entry(j, i));
  }
  __syncthreads();
  // Cholesky G = L L^H, column by column
  for (int k = 0; k < r; ++k) {
    const double d = sqrt(fmax(L[k][k].x, 1e-300));
    const double2 lik = in && i > k ? L[i][k] : make_double2(0.0, 0.0);
    const double2 ljk = in && j > k ? L[j][k] : make_double2(0.0, 0.0);
    __syncthreads();
    if (in && j == k) {
      if (i == k) L[k][k] = make_double2(d, 0.0);
      else if (i > k) L[i][k] = make_double2(lik.x / d, lik.y / d);
    }
    if (in && j > k && i >= j) {
      const double2 u = make_double2(lik.x / d, lik.y / d), v = make_double2(ljk.x / d, -ljk.y / d);
      L[i][j] = dsub(L[i][j], dmul(u, v));
    }
    __syncthreads();
  }
  // Li = L^-1, one thread per column; Gi = Li^H Li
  if (i == 0 && j < r) {
    for (int p = 0; p < r; ++p) {
      double2 s = make_double2(p == j ? 1.0 : 0.0, 0.0);
      for (int k = j; k < p; ++k) s = dsub(s, dmul(L[p][k], Li[k][j]));
      Li[p][j] = p < j ? make_double2(0.0, 0.0) : make_double2(s.x / L[p][p].x, s.y / L[p][p].x);
    }
  }
  __syncthreads();
  double2 g = make_double2(0.0, 0.0);
  if (in)
    for (int k = max(i, j); k < r; ++k) g = dadd(g, djmul(Li[k][i], Li[k][j]));
  Gi[i][j] = g;
  __syncthreads();
  // P1 = C^H Gi; X = Gi C; P2 = X X^H; loss = r - tr(Gi C C^H) = r - tr(C^H X)
  double2* P1 = a.P + (long)b * 2 * r * r;
  double2* P2 = P1 + r * r;
  double2 x = make_double2(0.0, 0.0), p1 = x;
  if (in) {
    for (int k = 0; k < r; ++k) {
      x = dadd(x, dmul(Gi[i][k], Cm[k][j]));
      p1 = dadd(p1, djmul(Cm[k][i], Gi[k][j]));
    }
    P1[i * r + j] = p1;
  }
  X[i][j] = x;
  __syncthreads();
  if (in) {
    double2 p2 = make_double2(0.0, 0.0);
    for (int k = 0; k < r; ++k) p2 = dadd(p2, dmul(X[i][k], dconj(X[j][k])));
    P2[i * r + j] = p2;
  }
  if (tid == 0) {
    double lt = 0.0;
    for (int p = 0; p < r; ++p)
      for (int k = 0; k < r; ++k) lt += djmul(Cm[p][k], X[p][k]).x;
    a.loss_b[b] = r - lt;
  }
}

// dL/d conj(M) = M P2 - U P1; output-channel gradient (2 Re, 2 Im) * scale.
// RT >= r columns; P1 and P2 in LDS.  The first workgroup also forms the
// mean loss (sequences in order).
template <int RT>
__global__ __launch_bounds__(256) void k_loss_grad(LossArgs a) {
  __shared__ double2 P[2 * 256];
  const int b = blockIdx.y, r = a.r;
  for (int e = threadIdx.x; e < 2 * r * r; e += 256) P[e] = a.P[(long)b * 2 * r * r + e];
  __syncthreads();
  if (blockIdx.x == 0 && b == 0 && threadIdx.x == 0) {
    double s = 0.0;
    for (int k = 0; k < a.batch; ++k) s += a.loss_b[k];
    *a.loss = s / a.batch;
  }
  const long p = (long)blockIdx.x * 256 + threadIdx.x;
  if (p >= a.n) return;
  const float* Yb = a.Y4 + (long)b * 2 * r * a.n;
  const float2* Ub = a.Ut + (long)b * r * a.n;
  const double2* P1 = P;
  const double2* P2 = P + r * r;
  float* dY = a.dY4 + (long)b * 2 * r * a.n;
  float2 Mp[RT], Up[RT];
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    const int ic = min(i, r - 1);
    Mp[i] = make_float2(Yb[(long)(2 * ic) * a.n + p], Yb[(long)(2 * ic + 1) * a.n + p]);
    Up[i] = Ub[(long)ic * a.n + p];
  }
  for (int j = 0; j < r; ++j) {
    double2 s = make_double2(0.0, 0.0);
#pragma unroll
    for (int i = 0; i < RT; ++i)
      if (i < r) s = dadd(s, dsub(dmul(f2d(Mp[i]), P2[i * r + j]), dmul(f2d(Up[i]), P1[i * r + j])));
    dY[(long)(2 * j) * a.n + p] = (float)(2.0 * s.x * a.scale);
    dY[(long)(2 * j + 1) * a.n + p] = (float)(2.0 * s.y * a.scale);
  }
}

// network output -> M, n x r column-major complex per sequence
__global__ void k_cnn_to_M(const float* Y4, int r, long n, int batch, float2* M) {
  const long total = (long)batch * r * n;
  for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (long)gridDim.x * blockDim.x) {
    const long b = e / ((long)r * n), rem = e % ((long)r * n);
    const int j = (int)(rem / n);
    const long p = rem % n;
    const float* Yb = Y4 + b * 2 * r * n;
    M[e] = make_float2(Yb[(long)(2 * j) * n + p], Yb[(long)(2 * j + 1) * n + p]);
  }
}

__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, long n, float lr, float b1, float b2, float c1, float c2, float eps) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
size_t cnn_pack_bytes(int cin) { return (size_t)((cin + CV_CH - 1) / CV_CH) * 9 * 2 * 512 * 2; }

hipError_t launch_cnn_pack(const CnnLayers& a, hipStream_t s) {
  hipLaunchKernelGGL(k_cnn_pack, dim3(32, 8), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_conv(const ConvArgs& a, int batch, hipStream_t s) {
  // tiles of 64 pixels up to four of them a compute unit: a quarter of the
  // work a workgroup and four times the workgroups, where the larger tiles
  // leave the chip idle.  A forward pass in either, us: one sequence of 64 x 64
  // 29 / 55, 128 x 128 35 / 70, 256 x 256 (1,024 tiles) 63 / 78; two of 256 x 256
  // 106 / 92, 16 of 64 x 64 (1,024) 51 / 63, eight of 128 x 128 (2,048) 105 / 98.
  const long small = (long)((a.H + 3) / 4) * ((a.W + 15) / 16);
  if (small * batch <= 1024) {
    hipLaunchKernelGGL((k_conv<16, 4>), dim3((unsigned)small, batch), dim3(256), 0, s, a);
    return hipGetLastError();
  }
  // the tile whose padded image is the smallest; among equals the widest,
  // which writes whole cache lines (128 x 128, 16 sequences, 96 channels in:
  // 64 x 4 54 us, 32 x 8 64 us, 16 x 16 66 us; 32 channels in: 28, 31 and 29 us)
  int best = 16;
  long area = 0;
  for (int tw = 64; tw >= 16; tw /= 2) {
    const int th = 256 / tw;
    const long p = (long)((a.H + th - 1) / th * th) * ((a.W + tw - 1) / tw * tw);
    if (area == 0 || p < area) {
      area = p;
      best = tw;
    }
  }
  const dim3 g(((a.H + 256 / best - 1) / (256 / best)) * ((a.W + best - 1) / best), batch);
  if (best == 64) hipLaunchKernelGGL((k_conv<64, 4>), g, dim3(256), 0, s, a);
  else if (best == 32) hipLaunchKernelGGL((k_conv<32, 8>), g, dim3(256), 0, s, a);
  else hipLaunchKernelGGL((k_conv<16, 16>), g, dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_wgrad(const WgradArgs& a, int batch, hipStream_t s) {
  const int cit = std::min(3, (a.cin + 31) / 32);  // 32 cit input channels per workgroup
  const dim3 g(a.H / CNN_BAND, batch, (a.cin + 32 * cit - 1) / (32 * cit));
  if (cit == 1) hipLaunchKernelGGL(k_conv_wgrad<1>, g, dim3(256), 0, s, a);
  else if (cit == 2) hipLaunchKernelGGL(k_conv_wgrad<2>, g, dim3(256), 0, s, a);
  else hipLaunchKernelGGL(k_conv_wgrad<3>, g, dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_wgrad_reduce(const CnnLayers& a, hipStream_t s) {
  int rows = 0;
  for (int l = 0; l < 4; ++l) rows = std::max(rows, 9 * a.cin[l] + 1);
  hipLaunchKernelGGL(k_wgrad_reduce, dim3(rows, 4), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_loss(const LossArgs& a, hipStream_t s) {
  const dim3 gg(a.nchunks, a.batch), gp((unsigned)((a.n + 255) / 256), a.batch), b(256);
  switch ((4 * a.r + 15) / 16) {  // tiles of the 4r real columns
    case 1: hipLaunchKernelGGL(k_loss_gram<1>, gg, b, 0, s, a); break;
    case 2: hipLaunchKernelGGL(k_loss_gram<2>, gg, b, 0, s, a); break;
    case 3: hipLaunchKernelGGL(k_loss_gram<3>, gg, b, 0, s, a); break;
    default: hipLaunchKernelGGL(k_loss_gram<4>, gg, b, 0, s, a); break;
  }
  hipLaunchKernelGGL(k_loss_small, dim3(a.batch), b, 0, s, a);
  if (a.r <= 4) hipLaunchKernelGGL(k_loss_grad<4>, gp, b, 0, s, a);
  else if (a.r <= 8) hipLaunchKernelGGL(k_loss_grad<8>, gp, b, 0, s, a);
  else hipLaunchKernelGGL(k_loss_grad<16>, gp, b, 0, s, a);
  return hipGetLastError();
}

hipError_t launch_cnn_to_M(const float* Y4, int r, long n, int batch, float2* M, hipStream_t s) {
  hipLaunchKernelGGL(k_cnn_to_M, dim3(1024), dim3(256), 0, s, Y4, r, n, batch, M);
  return hipGetLastError();
}

hipError_t launch_adam(float* p, const float* g, float* m, float* v, long n, float lr, int step, hipStream_t s) {
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = (float)(1.0 - pow(0.9, step)), c2 = (float)(1.0 - pow(0.999, step));
  hipLaunchKernelGGL(k_adam, dim3(256), dim3(256), 0, s, p, g, m, v, n, lr, b1, b2, c1, c2, 1e-8f);
  return hipGetLastError();
}

// L1: 2q planes (Re, Im of column k of X = A^H(y)) divided by their RMS.
// Pass 1: FP64 partial sums of squares per workgroup; pass 2: every
// workgroup re-sums the partials and writes its share.
__global__ __launch_bounds__(256) void k_planes_sumsq(const float2* X, long total, double* partial) {
  __shared__ double red[256];
  double s = 0.0;
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < total; e += (long)gridDim.x * 256) {
    const float2 v = X[e];
    s += (double)v.x * v.x + (double)v.y * v.y;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(256) void k_planes_write(const float2* X, long n, int q, const double* partial,
                                                      int nparts, float* out) {
  __shared__ float s_inv;
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int i = 0; i < nparts; ++i) s += partial[i];
    const double rms = sqrt(s / (2.0 * q * n));
    s_inv = rms > 0.0 ? (float)(1.0 / rms) : 1.f;
  }
  __syncthreads();
  const float inv = s_inv;
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < (long)q * n; e += (long)gridDim.x * 256) {
    const long k = e / n, p = e % n;
    const float2 v = X[e];
    out[(2 * k) * n + p] = v.x * inv;
    out[(2 * k + 1) * n + p] = v.y * inv;
  }
}

hipError_t launch_cnn_planes(const float2* X, long n, int q, double* partial, float* out, hipStream_t s) {
  hipLaunchKernelGGL(k_planes_sumsq, dim3(256), dim3(256), 0, s, X, n * q, partial);
  hipLaunchKernelGGL(k_planes_write, dim3(256), dim3(256), 0, s, X, n, q, partial, 256, out);
  return hipGetLastError();
}

}  // namespace ag
