// Kernel argument blocks and launch helpers shared by the host code and the
// kernel translation units.
#pragma once

#include "common.hpp"

namespace ag {

// The column and row passes of the measurement operators: CT image columns
// (or CT contiguous rows) per workgroup of NT threads, such that every thread
// has a whole radix group in both passes of the transform and the LDS tile
// stays at 32 KB or less (512: three passes).
template <int N> struct OpTile;
template <> struct OpTile<8>   { static constexpr int CT = 64, NT = 64;  };
template <> struct OpTile<16>  { static constexpr int CT = 16, NT = 64;  };
template <> struct OpTile<32>  { static constexpr int CT = 32, NT = 128; };
template <> struct OpTile<64>  { static constexpr int CT = 16, NT = 128; };
template <> struct OpTile<128> { static constexpr int CT = 16, NT = 128; };
template <> struct OpTile<256> { static constexpr int CT = 16, NT = 256; };
template <> struct OpTile<512> { static constexpr int CT = 8,  NT = 256; };
int op_tile(int N);  // OpTile<N>::CT

// conjugate gradients, one system per image (the mean image: one; MEC-1: one
// per frame): the scalars after an iteration's stop test
struct FrameCg {
  double gamma, gamma0;  // ||s||^2 now and at the start
  int32_t iters, done;
  int32_t brk, pad;      // set by the step: ||A p|| = 0
};

// one CG iteration's scalars: iteration it reads slot (it - 1) & 1 and writes slot it & 1
struct CgArgs {
  const FrameCg* in;
  FrameCg* out;
  const double* nrm;  // [image][nnrm]: shares of ||s||^2
  int nnrm, it;
  double tol;
};

// ISTA (MEC-2)
struct IstaState {
  double omega, last_change;
  int32_t iters, done;
};

struct RowArgs {
  const float2* src;
  float2* dst;
  const float2* tw;
  long nrows;
  const int32_t* m_k;  // null: every row valid
  int nc, lmax;        // measurement-line layout when m_k != null
  float scale;
  int trunc;           // zero samples with |v|^2 > gamma before the transform
  const DevState* st;
  int32_t* trunc_count;  // non-null with trunc: receives the number of samples zeroed
  const float2* sub;   // non-null: store sub - result on the valid rows
};

__device__ __forceinline__ bool row_valid(const RowArgs& a, long rho, int N) {
  if (!a.m_k) return true;
  const long per_k = (long)a.nc * a.lmax;
  const int k = (int)(rho / per_k);
  const int l = (int)(rho % a.lmax);
  return l < a.m_k[k] / N;
}

// image columns -> k-space rows
struct ColFwdArgs {
  const float2* src;       // images, n apart (null: zero)
  const float2* add;       // non-null: one image added to every src image
  const float2* coils;
  long n;
  int nx, nc;
  int cgs;                 // coils per workgroup
  const float2* tw;
  float2* dst;
  long dst_c_stride, dst_img_stride;
  const int32_t* rows;     // ky of each output row of an image (null: all rows)
  long rows_img_stride;
  const int32_t* m_k;      // with rows: n_rows = m_k[img]/nx
  int pad_rows;            // with rows: zeros written for rows n_rows..pad_rows-1
  float scale;
  int img0;                // first image (src, rows, CG systems); dst starts at it
  // CG: src is s, p = s + beta p_old is transformed and stored
  const float2* p_old;
  float2* p_new;
  double* dot;             // with rows: [image][parts] shares of ||A p||^2
  CgArgs cg;
  const IstaState* ista;   // non-null: nothing to do once its done is set
  const DevState* st;
};

// k-space rows -> image columns, with the coil combine
struct ColAdjArgs {
  const float2* src;
  long src_c_stride, src_img_stride;
  const int32_t* rows;     // as in ColFwdArgs
  long rows_img_stride;
  const int32_t* m_k;
  const float2* coils;
  long n;
  int nx, nc;
  const float2* tw;
  float2* dst;
  long dst_img_stride;
  int cgs;                    // coils per workgroup (0: all); group g writes dst + g*dst_part_stride
  long dst_part_stride;
  const int32_t* m_k_scale;   // non-null: scale by 1/sqrt(m_k[img] * mbar)
  float scale;
  int img0;
  // CGLS: x = 0 (first) or x += alpha p; with rows also r -= alpha q before the transform
  int first;
  float2 *x, *r;              // r: src, updated in place
  const float2 *p, *q;
  FrameCg* cg;                // this iteration's slot
  const double* dot;
  int ndot;
  double* nrm;                // one coil group: [image][tiles] shares of ||s||^2, s = the result
  const IstaState* ista;
  const DevState* st;
};

// general masks: a row pass between the k-space rows T[image][c][ky][x] and
// the measurements y[k][c][m_max]; imap[k][location] is the sample's position
// in its frame, -1 where the frame does not sample
struct IndexRowArgs {
  float2* T;
  const int32_t* imap;
  long n;
  int nc, ny, m_max, img0;
  const int32_t* m_k;
  const float2* tw;
  float scale;
  float2* y;               // forward: out
  const float2* yin;       // adjoint: in; forward: stored as yin - result when non-null
  int trunc;
  int32_t* trunc_count;
  // CGLS: forward adds its shares of ||q||^2; adjoint takes r - alpha q (stored)
  double* dot;
  FrameCg* cg;
  float2* r;
  const float2* q;
  int ndot;
  const IstaState* ista;
  const DevState* st;
};

hipError_t launch_rows(int N, const RowArgs& a, bool inv, hipStream_t st);
hipError_t launch_cols_fwd(int N, const ColFwdArgs& a, bool cg, int images, hipStream_t st);
hipError_t launch_cols_adj(int N, const ColAdjArgs& a, bool cgls, int images, hipStream_t st);
enum { IDX_FWD = 0, IDX_ADJ = 1, IDX_RES = 2 };  // T -> y; y -> T; T -> F^H(y - F T) in T
hipError_t launch_index_rows(int N, const IndexRowArgs& a, int mode, bool cgls, int images, hipStream_t st);

}  // namespace ag
