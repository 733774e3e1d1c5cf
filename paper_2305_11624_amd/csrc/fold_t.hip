// Fold and fold-back of the TransposedConv-BN block (Sec. 3.2.1: the associative law behind Tune mode
// holds for transposed convolution as well; Sec. 3.3 and Table 2 "Tune" with the per-channel scale on
// the weight's OUTPUT-channel index, which is the innermost one of the transposed block's weight):
//   W      [Ci][taps][Co]     (the channels-last order of the logical [Ci, Co, kH, kW])
//   fold   w_same[ci][tap][co] = s[co] W[ci][tap][co]      read by the backward's input-gradient pass
//          w_swap[co][tap][ci] = s[co] W[ci][tap][co]      read by the forward pass (or [tap][co][ci] where the
//                                                          forward pass is a single product, see conv_pw.hip)
//          b'[co] = (b[co] - mu[co]) s[co] + beta[co]
//   back   dW[ci][tap][co] = s[co] dw'[ci][tap][co],  dgamma[co] = (sum_{ci,tap} dw' W + r (b - mu)) / sqrt(var + eps),
//          dbeta = r, db = s r
// Both are memory-bound passes over the weight; threads run along co, so every access is contiguous.
#include "fold_back_t_tile.h"

namespace convbn {

namespace {

constexpr int TT = 32;   // tile edge of the ci <-> co transpose

// grid (ceil(Co/TT), ceil(Ci/TT), taps)
template <typename T>
__global__ __launch_bounds__(256) void fold_t_kernel(const T* __restrict__ W, const float* __restrict__ b,
                                                     const float* __restrict__ gamma, const float* __restrict__ beta,
                                                     const float* __restrict__ mean, const float* __restrict__ var,
                                                     float eps, int Ci, int Co, int taps, int tap_major,
                                                     T* __restrict__ w_same, T* __restrict__ w_swap,
                                                     float* __restrict__ bfold) {
  __shared__ float tile[TT][TT + 1];
  const int tx = threadIdx.x % TT, ty = threadIdx.x / TT;   // ty in [0, 8)
  const int co0 = blockIdx.x * TT, ci0 = blockIdx.y * TT, tap = blockIdx.z;
  const int co = co0 + tx;
  // all four rows are asked for at once, out of range the last one inside (reads behind a condition wait for each other:
  // 512 -> 256 channels, 4 x 4, 6.7 -> 5.8 us; 256 -> 128, 2 x 2, a forward pass 10.6 -> 8.5)
  const int cc = co < Co ? co : 0;
  T wv[TT / 8];
  size_t idx[TT / 8];
  bool ok[TT / 8];
#pragma unroll
  for (int e = 0; e < TT / 8; ++e) {
    const int ci = ci0 + ty + 8 * e;
    ok[e] = ci < Ci && co < Co;
    idx[e] = ((size_t)min(ci, Ci - 1) * taps + tap) * Co + cc;
    wv[e] = W[idx[e]];
  }
  // gamma == nullptr (the Eval comparison path): s = 1 and b' = b, i.e. a pure reordering of the weight
  const float s = gamma ? gamma[cc] / sqrtf(var[cc] + eps) : 1.f;
#pragma unroll
  for (int e = 0; e < TT / 8; ++e) {
    // the scaled weight is rounded once, to the storage type, exactly as it is stored
    const T r = from_f32<T>(to_f32(wv[e]) * s);
    if (ok[e] && w_same) w_same[idx[e]] = r;
    tile[ty + 8 * e][tx] = to_f32(r);
  }
  if (bfold && blockIdx.y == 0 && (tap == 0 || tap_major) && ty == 0 && co < Co)
    bfold[(tap_major ? tap * Co : 0) + co] = gamma ? ((b ? b[co] : 0.f) - mean[co]) * s + beta[co] : (b ? b[co] : 0.f);
  if (!w_swap) return;
  __syncthreads();
#pragma unroll
  for (int e = 0; e < TT / 8; ++e) {
    const int oc = co0 + ty + 8 * e, ic = ci0 + tx;
    if (oc < Co && ic < Ci)
      w_swap[(tap_major ? (size_t)tap * Co + oc : (size_t)oc * taps + tap) * Ci + ic] = from_f32<T>(tile[tx][ty + 8 * e]);
  }
}

// How the fold-back is split.  W is rows = Ci*taps of Co columns, P = rows*Co; a workgroup leaves one row of dot_part.
//  * Co % 4 != 0: 8 rows of 64 columns, an element per thread.
//  * few partial copies (under 8, under 16 of a large weight: 256 -> 128 channels, 4 x 4, 8 copies, a backward pass 80.5 us
//    this way and 83.5 the other): 256 columns, four per lane, and 8 rows, or 32 (fewer rows for the finish to read) where
//    that still makes 256 workgroups.  512 -> 256 channels, 4 x 4 (8192 rows, 2 copies): a backward pass 85.0 us with 8 rows, 81.9
//    with 32; 2 x 2 (2048 rows): 27.9 with 8, 34.4 with 32.
//  * else the copies are the work: el columns of four, and the 256 / el threads of each share the copies.  el = 16, or 64 where
//    P is large enough to keep every compute unit busy.  128 -> 64 channels, 2 x 2 (512 rows, 100 copies): 5.4 us (a
//    lane reading all the copies of its columns 14.2); 64 -> 32 channels, 4 x 4 (1024 rows, 62 copies): 7.9 (10.8).
struct BackPlan { int el, rows, cols, ncol, chunks; };   // el: 0 = the first two ways
BackPlan back_plan(int rows, int Co, int nsplit) {
  BackPlan p{0, 8, 256, 0, 0};
  if (Co % 4 != 0) {
    p.cols = 64;
  } else if (nsplit >= ((size_t)rows * Co >= (size_t)131072 ? 16 : 8)) {
    p.el = (size_t)rows * Co >= (size_t)131072 ? 64 : 16;
    const int cw = Co / 4 < p.el ? Co / 4 : p.el;
    p.rows = p.el / cw;
    p.cols = 4 * cw;
  } else if (ceil_div(rows, 32) * ceil_div(Co, 256) >= 256) {
    p.rows = 32;
  }
  p.ncol = ceil_div(Co, p.cols);
  p.chunks = ceil_div(rows, p.rows);
  return p;
}

template <typename T>
__global__ __launch_bounds__(256) void fold_back_t_kernel(FoldBackTArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[FBT_SMEM];
  const int block = blockIdx.x;
  if (block < a.rs.blocks) fbt_colsum(a.rs, a.Co, block, threadIdx.x, smem);
  else fbt_block<T, 4>(a, block - a.rs.blocks, threadIdx.x, true, smem);
}

// Any Co.  grid (ceil(Co/64), ceil(rows/8)).  Thread -> column tid%64, row lane tid/64.
template <typename T>
__global__ __launch_bounds__(256) void fold_back_t_scalar_kernel(const float* __restrict__ part, int nsplit,
                                                                 const T* __restrict__ W,
                                                                 const float* __restrict__ gamma,
                                                                 const float* __restrict__ var, float eps, int rows,
                                                                 int Co, T* __restrict__ dW,
                                                                 float* __restrict__ dot_part) {
  __shared__ float red[4][64];
  const int c = threadIdx.x & 63, rl = threadIdx.x >> 6;
  const int co = blockIdx.x * 64 + c;
  const int r0 = blockIdx.y * 8, r1 = min(rows, r0 + 8);
  const size_t P = (size_t)rows * Co;
  float dot = 0.f;
  if (co < Co) {
    const float s = gamma ? gamma[co] / sqrtf(var[co] + eps) : 1.f;
    for (int r = r0 + rl; r < r1; r += 4) {
      const size_t idx = (size_t)r * Co + co;
      float dw = 0.f;
      for (int sp = 0; sp < nsplit; ++sp) dw += part[sp * P + idx];
      dW[idx] = from_f32<T>(s * dw);
      dot += dw * to_f32(W[idx]);
    }
  }
  if (!dot_part) return;
  red[rl][c] = dot;
  __syncthreads();
  if (rl == 0 && co < Co) dot_part[(size_t)blockIdx.y * Co + co] = red[0][c] + red[1][c] + red[2][c] + red[3][c];
}

// grid Co/V, V = 4 columns where Co % 4 == 0, else one; a thread takes every 256th partial row, four of them and its one
// of r's (there are at most 256) in flight: the rows lie Co floats apart, and each load is a round trip to memory.  512 -> 256 channels, 4 x 4 (256
// partial rows): 4.9 us, of which a launch is about 2.5 (16 columns a workgroup and 64 of 1024 rows a thread: 7.7).
template <int V>
__global__ __launch_bounds__(256) void fold_back_t_finish_kernel(const float* __restrict__ dot_part, int nchunks,
                                                                 const float* __restrict__ r_part, int nrpart,
                                                                 const float* __restrict__ b,
                                                                 const float* __restrict__ gamma,
                                                                 const float* __restrict__ mean,
                                                                 const float* __restrict__ var, float eps, int Co,
                                                                 float* __restrict__ db, float* __restrict__ dgamma,
                                                                 float* __restrict__ dbeta) {
  struct __attribute__((aligned(4 * V))) Vec { float v[V]; };
  __shared__ float red[4][2 * V];
  const int tid = threadIdx.x, co = blockIdx.x * V;
  const int c = co + (tid < V ? tid : 0);   // the column this thread finishes
  const float fv = var[c], fm = mean[c], fb = b ? b[c] : 0.f, fg = gamma[c];
  const Vec r0 = *reinterpret_cast<const Vec*>(r_part + (size_t)min(tid, nrpart - 1) * Co + co);   // (nrpart <= 256)
  float sum[2 * V] = {};   // dot and r
  for (int k = tid; k < nchunks; k += 4 * 256) {
    Vec a[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) a[j] = *reinterpret_cast<const Vec*>(dot_part + (size_t)min(k + 256 * j, nchunks - 1) * Co + co);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < V; ++e) sum[e] += k + 256 * j < nchunks ? a[j].v[e] : 0.f;
  }
#pragma unroll
  for (int e = 0; e < V; ++e) sum[V + e] = tid < nrpart ? r0.v[e] : 0.f;
#pragma unroll
  for (int e = 0; e < 2 * V; ++e) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum[e] += __shfl_xor(sum[e], o);
    if ((tid & 63) == 0) red[tid >> 6][e] = sum[e];
  }
  __syncthreads();
  if (tid >= V) return;
  const float dot = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
  const float r = (red[0][V + tid] + red[1][V + tid]) + (red[2][V + tid] + red[3][V + tid]);
  const float sd = sqrtf(fv + eps);
  dgamma[c] = (dot + r * (fb - fm)) / sd;
  dbeta[c] = r;
  if (db) db[c] = fg / sd * r;
}

}  // namespace

hipError_t launch_fold_t(int dtype, int Ci, int Co, int taps, const void* W, const float* b, const float* gamma,
                         const float* beta, const float* mean, const float* var, float eps, int tap_major,
                         void* w_same, void* w_swap, float* bfold, hipStream_t st) {
  const dim3 grid(ceil_div(Co, TT), ceil_div(Ci, TT), taps);
  if (dtype == CONVBN_BF16)
    hipLaunchKernelGGL(fold_t_kernel<bf16_t>, grid, dim3(256), 0, st, (const bf16_t*)W, b, gamma, beta, mean, var, eps,
                       Ci, Co, taps, tap_major, (bf16_t*)w_same, (bf16_t*)w_swap, bfold);
  else
    hipLaunchKernelGGL(fold_t_kernel<float>, grid, dim3(256), 0, st, (const float*)W, b, gamma, beta, mean, var, eps,
                       Ci, Co, taps, tap_major, (float*)w_same, (float*)w_swap, bfold);
  return hipGetLastError();
}

int fold_back_t_chunks(int Ci, int Co, int taps, int nsplit) { return back_plan(Ci * taps, Co, nsplit).chunks; }

namespace {
bool sums_aside(int dtype, int Co) { return dtype == CONVBN_BF16 && Co % 8 == 0 && Co <= 2048; }
FoldBackTArgs back_args(int dtype, int Ci, int Co, int taps, const float* dwf_part, int nsplit, const Geom& zrows, const void* dz,
                        float* r_part, const void* W, const float* gamma, const float* var, float eps, float* dot_part, void* dW) {
  const int rows = Ci * taps;
  const BackPlan bp = back_plan(rows, Co, nsplit);
  const int nrpart = colsum_parts(zrows);
  FoldBackTArgs a{};
  if (gamma && sums_aside(dtype, Co)) a.rs = {static_cast<const uint4*>(dz), r_part, zrows.M, ceil_div(zrows.M, nrpart), nrpart};
  a.part = dwf_part; a.W = W; a.gamma = gamma; a.var = var; a.dW = dW; a.dot_part = dot_part; a.eps = eps;
  a.nsplit = nsplit; a.rows = rows; a.Co = Co; a.ncol = bp.ncol; a.cw = bp.cols / 4;
  a.kind = bp.el == 64 ? FBT_SPLIT_64 : bp.el == 16 ? FBT_SPLIT_16 : bp.rows == 32 ? FBT_ROWS_8 : FBT_ROWS_2;
  a.blocks = bp.ncol * bp.chunks;
  return a;
}
}  // namespace

bool fold_back_t_side(int dtype, int Ci, int Co, int taps, const float* dwf_part, int nsplit, const Geom& zrows, const void* dz,
                      float* r_part, const void* W, const float* gamma, const float* var, float eps, float* dot_part, void* dW,
                      FoldBackTArgs* a) {
  if (!sums_aside(dtype, Co)) return false;
  *a = back_args(dtype, Ci, Co, taps, dwf_part, nsplit, zrows, dz, r_part, W, gamma, var, eps, dot_part, dW);
  return true;
}
hipError_t launch_fold_back_t_finish(int Ci, int Co, int taps, int nsplit, const Geom& zrows, const float* r_part, const float* b,
                                     const float* gamma, const float* mean, const float* var, float eps, const float* dot_part,
                                     float* db, float* dgamma, float* dbeta, hipStream_t st) {
  const int chunks = fold_back_t_chunks(Ci, Co, taps, nsplit), nrpart = colsum_parts(zrows);
#define FINISH(V)                                                                                                      \
  hipLaunchKernelGGL(fold_back_t_finish_kernel<V>, dim3(Co / V), dim3(256), 0, st, dot_part, chunks, r_part, nrpart, b, \
                     gamma, mean, var, eps, Co, db, dgamma, dbeta)
  if (Co % 4 == 0) FINISH(4); else FINISH(1);
#undef FINISH
  return hipGetLastError();
}

hipError_t launch_fold_back_t(int dtype, int Ci, int Co, int taps, const float* dwf_part, int nsplit,
                              const Geom& zrows, const void* dz, float* r_part, const void* W, const float* b,
                              const float* gamma, const float* mean, const float* var, float eps, float* dot_part, void* dW,
                              float* db, float* dgamma, float* dbeta, hipStream_t st) {
  const FoldBackTArgs a = back_args(dtype, Ci, Co, taps, dwf_part, nsplit, zrows, dz, r_part, W, gamma, var, eps, dot_part, dW);
  if (gamma && a.rs.blocks == 0)
    if (hipError_t e = launch_colsum(zrows, dtype, dz, r_part, st); e != hipSuccess) return e;
  const dim3 grid(a.rs.blocks + a.blocks), scalar(a.ncol, a.blocks / a.ncol);
  if (dtype == CONVBN_BF16) {
    if (Co % 4 == 0) hipLaunchKernelGGL(fold_back_t_kernel<bf16_t>, grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL(fold_back_t_scalar_kernel<bf16_t>, scalar, dim3(256), 0, st, dwf_part, nsplit, (const bf16_t*)W, gamma,
                            var, eps, a.rows, Co, (bf16_t*)dW, dot_part);
  } else {
    if (Co % 4 == 0) hipLaunchKernelGGL(fold_back_t_kernel<float>, grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL(fold_back_t_scalar_kernel<float>, scalar, dim3(256), 0, st, dwf_part, nsplit, (const float*)W, gamma,
                            var, eps, a.rows, Co, (float*)dW, dot_part);
  }
  if (hipError_t e = hipGetLastError(); e != hipSuccess || !gamma) return e;   // no gamma: dW = sum of the partial copies, nothing else
  return launch_fold_back_t_finish(Ci, Co, taps, nsplit, zrows, r_part, b, gamma, mean, var, eps, dot_part, db, dgamma, dbeta, st);
}

}  // namespace convbn
