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
#include "fold_tile.h"

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

__device__ __forceinline__ void load4(const float* p, float (&v)[4]) {
  const float4 t = *reinterpret_cast<const float4*>(p);
  v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
}
__device__ __forceinline__ void load4(const bf16_t* p, float (&v)[4]) {
  const uint2 t = *reinterpret_cast<const uint2*>(p);
  v[0] = bf16_lo(t.x); v[1] = bf16_hi(t.x); v[2] = bf16_lo(t.y); v[3] = bf16_hi(t.y);
}
__device__ __forceinline__ void store4(float* p, const float (&v)[4]) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ void store4(bf16_t* p, const float (&v)[4]) {
  *reinterpret_cast<uint2*>(p) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
}

// The first rs.blocks workgroups of a fold-back (bf16 with Co % 8 == 0, Co <= 2048; else none, and a launch before this one)
// sum dZ's columns: that reads dZ while the others read the copies, and needs nothing of theirs.  512 -> 256 channels, 4 x 4,
// 14 x 14, 32 images: 7.8 us, 38 MB (the sums in a launch of their own: 6.3 + 7.3).
struct RSum { const uint4* dz; float* part; int M, rows, blocks; };
__device__ __forceinline__ bool colsum_block(const RSum& rs, int Co, float (*red)[9]) {
  const int block = blockIdx.x;
  if (block >= rs.blocks) return false;
  const int m0 = block * rs.rows;
  colsum_slice_bf16x8(rs.dz, m0, min(rs.M, m0 + rs.rows), Co, threadIdx.x, red, rs.part + (size_t)block * Co);
  return true;
}

// A wave owns RW rows of its workgroup's 4 RW, all asked for at once, and a lane four consecutive columns.
template <typename T, int RW>
__global__ __launch_bounds__(256) void fold_back_t_kernel(RSum rs, const float* __restrict__ part, int nsplit,
                                                          const T* __restrict__ W, const float* __restrict__ gamma,
                                                          const float* __restrict__ var, float eps, int rows, int Co, int ncol,
                                                          T* __restrict__ dW, float* __restrict__ dot_part) {
  __shared__ float red[256][9];
  if (colsum_block(rs, Co, red)) return;
  const int block = blockIdx.x - rs.blocks;
  const int bx = block % ncol, by = block / ncol;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = bx * 256 + lane * 4;
  const int r0 = by * 4 * RW + wave;   // and every fourth row behind it
  const size_t P = (size_t)rows * Co;
  float dot[4] = {0.f, 0.f, 0.f, 0.f};
  if (col < Co && r0 < rows) {
    size_t at[RW];
    bool in[RW];
    float w[RW][4], dw[RW][4] = {};
    float s[4] = {1.f, 1.f, 1.f, 1.f}, v[4] = {1.f, 1.f, 1.f, 1.f};   // no gamma: plain sum
    if (gamma) { load4(gamma + col, s); load4(var + col, v); }
#pragma unroll
    for (int i = 0; i < RW; ++i) {
      in[i] = r0 + 4 * i < rows;
      at[i] = (size_t)(in[i] ? r0 + 4 * i : r0) * Co + col;
      load4(W + at[i], w[i]);
    }
#pragma unroll 4
    for (int sp = 0; sp < nsplit; ++sp)
#pragma unroll
      for (int i = 0; i < RW; ++i) {
        const float4 t = *reinterpret_cast<const float4*>(part + sp * P + at[i]);
        dw[i][0] += t.x; dw[i][1] += t.y; dw[i][2] += t.z; dw[i][3] += t.w;
      }
    if (gamma)
#pragma unroll
      for (int e = 0; e < 4; ++e) s[e] /= sqrtf(v[e] + eps);
#pragma unroll
    for (int i = 0; i < RW; ++i) {
      if (!in[i]) continue;
      float o[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) { o[e] = s[e] * dw[i][e]; dot[e] += dw[i][e] * w[i][e]; }
      store4(dW + at[i], o);
    }
  }
  if (!dot_part) return;
  float* const sum = &red[0][0];   // [wave][256]
#pragma unroll
  for (int e = 0; e < 4; ++e) sum[wave * 256 + lane * 4 + e] = dot[e];
  __syncthreads();
  const int c = threadIdx.x, co = bx * 256 + c;
  if (co < Co) dot_part[(size_t)by * Co + co] = sum[c] + sum[256 + c] + sum[512 + c] + sum[768 + c];
}

// Thread -> column group el (of EL / cw rows, cw columns of four each) and every (256 / EL)-th partial copy.
template <typename T, int EL>
__global__ __launch_bounds__(256) void fold_back_t_split_kernel(RSum rs, const float* __restrict__ part, int nsplit,
                                                                const T* __restrict__ W, const float* __restrict__ gamma,
                                                                const float* __restrict__ var, float eps, int rows, int Co,
                                                                int ncol, int cw, T* __restrict__ dW,
                                                                float* __restrict__ dot_part) {
  constexpr int SL = 256 / EL;
  __shared__ union { float r[256][9]; struct { float copy[SL][EL * 4], dot[EL * 4]; } s; } red;
  if (colsum_block(rs, Co, red.r)) return;
  const int block = blockIdx.x - rs.blocks, bx = block % ncol, by = block / ncol;
  const int nr = EL / cw;
  const size_t P = (size_t)rows * Co;
  // element `el` of the workgroup: its offset in a copy (one inside where there is none) and whether there is one
  auto element = [&](int el, size_t& at) {
    const int rr = el / cw, row = by * nr + rr, c = (bx * cw + el - rr * cw) * 4;
    const bool in = rr < nr && row < rows && c < Co;
    at = in ? (size_t)row * Co + c : 0;
    return in;
  };
  const int tid = threadIdx.x;
  // the element this thread finishes: column e of group fe
  const int fe = tid >> 2, fc = (bx * cw + fe % cw) * 4 + (tid & 3);
  size_t fat = 0;
  const bool fin = tid < EL * 4 && element(fe, fat);
  fat += tid & 3;
  const float fw = fin ? to_f32(W[fat]) : 0.f;
  const float fg = fin && gamma ? gamma[fc] : 1.f, fv = fin && gamma ? var[fc] : 1.f;
  {
    const int el = tid % EL, sl = tid / EL;
    size_t at;
    const bool in = element(el, at);
    float dw[4] = {0.f, 0.f, 0.f, 0.f};
    for (int sp = sl; sp < nsplit; sp += 4 * SL) {
      float4 t[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) t[j] = *reinterpret_cast<const float4*>(part + (size_t)min(sp + j * SL, nsplit - 1) * P + at);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (sp + j * SL >= nsplit) t[j] = make_float4(0.f, 0.f, 0.f, 0.f);
        dw[0] += t[j].x; dw[1] += t[j].y; dw[2] += t[j].z; dw[3] += t[j].w;
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) red.s.copy[sl][el * 4 + e] = in ? dw[e] : 0.f;
  }
  __syncthreads();
  if (tid < EL * 4) {
    float dw = 0.f;
#pragma unroll
    for (int l = 0; l < SL; ++l) dw += red.s.copy[l][tid];
    if (fin) dW[fat] = from_f32<T>(gamma ? fg / sqrtf(fv + eps) * dw : dw);
    red.s.dot[tid] = fin ? dw * fw : 0.f;
  }
  if (!dot_part) return;
  __syncthreads();
  if (!fin || fe >= cw) return;
  float dot = 0.f;
  for (int rr = 0; rr < nr; ++rr) dot += red.s.dot[rr * cw * 4 + tid];
  dot_part[(size_t)by * Co + fc] = dot;
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

hipError_t launch_fold_back_t(int dtype, int Ci, int Co, int taps, const float* dwf_part, int nsplit,
                              const Geom& zrows, const void* dz, float* r_part, const void* W, const float* b,
                              const float* gamma, const float* mean, const float* var, float eps, float* dot_part, void* dW,
                              float* db, float* dgamma, float* dbeta, hipStream_t st) {
  const int rows = Ci * taps;
  const BackPlan bp = back_plan(rows, Co, nsplit);
  const int chunks = bp.chunks, ncol = bp.ncol;
  const int nrpart = gamma ? colsum_parts(zrows) : 0;
  RSum rs{};
  if (gamma && dtype == CONVBN_BF16 && Co % 8 == 0 && Co <= 2048)
    rs = {static_cast<const uint4*>(dz), r_part, zrows.M, ceil_div(zrows.M, nrpart), nrpart};
  else if (gamma)
    if (hipError_t e = launch_colsum(zrows, dtype, dz, r_part, st); e != hipSuccess) return e;
  const bool vec = Co % 4 == 0;
  const dim3 grid(rs.blocks + (unsigned)ncol * chunks);
#define FBT_ROWS(T, RW)                                                                                                  \
  hipLaunchKernelGGL((fold_back_t_kernel<T, RW>), grid, dim3(256), 0, st, rs, dwf_part, nsplit, (const T*)W, gamma, var, \
                     eps, rows, Co, ncol, (T*)dW, dot_part)
#define FBT_SPLIT(T, EL)                                                                                               \
  hipLaunchKernelGGL((fold_back_t_split_kernel<T, EL>), grid, dim3(256), 0, st, rs, dwf_part, nsplit, (const T*)W, gamma, \
                     var, eps, rows, Co, ncol, bp.cols / 4, (T*)dW, dot_part)
#define FBT(T)                                                                                                         \
  do {                                                                                                                 \
    if (!vec) hipLaunchKernelGGL(fold_back_t_scalar_kernel<T>, dim3(ncol, chunks), dim3(256), 0, st, dwf_part, nsplit, \
                                 (const T*)W, gamma, var, eps, rows, Co, (T*)dW, dot_part);                           \
    else if (bp.el == 64) FBT_SPLIT(T, 64);                                                                            \
    else if (bp.el == 16) FBT_SPLIT(T, 16);                                                                            \
    else if (bp.rows == 32) FBT_ROWS(T, 8);                                                                            \
    else FBT_ROWS(T, 2);                                                                                               \
  } while (0)
  if (dtype == CONVBN_BF16) FBT(bf16_t);
  else FBT(float);
#undef FBT
#undef FBT_SPLIT
#undef FBT_ROWS
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !gamma) return e;   // no gamma: dW = sum of the partial copies, nothing else
#define FINISH(V)                                                                                                      \
  hipLaunchKernelGGL(fold_back_t_finish_kernel<V>, dim3(Co / V), dim3(256), 0, st, dot_part, chunks, r_part, nrpart, b, \
                     gamma, mean, var, eps, Co, db, dgamma, dbeta)
  if (vec) FINISH(4); else FINISH(1);
#undef FINISH
  return hipGetLastError();
}

}  // namespace convbn
