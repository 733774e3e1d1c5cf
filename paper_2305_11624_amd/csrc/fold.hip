// Memory-bound kernels around the convolution:
//   fold        w' = s w, b' = (b - mu) s + beta            (Sec. 3.3, definitions of w', b')
//   fold-back   dW = s dw', dgamma, dbeta, db               (Table 2, row "Tune")
//   colsum      r_c = sum_{n,h,w} dZ                        (App. B: backward of a broadcast)
//   bn_affine   Z = gamma (Y - mu)/sqrt(var+eps) + beta     (Sec. 3.1; Eval comparison path)
//   bn_bwd      dY = s dZ and the per-channel sums of Table 2, row "Eval"
#include "common.h"
#include "fold_tile.h"

#include <cstring>

namespace convbn {

namespace {

constexpr int FOLD_TCO = 32;  // output channels per tile
constexpr int FOLD_TK = 64;   // reduction-index (tap, ci) entries per tile

// One tile = FOLD_TCO rows of W x FOLD_TK columns.  Rows of W ([Cout][K], K = taps*Cin)
// are read coalesced along K, scaled, written back in the same order (w_krsc) and,
// through an LDS transpose, as [Cin][taps][Cout] (w_crsk) with Cout contiguous.
template <typename T>
__global__ __launch_bounds__(256) void fold_kernel(const T* __restrict__ W, const float* __restrict__ b,
                                                   const float* __restrict__ gamma,
                                                   const float* __restrict__ beta,
                                                   const float* __restrict__ mean,
                                                   const float* __restrict__ var, float eps,
                                                   int identity, int Cout, int K, int Cin, int taps,
                                                   T* __restrict__ w_krsc, T* __restrict__ w_crsk,
                                                   float* __restrict__ bfold) {
  __shared__ T tile[FOLD_TK][FOLD_TCO + 2];
  const int tid = threadIdx.x;
  const int co0 = blockIdx.y * FOLD_TCO;
  const int k0 = blockIdx.x * FOLD_TK;
  // Every load of the kernel (weights, the per-row BN vectors, the inputs of b') is issued before the
  // first use, so the kernel pays one memory round trip, not one per dependent stage.
  const bool do_bias = blockIdx.x == 0 && tid < FOLD_TCO && bfold && co0 + tid < Cout;
  float bg = 1.f, bv = 1.f, bm = 0.f, bb = 0.f, bc = 0.f;
  if (do_bias) {
    const int co = co0 + tid;
    if (!identity) { bg = gamma[co]; bv = var[co]; bm = mean[co]; bb = beta[co]; }
    if (b) bc = b[co];
  }
  // read + scale: a wave reads 64 consecutive columns of one row; rows tid/64 + 4e
  {
    const int kc = tid & 63;
    const int k = k0 + kc;
    T wv[FOLD_TCO / 4];
    float gv[FOLD_TCO / 4], vv[FOLD_TCO / 4];
#pragma unroll
    for (int e = 0; e < FOLD_TCO / 4; ++e) {
      const int co = co0 + (tid >> 6) + 4 * e;
      const bool ok = co < Cout && k < K;
      wv[e] = ok ? W[(size_t)co * K + k] : from_f32<T>(0.f);
      gv[e] = (ok && !identity) ? gamma[co] : 1.f;
      vv[e] = (ok && !identity) ? var[co] : 1.f - eps;
    }
#pragma unroll
    for (int e = 0; e < FOLD_TCO / 4; ++e) {
      const int r = (tid >> 6) + 4 * e;
      const int co = co0 + r;
      const float sc = identity ? 1.f : gv[e] / sqrtf(vv[e] + eps);
      const T v = from_f32<T>(to_f32(wv[e]) * sc);
      if (co < Cout && k < K && w_krsc) w_krsc[(size_t)co * K + k] = v;
      tile[kc][r] = v;
    }
  }
  if (do_bias) {
    const float sc = identity ? 1.f : bg / sqrtf(bv + eps);
    bfold[co0 + tid] = identity ? bc : (bc - bm) * sc + bb;
  }
  if (!w_crsk) return;
  __syncthreads();
  // transposed write: thread -> (k row = tid/4, co cols (tid%4)*8 .. +8)
  {
    const int kr = tid >> 2;
    const int cc = (tid & 3) * 8;
    const int k = k0 + kr;
    if (k < K) {
      const int tap = k / Cin, ci = k - tap * Cin;
      T* dst = w_crsk + ((size_t)ci * taps + tap) * Cout + co0;
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (co0 + cc + e < Cout) dst[cc + e] = tile[kr][cc + e];
    }
  }
}

__global__ __launch_bounds__(256) void fold_bf16x8_kernel(FoldArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned short tile[64][72];   // [k][co], 144-byte rows
  fold_tile_bf16x8(a, blockIdx.x, blockIdx.y, threadIdx.x, tile);
}

// The folds of several blocks in one launch (Sec. 3.3: a training step starts by folding every block's
// BatchNorm into its weights; one launch per block would be bound by the launches, not by memory).
// items[i] covers blocks [first_block, first_block + tiles): tile t of item i is (t % tiles_k, t / tiles_k).
struct FoldGroupItem { FoldArgs a; int first_block, tiles_k; };
__global__ __launch_bounds__(256) void fold_group_kernel(const FoldGroupItem* __restrict__ items, int n) {
  __shared__ __attribute__((aligned(16))) unsigned short tile[64][72];
  int lo = 0, hi = n - 1;   // last item whose first_block <= blockIdx.x
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (items[mid].first_block <= (int)blockIdx.x) lo = mid; else hi = mid - 1;
  }
  const FoldGroupItem it = items[lo];
  const int t = blockIdx.x - it.first_block;
  fold_tile_bf16x8(it.a, t % it.tiles_k, t / it.tiles_k, threadIdx.x, tile);
}

template <typename T, int NTHR, RowKind ROW, RowLen LEN>
__global__ __launch_bounds__(NTHR) void fold_back_kernel(FoldBackArgs a) {
  __shared__ float4 red4[NTHR];
  __shared__ float red[2 * NTHR / 64];
  fold_back_row<T, 16, 1, ROW, LEN>(a, blockIdx.x, threadIdx.x, NTHR, red4, red);
}

// The fold-backs of several blocks in one launch (Table 2 "Tune", last four lines, for every block of a group):
// workgroup w handles output channel w - first_block of the item it falls into.  Same arithmetic, in the same
// order, as the 256-thread single-block kernel.
struct FoldBackGroupItem {
  FoldBackArgs a;
  int first_block;
};
__global__ __launch_bounds__(256) void fold_back_group_kernel(const FoldBackGroupItem* __restrict__ items, int n) {
  __shared__ float4 red4[256];
  __shared__ float red[8];
  int lo = 0, hi = n - 1;   // last item whose first_block <= blockIdx.x
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (items[mid].first_block <= (int)blockIdx.x) lo = mid; else hi = mid - 1;
  }
  const FoldBackArgs a = items[lo].a;
  fold_back_row<bf16_t, 16, 1, ROW_VEC>(a, blockIdx.x - items[lo].first_block, threadIdx.x, 256, red4, red);
}

// Column reductions over a [M][Cout] channels-last tensor.  `cw` threads walk the
// channel dimension (coalesced), 256/cw row lanes stride over this block's rows.
__device__ __forceinline__ int pow2_cw(int Cout) {
  int cw = 1;
  while (cw < Cout && cw < 256) cw <<= 1;
  return cw;
}

template <typename T>
__global__ __launch_bounds__(256) void colsum_kernel(const T* __restrict__ dz, int M, int Cout,
                                                     int rows_per_block, float* __restrict__ part) {
  __shared__ float red[256];
  const int cw = pow2_cw(Cout);
  const int lanes = 256 / cw;
  const int tc = threadIdx.x % cw, tr = threadIdx.x / cw;
  const int m0 = blockIdx.x * rows_per_block;
  const int m1 = min(M, m0 + rows_per_block);
  for (int c0 = 0; c0 < Cout; c0 += cw) {
    const int co = c0 + tc;
    float acc = 0.f;
    if (co < Cout)
      for (int m = m0 + tr; m < m1; m += lanes) acc += to_f32(dz[(size_t)m * Cout + co]);
    red[threadIdx.x] = acc;
    __syncthreads();
    if (tr == 0 && co < Cout) {
      for (int l = 1; l < lanes; ++l) acc += red[l * cw + tc];
      part[(size_t)blockIdx.x * Cout + co] = acc;
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void colsum_bf16x8_kernel(const uint4* __restrict__ dz, int M, int Cout,
                                                            int rows_per_block, float* __restrict__ part) {
  __shared__ float red[256][9];
  const int m0 = blockIdx.x * rows_per_block;
  colsum_slice_bf16x8(dz, m0, min(M, m0 + rows_per_block), Cout, threadIdx.x, red, part + (size_t)blockIdx.x * Cout);
}

template <typename T>
__global__ __launch_bounds__(256) void bn_affine_fwd_kernel(const T* __restrict__ y,
                                                            const float* __restrict__ gamma,
                                                            const float* __restrict__ beta,
                                                            const float* __restrict__ mean,
                                                            const float* __restrict__ var, float eps,
                                                            size_t total, int Cout, T* __restrict__ z) {
  const size_t stride = (size_t)gridDim.x * 256;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += stride) {
    const int co = (int)(i % Cout);
    const float ybar = (to_f32(y[i]) - mean[co]) / sqrtf(var[co] + eps);
    z[i] = from_f32<T>(gamma[co] * ybar + beta[co]);
  }
}

// 8 bf16 per thread, Cout % 8 == 0; per-channel scale/shift staged in LDS (2*Cout floats).
__global__ __launch_bounds__(256) void bn_affine_fwd_bf16x8_kernel(
    const uint4* __restrict__ y, const float* __restrict__ gamma, const float* __restrict__ beta,
    const float* __restrict__ mean, const float* __restrict__ var, float eps, size_t nvec, int Cout,
    uint4* __restrict__ z, int relu, const uint4* __restrict__ add) {
  extern __shared__ float sm[];
  float* s_s = sm;
  float* s_t = sm + Cout;
  for (int c = threadIdx.x; c < Cout; c += 256) {
    const float s = gamma[c] / sqrtf(var[c] + eps);
    s_s[c] = s;
    s_t[c] = beta[c] - mean[c] * s;
  }
  __syncthreads();
  const size_t stride = (size_t)gridDim.x * 256;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < nvec; i += stride) {
    const int co = (int)((i * 8) % Cout);
    const uint4 v = y[i];
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    uint32_t o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int c = co + 2 * e;
      o[e] = pack_bf16x2(bf16_lo(w[e]) * s_s[c] + s_t[c], bf16_hi(w[e]) * s_s[c + 1] + s_t[c + 1]);
    }
    uint4 r = make_uint4(o[0], o[1], o[2], o[3]);
    if (add) r = add8(r, add[i]);   // (an addend and a ReLU behind the block: the descriptor's activation bits)
    z[i] = relu ? relu8(r) : r;
  }
}

template <typename T>
__global__ __launch_bounds__(256) void bn_bwd_kernel(const T* __restrict__ dz, const T* __restrict__ y,
                                                     const float* __restrict__ gamma,
                                                     const float* __restrict__ mean,
                                                     const float* __restrict__ var, float eps, int M,
                                                     int Cout, int rows_per_block, T* __restrict__ dy,
                                                     float* __restrict__ part) {
  __shared__ float red0[256];
  __shared__ float red1[256];
  const int cw = pow2_cw(Cout);
  const int lanes = 256 / cw;
  const int tc = threadIdx.x % cw, tr = threadIdx.x / cw;
  const int m0 = blockIdx.x * rows_per_block;
  const int m1 = min(M, m0 + rows_per_block);
  for (int c0 = 0; c0 < Cout; c0 += cw) {
    const int co = c0 + tc;
    float a0 = 0.f, a1 = 0.f;
    if (co < Cout) {
      const float sd = sqrtf(var[co] + eps);
      const float s = gamma[co] / sd, mu = mean[co];
      for (int m = m0 + tr; m < m1; m += lanes) {
        const size_t idx = (size_t)m * Cout + co;
        const float g = to_f32(dz[idx]);
        dy[idx] = from_f32<T>(s * g);
        a0 += g;
        a1 += g * ((to_f32(y[idx]) - mu) / sd);
      }
    }
    red0[threadIdx.x] = a0;
    red1[threadIdx.x] = a1;
    __syncthreads();
    if (tr == 0 && co < Cout) {
      for (int l = 1; l < lanes; ++l) {
        a0 += red0[l * cw + tc];
        a1 += red1[l * cw + tc];
      }
      part[((size_t)blockIdx.x * 2 + 0) * Cout + co] = a0;
      part[((size_t)blockIdx.x * 2 + 1) * Cout + co] = a1;
    }
    __syncthreads();
  }
}

// bf16, Cout % 8 == 0, Cout <= 2048: 16 bytes (8 channels) per thread per row, as colsum_bf16x8_kernel.
__global__ __launch_bounds__(256) void bn_bwd_bf16x8_kernel(const uint4* __restrict__ dz, const uint4* __restrict__ y,
                                                            const float* __restrict__ gamma,
                                                            const float* __restrict__ mean,
                                                            const float* __restrict__ var, float eps, int M,
                                                            int Cout, int rows_per_block, uint4* __restrict__ dy,
                                                            float* __restrict__ part) {
  __shared__ float red0[256][9];
  __shared__ float red1[256][9];
  const int c8 = Cout >> 3;
  const int lanes = 256 / c8;
  const int tc = threadIdx.x % c8, tr = threadIdx.x / c8;
  const int m0 = blockIdx.x * rows_per_block;
  const int m1 = min(M, m0 + rows_per_block);
  float a0[8], a1[8], sc[8], mu[8], isd[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    a0[e] = 0.f; a1[e] = 0.f;
    const int c = min(tc * 8 + e, Cout - 1);
    isd[e] = 1.f / sqrtf(var[c] + eps);
    sc[e] = gamma[c] * isd[e];
    mu[e] = mean[c];
  }
  if (tr < lanes)
    for (int m = m0 + tr; m < m1; m += lanes) {
      const size_t idx = (size_t)m * c8 + tc;
      const uint4 g4 = dz[idx], y4 = y[idx];
      const uint32_t gw[4] = {g4.x, g4.y, g4.z, g4.w}, yw[4] = {y4.x, y4.y, y4.z, y4.w};
      uint32_t ow[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float g0 = bf16_lo(gw[e]), g1 = bf16_hi(gw[e]);
        const float y0 = bf16_lo(yw[e]), y1 = bf16_hi(yw[e]);
        ow[e] = pack_bf16x2(sc[2 * e] * g0, sc[2 * e + 1] * g1);
        a0[2 * e] += g0; a0[2 * e + 1] += g1;
        a1[2 * e] += g0 * ((y0 - mu[2 * e]) * isd[2 * e]);
        a1[2 * e + 1] += g1 * ((y1 - mu[2 * e + 1]) * isd[2 * e + 1]);
      }
      dy[idx] = make_uint4(ow[0], ow[1], ow[2], ow[3]);
    }
#pragma unroll
  for (int e = 0; e < 8; ++e) { red0[threadIdx.x][e] = a0[e]; red1[threadIdx.x][e] = a1[e]; }
  __syncthreads();
  for (int c = threadIdx.x; c < Cout; c += 256) {
    float s0 = 0.f, s1 = 0.f;
    for (int l = 0; l < lanes; ++l) {
      s0 += red0[l * c8 + (c >> 3)][c & 7];
      s1 += red1[l * c8 + (c >> 3)][c & 7];
    }
    part[((size_t)blockIdx.x * 2 + 0) * Cout + c] = s0;
    part[((size_t)blockIdx.x * 2 + 1) * Cout + c] = s1;
  }
}

// Sums the per-workgroup partial (dbeta, dgamma) rows: 64 channels per workgroup, 16 waves each take
// every 16th partial row, then a fixed-order reduction through LDS (deterministic).
__global__ __launch_bounds__(1024) void bn_bwd_finalize_kernel(const float* __restrict__ part, int parts,
                                                               const float* __restrict__ gamma,
                                                               const float* __restrict__ var, float eps,
                                                               int Cout, float* __restrict__ dgamma,
                                                               float* __restrict__ dbeta,
                                                               float* __restrict__ db) {
  __shared__ float red[2][16][64];
  const int lane = threadIdx.x & 63, slice = threadIdx.x >> 6;
  const int co = blockIdx.x * 64 + lane;
  float a0 = 0.f, a1 = 0.f;
  if (co < Cout) {
#pragma unroll 4
    for (int p = slice; p < parts; p += 16) {
      a0 += part[((size_t)p * 2 + 0) * Cout + co];
      a1 += part[((size_t)p * 2 + 1) * Cout + co];
    }
  }
  red[0][slice][lane] = a0;
  red[1][slice][lane] = a1;
  __syncthreads();
  if (slice != 0 || co >= Cout) return;
  a0 = 0.f; a1 = 0.f;
#pragma unroll
  for (int q = 0; q < 16; ++q) { a0 += red[0][q][lane]; a1 += red[1][q][lane]; }
  dbeta[co] = a0;
  dgamma[co] = a1;
  if (db) db[co] = gamma[co] / sqrtf(var[co] + eps) * a0;
}

template <typename E>
__global__ __launch_bounds__(256) void repitch_kernel(const E* __restrict__ src, E* __restrict__ dst, size_t total,
                                                      size_t inner_in, size_t inner_out) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) {
    const size_t row = i / inner_out, c = i - row * inner_out;
    dst[i] = c < inner_in ? src[row * inner_in + c] : E(0);
  }
}

int rows_per_block_for(int M, int parts) { return ceil_div(M, parts); }

}  // namespace

hipError_t launch_repitch(int elem_bytes, size_t rows, size_t inner_in, size_t inner_out, const void* src,
                          void* dst, hipStream_t st) {
  const size_t total = rows * inner_out;
  const int blocks = (int)((total + 255) / 256 < 4096 ? (total + 255) / 256 : 4096);
  if (elem_bytes == 2)
    hipLaunchKernelGGL(repitch_kernel<unsigned short>, dim3(blocks), dim3(256), 0, st, (const unsigned short*)src,
                       (unsigned short*)dst, total, inner_in, inner_out);
  else
    hipLaunchKernelGGL(repitch_kernel<unsigned int>, dim3(blocks), dim3(256), 0, st, (const unsigned int*)src,
                       (unsigned int*)dst, total, inner_in, inner_out);
  return hipGetLastError();
}

hipError_t launch_fold(const Geom& g, int dtype, const void* W, const float* b, const float* gamma,
                       const float* beta, const float* mean, const float* var, int identity,
                       void* w_krsc, void* w_crsk, float* bfold, hipStream_t st) {
  dim3 grid(ceil_div(g.K, FOLD_TK), ceil_div(g.Cout, FOLD_TCO));
  const int taps = g.kH * g.kW;
  if (dtype == CONVBN_BF16 && g.K % 8 == 0 && g.Cout % 8 == 0)
    hipLaunchKernelGGL(fold_bf16x8_kernel, dim3(ceil_div(g.K, 64), ceil_div(g.Cout, 64)), dim3(256), 0, st,
                       FoldArgs{(const bf16_t*)W, b, gamma, beta, mean, var, (bf16_t*)w_krsc, (bf16_t*)w_crsk, bfold,
                                g.eps, identity, g.Cout, g.K, g.Cin, taps});
  else if (dtype == CONVBN_BF16)
    hipLaunchKernelGGL(fold_kernel<bf16_t>, grid, dim3(256), 0, st, (const bf16_t*)W, b, gamma, beta,
                       mean, var, g.eps, identity, g.Cout, g.K, g.Cin, taps, (bf16_t*)w_krsc,
                       (bf16_t*)w_crsk, bfold);
  else
    hipLaunchKernelGGL(fold_kernel<float>, grid, dim3(256), 0, st, (const float*)W, b, gamma, beta,
                       mean, var, g.eps, identity, g.Cout, g.K, g.Cin, taps, (float*)w_krsc,
                       (float*)w_crsk, bfold);
  return hipGetLastError();
}

size_t fold_group_item_bytes() { return sizeof(FoldGroupItem); }

bool fold_group_item(const Geom& g, int dtype, const void* W, const float* b, const float* gamma, const float* beta,
                     const float* mean, const float* var, int identity, void* w_krsc, void* w_crsk, float* bfold,
                     int first_block, void* item_out, int* blocks) {
  if (dtype != CONVBN_BF16 || g.K % 8 != 0 || g.Cout % 8 != 0) return false;
  FoldGroupItem it{};
  it.a = FoldArgs{(const bf16_t*)W, b, gamma, beta, mean, var, (bf16_t*)w_krsc, (bf16_t*)w_crsk, bfold,
                  g.eps, identity, g.Cout, g.K, g.Cin, g.kH * g.kW};
  it.first_block = first_block;
  it.tiles_k = ceil_div(g.K, 64);
  *blocks = it.tiles_k * ceil_div(g.Cout, 64);
  memcpy(item_out, &it, sizeof(it));
  return true;
}

hipError_t launch_fold_group(const void* items_dev, int n, int grid_blocks, hipStream_t st) {
  hipLaunchKernelGGL(fold_group_kernel, dim3(grid_blocks), dim3(256), 0, st, (const FoldGroupItem*)items_dev, n);
  return hipGetLastError();
}

size_t fold_back_group_item_bytes() { return sizeof(FoldBackGroupItem); }

bool fold_back_group_item(const Geom& g, int dtype, const float* dwf_part, int nsplit, const float* r_part, int nrpart,
                          const void* W, const float* b, const float* gamma, const float* mean, const float* var,
                          void* dW, float* db, float* dgamma, float* dbeta, int first_block, void* item_out,
                          int* blocks) {
  if (dtype != CONVBN_BF16 || g.K % 4 != 0) return false;
  const FoldBackGroupItem it{{dwf_part, r_part, W, b, gamma, mean, var, dW, db, dgamma, dbeta, g.eps, nsplit, nrpart, 0, g.Cout, g.K, 0},
                             first_block};
  *blocks = g.Cout;
  memcpy(item_out, &it, sizeof(it));
  return true;
}

hipError_t launch_fold_back_group(const void* items_dev, int n, int grid_blocks, hipStream_t st) {
  hipLaunchKernelGGL(fold_back_group_kernel, dim3(grid_blocks), dim3(256), 0, st, (const FoldBackGroupItem*)items_dev, n);
  return hipGetLastError();
}

hipError_t launch_fold_back(const Geom& g, int dtype, const float* dwf_part, int nsplit,
                            const float* r_part, int nrpart, const void* W, const float* b,
                            const float* gamma, const float* mean, const float* var, int identity,
                            void* dW, float* db, float* dgamma, float* dbeta, hipStream_t st) {
  const FoldBackArgs a{dwf_part, r_part, W, b, gamma, mean, var, dW, db, dgamma, dbeta, g.eps, nsplit, nrpart, identity, g.Cout, g.K, 0};
#define FB_LAUNCH(NTHR, ROW, LEN)                                                                                       \
  do {                                                                                                                  \
    if (dtype == CONVBN_BF16) hipLaunchKernelGGL((fold_back_kernel<bf16_t, NTHR, ROW, LEN>), dim3(g.Cout), dim3(NTHR), 0, st, a); \
    else hipLaunchKernelGGL((fold_back_kernel<float, NTHR, ROW, LEN>), dim3(g.Cout), dim3(NTHR), 0, st, a);              \
  } while (0)
  // few output channels and many partial copies: a 1024-thread block per channel (16 waves share
  // the copies) keeps enough loads in flight on the few CUs such a grid occupies
  const bool wide = g.Cout <= 128 && nsplit >= 16 && ceil_div(g.K, 4) < 256;
  if (g.K % 4 == 0) {
    if (wide) FB_LAUNCH(1024, ROW_VEC, LEN_SHORT);
    else if (g.K / 4 < 256) FB_LAUNCH(256, ROW_VEC, LEN_SHORT);
    else FB_LAUNCH(256, ROW_VEC, LEN_LONG);
  } else if (wide && g.K >= 4) FB_LAUNCH(1024, ROW_ANY, LEN_SHORT);
  else if (g.K < 256) FB_LAUNCH(256, ROW_ELEM, LEN_SHORT);
  else FB_LAUNCH(256, ROW_ELEM, LEN_LONG);
#undef FB_LAUNCH
  return hipGetLastError();
}

int colsum_parts(const Geom& g) { return g.M < 256 * 64 ? ceil_div(g.M, 64) : 256; }

hipError_t launch_colsum(const Geom& g, int dtype, const void* dz, float* r_part, hipStream_t st) {
  const int parts = colsum_parts(g);
  const int rpb = rows_per_block_for(g.M, parts);
  if (dtype == CONVBN_BF16 && g.Cout % 8 == 0 && g.Cout <= 2048)
    hipLaunchKernelGGL(colsum_bf16x8_kernel, dim3(parts), dim3(256), 0, st, (const uint4*)dz, g.M, g.Cout,
                       rpb, r_part);
  else if (dtype == CONVBN_BF16)
    hipLaunchKernelGGL(colsum_kernel<bf16_t>, dim3(parts), dim3(256), 0, st, (const bf16_t*)dz, g.M,
                       g.Cout, rpb, r_part);
  else
    hipLaunchKernelGGL(colsum_kernel<float>, dim3(parts), dim3(256), 0, st, (const float*)dz, g.M,
                       g.Cout, rpb, r_part);
  return hipGetLastError();
}

hipError_t launch_bn_affine_fwd(const Geom& g, int dtype, const void* y, const float* gamma,
                                const float* beta, const float* mean, const float* var, void* z,
                                hipStream_t st) {
  const size_t total = (size_t)g.M * g.Cout;
  if (dtype == CONVBN_BF16 && g.Cout % 8 == 0 && g.Cout <= 4096) {
    const size_t nvec = total / 8;
    const int blocks = (int)min((size_t)2048, (nvec + 255) / 256);
    hipLaunchKernelGGL(bn_affine_fwd_bf16x8_kernel, dim3(blocks), dim3(256), 2 * g.Cout * sizeof(float), st, (const uint4*)y,
                       gamma, beta, mean, var, g.eps, nvec, g.Cout, (uint4*)z, g.post_relu, (const uint4*)g.post_add);
  } else {
    const int blocks = (int)min((size_t)4096, (total + 255) / 256);
    if (dtype == CONVBN_BF16)
      hipLaunchKernelGGL(bn_affine_fwd_kernel<bf16_t>, dim3(blocks), dim3(256), 0, st,
                         (const bf16_t*)y, gamma, beta, mean, var, g.eps, total, g.Cout, (bf16_t*)z);
    else
      hipLaunchKernelGGL(bn_affine_fwd_kernel<float>, dim3(blocks), dim3(256), 0, st, (const float*)y,
                         gamma, beta, mean, var, g.eps, total, g.Cout, (float*)z);
    if (g.post_add && hipGetLastError() == hipSuccess) {
      const hipError_t e = launch_eltwise(3 /* a + b */, dtype, z, g.post_add, nullptr, total, st);
      if (e != hipSuccess) return e;
    }
    if (g.post_relu && hipGetLastError() == hipSuccess) return launch_eltwise(0 /* max(a, 0) */, dtype, z, nullptr, nullptr, total, st);
  }
  return hipGetLastError();
}

int bn_bwd_parts(const Geom& g) { return colsum_parts(g); }

hipError_t launch_bn_bwd(const Geom& g, int dtype, const void* dz, const void* y, const float* gamma,
                         const float* mean, const float* var, void* dy, float* part, hipStream_t st) {
  const int parts = bn_bwd_parts(g);
  const int rpb = rows_per_block_for(g.M, parts);
  if (dtype == CONVBN_BF16 && g.Cout % 8 == 0 && g.Cout <= 2048)
    hipLaunchKernelGGL(bn_bwd_bf16x8_kernel, dim3(parts), dim3(256), 0, st, (const uint4*)dz, (const uint4*)y,
                       gamma, mean, var, g.eps, g.M, g.Cout, rpb, (uint4*)dy, part);
  else if (dtype == CONVBN_BF16)
    hipLaunchKernelGGL(bn_bwd_kernel<bf16_t>, dim3(parts), dim3(256), 0, st, (const bf16_t*)dz,
                       (const bf16_t*)y, gamma, mean, var, g.eps, g.M, g.Cout, rpb, (bf16_t*)dy, part);
  else
    hipLaunchKernelGGL(bn_bwd_kernel<float>, dim3(parts), dim3(256), 0, st, (const float*)dz,
                       (const float*)y, gamma, mean, var, g.eps, g.M, g.Cout, rpb, (float*)dy, part);
  return hipGetLastError();
}

hipError_t launch_bn_bwd_finalize(const Geom& g, const float* part, int parts, const float* gamma,
                                  const float* var, float* dgamma, float* dbeta, float* db,
                                  hipStream_t st) {
  hipLaunchKernelGGL(bn_bwd_finalize_kernel, dim3(ceil_div(g.Cout, 64)), dim3(1024), 0, st, part, parts,
                     gamma, var, g.eps, g.Cout, dgamma, dbeta, db);
  return hipGetLastError();
}

}  // namespace convbn
