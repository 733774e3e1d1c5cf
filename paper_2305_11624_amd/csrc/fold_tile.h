// Pieces of the parameter-side kernels that run inside several launches: the fold of a bf16 weight, one 64 x 64 tile at a
// time (the fold kernels, and forward convolutions whose launch folds on the side), and a slice of dZ's column sums.
#pragma once
#include "common.h"

namespace convbn {

// bf16 fast path (K and Cout multiples of 8): 64 x 64 tiles, every global access is a 16-byte vector --
// rows of W are read and written back eight columns per thread, the transposed copy leaves through an
// LDS tile as rows of 64 consecutive output channels.
struct FoldArgs {
  const bf16_t* W; const float* b; const float* gamma; const float* beta; const float* mean; const float* var;
  bf16_t* w_krsc; bf16_t* w_crsk; float* bfold;
  float eps; int identity, Cout, K, Cin, taps;
};
// One 64 x 64 tile (bx along K, by along Cout) of one block's fold, by 256 threads `tid` of a workgroup all of whose
// threads call this (there is a barrier inside); a tile outside the matrix does nothing.
__device__ __forceinline__ void fold_tile_bf16x8(const FoldArgs& a, int bx, int by, int tid, unsigned short (*tile)[72]) {
  const bf16_t* __restrict__ W = a.W;
  const float* __restrict__ b = a.b; const float* __restrict__ gamma = a.gamma; const float* __restrict__ beta = a.beta;
  const float* __restrict__ mean = a.mean; const float* __restrict__ var = a.var;
  bf16_t* __restrict__ w_krsc = a.w_krsc; bf16_t* __restrict__ w_crsk = a.w_crsk; float* __restrict__ bfold = a.bfold;
  const float eps = a.eps;
  const int identity = a.identity, Cout = a.Cout, K = a.K, Cin = a.Cin, taps = a.taps;
  const int co0 = by * 64;
  const int k0 = bx * 64;
  const bool do_bias = bx == 0 && tid < 64 && bfold && co0 + tid < Cout;
  float bg = 1.f, bv = 1.f, bm = 0.f, bb = 0.f, bc = 0.f;
  if (do_bias) {
    const int co = co0 + tid;
    if (!identity) { bg = gamma[co]; bv = var[co]; bm = mean[co]; bb = beta[co]; }
    if (b) bc = b[co];
  }
  const int kv = (tid & 7) * 8, r = tid >> 3;
  uint4 wv[2];
  float gv[2], vv[2];
  bool ok[2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int co = co0 + r + 32 * e;
    ok[e] = co < Cout && k0 + kv < K;
    wv[e] = ok[e] ? *reinterpret_cast<const uint4*>(W + (size_t)co * K + k0 + kv) : make_uint4(0u, 0u, 0u, 0u);
    gv[e] = (ok[e] && !identity) ? gamma[co] : 1.f;
    vv[e] = (ok[e] && !identity) ? var[co] : 1.f - eps;
  }
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const float sc = identity ? 1.f : gv[e] / sqrtf(vv[e] + eps);
    const uint32_t in[4] = {wv[e].x, wv[e].y, wv[e].z, wv[e].w};
    uint32_t out[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      out[i] = pack_bf16x2(bf16_lo(in[i]) * sc, bf16_hi(in[i]) * sc);
      tile[kv + 2 * i][r + 32 * e] = (unsigned short)(out[i] & 0xffffu);
      tile[kv + 2 * i + 1][r + 32 * e] = (unsigned short)(out[i] >> 16);
    }
    if (ok[e] && w_krsc)
      *reinterpret_cast<uint4*>(w_krsc + (size_t)(co0 + r + 32 * e) * K + k0 + kv) = make_uint4(out[0], out[1], out[2], out[3]);
  }
  if (do_bias) {
    const float sc = identity ? 1.f : bg / sqrtf(bv + eps);
    bfold[co0 + tid] = identity ? bc : (bc - bm) * sc + bb;
  }
  __syncthreads();
  if (!w_crsk) return;
  const int kl = tid >> 2, c16 = (tid & 3) * 16;
  const int k = k0 + kl;
  if (k < K) {
    const int tap = k / Cin, ci = k - tap * Cin;
    bf16_t* dst = w_crsk + ((size_t)ci * taps + tap) * Cout + co0 + c16;
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (co0 + c16 + 8 * h < Cout)
        *reinterpret_cast<uint4*>(dst + 8 * h) = *reinterpret_cast<const uint4*>(&tile[kl][c16 + 8 * h]);
  }
}

constexpr int FOLD_TILE_BYTES = 64 * 72 * 2;

// A forward launch that is given the unfolded weight leaves w' = s w ([Cin][taps][Cout], what Tune mode keeps for
// backward, Sec. 3.4.2) with workgroups of its own behind the convolution's: they need compute units only as those free
// up, and the fold is no launch (3.5-4.5 us) any more.  A workgroup of 512 threads takes two tiles.
inline int fold_side_blocks(const BnEpilogue& bn) {
  if (!bn.gamma || !bn.w_folded_out) return 0;
  return ceil_div(ceil_div(bn.taps * bn.Cin, 64) * ceil_div(bn.Cout, 64), 2);
}
// smem: 2 * FOLD_TILE_BYTES
__device__ __forceinline__ void fold_side(const BnEpilogue& bn, const bf16_t* wgt, int wg, unsigned char* smem) {
  const FoldArgs a{wgt, nullptr, bn.gamma, bn.beta, bn.mean, bn.var, nullptr, static_cast<bf16_t*>(bn.w_folded_out), nullptr,
                   bn.eps, 0, bn.Cout, bn.taps * bn.Cin, bn.Cin, bn.taps};
  const int half = (int)threadIdx.x >> 8, tk = (a.K + 63) / 64;
  const int t = wg * 2 + half;
  fold_tile_bf16x8(a, t % tk, t / tk, (int)threadIdx.x & 255,
                   reinterpret_cast<unsigned short (*)[72]>(smem + half * FOLD_TILE_BYTES));
}

// Column sums of rows [m0, m1) of a bf16 matrix [..][Cout], Cout % 8 == 0 and at most 2048, by 256 threads: a thread reads 8
// channels (16 bytes) of a row, Cout / 8 threads cover one, the others stride over rows.  Eight rows of a thread are asked for
// at once: one at a time, a block of 98 rows of 256 channels was 13 trips to memory in a row.
__device__ __forceinline__ void colsum_slice_bf16x8(const uint4* __restrict__ dz, int m0, int m1, int Cout, int tid,
                                                    float (*red)[9], float* __restrict__ out) {
  const int c8 = Cout >> 3, lanes = 256 / c8;
  const int tc = tid % c8, tr = tid / c8;
  float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (tr < lanes)
    for (int m = m0 + tr; m < m1; m += 8 * lanes) {
      uint4 v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = dz[(size_t)min(m + j * lanes, m1 - 1) * c8 + tc];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        if (m + j * lanes >= m1) v[j] = make_uint4(0u, 0u, 0u, 0u);
        a[0] += bf16_lo(v[j].x); a[1] += bf16_hi(v[j].x); a[2] += bf16_lo(v[j].y); a[3] += bf16_hi(v[j].y);
        a[4] += bf16_lo(v[j].z); a[5] += bf16_hi(v[j].z); a[6] += bf16_lo(v[j].w); a[7] += bf16_hi(v[j].w);
      }
    }
#pragma unroll
  for (int e = 0; e < 8; ++e) red[tid][e] = a[e];
  __syncthreads();
  for (int c = tid; c < Cout; c += 256) {
    float acc = 0.f;
    for (int l = 0; l < lanes; ++l) acc += red[l * c8 + (c >> 3)][c & 7];
    out[c] = acc;
  }
}

}  // namespace convbn
