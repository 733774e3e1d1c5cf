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

// ---- fold-back: the partial copies of dw' of one output channel summed, dW = s dw', dgamma, dbeta, db (Table 2 "Tune")
struct __attribute__((packed, aligned(4))) F4u { float x, y, z, w; };
__device__ __forceinline__ float4 ld4u(const float* p) {   // 16 bytes from any element
  const F4u v = *reinterpret_cast<const F4u*>(p);
  return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void fb_load4(const float* p, float (&w)[4]) {
  const float4 v = *reinterpret_cast<const float4*>(p);
  w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
}
__device__ __forceinline__ void fb_load4(const bf16_t* p, float (&w)[4]) {
  const uint2 v = *reinterpret_cast<const uint2*>(p);
  w[0] = bf16_lo(v.x); w[1] = bf16_hi(v.x); w[2] = bf16_lo(v.y); w[3] = bf16_hi(v.y);
}
__device__ __forceinline__ void fb_store4(float* p, const float (&w)[4]) {
  *reinterpret_cast<float4*>(p) = make_float4(w[0], w[1], w[2], w[3]);
}
__device__ __forceinline__ void fb_store4(bf16_t* p, const float (&w)[4]) {
  *reinterpret_cast<uint2*>(p) = make_uint2(pack_bf16x2(w[0], w[1]), pack_bf16x2(w[2], w[3]));
}

// Output channel co by `nthr` threads (a multiple of 64, tid counts them; all threads of the workgroup call this together,
// there are barriers inside; co >= Cout does nothing but meet them).  A thread owns columns of four elements of the row (one,
// where a row's length is no multiple of 4 and there are few copies); ROW_ANY: the last column then starts early and counts
// only its own elements (7 x 7 x 3 rows, 512 copies, a launch: 11.5 us
// with one element a thread, 8.5 with four).  The `nsplit` partial copies of a
// column lie far apart in memory, so every load is a latency round trip of its own: short rows (fewer columns than threads)
// keep FLIGHT copies of a column in flight per thread, the copies are divided over as many thread groups as there are
// threads for, and the groups meet in LDS; long rows take COLS columns at once, four copies of each in flight (one column after the other, 512 columns on 64
// threads and two copies beside an input gradient of 208 workgroups: that launch 21.7 us, 16.9).  Four copies are added in pairs.
// red4: nthr entries, red: 2 per wave, of these threads' own.
enum RowKind { ROW_VEC, ROW_ANY, ROW_ELEM };   // columns of four elements, K % 4 == 0; ... K >= 4; columns of one
// LEN: how many columns a row has, where the launch knows: each form alone takes fewer registers and less code (1024 -> 2048, 1 x 1,
// one copy, a launch: 6.5 us with both in the kernel, 5.3).
enum RowLen { LEN_ANY, LEN_SHORT, LEN_LONG };   // ...; fewer than threads; at least as many
template <typename T, int FLIGHT, int COLS, RowKind ROW, RowLen LEN = LEN_ANY>
__device__ __forceinline__ void fold_back_row(const FoldBackArgs& a, int co, int tid, int nthr, float4* red4, float* red) {
  const bool live = co < a.Cout;
  co = min(co, a.Cout - 1);
  const int K = a.K, nsplit = a.nsplit;
  const T* const W = static_cast<const T*>(a.W) + (size_t)co * K;
  T* const dW = static_cast<T*>(a.dW) + (size_t)co * K;
  const size_t P = (size_t)a.Cout * K;
  const float* const row = a.part + (size_t)co * K;
  // Every trip to memory that does not depend on another starts here: with the weight, r and the channel's vectors read where
  // they are used, four trips in a row, a launch took 4.6 us on 72 -> 136 channels at 27 x 33 and 5.6 on 64 -> 64 at 56 x 56;
  // now 4.0 and 5.0.
  constexpr bool VEC = ROW == ROW_VEC, ELEM = ROW == ROW_ELEM;
  float s = 1.f, sd = 1.f, mu = 0.f, bc = 0.f, r = 0.f;
  if (!a.identity) {
    const float ga = a.gamma[co], va = a.var[co];
    mu = a.mean[co];
    if (a.b) bc = a.b[co];
    if (tid < a.nrpart) r = a.r_part[(size_t)tid * a.Cout + co];
    sd = sqrtf(va + a.eps);
    s = ga / sd;
  }
  float dot = 0.f;
  const float4 zero4 = make_float4(0.f, 0.f, 0.f, 0.f);
  const int K4 = ELEM ? K : (K + 3) >> 2;
  auto at = [&](int c) { return ELEM ? c : VEC ? 4 * c : min(4 * c, K - 4); };   // first element of column c
  auto load_w = [&](int c, float (&w4)[4]) {
    if constexpr (VEC) {
      fb_load4(W + 4 * c, w4);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) w4[e] = !ELEM || e == 0 ? to_f32(W[at(c) + e]) : 0.f;
    }
  };
  auto load_part = [&](const float* p) {
    if constexpr (ELEM) return make_float4(p[0], 0.f, 0.f, 0.f);
    else if constexpr (VEC) return *reinterpret_cast<const float4*>(p);
    else return ld4u(p);
  };
  auto finish = [&](int c, const float4& v, const float (&w4)[4]) {   // dW = s dw', <dw', w> of one column
    const float g4[4] = {v.x, v.y, v.z, v.w};
    float o4[4];
    const int k = at(c), skip = VEC || ELEM ? 0 : 4 * c - k;   // (its first `skip` elements are the column before's)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      o4[e] = s * g4[e];
      if (e >= skip && (!ELEM || e == 0)) dot += g4[e] * w4[e];
    }
    // (The sum stays in front of the store: the compiler had moved it behind the branch, and there its wait for W was one for the
    // store too, in every column.  512 -> 512, 3 x 3, one copy, a launch: 6.95 us, 5.85; 128 -> 128, 14 copies 5.7, 5.1.)
    asm volatile("" : "+v"(dot));
    if (!live) return;
    if constexpr (VEC) {
      fb_store4(dW + k, o4);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e >= skip && (!ELEM || e == 0)) dW[k + e] = from_f32<T>(o4[e]);
    }
  };
  if (LEN == LEN_LONG || (LEN == LEN_ANY && K4 >= nthr)) {
    for (int c0 = tid; c0 < K4; c0 += COLS * nthr) {
      float4 v[COLS];
      float w4[COLS][4];
#pragma unroll
      for (int i = 0; i < COLS; ++i) {
        v[i] = zero4;
        if (i == 0 || c0 + i * nthr < K4) load_w(c0 + i * nthr, w4[i]);
      }
      auto add = [&](float4& u, const float4& o) { u.x += o.x; u.y += o.y; u.z += o.z; u.w += o.w; };
      auto pairs = [&](float4& u, float4* t) {   // u + ((t0 + t1) + (t2 + t3))
        add(t[0], t[1]);
        add(t[2], t[3]);
        add(t[0], t[2]);
        add(u, t[0]);
      };
      if constexpr (LEN == LEN_LONG) {
        static_assert(COLS == 1);
        int sp = 0;
        for (; sp + 3 < nsplit; sp += 4) {
          float4 t[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) t[j] = load_part(row + (size_t)(sp + j) * P + at(c0));
          pairs(v[0], t);
        }
        float4 t[3];
#pragma unroll
        for (int j = 0; j < 3; ++j)
          if (sp + j < nsplit) t[j] = load_part(row + (size_t)(sp + j) * P + at(c0));
#pragma unroll
        for (int j = 0; j < 3; ++j)
          if (sp + j < nsplit) add(v[0], t[j]);
      } else {   // (in the form above an input gradient with a fold-back beside it takes 1 - 4 us more, in this one a launch of its own 1 us)
        for (int sp = 0; sp < nsplit; sp += 4) {
          float4 t[COLS][4];
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (sp + j < nsplit)
#pragma unroll
              for (int i = 0; i < COLS; ++i)
                if (i == 0 || c0 + i * nthr < K4) t[i][j] = load_part(row + (size_t)(sp + j) * P + at(c0 + i * nthr));
          if (sp + 3 < nsplit) {
#pragma unroll
            for (int i = 0; i < COLS; ++i) pairs(v[i], t[i]);
          } else {
#pragma unroll
            for (int j = 0; j < 3; ++j)
              if (sp + j < nsplit)
#pragma unroll
                for (int i = 0; i < COLS; ++i) add(v[i], t[i][j]);
          }
        }
      }
#pragma unroll
      for (int i = 0; i < COLS; ++i)
        if (c0 + i * nthr < K4) finish(c0 + i * nthr, v[i], w4[i]);
    }
  } else {
    // thread -> (column c, group g of the partial copies); a group more is a read from LDS in a row more, at the end
    const int G = min(nthr / K4, (nsplit + FLIGHT - 1) / FLIGHT);
    const int c = tid % K4, g = tid / K4;
    float4 v = zero4;
    float w4[4] = {0.f, 0.f, 0.f, 0.f};
    if (g == 0) load_w(c, w4);
    if (g < G) {
      const float* const col = row + at(c);
      for (int sp0 = g; sp0 < nsplit; sp0 += FLIGHT * G) {
        float4 t[FLIGHT];
#pragma unroll
        for (int j = 0; j < FLIGHT; ++j) t[j] = sp0 + j * G < nsplit ? load_part(col + (size_t)(sp0 + j * G) * P) : zero4;
#pragma unroll
        for (int j = 0; j < FLIGHT; j += 4) {
          v.x += (t[j].x + t[j + 1].x) + (t[j + 2].x + t[j + 3].x);
          v.y += (t[j].y + t[j + 1].y) + (t[j + 2].y + t[j + 3].y);
          v.z += (t[j].z + t[j + 1].z) + (t[j + 2].z + t[j + 3].z);
          v.w += (t[j].w + t[j + 1].w) + (t[j + 2].w + t[j + 3].w);
        }
      }
    }
    red4[tid] = v;
    __syncthreads();
    if (g == 0) {
      for (int l = 1; l < G; ++l) {
        const float4 o = red4[l * K4 + c];
        v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w;
      }
      finish(c, v, w4);
    }
  }
  if (a.identity) return;
#pragma unroll 4
  for (int q = tid + nthr; q < a.nrpart; q += nthr) r += a.r_part[(size_t)q * a.Cout + co];
  dot = wave_sum(dot);
  r = wave_sum(r);
  if ((tid & 63) == 0) { red[2 * (tid >> 6)] = dot; red[2 * (tid >> 6) + 1] = r; }
  __syncthreads();
  if (tid == 0 && live) {
    dot = 0.f;
    r = 0.f;
    for (int l = 0; l < nthr >> 6; ++l) { dot += red[2 * l]; r += red[2 * l + 1]; }
    a.dbeta[co] = r;
    a.dgamma[co] = (dot + r * (bc - mu)) / sd;
    if (a.db) a.db[co] = s * r;
  }
}

// An input gradient launched behind the weight gradient takes the fold-back along, on workgroups of its own behind the product's:
// they find the compute units that the product leaves idle, or that its first tiles have left, and the fold-back is no launch
// (4 - 5 us; a pass: 256 -> 64 channels at 56 x 56, 32 images 46.8 -> 43.8 us, at 46 x 40, 13 images 23.5 -> 19.5; 3 -> 32, 3 x 3
// / 2 at 172 x 172, 17 images 34.5 -> 29.4).  A workgroup of `threads` takes as many channels as leave a thread about sixteen loads.
constexpr int FOLD_BACK_SIDE_BYTES(int threads) { return threads * 16 + threads / 64 * 8; }
inline int fold_back_side_threads(int K, int nsplit, int threads) {   // of a channel
  const long long loads = (long long)ceil_div(K, 4) * nsplit;
  int per = 64;
  while (per < threads && loads > 16LL * per) per *= 2;
  return per;
}
inline int fold_back_side_blocks(int K, int nsplit, int Cout, int threads) {
  return ceil_div(Cout, threads / fold_back_side_threads(K, nsplit, threads));
}
inline int fold_back_side_blocks(FoldBackArgs& a, int threads) {
  a.per = fold_back_side_threads(a.K, a.nsplit, threads);
  return ceil_div(a.Cout, threads / a.per);
}
// smem: FOLD_BACK_SIDE_BYTES(THREADS)
template <int THREADS, RowKind ROW = ROW_VEC, int FLIGHT = 16, int COLS = 4>
__device__ __forceinline__ void fold_back_side(const FoldBackArgs& a, int wg, unsigned char* smem) {
  const int group = (int)threadIdx.x / a.per, tid = (int)threadIdx.x - group * a.per;
  float4* const red4 = reinterpret_cast<float4*>(smem);
  float* const red = reinterpret_cast<float*>(smem + THREADS * 16);
  fold_back_row<bf16_t, FLIGHT, COLS, ROW>(a, wg * (THREADS / a.per) + group, tid, a.per, red4 + group * a.per, red + group * (a.per >> 5));
}

}  // namespace convbn
