// The fold-back of a transposed block by workgroups of 256 threads, or by the halves of a workgroup of 512 that rides in
// another launch: dW = s dw' from the partial copies, a row of partial <dw', w> per workgroup, and dZ's column sums.
#pragma once
#include "fold_tile.h"

namespace convbn {

// W is rows = Ci taps rows of Co columns.  kind: FBT_ROWS_2 / _8: rows of a wave; FBT_SPLIT_16 / _64: column groups whose copies
// the threads share (fold_t.hip says when)
enum { FBT_ROWS_2, FBT_ROWS_8, FBT_SPLIT_16, FBT_SPLIT_64 };
// The first rs.blocks workgroups (bf16 with Co % 8 == 0, Co <= 2048; else none, and a launch before this one)
// sum dZ's columns: that reads dZ while the others read the copies, and needs nothing of theirs.  512 -> 256 channels, 4 x 4,
// 14 x 14, 32 images: 7.8 us, 38 MB (the sums in a launch of their own: 6.3 + 7.3).
struct RSum { const uint4* dz; float* part; int M, rows, blocks; };
struct FoldBackTArgs {
  static constexpr bool BACK = true;
  RSum rs;
  const float* part; const void* W; const float* gamma; const float* var;
  void* dW; float* dot_part;
  float eps;
  int nsplit, rows, Co, ncol, cw, kind;
  int blocks;   // of the fold-back, behind rs.blocks
};
constexpr int FBT_SMEM = 256 * 9 * 4;
__device__ __forceinline__ void fbt_colsum(const RSum& rs, int Co, int block, int tid, unsigned char* smem) {
  const int m0 = block * rs.rows;
  colsum_slice_bf16x8(rs.dz, m0, min(rs.M, m0 + rs.rows), Co, tid, reinterpret_cast<float (*)[9]>(smem), rs.part + (size_t)block * Co);
}

// A wave owns RW rows of its workgroup's 4 RW, UN copies of them all asked for at once, and a lane four consecutive columns.
template <typename T, int RW, int UN>
__device__ __forceinline__ void fbt_rows(const FoldBackTArgs& a, int block, int tid, bool live, unsigned char* smem) {
  const float* const part = a.part; const T* const W = static_cast<const T*>(a.W); T* const dW = static_cast<T*>(a.dW);
  const float* const gamma = a.gamma;
  const int nsplit = a.nsplit, rows = a.rows, Co = a.Co;
  const int bx = block % a.ncol, by = block / a.ncol;
  const int lane = tid & 63, wave = tid >> 6;
  const int col = bx * 256 + lane * 4;
  const int r0 = by * 4 * RW + wave;   // and every fourth row behind it
  const size_t P = (size_t)rows * Co;
  float dot[4] = {0.f, 0.f, 0.f, 0.f};
  if (col < Co && r0 < rows) {
    size_t at[RW];
    bool in[RW];
    float w[RW][4], dw[RW][4] = {};
    float s[4] = {1.f, 1.f, 1.f, 1.f}, v[4] = {1.f, 1.f, 1.f, 1.f};   // no gamma: plain sum
    if (gamma) { fb_load4(gamma + col, s); fb_load4(a.var + col, v); }
#pragma unroll
    for (int i = 0; i < RW; ++i) {
      in[i] = r0 + 4 * i < rows;
      at[i] = (size_t)(in[i] ? r0 + 4 * i : r0) * Co + col;
      fb_load4(W + at[i], w[i]);
    }
#pragma unroll UN
    for (int sp = 0; sp < nsplit; ++sp)
#pragma unroll
      for (int i = 0; i < RW; ++i) {
        const float4 t = *reinterpret_cast<const float4*>(part + sp * P + at[i]);
        dw[i][0] += t.x; dw[i][1] += t.y; dw[i][2] += t.z; dw[i][3] += t.w;
      }
    if (gamma)
#pragma unroll
      for (int e = 0; e < 4; ++e) s[e] /= sqrtf(v[e] + a.eps);
#pragma unroll
    for (int i = 0; i < RW; ++i) {
      if (!in[i] || !live) continue;
      float o[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) { o[e] = s[e] * dw[i][e]; dot[e] += dw[i][e] * w[i][e]; }
      fb_store4(dW + at[i], o);
    }
  }
  if (!a.dot_part) return;
  float* const sum = reinterpret_cast<float*>(smem);   // [wave][256]
#pragma unroll
  for (int e = 0; e < 4; ++e) sum[wave * 256 + lane * 4 + e] = dot[e];
  __syncthreads();
  const int c = tid, co = bx * 256 + c;
  if (live && co < Co) a.dot_part[(size_t)by * Co + co] = sum[c] + sum[256 + c] + sum[512 + c] + sum[768 + c];
}

// Thread -> column group el (of EL / cw rows, cw columns of four each) and every (256 / EL)-th partial copy.
template <typename T, int EL>
__device__ __forceinline__ void fbt_split(const FoldBackTArgs& a, int block, int tid, bool live, unsigned char* smem) {
  constexpr int SL = 256 / EL;
  struct Red { float copy[SL][EL * 4], dot[EL * 4]; };
  static_assert(sizeof(Red) <= FBT_SMEM, "LDS of 256 threads");
  struct { Red& s; } red{*reinterpret_cast<Red*>(smem)};
  const float* const part = a.part; const T* const W = static_cast<const T*>(a.W); T* const dW = static_cast<T*>(a.dW);
  const float* const gamma = a.gamma;
  const int nsplit = a.nsplit, rows = a.rows, Co = a.Co, cw = a.cw;
  const int bx = block % a.ncol, by = block / a.ncol;
  const int nr = EL / cw;
  const size_t P = (size_t)rows * Co;
  // element `el` of the workgroup: its offset in a copy (one inside where there is none) and whether there is one
  auto element = [&](int el, size_t& at) {
    const int rr = el / cw, row = by * nr + rr, c = (bx * cw + el - rr * cw) * 4;
    const bool in = rr < nr && row < rows && c < Co;
    at = in ? (size_t)row * Co + c : 0;
    return in;
  };
    // the element this thread finishes: column e of group fe
  const int fe = tid >> 2, fc = (bx * cw + fe % cw) * 4 + (tid & 3);
  size_t fat = 0;
  const bool fin = live && tid < EL * 4 && element(fe, fat);
  fat += tid & 3;
  const float fw = fin ? to_f32(W[fat]) : 0.f;
  const float fg = fin && gamma ? gamma[fc] : 1.f, fv = fin && gamma ? a.var[fc] : 1.f;
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
    if (fin) dW[fat] = from_f32<T>(gamma ? fg / sqrtf(fv + a.eps) * dw : dw);
    red.s.dot[tid] = fin ? dw * fw : 0.f;
  }
  if (!a.dot_part) return;
  __syncthreads();
  if (!fin || fe >= cw) return;
  float dot = 0.f;
  for (int rr = 0; rr < nr; ++rr) dot += red.s.dot[rr * cw * 4 + tid];
  a.dot_part[(size_t)by * Co + fc] = dot;
}


// block of the fold-back proper, by 256 threads; UN copies of eight rows in flight a thread; !live: nothing is stored
template <typename T, int UN>
__device__ __forceinline__ void fbt_block(const FoldBackTArgs& a, int block, int tid, bool live, unsigned char* smem) {
  if (a.kind == FBT_ROWS_2) fbt_rows<T, 2, 4>(a, block, tid, live, smem);
  else if (a.kind == FBT_ROWS_8) fbt_rows<T, 8, UN>(a, block, tid, live, smem);
  else if (a.kind == FBT_SPLIT_16) fbt_split<T, 16>(a, block, tid, live, smem);
  else fbt_split<T, 64>(a, block, tid, live, smem);
}

// Along with the block's input gradient (a convolution of dZ), as fold_back_side in fold_tile.h: workgroup `wg` of 512 threads
// takes two blocks, both of the column sums or both of the fold-back (the halves meet at the same barriers); where
// there is an odd one the second half only meets the barriers and stores nothing (dW may take the place of W, which the first half
// still reads then).  bf16.  FLIGHT as there.  smem: 2 FBT_SMEM.
inline int fold_back_side_blocks(const FoldBackTArgs& a, int) { return ceil_div(a.rs.blocks, 2) + ceil_div(a.blocks, 2); }
template <int THREADS, RowKind, int FLIGHT, int>
__device__ __forceinline__ void fold_back_side(const FoldBackTArgs& a, int wg, unsigned char* smem) {
  static_assert(THREADS == 512, "two halves");
  const int half = (int)threadIdx.x >> 8, tid = (int)threadIdx.x & 255, sums = (a.rs.blocks + 1) >> 1;
  unsigned char* const mine = smem + half * FBT_SMEM;
  if (wg < sums) {
    fbt_colsum(a.rs, a.Co, min(2 * wg + half, a.rs.blocks - 1), tid, mine);
  } else {
    const int block = 2 * (wg - sums) + half;
    fbt_block<bf16_t, FLIGHT < 16 ? 1 : 4>(a, min(block, a.blocks - 1), tid, block < a.blocks, mine);
  }
}

}  // namespace convbn
