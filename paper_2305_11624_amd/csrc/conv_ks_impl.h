// The window product (conv_win_impl.h) for few pixels: small tiles whose reduction is split over the eight waves of a
// workgroup.  Forward and input gradient, any window, stride and channel counts that are multiples of 8; the problem's
// description, the residue classes of a strided input gradient and what rides behind the product are that file's.
//
// What bounds the layers it is for.  A 3 x 3 layer with 512 -> 512 channels over 8 images of 6 x 6 pixels has eighteen
// 128 x 64 tiles, each a chain of 72 chunks of 24 KB that one compute unit copies, at about 50 bytes a clock, one barrier after
// the other: 25 us, with most of the chip idle.  A TM x TN tile needs (TM + TN) K elements copied, and the copies of all
// tiles run at once as long as there are no more tiles than compute units: 32 x 32 tiles are a third of the chain each, on eight
// times the compute units.  Small tiles have too little work per chunk to share it, so each wave takes every eighth chunk for
// itself: it copies the chunk global -> LDS into memory of its own (8 rows x 128 bytes per instruction, granules
// permuted by (row / 2) % 8 as in conv_win_impl.h), reads the operands, asks for its next chunk and multiplies.  No
// barrier in the loop: a wave waits for its own copies only, and while it does the others copy.  The eight sums meet in
// LDS, always in the same order.  (A second chunk per wave in LDS: 32 x 32 tiles, the same time, and one workgroup per compute
// unit instead of two.)
//
// Forward, us (before: 128 x 64 tiles, or the LDS-tile kernel's split sums and a fold launch; in brackets the tile):
//   3 x 3, 512 -> 512 at 6 x 6, 8 images      21.3 ->  8.9 (32 x 32)     3 x 3 / 2, 512 -> 512 at 6 x 6, 4 images  25.3 ->  8.4 (32 x 32)
//   3 x 3, 512 -> 512 at 7 x 7, 20 images     25.0 -> 12.1 (64 x 32)     3 x 3, 256 -> 256 at 18 x 18, 1 image    15.2 ->  6.2 (32 x 32)
//   1 x 1, 2048 -> 512 at 9 x 9, 3 images     13.2 ->  6.1 (32 x 32)     3 x 3, 72 -> 136 at 27 x 33, 5 images      8.3 ->  6.8 (64 x 64)
// A chunk of a 64 x 64 tile takes 0.127 us (36 and 72 of them, ks_us below) for its 16 KB, some 62 bytes a clock at 2.1 GHz: what a
// compute unit's copies get out of the L2.
#pragma once
#include "conv_win_impl.h"

namespace convbn {
namespace win {

template <int TM, int TN>
struct KsCfg {
  static constexpr int AU = TM / 8, WU = TN / 8;                     // copies of a chunk: activation rows, weight rows
  static constexpr int NPS = TM / 32, NCS = TN / 32;
  static constexpr int STAGE = (TM + TN) * 128;                      // a wave's chunk, and its sums afterwards
  static constexpr int OFF_BIAS = NWAVES * STAGE;                    // [TN] bias, [TN] scale
  static constexpr int LDS_BYTES = OFF_BIAS + 2 * TN * 4;
  static constexpr int GRANULES = TM * TN / 8;                       // 16-byte stores of a tile, one a thread
  static_assert(TM * TN * 4 <= STAGE && GRANULES <= 64 * NWAVES, "a wave's sums take the place of its chunks");
  static_assert(2 * FOLD_TILE_BYTES <= LDS_BYTES && FOLD_BACK_SIDE_BYTES(64 * NWAVES) <= LDS_BYTES && 2 * FBT_SMEM <= LDS_BYTES, "what folds on the side");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS of a compute unit");
  static constexpr int SHARED = shared_cu(LDS_BYTES), WAVES_SIMD = SHARED ? NWAVES / 2 : NWAVES / 4;
};

template <int TM, int TN, class Side>
__device__ __forceinline__ void ks_body(const WnParams& p, const Side& side, const int wg, unsigned char* smem) {
  using Cfg = KsCfg<TM, TN>;
  constexpr int AU = Cfg::AU, WU = Cfg::WU, NPS = Cfg::NPS, NCS = Cfg::NCS, STAGE = Cfg::STAGE;
  if (wg >= p.nconv) {
    if constexpr (Side::BACK) fold_back_aside<Cfg::SHARED>(side, wg - p.nconv, smem);
    else fold_side(p.bn, p.wgt, wg - p.nconv, smem);
    return;
  }
  float* biasl = reinterpret_cast<float*>(smem + Cfg::OFF_BIAS);
  const int k = class_of(p, wg);
  const Window cv = p.c[k].cv;
  const FastDiv dHW = p.c[k].dHW, dW = p.c[k].dW;
  const int M = p.c[k].M, nchunks = p.c[k].nchunks;
  const int block = wg - p.c[k].first;
  if (nchunks == 0) {
    store_untapped(p, k, block);
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int r0, m0;
  if (!tile_of<TM, TN>(p, k, block, r0, m0)) return;
  const __amdgpu_buffer_rsrc_t act_rsrc = make_rsrc(p.act, p.act_bytes);
  const __amdgpu_buffer_rsrc_t wgt_rsrc = make_rsrc(p.wgt, p.wgt_bytes);
  if (tid < TN) bias_and_scale<TN>(p, r0, tid, biasl);

  // ---- the output this thread stores: granule og (8 channels) of pixel opx of the tile; its addend and mask are requested here
  const int opx = tid % TM, og = tid / TM;
  const unsigned hw = (unsigned)(cv.oHo * cv.oWo);
  long long out_at = -1;
  if (og < TN / 8 && m0 + opx < M && r0 + og * 8 < p.R) {
    const int m = m0 + opx, ch = r0 + og * 8;
    if (!cv.out_strided) {
      out_at = (long long)m * p.R + ch;
    } else {
      const unsigned n = fdiv((unsigned)m, dHW), rem = (unsigned)m - n * hw;
      const unsigned ho = fdiv(rem, dW), wo = rem - ho * (unsigned)cv.oWo;
      out_at = (long long)cv.out_base + (long long)n * cv.out_n + (long long)ho * cv.out_h + (long long)wo * cv.out_w + ch;
    }
  }
  uint4 addv = make_uint4(0u, 0u, 0u, 0u), maskv = addv;
  if (p.add && out_at >= 0) addv = *reinterpret_cast<const uint4*>(p.add + out_at);
  if (p.mask && out_at >= 0) maskv = *reinterpret_cast<const uint4*>(p.mask + out_at);
  asm volatile("" ::: "memory");

  // ---- copies: unit j covers rows 8 j .. 8 j + 7; lane l writes LDS granule l % 8 of row 8 j + l / 8 and fetches the granule
  // that belongs there, (l % 8) ^ key(row), key = (row / 2) % 8: one for even j, its fourth neighbour for odd j
  const int crow = lane >> 3;
  unsigned base_a[AU], base_w[WU];
  int cv_h[AU], cv_w[AU];   // window origin of the row's pixel
#pragma unroll
  for (int j = 0; j < AU; ++j) {
    const int row = 8 * j + crow;
    const unsigned m = (unsigned)min(m0 + row, M - 1);
    const unsigned n = fdiv(m, dHW), rem = m - n * hw;
    const unsigned ho = fdiv(rem, dW), wo = rem - ho * (unsigned)cv.oWo;
    cv_h[j] = m0 + row < M ? (int)ho * cv.csh - cv.cph : -(1 << 20);   // rows past the last pixel: never inside the grid
    cv_w[j] = (int)wo * cv.csw - cv.cpw;
    base_a[j] = (n * (unsigned)cv.a_n + (unsigned)cv_h[j] * (unsigned)cv.a_h + (unsigned)cv_w[j] * (unsigned)cv.a_w) * 2u;
  }
#pragma unroll
  for (int j = 0; j < WU; ++j) {
    const int row = r0 + 8 * j + crow;
    base_w[j] = row < p.R ? (unsigned)row * (unsigned)cv.wrow * 2u : OOB;
  }
  // the granules (tap, eight channels) of the chunk to be issued next, for even and odd units; a wave's next chunk is 64 further
  const int C8 = p.C >> 3;
  int f_c[2], f_i[2], f_j[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int g = wave * 8 + ((lane & 7) ^ (crow >> 1) ^ (q << 2));
    const int t = g / C8;
    f_c[q] = g - t * C8;
    f_i[q] = t / cv.kW;
    f_j[q] = t - f_i[q] * cv.kW;
  }
  const int step_t = 64 / C8, s_c = 64 - step_t * C8, s_i = step_t / cv.kW, s_j = step_t - s_i * cv.kW;
  unsigned char* const mine = smem + wave * STAGE;
  auto issue_chunk = [&]() {
    unsigned off_a[2], off_w[2];
    bool in[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      in[q] = f_i[q] < cv.kH;
      off_a[q] = (unsigned)((f_i[q] * cv.a_h + f_j[q] * cv.a_w + f_c[q] * 8) * 2);
      off_w[q] = (unsigned)(((cv.wt0 + f_i[q] * cv.wt_row + f_j[q] * cv.wt_col) * p.C + f_c[q] * 8) * 2);
    }
#pragma unroll
    for (int j = 0; j < AU; ++j) {
      const int q = j & 1;
      const bool ok = in[q] && (unsigned)(cv_h[j] + f_i[q]) < (unsigned)cv.aH && (unsigned)(cv_w[j] + f_j[q]) < (unsigned)cv.aW;
      dma16(act_rsrc, ok ? base_a[j] + off_a[q] : OOB, 0u, mine + j * 1024);
    }
#pragma unroll
    for (int j = 0; j < WU; ++j) {
      const int q = j & 1;
      dma16(wgt_rsrc, in[q] && base_w[j] != OOB ? base_w[j] + off_w[q] : OOB, 0u, mine + TM * 128 + j * 1024);
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      f_c[q] += s_c; f_j[q] += s_j; f_i[q] += s_i;
      if (f_c[q] >= C8) { f_c[q] -= C8; ++f_j[q]; }
      if (f_j[q] >= cv.kW) { f_j[q] -= cv.kW; ++f_i[q]; }
    }
  };

  // ---- operands: row l % 32 of a subtile, granule 2 kk + l / 32 of the chunk, at position (2 kk) ^ (l / 32 ^ key)
  const int kb = lane >> 5, rl = lane & 31;
  const unsigned lane_off = (unsigned)(rl * 128 + (((kb ^ ((rl >> 1) & 7)) & 7) << 4));
  f32x16 acc[NCS][NPS];
#pragma unroll
  for (int i = 0; i < NCS; ++i)
#pragma unroll
    for (int ps = 0; ps < NPS; ++ps)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][ps][e] = 0.f;

  const int mychunks = (nchunks - wave + NWAVES - 1) / NWAVES;   // chunks wave, wave + 8, ...
  if (mychunks > 0) issue_chunk();
  for (int t = 0; t < mychunks; ++t) {
    wait_vm<0>();
    bf16x8 fa[KK][NCS], fb[KK][NPS];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
#pragma unroll
      for (int ps = 0; ps < NPS; ++ps) fb[kk][ps] = *reinterpret_cast<const bf16x8*>(mine + ps * 4096 + (lane_off ^ (unsigned)(kk << 5)));
#pragma unroll
      for (int i = 0; i < NCS; ++i) fa[kk][i] = *reinterpret_cast<const bf16x8*>(mine + TM * 128 + i * 4096 + (lane_off ^ (unsigned)(kk << 5)));
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the operands are in registers: their place can be filled again
    __builtin_amdgcn_sched_barrier(0);
    if (t + 1 < mychunks) issue_chunk();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
#pragma unroll
      for (int i = 0; i < NCS; ++i)
#pragma unroll
        for (int ps = 0; ps < NPS; ++ps) acc[i][ps] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kk][i], fb[kk][ps], acc[i][ps], 0, 0, 0);
  }

  // ---- sums.  Accumulator element e of lane l in subtile (i, ps): channel 32 i + 8 (e / 4) + 4 (l / 32) + e % 4, pixel
  // 32 ps + l % 32: four channels at a time, [subtile][e / 4][l]
  {
    float4* const red = reinterpret_cast<float4*>(mine);
#pragma unroll
    for (int i = 0; i < NCS; ++i)
#pragma unroll
      for (int ps = 0; ps < NPS; ++ps)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          red[((i * NPS + ps) * 4 + q) * 64 + lane] = make_float4(acc[i][ps][q * 4], acc[i][ps][q * 4 + 1], acc[i][ps][q * 4 + 2], acc[i][ps][q * 4 + 3]);
  }
  __syncthreads();
  if (out_at < 0) return;
  float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const int at = (((og >> 2) * NPS + (opx >> 5)) * 4 + (og & 3)) * 64 + (opx & 31);
#pragma unroll
  for (int w = 0; w < NWAVES; ++w) {
    const float4* const red = reinterpret_cast<const float4*>(smem + w * STAGE);
    const float4 lo = red[at], hi = red[at + 32];
    v[0] += lo.x; v[1] += lo.y; v[2] += lo.z; v[3] += lo.w;
    v[4] += hi.x; v[5] += hi.y; v[6] += hi.z; v[7] += hi.w;
  }
  const float* const bb = biasl + og * 8;
  const float* const sc = bb + TN;
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = fmaf(v[e], sc[e], bb[e]);
  uint4 o = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
  if (p.add) o = add8(o, addv);
  if (p.relu) o = relu8(o);
  if (p.mask) o = mask8(o, maskv);
  *reinterpret_cast<uint4*>(p.out + out_at) = o;
}

// An estimate of a laid-out launch of one round: a fixed part and what a chunk's copies take.  Fitted to launches of 4 to 72
// chunks: 32 x 32 4.2, 6.2, 8.9 us with 4, 36, 72; 64 x 32 7.8, 11.3 with 36, 72; 64 x 64 9.7, 14.3.
inline float ks_us(int tm, int tn, const WnParams& p) {
  int chunks = 0;
  for (int i = 0; i < p.ncls; ++i) chunks = p.c[i].nchunks > chunks ? p.c[i].nchunks : chunks;
  return tm == 32 ? 3.4f + 0.077f * chunks : tn == 32 ? 4.3f + 0.098f * chunks : 5.2f + 0.127f * chunks;
}

}  // namespace win
}  // namespace convbn
