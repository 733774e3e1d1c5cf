// bf16 convolution as a tiled matrix product, any window: the activation rows of every tap are gathered per output pixel
// (no window tile in LDS),
//     out[m][r] = sum_{tap, c} act[row(m, tap)][c] wgt[r][tap][c] (+ bias[r]),     m over the output pixels,
// for the layers the other kernels have no tile for: strided windows (which hardly overlap, so a window tile would buy
// little), channel counts that are no multiple of 32 or 64, and few pixels.  Forward and input gradient, like conv_gm.hip,
// whose pipeline this is: chunks of 64 reduced channels copied global -> LDS (1 KB per instruction: 8 rows x 128 bytes,
// granules permuted by (row / 2) % 8) into a ring, one barrier per chunk, eight waves on a TM pixel x TN channel tile.
//
// What is particular here:
//  * One launch runs up to four problems that share the operands: the residue classes of input positions of a strided
//    input gradient (each a stride-1 window with a subset of the taps), the longest reduction first.  A class that no
//    tap reaches is stored by workgroups of its own: the bias (an input gradient: zeros) and the post-operation.
//    (One launch per class: 128 channels at 34 x 34 / 2, 42 images: 4 x 7.0 us.)
//  * FLAT: the reduced index runs over (tap, channel) without a gap, 8 channels (one granule) at a time, so a layer with
//    72 channels does not multiply 56 zeros per tap.  A lane keeps the tap and the channels its next granule belongs to.
//  * The ring is three stages deep where several workgroups share a compute unit, six where one has it to itself: few
//    pixels, and the launch then lasts as long as one workgroup's chain of chunks, i.e. as long as its copies take.
//  * The weight's rows beyond R, and granules beyond the reduction, are zero-fill copies; R and C are multiples of 8.
//  * A forward launch given the unfolded weight applies s and b' in the epilogue and folds on the side (fold_tile.h).
#pragma once
#include "common.h"
#include "fold_back_t_tile.h"

namespace convbn {
namespace win {

constexpr int NWAVES = 8;
constexpr int CB = 64;                 // reduced channels per chunk
constexpr int KK = CB / 16;
constexpr unsigned OOB = 0x80000000u;  // beyond any buffer: the load returns zeros
constexpr int MAXC = 4;                // problems of a launch
constexpr int ZROWS = 16;              // 16-byte stores per thread of a workgroup that has no product to compute

struct FastDiv {   // exact n / d for 0 <= n < 2^31, without a branch: (hi(n mul) + n add) >> shr
  unsigned mul, shr, add;
};
inline FastDiv make_fastdiv(int d) {
  FastDiv f{0u, 0u, 1u};   // d = 1: n itself
  if (d <= 1) return f;
  f.add = 0u;
  unsigned s = 0;
  while ((1ull << (s + 1)) < (unsigned long long)d) ++s;   // 2^s < d <= 2^(s+1)
  f.shr = s;
  f.mul = (unsigned)((((unsigned long long)1 << (32 + s)) + d - 1) / d);
  return f;
}
__device__ __forceinline__ unsigned fdiv(unsigned n, const FastDiv& f) {
  return (__umulhi(n, f.mul) + n * f.add) >> f.shr;
}

// A kH x kW window slides with stride (csh, csw) and padding (cph, cpw) over an [N][aH][aW] activation grid with element
// strides a_n, a_h, a_w; output pixel (n, ho, wo) of an [N][oHo][oWo] grid is stored at element out_base + n out_n +
// ho out_h + wo out_w (out_strided) or at row m of a dense [M][R] tensor; window position (ti, tj) multiplies with tap
// wt0 + ti wt_row + tj wt_col of the weight tensor, whose rows (one per output channel) have wrow elements.
struct Window {
  int kH, kW, cph, cpw, csh, csw, aH, aW;
  int a_n, a_h, a_w;
  int oHo, oWo;
  int wt0, wt_row, wt_col, wrow;
  int out_strided, out_base, out_n, out_h, out_w;
};
struct WnClass {
  Window cv;
  int M, nchunks;
  int first;      // first workgroup
  FastDiv dHW, dW, dTiles;   // oHo oWo, oWo; pixel tiles (ORDER by channel) or channel tiles
};
struct WnParams {
  const bf16_t* act; const bf16_t* wgt; const float* bias;
  BnEpilogue bn;         // bn.gamma != null: the weight is unfolded, the epilogue applies s and b' (bias unused)
  bf16_t* out;
  const bf16_t* mask; const bf16_t* add;   // laid out like the output, or null
  int relu;
  unsigned act_bytes, wgt_bytes;
  int C, R, ntr;         // ntr: channel tiles
  int by_channel;        // which operand an XCD keeps to itself, see the kernel
  int ncls, nconv;       // nconv: the convolution's workgroups, those behind it fold, or fold back
  WnClass c[MAXC];
};

typedef __attribute__((address_space(3))) void* lds_ptr_t;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
// 1 KB copy: lane l fetches 16 bytes at voff (per lane, range-checked) + soff (wave-uniform) and writes them to LDS
// at lds_wave_base + 16 l.  The compiler barrier keeps every copy in the instruction stream: the waits count copies.
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t rsrc, unsigned voff, unsigned soff, void* lds_wave_base) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr_t)lds_wave_base, 16, (int)voff, (int)soff, 0, 0);
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void block_barrier() {   // no memory fence: that would drain the copies
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
template <int N> __device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit field");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Tiles whose LDS leaves room for a second workgroup on the compute unit leave it the registers too, at most 128 a lane: what folds
// back on the side then has fewer loads in flight.  (With the 16 and 4 of the larger tiles such kernels had 162 to 168 registers and
// a compute unit to each workgroup, in an input gradient of thousands of them: 3 x 3 / 2, 64 -> 64 at 112 x 112, 64 images 152.5 us
// a pass, 129.7 like this; at 56 x 56, 128 images 86.2, 73.8; transposed 4 x 4 / 2, 64 -> 32 at 56 x 56, 32 images 81.6, 71.2.)
constexpr bool shared_cu(int lds) { return 2 * lds <= 160 * 1024; }
template <bool SHARED, class Side>
__device__ __forceinline__ void fold_back_aside(const Side& side, int wg, unsigned char* smem) {
  fold_back_side<64 * NWAVES, ROW_VEC, SHARED ? 8 : 16, SHARED ? 2 : 4>(side, wg, smem);
}

template <int TM, int TN, int NST>
struct WnCfg {
  static constexpr int CW = TN / 2;                     // channels per wave
  static constexpr int NPS = TM / 128;                  // 32-pixel subtiles per wave
  static constexpr int NCS = CW / 32;                   // 32-channel subtiles per wave
  static constexpr int AUW = TM / 8 / NWAVES;           // activation copies (8 rows each) per wave and chunk
  static constexpr int WUW = TN / 8 / NWAVES;           // weight copies per wave and chunk
  static constexpr int CPW = AUW + WUW;
  static constexpr int STAGE = (TM + TN) * 128;
  static constexpr int OFF_BIAS = NST * STAGE;          // [TN] bias, [TN] scale
  static constexpr int LDS_BYTES = OFF_BIAS + 2 * TN * 4;
  static_assert(NWAVES * 32 * CW * 2 <= STAGE * NST, "the epilogue stages every wave's outputs in the ring");
  static_assert(2 * FOLD_TILE_BYTES <= LDS_BYTES && FOLD_BACK_SIDE_BYTES(64 * NWAVES) <= LDS_BYTES && 2 * FBT_SMEM <= LDS_BYTES, "what folds on the side");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS of a compute unit");
  static constexpr int SHARED = shared_cu(LDS_BYTES), WAVES_SIMD = SHARED ? NWAVES / 2 : NWAVES / 4;
};

// ---- what a workgroup is for
__device__ __forceinline__ int class_of(const WnParams& p, int wg) {
  int k = 0;
#pragma unroll
  for (int i = 1; i < MAXC; ++i)
    if (i < p.ncls && wg >= p.c[i].first) k = i;
  return k;
}
// Positions that no tap reaches: block `block` of a class stores their rows, 16 bytes at a time.
__device__ __forceinline__ void store_untapped(const WnParams& p, int k, int block) {
  const Window cv = p.c[k].cv;
  const int R8 = p.R >> 3;
  const unsigned hw = (unsigned)(cv.oHo * cv.oWo), total = (unsigned)p.c[k].M * (unsigned)R8;
  for (int e = 0; e < ZROWS; ++e) {
    const unsigned i = ((unsigned)block * ZROWS + e) * (64 * NWAVES) + threadIdx.x;
    if (i >= total) break;
    const unsigned m = i / (unsigned)R8, ch = (i - m * R8) * 8;
    const unsigned n = fdiv(m, p.c[k].dHW), rem = m - n * hw;
    const unsigned ho = fdiv(rem, p.c[k].dW), wo = rem - ho * (unsigned)cv.oWo;
    const size_t o = (size_t)cv.out_base + (size_t)n * cv.out_n + (size_t)ho * cv.out_h + (size_t)wo * cv.out_w + ch;
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (p.bias) {
      const float* b = p.bias + ch;
      v = make_uint4(pack_bf16x2(b[0], b[1]), pack_bf16x2(b[2], b[3]), pack_bf16x2(b[4], b[5]), pack_bf16x2(b[6], b[7]));
    }
    *reinterpret_cast<uint4*>(p.out + o) = post_op8(v, p.relu, p.mask, p.add, o);
  }
}
// Workgroups are handed to the eight XCDs in turn (id % 8), and each XCD has its own L2, which what its workgroups share
// should fit: the tiles are split into eight contiguous runs, along the channels where the weight is the larger operand
// (an XCD then reads its channel tiles' rows and all activations), else along the pixels.  False: none left for this one.
template <int TM, int TN>
__device__ __forceinline__ bool tile_of(const WnParams& p, int k, int block, int& r0, int& m0) {
  const int npt = (p.c[k].M + TM - 1) / TM, ntiles = npt * p.ntr;
  const int tile = (block & 7) * ((ntiles + 7) >> 3) + (block >> 3);
  if (tile >= min(ntiles, ((block & 7) + 1) * ((ntiles + 7) >> 3))) return false;
  const int q = (int)fdiv((unsigned)tile, p.c[k].dTiles);
  const int ptile = p.by_channel ? tile - q * npt : q, ctile = p.by_channel ? q : tile - q * p.ntr;
  r0 = ctile * TN;
  m0 = ptile * TM;
  return true;
}
// bias and scale of channel r0 + c of a tile
template <int TN>
__device__ __forceinline__ void bias_and_scale(const WnParams& p, int r0, int c, float* biasl) {
  const int ch = min(r0 + c, p.R - 1);
  float bias_v = p.bias ? p.bias[ch] : 0.f, scale_v = 1.f;
  if (p.bn.gamma) {   // Z = s (w (*) X) + b' (Sec. 3.3), s and b' worked out here
    scale_v = p.bn.gamma[ch] / sqrtf(p.bn.var[ch] + p.bn.eps);
    bias_v = ((p.bn.b ? p.bn.b[ch] : 0.f) - p.bn.mean[ch]) * scale_v + p.bn.beta[ch];
  }
  biasl[c] = bias_v;
  biasl[TN + c] = scale_v;
}

// Workgroup `wg` of the product (and, behind its workgroups, of the fold or the fold-back on the side); smem: WnCfg::LDS_BYTES
template <int TM, int TN, int NST, bool FLAT, class Side>
__device__ __forceinline__ void body(const WnParams& p, const Side& side, const int wg, unsigned char* smem) {
  using Cfg = WnCfg<TM, TN, NST>;
  constexpr int CW = Cfg::CW;
  constexpr int GR = CW / 8;          // 16-byte granules of a wave's staged output row
  constexpr int RPI = 64 / GR;        // rows one store instruction covers
  constexpr int ITS = 32 / RPI;       // store instructions per 32-pixel subtile
  constexpr int NPS = Cfg::NPS, NCS = Cfg::NCS, AUW = Cfg::AUW, WUW = Cfg::WUW, CPW = Cfg::CPW, STAGE = Cfg::STAGE;
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
  const int block = wg - p.c[k].first;   // (a class starts at a multiple of eight)

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;      // pixel group, channel group
  if (nchunks == 0) {
    store_untapped(p, k, block);
    return;
  }
  int r0, m0;
  if (!tile_of<TM, TN>(p, k, block, r0, m0)) return;
  const __amdgpu_buffer_rsrc_t act_rsrc = make_rsrc(p.act, p.act_bytes);
  const __amdgpu_buffer_rsrc_t wgt_rsrc = make_rsrc(p.wgt, p.wgt_bytes);

  if (tid < TN) bias_and_scale<TN>(p, r0, tid, biasl);

  // ---- copies of this wave: unit u covers rows 8 u .. 8 u + 7 of its tile; lane l writes LDS granule l % 8 of row
  // 8 u + l / 8 and fetches the granule that belongs there, (l % 8) ^ key(row), key = (row / 2) % 8: u = wave + 8 j, so
  // a lane fetches the same granule of every row it copies
  const int crow = lane >> 3;
  const int gr = (lane & 7) ^ ((wave * 4 + (crow >> 1)) & 7);
  unsigned voff_a[AUW], voff_w[WUW];
  int cv_h[AUW], cv_w[AUW];   // the row's window origin (h, w of window position (0, 0)); voff_a holds its image
  const unsigned hw = (unsigned)(cv.oHo * cv.oWo);
#pragma unroll
  for (int j = 0; j < AUW; ++j) {
    const int row = (wave + NWAVES * j) * 8 + crow;
    const unsigned m = (unsigned)min(m0 + row, M - 1);
    const unsigned n = fdiv(m, dHW), rem = m - n * hw;
    const unsigned ho = fdiv(rem, dW), wo = rem - ho * (unsigned)cv.oWo;
    cv_h[j] = m0 + row < M ? (int)ho * cv.csh - cv.cph : -(1 << 20);   // rows past the last pixel: never inside the grid
    cv_w[j] = (int)wo * cv.csw - cv.cpw;
    voff_a[j] = n * (unsigned)cv.a_n * 2u;
  }
#pragma unroll
  for (int j = 0; j < WUW; ++j) {
    const int row = r0 + (wave + NWAVES * j) * 8 + crow;
    voff_w[j] = row < p.R ? (unsigned)row * (unsigned)cv.wrow * 2u : OOB;
  }
  // the step whose copies are issued next.  FLAT: per lane, its granule's channels (in eights) and tap; else uniform,
  // chunk and tap
  const int C8 = p.C >> 3;
  const int cpt = (p.C + CB - 1) / CB;
  int f_k = 0, f_c = 0, f_i = 0, f_j = 0;
  int s_c = 0, s_i = 0, s_j = 0;
  if constexpr (FLAT) {
    const int t = gr / C8;
    f_c = gr - t * C8;
    f_i = t / cv.kW;
    f_j = t - f_i * cv.kW;
    const int st = 8 / C8;   // a chunk further: st taps and s_c eights
    s_c = 8 - st * C8;
    s_i = st / cv.kW;
    s_j = st - s_i * cv.kW;
  }
  // offsets of this lane's granule of every row in the step to be issued; not FLAT: the tap's, a chunk adds to the
  // instruction's scalar offset (no part of the range check, so OOB stays OOB)
  unsigned cur_a[AUW], cur_w[WUW];
  auto enter_tap = [&]() {
    const int c = FLAT ? f_c * 8 : gr * 8;
    const bool tap_ok = !FLAT || f_i < cv.kH;
#pragma unroll
    for (int j = 0; j < AUW; ++j) {
      const int h = cv_h[j] + f_i, w = cv_w[j] + f_j;
      const bool ok = (unsigned)h < (unsigned)cv.aH && (unsigned)w < (unsigned)cv.aW && tap_ok;
      cur_a[j] = ok ? voff_a[j] + (unsigned)((h * cv.a_h + w * cv.a_w + c) * 2) : OOB;
    }
    const unsigned off = (unsigned)(((cv.wt0 + f_i * cv.wt_row + f_j * cv.wt_col) * p.C + c) * 2);
#pragma unroll
    for (int j = 0; j < WUW; ++j) cur_w[j] = tap_ok ? voff_w[j] + off : OOB;
  };
  enter_tap();
  auto issue_copy = [&](int i, unsigned char* stage) {
    const unsigned soff = FLAT ? 0u : (unsigned)(f_c * (CB * 2));
    if (i < AUW) dma16(act_rsrc, cur_a[i < AUW ? i : 0], soff, stage + (wave + NWAVES * i) * 1024);
    else dma16(wgt_rsrc, cur_w[i - AUW < WUW ? i - AUW : 0], soff, stage + TM * 128 + (wave + NWAVES * (i - AUW)) * 1024);
  };
  auto advance_fill = [&]() {       // to the step after it (the last step stays)
    if (f_k + 1 >= nchunks) return;
    ++f_k;
    if constexpr (FLAT) {
      f_c += s_c; f_j += s_j; f_i += s_i;
      if (f_c >= C8) { f_c -= C8; ++f_j; }
      if (f_j >= cv.kW) { f_j -= cv.kW; ++f_i; }
      enter_tap();
    } else {
      if (++f_c == cpt) {
        f_c = 0;
        if (++f_j == cv.kW) { f_j = 0; ++f_i; }
        enter_tap();
      }
    }
  };

  // ---- operand addresses: row l % 32 of a subtile, granule 2 kk + l / 32 of the chunk, which sits at position
  // (2 kk + kb) ^ key = (2 kk) ^ (kb ^ key); key depends on l % 32 only (subtiles start at multiples of 32 rows)
  const int kb = lane >> 5;
  const int rl = lane & 31;
  const unsigned lane_off = (unsigned)(rl * 128 + (((kb ^ ((rl >> 1) & 7)) & 7) << 4));
  unsigned boff[NPS], aoff[NCS];
#pragma unroll
  for (int ps = 0; ps < NPS; ++ps) boff[ps] = (unsigned)((wm * (32 * NPS) + ps * 32) * 128) + lane_off;
#pragma unroll
  for (int i = 0; i < NCS; ++i) aoff[i] = (unsigned)(TM * 128 + (wn * CW + i * 32) * 128) + lane_off;

  f32x16 acc[NCS][NPS];
#pragma unroll
  for (int i = 0; i < NCS; ++i)
#pragma unroll
    for (int ps = 0; ps < NPS; ++ps)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][ps][e] = 0.f;

  constexpr bool ONE = NCS * NPS == 1;   // one subtile per wave
  constexpr int FB = ONE ? KK : 2;       // k-steps whose operands are in registers
  bf16x8 fa[FB][NCS], fb[FB][NPS];
  auto load_frags = [&](int buf, const unsigned char* stage, int kk) {
#pragma unroll
    for (int ps = 0; ps < NPS; ++ps) fb[buf][ps] = *reinterpret_cast<const bf16x8*>(stage + (boff[ps] ^ (unsigned)(kk << 5)));
#pragma unroll
    for (int i = 0; i < NCS; ++i) fa[buf][i] = *reinterpret_cast<const bf16x8*>(stage + (aoff[i] ^ (unsigned)(kk << 5)));
  };

  // ---- the addend and the mask of this lane's outputs (see the epilogue for the lane -> output map) are requested
  // before the first copy, so that they arrive while the product runs instead of holding up every store
  auto out_off = [&](int ps, int it) -> long long {
    const int row = it * RPI + lane / GR;
    const int ch = r0 + wn * CW + ((lane % GR) ^ ((row >> 1) & (GR - 1))) * 8;
    const int m = m0 + wm * (32 * NPS) + ps * 32 + row;
    if (m >= M || ch >= p.R) return -1;
    if (!cv.out_strided) return (long long)m * p.R + ch;
    const unsigned n = fdiv((unsigned)m, dHW), rem = (unsigned)m - n * hw;
    const unsigned ho = fdiv(rem, dW), wo = rem - ho * (unsigned)cv.oWo;
    return (long long)cv.out_base + (long long)n * cv.out_n + (long long)ho * cv.out_h + (long long)wo * cv.out_w + ch;
  };
  uint4 addv[NPS][ITS], maskv[NPS][ITS];
  if (p.add || p.mask) {
#pragma unroll
    for (int ps = 0; ps < NPS; ++ps)
#pragma unroll
      for (int it = 0; it < ITS; ++it) {
        const long long o = out_off(ps, it);
        addv[ps][it] = (p.add && o >= 0) ? *reinterpret_cast<const uint4*>(p.add + o) : make_uint4(0u, 0u, 0u, 0u);
        maskv[ps][it] = (p.mask && o >= 0) ? *reinterpret_cast<const uint4*>(p.mask + o) : make_uint4(0u, 0u, 0u, 0u);
      }
    asm volatile("" ::: "memory");
  }

  // ---- prologue: NST - 1 chunks (a chunk past the end is the last one again, into a stage nobody reads)
#pragma unroll
  for (int s = 0; s < NST - 1; ++s) {
#pragma unroll
    for (int i = 0; i < CPW; ++i) issue_copy(i, smem + s * STAGE);
    advance_fill();
  }
  int st_cur = 0;   // stage of the current chunk
  for (int c = 0; c < nchunks; ++c) {
    wait_vm<CPW * (NST - 2)>();    // this chunk has landed (the later ones' copies may be in flight) ...
    block_barrier();   // ... for every wave, and everybody is done with the stage refilled below
    const unsigned char* const stage = smem + st_cur * STAGE;
    unsigned char* const fill = smem + (st_cur >= 1 ? st_cur - 1 : NST - 1) * STAGE;
    if constexpr (ONE) {
      // One subtile: the four multiplies of a chunk depend on each other and are all a wave has to hide behind, so the
      // chunk's operands are all requested first, then its copies, and the multiplies follow as the operands arrive.
      // (Interleaved as below, a chunk of a 72-chunk layer, 96 workgroups, took 1000 clocks.)
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) load_frags(kk, stage, kk);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < CPW; ++i) issue_copy(i, fill);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kk][0], fb[kk][0], acc[0][0], 0, 0, 0);
    } else {
      load_frags(0, stage, 0);
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        const int cur = kk & 1;
        if (kk + 1 < KK) load_frags(cur ^ 1, stage, kk + 1);
        __builtin_amdgcn_sched_barrier(0);
        // the copies of the chunk NST - 1 ahead, spread over the multiplies of this one
        constexpr int PER = (CPW + KK - 1) / KK;
        int issued = 0;
#pragma unroll
        for (int i = 0; i < NCS; ++i)
#pragma unroll
          for (int ps = 0; ps < NPS; ++ps) {
            acc[i][ps] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[cur][i], fb[cur][ps], acc[i][ps], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (issued < PER && kk * PER + issued < CPW) {
              issue_copy(kk * PER + issued, fill);
              ++issued;
              __builtin_amdgcn_sched_barrier(0);
            }
          }
#pragma unroll
        for (; issued < PER; ++issued)
          if (kk * PER + issued < CPW) issue_copy(kk * PER + issued, fill);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    st_cur = st_cur + 1 == NST ? 0 : st_cur + 1;
    advance_fill();
  }
  wait_vm<0>();      // trailing copies must not outlive the loop: the ring becomes the staging space
  __syncthreads();   // (and the bias is visible)

  // ---- epilogue.  Accumulator element e of lane l in subtile (i, ps): channel 32 i + 8 (e / 4) + 4 (l / 32) + e % 4,
  // pixel 32 ps + l % 32 of the wave's block.  Per 32-pixel subtile the wave rounds 32 pixels x CW channels to bf16
  // into its own 64 CW bytes ([pixel][CW ch], granules swizzled by pixel) and reads them back row-wise: every store is 16
  // bytes per lane, GR lanes cover one pixel's CW contiguous channels.
  unsigned char* const st = smem + wave * (32 * CW * 2);
  const int px = lane & 31, psw = (px >> 1) & (GR - 1);
#pragma unroll
  for (int ps = 0; ps < NPS; ++ps) {
#pragma unroll
    for (int i = 0; i < NCS; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int ch = i * 32 + q * 8 + kb * 4;
        const float4 bb = *reinterpret_cast<const float4*>(biasl + wn * CW + ch);
        const float4 sc = *reinterpret_cast<const float4*>(biasl + TN + wn * CW + ch);
        const uint2 v = make_uint2(pack_bf16x2(fmaf(acc[i][ps][q * 4 + 0], sc.x, bb.x), fmaf(acc[i][ps][q * 4 + 1], sc.y, bb.y)),
                                   pack_bf16x2(fmaf(acc[i][ps][q * 4 + 2], sc.z, bb.z), fmaf(acc[i][ps][q * 4 + 3], sc.w, bb.w)));
        *reinterpret_cast<uint2*>(st + px * (CW * 2) + (((ch >> 3) ^ psw) << 4) + ((ch & 7) << 1)) = v;
      }
#pragma unroll
    for (int it = 0; it < ITS; ++it) {
      const int row = it * RPI + lane / GR;
      uint4 v = *reinterpret_cast<const uint4*>(st + row * (CW * 2) + ((lane % GR) << 4));
      const long long o = out_off(ps, it);
      if (p.add) v = add8(v, addv[ps][it]);
      if (p.relu) v = relu8(v);
      if (p.mask) v = mask8(v, maskv[ps][it]);
      if (o >= 0) *reinterpret_cast<uint4*>(p.out + o) = v;
    }
  }
}

// Lays the workgroups of a launch out: fills ntr, nconv and the classes' chunks, first workgroups and divisors.
template <int TM, int TN, bool FLAT>
inline void lay_out(WnParams& p) {
  p.ntr = ceil_div(p.R, TN);
  int blocks = 0;
  for (int i = 0; i < p.ncls; ++i) {
    WnClass& c = p.c[i];
    const int steps = c.cv.kH * c.cv.kW, npt = ceil_div(c.M, TM);
    c.nchunks = FLAT ? ceil_div(steps * (p.C >> 3), CB / 8) : steps * ceil_div(p.C, CB);
    c.first = blocks;
    c.dHW = make_fastdiv(c.cv.oHo * c.cv.oWo);
    c.dW = make_fastdiv(c.cv.oWo);
    c.dTiles = make_fastdiv(p.by_channel ? npt : p.ntr);
    if (c.nchunks > 0) blocks += ceil_div(npt * p.ntr, 8) * 8;
    else blocks += (int)(((size_t)c.M * (p.R >> 3) + 64 * NWAVES * ZROWS - 1) / (64 * NWAVES * ZROWS) + 7) / 8 * 8;
  }
  p.nconv = blocks;
}

// The parameters of an input gradient whose residue classes fit one launch (no pointers); false: they do not.
bool dgrad_params(const Geom& g, WnParams* p);
// An estimate of the input gradient as a launch of its own, with a fold-back behind its workgroups where `back` (0: it has more
// residue classes than a launch takes).
float ks_dgrad_us(const Geom& g, bool back);

}  // namespace win
}  // namespace convbn
