// bf16 pointwise (1x1) convolution, with or without a stride, as a tiled matrix product
//     out[m][r] = sum_c act[m][c] wgt[r][c] (+ bias[r]):
//   forward conv   Z  = w' (*) X + b'   (Sec. 3.1 / 3.3)   act = x,   wgt = w' as [Cout][Cin]
//   input gradient dX = w'_rot (*) dZ   (Sec. 3.2.1)       act = dz,  wgt = w' as [Cin][Cout]   (stride 1)
//
// One output tile per workgroup, as large as still fills the chip: 256 (or 128) pixels x 128 channels, shared by
// EIGHT waves as 4 (2) pixel groups x 2 channel groups, so that a wave owns 64 x 64 (32 x 64) outputs and reads four
// (three) operand fragments for four (two) multiplies, and the matrix pipe of every SIMD is fed by two waves.  Channel
// counts that are no multiple of 128 get 128 x 64 tiles, and so do layers with too few 128 x 128 tiles for the chip.
//
// Pipeline.  The reduction runs over 64-channel chunks.  A chunk of
// the activation tile and of the weight tile is copied global -> LDS directly (1 KB per instruction: 8 rows x 128
// bytes) into one of three (two) stages, two (one) chunks ahead; every wave issues the same number of copies per chunk,
// so "at most that many copies outstanding" means the current chunk has landed; one barrier per chunk.  LDS rows are 128
// bytes, unpadded: the copy permutes the eight 16-byte granules of row r by (r / 2) % 8 (it chooses which granule
// each lane fetches), so that the 128-bit operand reads of 16 consecutive rows fall on distinct banks.  The copies of
// a chunk are issued between its multiplies; operands are double-buffered in registers one 16-channel step ahead.
// A copy's per-lane byte offset is free, which is all a stride needs: a strided layer gathers every stride-th pixel's row.
// A forward launch given the unfolded weight applies s and b' in the epilogue and folds on the side (fold_tile.h).
//
// Layers that are bound by their stores rather than by the product (64 or 128 reduced channels over tens of
// thousands of pixels) run a variant with all their one or two chunks resident: no ring, about 70 registers, 33 or
// 65 KB of LDS -- several workgroups share a compute unit, and one's stores overlap another's loads.
#include "common.h"
#include "fold_tile.h"

namespace convbn {

namespace {

constexpr int NWAVES = 8;
constexpr int CB = 64;                 // reduced channels per chunk
constexpr int KK = CB / 16;
constexpr unsigned OOB = 0x80000000u;  // beyond any buffer: the load returns zeros

enum { ORDER_TOGETHER, ORDER_PIXEL_RUNS, ORDER_CHANNEL_RUNS };
struct GmParams {
  const bf16_t* act;     // [M][C]
  const bf16_t* wgt;     // [R][C]
  const float* bias;     // [R] or null
  BnEpilogue bn;         // bn.gamma != null: the weight is unfolded, the epilogue applies s and b' (bias unused)
  bf16_t* out;           // [M][R]
  int relu;
  const bf16_t* mask;    // not null: [M][R], the output is zeroed where this is <= 0
  const bf16_t* add;     // not null: [M][R], added to the (rounded) output before the ReLU and the mask
  unsigned act_bytes, wgt_bytes;
  int M, C, R;
  int ntr;               // channel tiles
  int nchunks;
  int order;             // of the tiles, see the kernel
  int nconv;             // the product's workgroups, those behind it fold, or fold back
  // A pointwise layer with a stride (a downsampling shortcut) is the same product over the output pixels; gather: the
  // activation row of output pixel m = (n, ho, wo) is pixel (n, ho sh, wo sw) of an [N][Hs][Ws] tensor.
  int gather;
  int Ho, Wo, Hs, Ws, sh, sw;
};

// pixel index in the strided tensor of row m of the dense side
__device__ __forceinline__ size_t strided_row(const GmParams& p, int m) {
  const int hw = p.Ho * p.Wo;
  const int n = m / hw, rem = m - n * hw;
  const int ho = rem / p.Wo, wo = rem - ho * p.Wo;
  return ((size_t)n * p.Hs + (size_t)ho * p.sh) * p.Ws + (size_t)wo * p.sw;
}

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

// TM: pixels per workgroup (256: a wave owns 2 x 2 subtiles of 32 x 32; 128: 1 x 2).
// RES > 0: the reduction is RES chunks in all (64 or 128 channels), each with a stage of its own and requested at the
// start: no ring, few registers -- what such a layer needs is several workgroups per compute unit, so that one's
// stores and another's loads overlap.
// TN: output channels per workgroup (128; 64 for layers whose channel count is no multiple of 128 -- the two channel
// groups of waves then own 32 channels each).
// NS: stages of the ring.
template <int TM, int RES = 0, int TN = 128, int NS = 3>
struct GmCfg {
  static constexpr bool ONE = RES > 0;
  static constexpr int CW = TN / 2;                     // channels per wave
  static constexpr int NPS = TM / 128;                  // 32-pixel subtiles per wave
  static constexpr int NCS = CW / 32;                   // 32-channel subtiles per wave
  static constexpr int AUW = TM / 8 / NWAVES;           // activation copies (8 rows each) per wave and chunk
  static constexpr int WUW = TN / 8 / NWAVES;           // weight copies per wave and chunk
  static constexpr int CPW = AUW + WUW;
  static constexpr int STAGE = (TM + TN) * 128;
  static constexpr int OFF_BIAS = (RES ? RES : NS) * STAGE;   // [TN] bias, [TN] scale
  static constexpr int LDS_BYTES = OFF_BIAS + 2 * TN * 4;
  static constexpr bool SHARED = 2 * LDS_BYTES <= 160 * 1024;   // two workgroups, and more, share a compute unit
  static_assert(NWAVES * 32 * CW * 2 <= STAGE, "the epilogue stages every wave's outputs (32 pixels at a time) in the first stage");
};

// STREAM: non-temporal stores, see launch_gm.  Side: what the workgroups behind the product's do, FoldBackArgs (an input gradient) or
// FoldSide (the rest)
template <int TM, int RES, int TN, int NS, bool STREAM, class Side>
__global__ __launch_bounds__(64 * NWAVES) void conv_gm_kernel(GmParams p, Side side) {
  using Cfg = GmCfg<TM, RES, TN, NS>;
  constexpr bool ONE = Cfg::ONE;
  constexpr int CW = Cfg::CW;
  constexpr int GR = CW / 8;          // 16-byte granules of a wave's staged output row
  constexpr int RPI = 64 / GR;        // rows one store instruction covers
  constexpr int ITS = 32 / RPI;       // store instructions per 32-pixel subtile
  constexpr int NPS = Cfg::NPS, NCS = Cfg::NCS, AUW = Cfg::AUW, WUW = Cfg::WUW, CPW = Cfg::CPW, STAGE = Cfg::STAGE;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  float* biasl = reinterpret_cast<float*>(smem + Cfg::OFF_BIAS);
  if ((int)blockIdx.x >= p.nconv) {
    // (as many loads in flight as the registers of the workgroups that share a compute unit leave: 2048 -> 512 at 6 x 6, 41 images, a pass
    // 34.9 us with 8 and one column at a time on 128 x 128 tiles, 32.7; 1024 -> 256 at 17 x 20, 5 images, one and two columns on
    // 128 x 64 tiles 20.8, 20.3)
    if constexpr (Side::BACK) fold_back_side<64 * NWAVES, ROW_VEC, Cfg::SHARED ? 8 : 16, !Cfg::SHARED ? 4 : ONE || TN == 128 ? 1 : 2>(side, (int)blockIdx.x - p.nconv, smem);
    else fold_side(p.bn, p.wgt, (int)blockIdx.x - p.nconv, smem);
    return;
  }

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;      // pixel group, channel group
  // Workgroups are handed to the eight XCDs in turn (id % 8), and each XCD has its own L2, which what its workgroups share
  // should fit: the tiles are split into eight contiguous runs, along the channels where the weight is the larger operand
  // (an XCD then reads its channel tiles' rows and all activations), else along the pixels (2048 <- 512 channels at 7 x 7,
  // 64 images, whole step: 60.3 -> 57.0 us).  Long streams are read and written front to back by all XCDs together, a pixel
  // tile's channel tiles on one of them: eight far-apart streams cost 3 % (64 -> 256 channels, 253k pixels: 121.9 against
  // 125.7 us a step).
  const int npt = (p.M + TM - 1) / TM, ntiles = npt * p.ntr;
  const int xcd = (int)blockIdx.x & 7, kx = (int)blockIdx.x >> 3;
  int ptile, ctile;
  if (p.order == ORDER_TOGETHER) {
    ctile = kx % p.ntr;
    ptile = (kx / p.ntr) * 8 + xcd;
    if (ptile >= npt) return;
  } else {
    const int tile = xcd * ((ntiles + 7) >> 3) + kx;
    if (tile >= ntiles) return;
    if (p.order == ORDER_CHANNEL_RUNS) { ctile = tile / npt; ptile = tile - ctile * npt; }
    else { ptile = tile / p.ntr; ctile = tile - ptile * p.ntr; }
  }
  const int r0 = ctile * TN, m0 = ptile * TM;
  const __amdgpu_buffer_rsrc_t act_rsrc = make_rsrc(p.act, p.act_bytes);
  const __amdgpu_buffer_rsrc_t wgt_rsrc = make_rsrc(p.wgt, p.wgt_bytes);

  if (tid < TN) {
    const int ch = r0 + tid;
    float bias_v = p.bias ? p.bias[ch] : 0.f, scale_v = 1.f;
    if (p.bn.gamma) {   // Z = s (w (*) X) + b' (Sec. 3.3), s and b' worked out here
      scale_v = p.bn.gamma[ch] / sqrtf(p.bn.var[ch] + p.bn.eps);
      bias_v = ((p.bn.b ? p.bn.b[ch] : 0.f) - p.bn.mean[ch]) * scale_v + p.bn.beta[ch];
    }
    biasl[tid] = bias_v;
    biasl[TN + tid] = scale_v;
  }

  // ---- copies of this wave: unit u covers rows 8 u .. 8 u + 7 of its tile; lane l writes LDS granule l % 8 of row
  // 8 u + l / 8 and fetches the granule that belongs there, (l % 8) ^ key(row), key = (row / 2) % 8
  const int crow = lane >> 3, cpos = lane & 7;
  unsigned voff_a[AUW], voff_w[WUW];
#pragma unroll
  for (int j = 0; j < AUW; ++j) {
    const int row = (wave + NWAVES * j) * 8 + crow;
    const int g = cpos ^ ((row >> 1) & 7);
    const size_t arow = (p.gather && m0 + row < p.M) ? strided_row(p, m0 + row) : (size_t)(m0 + row);
    voff_a[j] = m0 + row < p.M ? (unsigned)((arow * p.C + g * 8) * 2) : OOB;   // rows past the last pixel: zeros
  }
#pragma unroll
  for (int j = 0; j < WUW; ++j) {
    const int row = (wave + NWAVES * j) * 8 + crow;
    const int g = cpos ^ ((row >> 1) & 7);
    voff_w[j] = (unsigned)(((size_t)(r0 + row) * p.C + g * 8) * 2);
  }
  // copy i (0 .. CPW-1) of a chunk
  auto issue_copy = [&](int i, int chunk, unsigned char* stage) {
    const unsigned soff = (unsigned)(chunk * (CB * 2));
    if (i < AUW) dma16(act_rsrc, voff_a[i < AUW ? i : 0], soff, stage + (wave + NWAVES * i) * 1024);
    else dma16(wgt_rsrc, voff_w[i - AUW < WUW ? i - AUW : 0], soff, stage + TM * 128 + (wave + NWAVES * (i - AUW)) * 1024);
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

  bf16x8 fa[2][NCS], fb[2][NPS];
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
    const int g = (lane % GR) ^ ((row >> 1) & (GR - 1));
    const int m = m0 + wm * (32 * NPS) + ps * 32 + row;
    if (m >= p.M) return -1;
    return (long long)((size_t)m * p.R + r0 + wn * CW + g * 8);
  };
  uint4 addv[NPS][ITS], maskv[NPS][ITS];
  if (!ONE && (p.add || p.mask)) {
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

  // ---- prologue: chunk 0 and, but for a ring of two stages, chunk 1 (a chunk past the end is the last one again, into a
  // stage nobody reads)
  const int nchunks = p.nchunks;
  int f_c = 0;   // the chunk whose copies are issued next; the last one stays
#pragma unroll
  for (int i = 0; i < CPW; ++i) issue_copy(i, f_c, smem);
  if (f_c + 1 < nchunks) ++f_c;
  if constexpr (ONE ? RES > 1 : NS > 2) {
#pragma unroll
    for (int i = 0; i < CPW; ++i) issue_copy(i, f_c, smem + STAGE);
    if (f_c + 1 < nchunks) ++f_c;
  }

  int st_cur = 0;   // stage of the current chunk
  for (int c = 0; c < nchunks; ++c) {
    if (ONE ? c == RES - 1 : NS == 2) wait_vm<0>();   // (nothing behind it: the last resident chunk; two stages)
    else wait_vm<CPW>();    // this chunk has landed (the next one's copies may be in flight) ...
    block_barrier();   // ... for every wave, and everybody is done with the stage refilled below
    const unsigned char* const stage = smem + st_cur * STAGE;
    const int st_fill = st_cur >= 1 ? st_cur - 1 : NS - 1;   // (c + NS - 1) % NS
    unsigned char* const fill = smem + st_fill * STAGE;
    load_frags(0, stage, 0);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const int cur = kk & 1;
      if (kk + 1 < KK) load_frags(cur ^ 1, stage, kk + 1);
      __builtin_amdgcn_sched_barrier(0);
      // the copies of the chunk NS - 1 ahead, spread over the multiplies of this one
      constexpr int PER = (CPW + KK - 1) / KK;
      int issued = 0;
#pragma unroll
      for (int i = 0; i < NCS; ++i)
#pragma unroll
        for (int ps = 0; ps < NPS; ++ps) {
          acc[i][ps] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[cur][i], fb[cur][ps], acc[i][ps], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
          if (!ONE && issued < PER && kk * PER + issued < CPW) {
            issue_copy(kk * PER + issued, f_c, fill);
            ++issued;
            __builtin_amdgcn_sched_barrier(0);
          }
        }
#pragma unroll
      for (; issued < PER; ++issued)
        if (!ONE && kk * PER + issued < CPW) issue_copy(kk * PER + issued, f_c, fill);
      __builtin_amdgcn_sched_barrier(0);
    }
    st_cur = st_cur + 1 == NS ? 0 : st_cur + 1;
    if (f_c + 1 < nchunks) ++f_c;
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
      if constexpr (ONE) {
        if (o >= 0) v = post_op8(v, p.relu, p.mask, p.add, (size_t)o);
      } else {
        if (p.add) v = add8(v, addv[ps][it]);
        if (p.relu) v = relu8(v);
        if (p.mask) v = mask8(v, maskv[ps][it]);
      }
      if (o >= 0) {
        if constexpr (STREAM) store_result(p.out + o, v);
        else *reinterpret_cast<uint4*>(p.out + o) = v;
      }
    }
  }
}

constexpr int MIN_TILES = 160;       // fewer 256-pixel tiles leave too many compute units without one: 128-pixel tiles then,
constexpr int MIN_TILES_SMALL = 96;  // down to this many (measured against the split-sum plans of the LDS-tile kernel:
                                     // 1024 -> 256 at 14 x 14, 98 tiles, 10.8 against 12.0 us)
constexpr int MAX_PIXELS = 32768;    // longer pixel ranges with short reductions stream through the weight-stationary kernel

// Bytes written, read and written, from which on the channel tiles of a pixel tile follow one another on an XCD
// (ORDER_TOGETHER) instead of each XCD taking a run of the tiles.  Forward, together / runs, ten channel counts from 64 to 2048:
// above the line 1-13 % in favour of together (64 -> 256, 160 MB 36.8 / 41.6 us; 1024 -> 256, 70 MB 22.5 / 22.7), but for launches
// whose pixel tiles, rounded up to eights, need one more round (512 -> 2048, 46 MB 38.5 / 34.0).  Below it the two are within 4 %
// for most, and that round costs more (512 -> 2048, 26 MB 26.2 / 20.9; 512 -> 512, 34 MB 24.4 / 21.1); 64 -> 256 and
// 128 -> 512 gain 4-9 % together from 14 MB on (20 MB 7.0 / 7.6).
constexpr size_t LONG_OUTPUT = 32u << 20, LONG_STREAM = 48u << 20;

struct GmPlan { int tm, res, tn, ns; };   // tm == 0: not taken

GmPlan choose_plan(int M, int C, int R) {
  GmPlan none{0, 0, 0, 3};
  if (M < 1 || C < CB || C % CB || R % 64) return none;
  if ((size_t)M * C * 2 >= OOB || (size_t)M * R * 2 >= OOB || (size_t)R * C * 2 >= OOB) return none;
  const int tn = R % 128 == 0 ? 128 : 64;
  const int ntr = R / tn;
  const long long t128 = (long long)ceil_div(M, 128) * ntr, t256 = (long long)ceil_div(M, 256) * ntr;
  // short reductions over many tiles: every chunk resident, several workgroups per compute unit
  if ((C == CB || C == 2 * CB) && t128 >= 3 * MIN_TILES) return GmPlan{128, C / CB, tn, 3};
  if (tn == 64) return t128 >= MIN_TILES_SMALL ? GmPlan{128, 0, 64, 3} : none;
  // (measured on the 56 x 56 stage: with 256 reduced channels the tile beats the streaming kernel, 21.9 against 26.1 us
  // for 256 -> 128; with 64 or 128 both are bound by their stores and take the same time)
  if (M > MAX_PIXELS && C < 256) return none;
  // many tiles: 256 x 128 ones in a ring of three stages need the whole LDS of a compute unit, so nothing covers a tile's
  // first loads and its stores; with up to four chunks these are most of its time, and 128 x 128 tiles with two stages, two
  // workgroups per compute unit, are faster although they read more operands per multiply (256 -> 1024 at 14 x 14 with an
  // addend: 128 images 53.0 -> 43.5 us, 64 images 21.8 -> 19.8; 256 -> 128 at 56 x 56, 128 images 79.5 -> 68.4, 32 images
  // 21.8 -> 19.4).  With eight chunks both take the same time (512 -> 256 at 28 x 28, 64 images: 22.5 and 22.8), with
  // sixteen the larger tile wins (1024 -> 256 at 14 x 14, 128 images: 17.8 against 19.3).
  if (t256 >= MIN_TILES) return C <= 4 * CB ? GmPlan{128, 0, 128, 2} : GmPlan{256, 0, 128, 3};
  // too few 128 x 128 tiles for the chip: twice as many of half the channels (measured: 1024 -> 256 at 14 x 14, 98 tiles,
  // 10.4 -> 9.0 us; 2048 -> 512 at 7 x 7, 52 tiles, 16.8 us on the split-sum tile kernel -> 12.6)
  if (t128 < MIN_TILES && 2 * t128 >= MIN_TILES_SMALL) return GmPlan{128, 0, 64, 3};
  if (t128 >= MIN_TILES_SMALL) return GmPlan{128, 0, 128, 3};
  return none;
}

template <int TM, int RES, int TN, int NS, bool STREAM, class Side>
hipError_t launch_inst(GmParams p, Side side, hipStream_t st) {
  static LdsLimitOnce lds_once;
  constexpr int lds = GmCfg<TM, RES, TN, NS>::LDS_BYTES;
  if (hipError_t e = set_lds_limit_once(lds_once, reinterpret_cast<const void*>(&conv_gm_kernel<TM, RES, TN, NS, STREAM, Side>), lds);
      e != hipSuccess) return e;
  static_assert(2 * FOLD_TILE_BYTES <= lds && FOLD_BACK_SIDE_BYTES(64 * NWAVES) <= lds, "what folds on the side");
  const int npt = ceil_div(p.M, TM);
  const size_t out_bytes = (size_t)p.M * p.R * 2;
  p.order = out_bytes > LONG_OUTPUT || out_bytes + p.act_bytes > LONG_STREAM ? ORDER_TOGETHER
            : p.wgt_bytes > p.act_bytes ? ORDER_CHANNEL_RUNS : ORDER_PIXEL_RUNS;
  p.nconv = p.order == ORDER_TOGETHER ? ceil_div(npt, 8) * 8 * p.ntr : ceil_div(npt * p.ntr, 8) * 8;
  int nside;
  if constexpr (Side::BACK) nside = fold_back_side_blocks(side, 64 * NWAVES); else nside = fold_side_blocks(p.bn);
  hipLaunchKernelGGL((conv_gm_kernel<TM, RES, TN, NS, STREAM, Side>), dim3(p.nconv + nside), dim3(64 * NWAVES), lds, st, p, side);
  return hipGetLastError();
}

}  // namespace

bool gm_supported(int M, int C, int R) { return choose_plan(M, C, R).tm != 0; }
bool gm_round_full(int M, int C, int R, int aside) {
  const GmPlan pl = choose_plan(M, C, R);
  if (pl.res > 0 || pl.tn != 128 || pl.ns != 3) return false;   // (the others share a compute unit)
  const long long tiles = (long long)ceil_div(M, pl.tm) * (R / 128);
  return tiles <= 256 && tiles + aside > 256;
}

hipError_t launch_gm(int M, int C, int R, const void* act, const void* wgt, const float* bias, const BnEpilogue* bn,
                     void* out, int relu, const void* mask, const void* add, hipStream_t st, const GmStride* sd, bool grad,
                     const FoldBackArgs* fb) {
  const GmPlan pl = choose_plan(M, C, R);
  if (pl.tm == 0) return hipErrorInvalidValue;
  GmParams p{};
  p.M = M; p.C = C; p.R = R;
  p.act_bytes = (unsigned)((size_t)M * C * 2);
  if (sd) {
    const size_t strided_pixels = (size_t)sd->N * sd->Hs * sd->Ws;
    if (strided_pixels * (size_t)C * 2 >= OOB) return hipErrorInvalidValue;
    p.gather = 1;
    p.Ho = sd->Ho; p.Wo = sd->Wo; p.Hs = sd->Hs; p.Ws = sd->Ws; p.sh = sd->sh; p.sw = sd->sw;
    p.act_bytes = (unsigned)(strided_pixels * C * 2);
  }
  p.wgt_bytes = (unsigned)((size_t)R * C * 2);
  p.ntr = R / pl.tn;
  p.nchunks = C / CB;
  p.act = (const bf16_t*)act; p.wgt = (const bf16_t*)wgt; p.bias = bias; p.out = (bf16_t*)out;
  if (bn) p.bn = *bn;
  // An input gradient of 16 MB and more is stored past the caches.  The weight gradient behind it takes what it took (14.4 us), it is
  // the next forward pass that finds more room (256 -> 64 at 56 x 56, 32 images: 21.2 -> 18.1).  A block on its own, inputs from
  // memory: 256 -> 64 at 56 x 56, 32 images (51 MB of dx) 62.1 -> 58.2 us a pass, 16 images 42.6 -> 40.1, 64 images 98.3 -> 91.7;
  // 512 -> 128 at 28 x 28, 32 images 47.1 -> 45.2; inputs still in the last-level cache from the pass before last 58.5 -> 52.2; the
  // same tensors again at once 51.0 -> 51.3.  Where the previous block reads dx next, it pays some of it back: three blocks in a
  // row, a step, 0.4 - 2 % longer from 17 to 103 MB (51 MB: 159.5 -> 162.5 us) and 5 % shorter at 206 MB (478 -> 454); the
  // backbone's training step 16 and 32 images 0.3 % longer (2813 -> 2822), 64 and 128 images 0.5 and 1 % shorter (7643 -> 7565).
  // Forward outputs stay in the caches: the backbone's forward pass, 32 images, takes 861 us with them there, 919 without.
  const bool stream = grad && (size_t)M * R * 2 >= ((size_t)16 << 20);
  p.relu = relu; p.mask = (const bf16_t*)mask; p.add = (const bf16_t*)add;
#define GM_CASE(TM_, RES_, TN_, NS_)                                                                                    \
  if (pl.tm == TM_ && pl.res == RES_ && pl.tn == TN_ && pl.ns == NS_) {                                                 \
    if (fb) return stream ? launch_inst<TM_, RES_, TN_, NS_, true>(p, *fb, st) : launch_inst<TM_, RES_, TN_, NS_, false>(p, *fb, st); \
    return stream ? launch_inst<TM_, RES_, TN_, NS_, true>(p, FoldSide{}, st) : launch_inst<TM_, RES_, TN_, NS_, false>(p, FoldSide{}, st); \
  }
  GM_CASE(128, 0, 128, 2) GM_CASE(256, 0, 128, 3) GM_CASE(128, 1, 128, 3) GM_CASE(128, 2, 128, 3)
  GM_CASE(128, 0, 64, 3) GM_CASE(128, 1, 64, 3) GM_CASE(128, 2, 64, 3)
  if (pl.tm == 128 && pl.res == 0 && pl.tn == 128 && pl.ns == 3)   // (under 2 MIN_TILES tiles: never 16 MB)
    return fb ? launch_inst<128, 0, 128, 3, false>(p, *fb, st) : launch_inst<128, 0, 128, 3, false>(p, FoldSide{}, st);
#undef GM_CASE
  return hipErrorInvalidValue;
}

}  // namespace convbn
