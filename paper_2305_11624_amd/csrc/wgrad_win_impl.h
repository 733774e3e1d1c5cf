// bf16 MFMA weight gradient of any window and stride, channels multiples of 8:
//   dw'[co][tap][ci] = sum_m dZ[m][co] * X[m (+) tap][ci]      (Sec. 3.2.1: dJ/dw = dJ/dY (.) X)
//   r[co]            = sum_m dZ[m][co]                         (App. B)
// as one tiled product over (output channel) x (tap, input channel), the second index flat in steps of 8 channels, reduced
// over the output pixels.  A workgroup owns a TA x TB tile (128 or 64 each) and a slice of the pixels.
//
// Per chunk of P pixels the dZ rows and, for every 64 columns, the X rows that the columns' taps read at those pixels are
// copied global -> LDS (1 KB per instruction: 8 pixels x 128 bytes; out-of-image rows, tails and columns past the end are
// zero fills through an out-of-range offset) into a ring, chunks ahead of the multiplies; a lane's column, hence its tap,
// never changes, only its pixel moves on, by P, with two carries.  The reduced index is the pixel, the strided direction of
// those rows, so operands are read with the transposing LDS load (ds_read_b64_tr_b16: a 16-lane group turns 4 pixels x 16
// channels into "lane = channel, 4 pixels").  Granules of a row are exchanged (0-3 with 4-7) for every other pair of
// pixels: the four 64-byte pieces that half a wave reads then fall on distinct banks.
//
// Eight waves own 64 x 64 outputs each (8 transposing reads for 4 multiplies): one, two or four of them make up the tile,
// the others take further pixels of the chunk, and their sums meet in LDS at the end.  What bounds it is the rate at which
// the copies fill the LDS (about 40 bytes per clock and compute unit for 128-byte rows): 32 KB per 128 x 128 x 64 chunk are
// 800 clocks for 512 of multiplies.  (4x4 / 2 layer, 512 x 4096 weights, 6272 pixels: ~80 us on the two-barrier implicit
// GEMM this replaces.)
#pragma once
#include "common.h"

namespace convbn {
namespace wgw {

constexpr int NWAVES = 8;
constexpr unsigned OOB = 0x80000000u;   // beyond any buffer: the load returns zeros

struct WwParams {
  const bf16_t* x; const bf16_t* dz;
  float* part;        // [slices][Co][K]
  float* r_part;      // [slices][Co] or null
  unsigned x_bytes, dz_bytes;
  int Cin, Co, K, M;
  int H, W, Ho, Wo, kH, kW, sh, sw, ph, pw;
  int nta, ntb;       // tiles
  int slices, per;    // pixel slices, pixels of one (a multiple of 128)
};

typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t rsrc, unsigned voff, void* lds_wave_base) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr_t)lds_wave_base, 16, (int)voff, 0, 0, 0);
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ unsigned lds_off(const void* p) {
  return (unsigned)(size_t)(__attribute__((address_space(3))) const void*)p;
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
// The operands of a 16-pixel step: channels 0-31 of a block's row half (f[0]) and the other half (f[1]), each as pixels 0-3
// and 4-7 of this lane's eight (512 bytes apart).  Inline asm: the compiler would hold every LDS read until the copies in
// flight have landed.  The wait is in the same block: registers that a read still writes are nothing the compiler knows of.
__device__ __forceinline__ void tr_read_step(unsigned a0, unsigned a1, unsigned b0, unsigned b1, i32x2 (&fa)[2][2], i32x2 (&fb)[2][2]) {
  asm volatile("ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %8 offset:512\n\t"
               "ds_read_b64_tr_b16 %2, %10\n\tds_read_b64_tr_b16 %3, %10 offset:512\n\t"
               "ds_read_b64_tr_b16 %4, %9\n\tds_read_b64_tr_b16 %5, %9 offset:512\n\t"
               "ds_read_b64_tr_b16 %6, %11\n\tds_read_b64_tr_b16 %7, %11 offset:512\n\t"
               "s_waitcnt lgkmcnt(0)"
               : "=&v"(fa[0][0]), "=&v"(fa[0][1]), "=&v"(fb[0][0]), "=&v"(fb[0][1]), "=&v"(fa[1][0]), "=&v"(fa[1][1]),
                 "=&v"(fb[1][0]), "=&v"(fb[1][1])
               : "v"(a0), "v"(a1), "v"(b0), "v"(b1) : "memory");
}

template <int TA, int TB>
struct WwCfg {
  static constexpr int NA = TA / 64, NB = TB / 64, WT = NA * NB;
  static constexpr int PS = NWAVES / WT;                // waves that share a 64 x 64 block, each its own pixels
  static constexpr int P = WT == 1 ? 128 : 64;          // pixels of a chunk
  static constexpr int U = P / (16 * PS);               // 16-pixel steps of a wave per chunk
  static constexpr int OCT = P / 64;                    // pixel octets a wave copies
  static constexpr int CPW = OCT * (NA + NB);           // copies per wave and chunk
  static constexpr int STAGE = (TA + TB) * P * 2;
  static constexpr int NST = WT == 2 ? 5 : 4;           // 128 or 120 KB
  static constexpr int LDS_BYTES = NST * STAGE;
  static_assert(U >= 1 && LDS_BYTES >= NWAVES * 8192, "the sums meet where the ring was");
};

// Workgroup `wg` of the launch; smem: WwCfg::LDS_BYTES
template <int TA, int TB>
__device__ __forceinline__ void body(const WwParams& p, const int wg, unsigned char* smem) {
  using Cfg = WwCfg<TA, TB>;
  constexpr int NA = Cfg::NA, NB = Cfg::NB, WT = Cfg::WT, PS = Cfg::PS, P = Cfg::P, U = Cfg::U, OCT = Cfg::OCT;
  constexpr int CPW = Cfg::CPW, STAGE = Cfg::STAGE, NST = Cfg::NST, BLK = P * 128;   // BLK: a 64-channel block of a stage
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // workgroups go to the eight XCDs in turn: contiguous runs, slices outermost -- the tiles of a slice read the same rows
  const int total = p.nta * p.ntb * p.slices, run = (total + 7) >> 3;
  const int id = (wg & 7) * run + (wg >> 3);
  if ((wg >> 3) >= run || id >= total) return;
  const int slice = id / (p.nta * p.ntb), tile = id - slice * (p.nta * p.ntb);
  const int ta = tile % p.nta, tb = tile / p.nta;
  const int co0 = ta * TA, k0 = tb * TB;
  const int m_beg = slice * p.per, m_end = min(p.M, m_beg + p.per);
  const int nchunks = (m_end - m_beg + P - 1) / P;
  const __amdgpu_buffer_rsrc_t x_rsrc = make_rsrc(p.x, p.x_bytes), z_rsrc = make_rsrc(p.dz, p.dz_bytes);

  // ---- copies of this wave: pixel octets wave, wave + 8, ...; lane l writes granule l % 8 of pixel l / 8's row
  const int prow = lane >> 3;
  const int gran = (lane & 7) ^ (((prow >> 1) & 1) << 2);
  unsigned za[NA];   // dZ: byte offset of this lane's channels in a row, OOB past the last channel
#pragma unroll
  for (int a = 0; a < NA; ++a) {
    const int c = co0 + a * 64 + gran * 8;
    za[a] = c < p.Co ? (unsigned)(c * 2) : OOB;
  }
  int bt_h[NB], bt_w[NB], bt_off[NB];   // X: this lane's tap and what it adds to the pixel's byte offset
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int q = k0 + b * 64 + gran * 8;
    const int tap = q / p.Cin, c = q - tap * p.Cin;
    const int ti = tap / p.kW, tj = tap - ti * p.kW;
    bt_h[b] = q < p.K ? ti : 1 << 20;   // (columns past the end: never inside the image)
    bt_w[b] = tj;
    bt_off[b] = ((ti * p.W + tj) * p.Cin + c) * 2;
  }
  int pm[OCT], pho[OCT], pwo[OCT], po[OCT];   // the octet's pixel of this lane: index, row, column, byte offset of its window origin in X
  const int cb = p.Cin * 2;
#pragma unroll
  for (int o = 0; o < OCT; ++o) {
    const int m = m_beg + (wave + NWAVES * o) * 8 + prow;
    const int q = (int)((unsigned)m / (unsigned)p.Wo);
    pm[o] = m;
    pwo[o] = m - q * p.Wo;
    const int n = (int)((unsigned)q / (unsigned)p.Ho);
    pho[o] = q - n * p.Ho;
    po[o] = ((n * p.H + pho[o] * p.sh - p.ph) * p.W + pwo[o] * p.sw - p.pw) * cb;
  }
  // P pixels further: columns, rows and images, and what the step and the carries add to the byte offset
  const int step_q = P / p.Wo, step_w = P - step_q * p.Wo, step_n = step_q / p.Ho, step_h = step_q - step_n * p.Ho;
  const int step_b = ((step_n * p.H + step_h * p.sh) * p.W + step_w * p.sw) * cb;
  const int carry_w = (p.sh * p.W - p.Wo * p.sw) * cb, carry_h = (p.H - p.Ho * p.sh) * p.W * cb;
  auto issue_copy = [&](int i, unsigned char* stage) {
    const int o = i / (NA + NB), j = i - o * (NA + NB);
    unsigned char* const dst = stage + (wave + NWAVES * o) * 1024;
    const bool live = pm[o] < m_end;
    if (j < NA) {
      const unsigned zo = za[j < NA ? j : 0];
      dma16(z_rsrc, live ? zo + (unsigned)pm[o] * (unsigned)(p.Co * 2) : OOB, dst + j * BLK);
    } else {
      const int b = j - NA < NB ? j - NA : 0;
      const int h = pho[o] * p.sh - p.ph + bt_h[b], w = pwo[o] * p.sw - p.pw + bt_w[b];
      const bool ok = live && (unsigned)h < (unsigned)p.H && (unsigned)w < (unsigned)p.W;
      dma16(x_rsrc, ok ? (unsigned)(po[o] + bt_off[b]) : OOB, dst + j * BLK);
    }
  };
  auto advance = [&]() {
#pragma unroll
    for (int o = 0; o < OCT; ++o) {
      pm[o] += P;
      int wo = pwo[o] + step_w, ho = pho[o] + step_h, d = step_b;
      if (wo >= p.Wo) { wo -= p.Wo; ++ho; d += carry_w; }
      if (ho >= p.Ho) { ho -= p.Ho; d += carry_h; }
      pwo[o] = wo; pho[o] = ho; po[o] += d;
    }
  };

  // ---- operands: this wave's 64 x 64 block and pixels; lane l addresses pixel (l % 16) / 4 (+ 8 for the upper half wave)
  // and four channels of a 32-channel half row
  const int wt = wave % WT, ps = wave / WT;
  const int wa = wt % NA, wb = wt / NA;
  const int kb = lane >> 5, ep = (lane & 15) >> 2;
  const unsigned rbase = lds_off(smem) + (unsigned)((ps * U * 16 + kb * 8 + ep) * 128 +
                                                    (((lane >> 4) & 1) * 2 + ((lane & 3) >> 1)) * 16 + (lane & 1) * 8);
  const unsigned h0 = (unsigned)((ep >> 1) & 1) << 6, h1 = h0 ^ 64u;   // where the row's first and second 32 channels are
  const unsigned a_blk = (unsigned)(wa * BLK), b_blk = (unsigned)((NA + wb) * BLK);

  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  const bool want_r = p.r_part && tb == 0 && wb == 0;
  float racc[2] = {0.f, 0.f};

#pragma unroll
  for (int s = 0; s < NST - 1; ++s) {
#pragma unroll
    for (int i = 0; i < CPW; ++i) issue_copy(i, smem + s * STAGE);
    advance();
  }
  int cur = 0;
  for (int c = 0; c < nchunks; ++c) {
    wait_vm<CPW * (NST - 2)>();
    block_barrier();
    const unsigned st = rbase + (unsigned)(cur * STAGE);
    unsigned char* const fill = smem + (cur >= 1 ? cur - 1 : NST - 1) * STAGE;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      i32x2 fa[2][2], fb[2][2];
      const unsigned a0 = st + a_blk + u * 2048, b0 = st + b_blk + u * 2048;
      tr_read_step(a0 + h0, a0 + h1, b0 + h0, b0 + h1, fa, fb);
      bf16x8 A[2], Bq[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        A[i] = __builtin_bit_cast(bf16x8, (i32x4){fa[i][0][0], fa[i][0][1], fa[i][1][0], fa[i][1][1]});
        Bq[i] = __builtin_bit_cast(bf16x8, (i32x4){fb[i][0][0], fb[i][0][1], fb[i][1][0], fb[i][1][1]});
      }
      // the copies of the chunk NST - 1 ahead, spread over the multiplies of this one: issued together behind the barrier they
      // keep every wave of the compute unit from its first multiply (transposed 4x4 / 2, 512 -> 256, 14 x 14: 38.8 -> 36.6 us)
      constexpr int PER = (CPW + U - 1) / U;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[i], Bq[j], acc[i][j], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
          const int k = i * 2 + j;
#pragma unroll
          for (int q = k * PER / 4; q < (k + 1) * PER / 4; ++q)
            if (u * PER + q < CPW) issue_copy(u * PER + q, fill);
          __builtin_amdgcn_sched_barrier(0);
        }
      if (want_r) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int e = 0; e < 2; ++e)
            racc[i] += (bf16_lo((uint32_t)fa[i][e][0]) + bf16_hi((uint32_t)fa[i][e][0])) +
                       (bf16_lo((uint32_t)fa[i][e][1]) + bf16_hi((uint32_t)fa[i][e][1]));
      }
    }
    cur = cur + 1 == NST ? 0 : cur + 1;
    advance();
  }
  wait_vm<0>();
  __syncthreads();

  // ---- sums of the waves that share a block.  Accumulator: lane = column l % 32, rows 8 (e / 4) + 4 (l / 32) + e % 4
  // (element (e, l) of a subtile; two subtiles of a wave at a time)
  float (*red)[2][16][64] = reinterpret_cast<float (*)[2][16][64]>(smem);   // [wave][columns 0-31, 32-63]
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    if (i > 0) __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) red[wave][j][e][lane] = acc[i][j][e];
    __syncthreads();
    // four columns a thread: block o, subtile j, register e, lanes l4 .. l4 + 3
    const int j = tid >> 8, e = (tid >> 4) & 15, l4 = (tid & 15) * 4;
#pragma unroll
    for (int o = 0; o < WT; ++o) {
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int s = 0; s < PS; ++s) {
        const float4 f = *reinterpret_cast<const float4*>(&red[s * WT + o][j][e][l4]);
        v.x += f.x; v.y += f.y; v.z += f.z; v.w += f.w;
      }
      const int co = co0 + (o % NA) * 64 + i * 32 + 8 * (e >> 2) + 4 * (l4 >> 5) + (e & 3);
      const int k = k0 + (o / NA) * 64 + j * 32 + (l4 & 31);
      if (co < p.Co && k < p.K) *reinterpret_cast<float4*>(p.part + ((size_t)slice * p.Co + co) * p.K + k) = v;   // (K % 8 == 0)
    }
  }
  if (p.r_part && tb == 0) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) red[wave][0][i][lane] = racc[i];
    __syncthreads();
    if (tid < TA && co0 + tid < p.Co) {
      const int a = tid >> 6, i = (tid >> 5) & 1, l = tid & 31;
      float v = 0.f;
#pragma unroll
      for (int s = 0; s < PS; ++s) v += red[s * WT + a][0][i][l] + red[s * WT + a][0][i][l + 32];
      p.r_part[(size_t)slice * p.Co + co0 + tid] = v;
    }
  }
}

// us: an estimate of the launch, fold_us: of what summing its copies takes (see wgrad_win.hip)
struct WwPlan { bool ok; int ta, tb; float us, fold_us; WwParams p; };
const WwPlan& plan(const Geom& g);
// the plan for at most that many workgroups; false: there is none
bool limited(const Geom& g, int workgroups, WwPlan* pl);

}  // namespace wgw
}  // namespace convbn
