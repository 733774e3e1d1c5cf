// Contractions with the reduction split over the waves of a workgroup: the fp32 path of a dense block.
//
// v_mfma_f32_32x32x2_f32 multiplies and accumulates in fp32 (no narrower type anywhere), 128 multiply-adds per clock and
// compute unit.  What bounds a problem of the sizes fp32 is used for is how much of the chip it keeps busy: a workgroup
// owns ONE 32 pixel x 32 channel tile and its eight waves take an eighth of the reduction each, added through LDS at the
// end -- 8 (M / 32)(R / 32) waves (8 images, 28 x 28, 64 -> 64 channels: 392 workgroups), and no barrier before the end:
// every wave copies its own operand stages (16 channels of 32 pixels and 32 output channels, 4 KB) into its own part of
// the LDS.  Measured on the forward pass above: one thread per output element 452 us; operands loaded straight into
// registers (a lane owns a row, the 64 lanes of a load touch 64 cache lines, and the address units set the pace) 13.7 us;
// this way 11, of which 3 us are multiplies at full rate and about 4 what any launch takes.
// A workgroup's pixels all belong to one residue class of input positions in a strided input gradient, so no multiply
// is spent on taps that do not reach them.
#include "common.h"

namespace convbn {

namespace {

constexpr unsigned OOB = 0x80000000u;   // beyond any buffer: the load returns zeros
constexpr int KS = 8;                   // waves of a workgroup = slices of its reduction
constexpr int STAGE = 4096;             // bytes of an operand stage: 64 rows (pixels, output channels) of 16 channels
constexpr int WAVE_LDS = STAGE;         // one: the next step's copies are asked for as soon as this one's operands are in registers.
                                        // With 33 KB of LDS and at most 80 registers three workgroups share a compute unit, and
                                        // their waves cover one another (64 -> 64, 28 x 28, 8 images, a step: two stages and
                                        // two workgroups 34.7 us, 31.5; 25 -> 87 at 23 x 17, 8 images 44.6, 33.4)

typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

struct WvParams {
  const void* act; const void* wgt; void* out;
  const void* mask; const void* add;
  const float* bias;
  BnEpilogue bn;
  int relu, dgrad;
  unsigned act_bytes, wgt_bytes;
  int N, C, R;                   // C reduced, R produced channels
  int aH, aW, oH, oW;            // activation and output planes
  int kH, kW, sh, sw, ph, pw;
  int ptiles, rtiles;            // pixel tiles of a class, channel tiles
  int ncls, ncw;                 // residue classes that have positions (input gradient), columns of them
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
// 1 KB copy: lane l fetches 16 bytes at byte offset voff and writes them to LDS at lds_wave_base + 16 l
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t rsrc, unsigned voff, void* lds_wave_base) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr_t)lds_wave_base, 16, (int)voff, 0, 0, 0);
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ unsigned lds_off(const void* p) {
  return (unsigned)(size_t)(__attribute__((address_space(3))) const void*)p;
}
// The operands of a stage: 16 bytes each at g0 and g1 (activations) and 2048 behind them (weights).  Inline asm: the compiler
// would hold the reads until the copies of the next stage have landed.  The wait is in the same block: registers that a
// read still writes are nothing the compiler knows of.
__device__ __forceinline__ void lds_read_stage(unsigned g0, unsigned g1, u32x4& x0, u32x4& w0, u32x4& x1, u32x4& w1) {
  asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:2048\n\tds_read_b128 %2, %5\n\t"
               "ds_read_b128 %3, %5 offset:2048\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(x0), "=&v"(w0), "=&v"(x1), "=&v"(w1) : "v"(g0), "v"(g1) : "memory");
}
__device__ __forceinline__ float ldf(__amdgpu_buffer_rsrc_t r, unsigned off) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
}

// acc += A B over the 8 reduced channels that 4 channels per lane hold: half a wave owns channels 0-3, the other half
// 4-7 (which channels an instruction multiplies is free as long as both operands agree)
__device__ __forceinline__ f32x16 mul(u32x4 w, u32x4 x, f32x16 acc) {
#pragma unroll
  for (int e = 0; e < 4; ++e)
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(w[e]), __uint_as_float(x[e]), acc, 0, 0, 0);
  return acc;
}

// w' = s w as [Cin][taps][Cout], slice `wg` of `nwg` (the fold kernel's values)
// (by the 64 * (KS - 4) threads of the waves that have no part in the epilogue)
__device__ __forceinline__ void emit_folded(const BnEpilogue& bn, const float* __restrict__ w, int wg, int nwg, int thr) {
  float* out = static_cast<float*>(bn.w_folded_out);
  const unsigned P = (unsigned)bn.Cout * bn.taps * bn.Cin;
  const unsigned per = (P + nwg - 1) / nwg;
  const unsigned end = min(P, (wg + 1) * per);
  for (unsigned j = wg * per + thr; j < end; j += 64 * (KS - 4)) {
    const unsigned rest = j / bn.Cout, co = j - rest * bn.Cout;
    const unsigned ci = rest / bn.taps, tap = rest - ci * bn.taps;
    const float s = bn.gamma[co] / sqrtf(bn.var[co] + bn.eps);
    out[j] = w[((size_t)co * bn.taps + tap) * bn.Cin + ci] * s;
  }
}

// One 32 pixel x 32 channel tile.  WHOLE: C is a multiple of 4 (else operands are loaded element by element).
template <bool WHOLE>
__device__ __forceinline__ void conv_body(const WvParams& p, const int block, const int nblocks, unsigned char* smem) {
  float* s_lds = reinterpret_cast<float*>(smem + KS * WAVE_LDS);
  float* b_lds = s_lds + 32;
  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rt = block % p.rtiles;
  const int pc = block / p.rtiles;
  const int cls = pc / p.ptiles, pt = pc - cls * p.ptiles;
  const int r0 = rt * 32;

  // window of this tile's pixels: act row = P csh + ch0 + ti dth, weight tap (i0 + ti wsh) kW + (j0 + tj wsw)
  int csh = p.sh, csw = p.sw, ch0 = -p.ph, cw0 = -p.pw, dth = 1, i0 = 0, j0 = 0, wsh = 1, wsw = 1, kh = p.kH, kw = p.kW;
  int qH = p.oH, qW = p.oW, osh = 1, osw = 1, oh0 = 0, ow0 = 0;
  if (p.dgrad) {
    const int a = cls / p.ncw, b = cls - a * p.ncw;
    i0 = (a + p.ph) % p.sh; j0 = (b + p.pw) % p.sw;
    ch0 = (a + p.ph - i0) / p.sh; cw0 = (b + p.pw - j0) / p.sw;
    csh = csw = 1; dth = -1; wsh = p.sh; wsw = p.sw;
    kh = i0 < p.kH ? 1 + (p.kH - 1 - i0) / p.sh : 0;
    kw = j0 < p.kW ? 1 + (p.kW - 1 - j0) / p.sw : 0;
    qH = 1 + (p.oH - 1 - a) / p.sh;
    qW = 1 + (p.oW - 1 - b) / p.sw;
    osh = p.sh; osw = p.sw; oh0 = a; ow0 = b;
  }
  const int npix = p.N * qH * qW;
  if (pt * 32 >= npix) return;   // (the whole workgroup: a class smaller than the largest)

  if (tid < 32) {
    const int r = min(r0 + tid, p.R - 1);
    float s = 1.f, b = p.bias ? p.bias[r] : 0.f;
    if (p.bn.gamma) {
      s = p.bn.gamma[r] / sqrtf(p.bn.var[r] + p.bn.eps);
      b = ((p.bn.b ? p.bn.b[r] : 0.f) - p.bn.mean[r]) * s + p.bn.beta[r];
    }
    s_lds[tid] = s;
    b_lds[tid] = b;
  }

  struct Pixel { int n, P, Q; bool ok; };
  auto pixel = [&](int m) {
    Pixel x;
    x.ok = m < npix;
    const unsigned mm = (unsigned)(x.ok ? m : npix - 1);
    x.n = (int)(mm / (unsigned)(qH * qW));
    const unsigned rem = mm - (unsigned)(x.n * qH * qW);
    x.P = (int)(rem / (unsigned)qW);
    x.Q = (int)(rem - (unsigned)(x.P * qW));
    return x;
  };
  const Pixel px = pixel(pt * 32 + l32);   // this lane's pixel of the accumulator
  const __amdgpu_buffer_rsrc_t ra = make_rsrc(p.act, p.act_bytes), rw = make_rsrc(p.wgt, p.wgt_bytes);
  const unsigned wrow_bytes = (unsigned)(p.kH * p.kW * p.C) * 4u;

  // rows this lane loads: WHOLE 16-row copies (row 16 i + lane / 4), else its own pixel and channel
  constexpr int NR = WHOLE ? 2 : 1;
  int rn[NR], rh[NR], rwc[NR];
  unsigned wrow[NR];
  bool rok[NR];
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int row = WHOLE ? 16 * i + (lane >> 2) : l32;
    const Pixel x = pixel(pt * 32 + row);
    rn[i] = x.n; rok[i] = x.ok;
    rh[i] = x.P * csh + ch0; rwc[i] = x.Q * csw + cw0;
    wrow[i] = r0 + row < p.R ? (unsigned)(r0 + row) * wrow_bytes : OOB;
  }

  constexpr int CH = WHOLE ? 16 : 8;             // channels of a step
  const int nch = (p.C + CH - 1) / CH;
  const int total = kh * kw * nch;               // steps: (tap, channels)
  const int lo = total * wave / KS, n_mine = total * (wave + 1) / KS - lo;
  int tap = lo / nch, cc = lo - tap * nch;       // position of the next step to load
  int ti = kw > 0 ? tap / kw : 0, tj = tap - ti * kw;
  unsigned aoff[NR], woff[NR];
  auto enter_tap = [&] {
    const unsigned wtap = (unsigned)(((i0 + ti * wsh) * p.kW + j0 + tj * wsw) * p.C) * 4u;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int h = rh[i] + ti * dth, w = rwc[i] + tj * dth;
      const bool ok = rok[i] && (unsigned)h < (unsigned)p.aH && (unsigned)w < (unsigned)p.aW;
      aoff[i] = ok ? (unsigned)((rn[i] * p.aH + h) * p.aW + w) * (unsigned)p.C * 4u : OOB;
      woff[i] = wrow[i] + wtap;
    }
  };
  auto advance = [&] {
    if (++cc == nch) {
      cc = 0;
      if (++tj == kw) { tj = 0; ++ti; }
      enter_tap();   // (one tap past the last: never loaded from)
    }
  };
  enter_tap();

  f32x16 acc = {};
  unsigned char* const mine = smem + wave * WAVE_LDS;
  if constexpr (WHOLE) {
    // a stage's rows are 64 bytes, their four granules permuted by bits 2-3 of the row: sixteen rows' reads of one
    // granule then fall on all banks
    const int gran = (lane & 3) ^ ((lane >> 4) & 3);
    const unsigned read_row = lds_off(mine) + (unsigned)l32 * 64u;
    const unsigned sw = (unsigned)((l32 >> 2) & 3);
    const unsigned g0 = read_row + (((unsigned)half ^ sw) * 16u), g1 = read_row + (((2u + half) ^ sw) * 16u);
    auto copy = [&] {
      const int g = cc * 4 + gran;
      const bool in = g * 4 < p.C;
      unsigned char* const dst = mine;
#pragma unroll
      for (int i = 0; i < 2; ++i) dma16(ra, in ? aoff[i] + g * 16u : OOB, dst + i * 1024);
#pragma unroll
      for (int i = 0; i < 2; ++i) dma16(rw, in ? woff[i] + g * 16u : OOB, dst + 2048 + i * 1024);
      advance();
    };
    const int last_full = (p.C & 15) == 0 || (p.C & 15) > 8;   // the last step of a tap has more than 8 channels
    int mc = cc;                                              // channels step that is multiplied
    if (n_mine > 0) copy();
    for (int s = 0; s < n_mine; ++s) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      u32x4 x0, w0, x1, w1;
      lds_read_stage(g0, g1, x0, w0, x1, w1);
      if (s + 1 < n_mine) copy();
      acc = mul(w0, x0, acc);
      if (mc + 1 < nch || last_full) acc = mul(w1, x1, acc);
      if (++mc == nch) mc = 0;
    }
  } else {
    constexpr int DEPTH = 4;   // steps in flight
    u32x4 xa[DEPTH], wa[DEPTH];
    auto load = [&](u32x4& x, u32x4& w) {
      const int c = cc * 8 + half * 4;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool in = c + e < p.C;
        x[e] = __float_as_uint(ldf(ra, in ? aoff[0] + (c + e) * 4 : OOB));
        w[e] = __float_as_uint(ldf(rw, in ? woff[0] + (c + e) * 4 : OOB));
      }
      advance();
    };
#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
      if (d < n_mine) load(xa[d], wa[d]);
    for (int it = 0; it < n_mine; it += DEPTH) {
#pragma unroll
      for (int d = 0; d < DEPTH; ++d) {
        if (it + d >= n_mine) break;
        acc = mul(wa[d], xa[d], acc);
        if (it + d + DEPTH < n_mine) load(xa[d], wa[d]);
      }
    }
  }

  // accumulator: lane = pixel l32, rows (channels) 8 q + 4 half + e in register 4 q + e; a wave leaves it where its
  // stages were
#pragma unroll
  for (int q = 0; q < 4; ++q)
    *reinterpret_cast<float4*>(mine + q * 1024 + lane * 16) = make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
  __syncthreads();
  if (wave >= 4) {
    if (p.bn.gamma && p.bn.w_folded_out) emit_folded(p.bn, static_cast<const float*>(p.wgt), block, nblocks, tid - 256);
    return;
  }
  float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    const float4 f = *reinterpret_cast<const float4*>(smem + s * WAVE_LDS + wave * 1024 + lane * 16);
    v[0] += f.x; v[1] += f.y; v[2] += f.z; v[3] += f.w;
  }
  const int rl = 8 * wave + 4 * half, rr = r0 + rl;
  if (!px.ok || rr >= p.R) return;
  // A tap in the padding takes no part in a pixel's sum (Sec. 3.1), but the product multiplies it with zeros, and zero
  // times an infinite weight is NaN: such a sum is formed again over the taps inside, up to its first NaN.  (8 images, 28 x 28, 64 -> 64
  // channels, forward and backward: 34.9 us without, 35.0 with.)
  const float nan = (v[0] + v[1]) + (v[2] + v[3]);
  if (__builtin_expect(nan != nan, 0)) {
    const int h0 = px.P * csh + ch0, w0 = px.Q * csw + cw0, h1 = h0 + (kh - 1) * dth, w1 = w0 + (kw - 1) * dth;
    const bool inside = (unsigned)h0 < (unsigned)p.aH && (unsigned)h1 < (unsigned)p.aH && (unsigned)w0 < (unsigned)p.aW &&
                        (unsigned)w1 < (unsigned)p.aW;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (inside || v[e] == v[e] || rr + e >= p.R) continue;
      float u = 0.f;
      for (int i = 0; i < kh && u == u; ++i)
        for (int j = 0; j < kw && u == u; ++j) {
          const int h = h0 + i * dth, w = w0 + j * dth;
          if ((unsigned)h >= (unsigned)p.aH || (unsigned)w >= (unsigned)p.aW) continue;
          const float* xp = static_cast<const float*>(p.act) + ((size_t)(px.n * p.aH + h) * p.aW + w) * p.C;
          const float* wp = static_cast<const float*>(p.wgt) +
                            ((size_t)((rr + e) * p.kH + i0 + i * wsh) * p.kW + j0 + j * wsw) * p.C;
          for (int c = 0; c < p.C; ++c) u = fmaf(xp[c], wp[c], u);
        }
      v[e] = u;
    }
  }
  const size_t o = ((size_t)(px.n * p.oH + px.P * osh + oh0) * p.oW + px.Q * osw + ow0) * p.R + rr;
  float* out = static_cast<float*>(p.out) + o;
  const float* add = p.add ? static_cast<const float*>(p.add) + o : nullptr;
  const float* mask = p.mask ? static_cast<const float*>(p.mask) + o : nullptr;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = v[e] * s_lds[rl + e] + b_lds[rl + e];
  if ((p.R & 3) == 0) {
    if (add) {
      const float4 t = *reinterpret_cast<const float4*>(add);
      v[0] += t.x; v[1] += t.y; v[2] += t.z; v[3] += t.w;
    }
    if (p.relu)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.f);
    if (mask) {
      const float4 t = *reinterpret_cast<const float4*>(mask);
      v[0] = t.x > 0.f ? v[0] : 0.f; v[1] = t.y > 0.f ? v[1] : 0.f;
      v[2] = t.z > 0.f ? v[2] : 0.f; v[3] = t.w > 0.f ? v[3] : 0.f;
    }
    *reinterpret_cast<float4*>(out) = make_float4(v[0], v[1], v[2], v[3]);
  } else {
    for (int e = 0; e < 4 && rr + e < p.R; ++e) {
      float u = v[e];
      if (add) u += add[e];
      if (p.relu) u = fmaxf(u, 0.f);
      if (mask) u = mask[e] > 0.f ? u : 0.f;
      out[e] = u;
    }
  }
}

// ---- weight gradient, fp32 -------------------------------------------------------------------------------
// dw'[co][tap][ci] = sum_m dZ[m][co] X[m (+) tap][ci] (Sec. 3.2.1), r[co] = sum_m dZ[m][co] (App. B).  The reduced index
// is the pixel: an instruction multiplies two pixels, half a wave each, and a load instruction is two rows of 32
// consecutive channels.  A workgroup owns 32 x 32 channel pairs of up to TG neighbouring taps (one dZ operand for all of
// them) over a slice of the pixels, its eight waves every eighth pair of pixels.
struct WgParams {
  const float* x; const float* dz;
  float* part;     // [slices][Cout][taps][Cin]
  float* r_part;   // [slices][Cout] or null
  unsigned x_bytes, dz_bytes;
  int Cin, Cout, H, W, Ho, Wo, M;
  int kH, kW, sh, sw, ph, pw;
  int nci, nco, ntg, per;   // tiles, tap groups, pixels of a slice
};

template <int TG>
__device__ __forceinline__ void wgrad_body(const WgParams& p, const int block, unsigned char* smem) {
  constexpr int WD = TG == 3 ? 3 : 4;   // pixel pairs in flight
  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int t = block;
  const int it_ci = t % p.nci; t /= p.nci;
  const int it_co = t % p.nco; t /= p.nco;
  const int tg = t % p.ntg, slice = t / p.ntg;
  const int taps = p.kH * p.kW;   // a multiple of TG
  const int co = it_co * 32 + l32, ci = it_ci * 32 + l32;
  const int m0 = slice * p.per, m1 = min(p.M, m0 + p.per);
  const __amdgpu_buffer_rsrc_t rx = make_rsrc(p.x, p.x_bytes), rz = make_rsrc(p.dz, p.dz_bytes);
  // the group's taps: TG neighbours of one window row (TG == 3: windows three wide), or one
  const int ti = tg * TG / p.kW, tj = tg * TG - ti * p.kW;
  f32x16 acc[TG] = {};
  float racc = 0.f;
  float za[WD], xa[WD][TG];
  int m = m0 + 2 * wave + half;
  int wo = (int)((unsigned)m % (unsigned)p.Wo), ho, n;
  {
    const int q = (int)((unsigned)m / (unsigned)p.Wo);
    ho = (int)((unsigned)q % (unsigned)p.Ho);
    n = (int)((unsigned)q / (unsigned)p.Ho);
  }
  const int step_w = 2 * KS % p.Wo, step_q = 2 * KS / p.Wo;   // 16 pixels further: rows and columns
  const int step_h = step_q % p.Ho, step_n = step_q / p.Ho;
  unsigned zoff = co < p.Cout ? (unsigned)(m * p.Cout + co) * 4u : OOB;
  const unsigned zstep = co < p.Cout ? (unsigned)(2 * KS * p.Cout) * 4u : 0u;
  const unsigned tap_bytes = (unsigned)p.Cin * 4u;
  auto load = [&](float& z, float (&x)[TG]) {
    const bool ok = m < m1;
    z = ldf(rz, ok ? zoff : OOB);
    const int h = ho * p.sh - p.ph + ti, w = wo * p.sw - p.pw + tj;
    const bool row_ok = ok && ci < p.Cin && (unsigned)h < (unsigned)p.H;
    const unsigned off = (unsigned)(((n * p.H + h) * p.W + w) * p.Cin + ci) * 4u;
#pragma unroll
    for (int u = 0; u < TG; ++u) x[u] = ldf(rx, row_ok && (unsigned)(w + u) < (unsigned)p.W ? off + u * tap_bytes : OOB);
    zoff += zstep;
    m += 2 * KS;
    wo += step_w; ho += step_h; n += step_n;
    if (wo >= p.Wo) { wo -= p.Wo; ++ho; }
    if (ho >= p.Ho) { ho -= p.Ho; ++n; }
  };
  const int steps = (m1 - m0 + 2 * KS - 1) / (2 * KS);
#pragma unroll
  for (int d = 0; d < WD; ++d)
    if (d < steps) load(za[d], xa[d]);
  for (int it = 0; it < steps; it += WD) {
#pragma unroll
    for (int d = 0; d < WD; ++d) {
      if (it + d >= steps) break;
      racc += za[d];
#pragma unroll
      for (int u = 0; u < TG; ++u) acc[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(za[d], xa[d][u], acc[u], 0, 0, 0);
      if (it + d + WD < steps) load(za[d], xa[d]);
    }
  }
  // accumulator: lane = input channel, rows (output channels) 8 (i / 4) + 4 half + i % 4
  float (*red)[16][64] = reinterpret_cast<float (*)[16][64]>(smem);
#pragma unroll
  for (int u = 0; u < TG; ++u) {
    if (u > 0) __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) red[wave][i][lane] = acc[u][i];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int i = wave + KS * e;
      float v = 0.f;
#pragma unroll
      for (int s = 0; s < KS; ++s) v += red[s][i][lane];
      const int c = it_co * 32 + 8 * (i >> 2) + 4 * half + (i & 3);
      if (__builtin_expect(v != v && c < p.Cout && ci < p.Cin, 0)) {   // (as in conv_body: an infinite dZ where the tap is in the padding)
        const int h0 = ti - p.ph, w0 = tj + u - p.pw;
        v = 0.f;
        for (int m = m0; m < m1 && v == v; ++m) {
          const int q = (int)((unsigned)m / (unsigned)p.Wo), img = (int)((unsigned)q / (unsigned)p.Ho);
          const int h = h0 + (q - img * p.Ho) * p.sh, w = w0 + (m - q * p.Wo) * p.sw;
          if ((unsigned)h >= (unsigned)p.H || (unsigned)w >= (unsigned)p.W) continue;
          v = fmaf(p.dz[(size_t)m * p.Cout + c], p.x[((size_t)(img * p.H + h) * p.W + w) * p.Cin + ci], v);
        }
      }
      if (c < p.Cout && ci < p.Cin)
        p.part[((size_t)slice * p.Cout + c) * taps * p.Cin + (size_t)(tg * TG + u) * p.Cin + ci] = v;
    }
  }
  if (p.r_part && it_ci == 0 && tg == 0) {   // (uniform over the workgroup)
    __syncthreads();
    red[wave][0][lane] = racc;
    __syncthreads();
    if (tid < 32 && it_co * 32 + tid < p.Cout) {
      float v = 0.f;
#pragma unroll
      for (int s = 0; s < KS; ++s) v += red[s][0][tid] + red[s][0][tid + 32];
      p.r_part[(size_t)slice * p.Cout + it_co * 32 + tid] = v;
    }
  }
}

constexpr int SMEM = KS * WAVE_LDS + 256;

template <bool WHOLE>
__global__ __launch_bounds__(64 * KS, 6) void wave_conv_kernel(WvParams p) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  conv_body<WHOLE>(p, blockIdx.x, gridDim.x, smem);
}
template <int TG>
__global__ __launch_bounds__(64 * KS, 6) void wave_wgrad_kernel(WgParams p) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  wgrad_body<TG>(p, blockIdx.x, smem);
}
// The two gradient passes are independent: one launch, the weight gradient's workgroups (the longer ones) first.
template <bool WHOLE, int TG>
__global__ __launch_bounds__(64 * KS, 6) void wave_pair_kernel(WgParams g, WvParams d, int ng) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  if ((int)blockIdx.x < ng) wgrad_body<TG>(g, blockIdx.x, smem);
  else conv_body<WHOLE>(d, blockIdx.x - ng, gridDim.x - ng, smem);
}

bool sizes_fit(const Geom& g) {
  const size_t lim = 0x7fffff00u;
  return (size_t)g.Min * g.Cin * 4 < lim && (size_t)g.M * g.Cout * 4 < lim && (size_t)g.Cout * g.K * 4 < lim;
}

WvParams fprop_params(const Geom& g) {
  WvParams p{};
  p.N = g.N; p.C = g.Cin; p.R = g.Cout; p.aH = g.Hin; p.aW = g.Win; p.oH = g.Hout; p.oW = g.Wout;
  p.kH = g.kH; p.kW = g.kW; p.sh = g.sh; p.sw = g.sw; p.ph = g.ph; p.pw = g.pw;
  p.act_bytes = (unsigned)((size_t)g.Min * g.Cin * 4);
  p.wgt_bytes = (unsigned)((size_t)g.Cout * g.K * 4);
  p.rtiles = ceil_div(g.Cout, 32);
  p.ptiles = ceil_div(g.M, 32);
  p.ncls = p.ncw = 1;
  p.relu = g.post_relu; p.mask = g.post_mask; p.add = g.post_add;
  return p;
}
WvParams dgrad_params(const Geom& g) {
  WvParams p{};
  p.dgrad = 1;
  p.N = g.N; p.C = g.Cout; p.R = g.Cin; p.aH = g.Hout; p.aW = g.Wout; p.oH = g.Hin; p.oW = g.Win;
  p.kH = g.kH; p.kW = g.kW; p.sh = g.sh; p.sw = g.sw; p.ph = g.ph; p.pw = g.pw;
  p.act_bytes = (unsigned)((size_t)g.M * g.Cout * 4);
  p.wgt_bytes = (unsigned)((size_t)g.Cout * g.K * 4);
  p.rtiles = ceil_div(g.Cin, 32);
  p.ptiles = ceil_div(g.N * (1 + (g.Hin - 1) / g.sh) * (1 + (g.Win - 1) / g.sw), 32);
  p.ncw = g.sw < g.Win ? g.sw : g.Win;
  p.ncls = (g.sh < g.Hin ? g.sh : g.Hin) * p.ncw;
  p.relu = g.post_relu; p.mask = g.post_mask; p.add = g.post_add;
  return p;
}
long long conv_blocks(const WvParams& p) { return (long long)p.ptiles * p.rtiles * p.ncls; }
constexpr long long MAX_BLOCKS = 0xffffffffLL / (64 * KS);   // a launch has fewer than 2^32 threads

// a tap group is a window row of a 3-wide window, else single taps
int tap_group(const Geom& g) { return g.kW == 3 ? 3 : 1; }
struct WgSplit { int slices, per; };
WgSplit wgrad_split(const Geom& g) {
  // one and a half workgroups per compute unit beside the input gradient's, no slice shorter than 64 pixels (four steps of a wave), and no more fp32 copies of
  // dw' than 16 MB: the fold-back reads them all
  const int units = ceil_div(g.Cin, 32) * ceil_div(g.Cout, 32) * ceil_div(g.kH * g.kW, tap_group(g));
  const size_t copy = (size_t)g.Cout * g.K * 4;
  int want = ceil_div(384, units);
  const int most = (int)(((size_t)16 << 20) / copy);
  if (want > most) want = most;
  if (want > ceil_div(g.M, 64)) want = ceil_div(g.M, 64);
  if (want < 1) want = 1;
  const int per = (ceil_div(g.M, want) + 2 * KS - 1) / (2 * KS) * (2 * KS);
  return {ceil_div(g.M, per), per};
}
WgParams wgrad_params(const Geom& g) {
  WgParams p{};
  p.Cin = g.Cin; p.Cout = g.Cout; p.H = g.Hin; p.W = g.Win; p.Ho = g.Hout; p.Wo = g.Wout; p.M = g.M;
  p.kH = g.kH; p.kW = g.kW; p.sh = g.sh; p.sw = g.sw; p.ph = g.ph; p.pw = g.pw;
  p.x_bytes = (unsigned)((size_t)g.Min * g.Cin * 4);
  p.dz_bytes = (unsigned)((size_t)g.M * g.Cout * 4);
  p.nci = ceil_div(g.Cin, 32); p.nco = ceil_div(g.Cout, 32); p.ntg = ceil_div(g.kH * g.kW, tap_group(g));
  p.per = wgrad_split(g).per;
  return p;
}
long long wgrad_blocks(const Geom& g, const WgParams& p) { return (long long)p.nci * p.nco * p.ntg * wgrad_split(g).slices; }

#define WAVE_LAUNCH(KERNEL, GRID, ...)                                                                            \
  do {                                                                                                            \
    static LdsLimitOnce lds_once;                                                                                 \
    if (hipError_t e = set_lds_limit_once(lds_once, reinterpret_cast<const void*>(&KERNEL), SMEM); e != hipSuccess) \
      return e;                                                                                                   \
    hipLaunchKernelGGL(KERNEL, dim3(GRID), dim3(64 * KS), SMEM, st, __VA_ARGS__);                                  \
    return hipGetLastError();                                                                                     \
  } while (0)

hipError_t launch_conv(const WvParams& p, hipStream_t st) {
  if (p.C % 4 == 0) WAVE_LAUNCH((wave_conv_kernel<true>), (unsigned)conv_blocks(p), p);
  WAVE_LAUNCH((wave_conv_kernel<false>), (unsigned)conv_blocks(p), p);
}

}  // namespace

bool wave_f32_supported(const Geom& g, int dtype) {
  if (dtype != CONVBN_F32 || !sizes_fit(g)) return false;
  return conv_blocks(fprop_params(g)) <= MAX_BLOCKS &&   // (the weight gradient's workgroups share the input gradient's launch)
         conv_blocks(dgrad_params(g)) + wgrad_blocks(g, wgrad_params(g)) <= MAX_BLOCKS;
}

hipError_t launch_fprop_wave(const Geom& g, const void* x, const void* w_krsc, const float* bias, void* z, hipStream_t st,
                             const BnEpilogue* bn) {
  WvParams p = fprop_params(g);
  p.act = x; p.wgt = w_krsc; p.bias = bias; p.out = z;
  if (bn) p.bn = *bn;
  return launch_conv(p, st);
}
hipError_t launch_dgrad_wave(const Geom& g, const void* dz, const void* w_crsk, const float* bias, void* dx,
                             hipStream_t st) {
  WvParams p = dgrad_params(g);
  p.act = dz; p.wgt = w_crsk; p.bias = bias; p.out = dx;
  return launch_conv(p, st);
}
int wave_wgrad_splits(const Geom& g) { return wgrad_split(g).slices; }
hipError_t launch_wgrad_wave(const Geom& g, const void* x, const void* dz, float* part, float* r_part, hipStream_t st) {
  WgParams p = wgrad_params(g);
  p.x = (const float*)x; p.dz = (const float*)dz; p.part = part; p.r_part = r_part;
  const int blocks = (int)wgrad_blocks(g, p);
  if (tap_group(g) == 3) WAVE_LAUNCH((wave_wgrad_kernel<3>), blocks, p);
  WAVE_LAUNCH((wave_wgrad_kernel<1>), blocks, p);
}
hipError_t launch_pair_wave(const Geom& g, const void* x, const void* dz, const void* w_crsk, void* dx, float* part,
                            float* r_part, hipStream_t st) {
  WgParams p = wgrad_params(g);
  p.x = (const float*)x; p.dz = (const float*)dz; p.part = part; p.r_part = r_part;
  WvParams d = dgrad_params(g);
  d.act = dz; d.wgt = w_crsk; d.out = dx;
  const int ng = (int)wgrad_blocks(g, p);
  const unsigned grid = ng + (unsigned)conv_blocks(d);
  const bool whole = g.Cout % 4 == 0;
  if (tap_group(g) == 3) {
    if (whole) WAVE_LAUNCH((wave_pair_kernel<true, 3>), grid, p, d, ng);
    WAVE_LAUNCH((wave_pair_kernel<false, 3>), grid, p, d, ng);
  }
  if (whole) WAVE_LAUNCH((wave_pair_kernel<true, 1>), grid, p, d, ng);
  WAVE_LAUNCH((wave_pair_kernel<false, 1>), grid, p, d, ng);
}

}  // namespace convbn
