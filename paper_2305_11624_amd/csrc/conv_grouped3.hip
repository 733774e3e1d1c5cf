// The three contractions of a grouped 3x3 block with groups of 4, 8, 16 or 32 channels (as many inputs as outputs), stride 1
// or 2, bf16 MFMA: the waves of a launch work on their own, without a tile that a workgroup shares.
//
// 32 consecutive channels hold whole groups, so the block is a stack of 32 -> 32 channel convolutions with a block-diagonal
// weight (conv_grouped.hip has the other widths and windows, and how that one works).  A wave takes one such chunk of 16
// (weight gradient: 32) neighbouring columns and slides down a strip of rows:
//  * forward / input gradient: the 18 weight fragments (9 taps x 2 x 16 output channels, 32 reduced channels each, zeros
//    outside the groups included) stay in registers; an input row is three fragments -- one per window column, 16 bytes of a
//    pixel per lane, loaded straight from memory two rows ahead, the overlap from the L1 -- and goes into the three output rows
//    that it reaches, 18 v_mfma_f32_16x16x32_bf16.  No LDS, no barrier.
//  * weight gradient: the reduced index is the pixel, so rows pass through LDS (a ring of the wave's own, filled by direct
//    copies) and are read with the transposing load; the fragments of the last three dZ rows stay in registers.
// What bounds them: these layers move 13-26 MB, a few microseconds of traffic, so a launch lasts as long as its chain of
// memory round trips.  The kernels that share a tile between the waves (fetch, barrier, LDS, multiply, store, in step, two
// or three tiles in a row) took 18.6, 18.6 and 17.5 us for the three passes of 256 channels at 28 x 28, 32 images; here forward
// takes 12.5, both gradients as one launch 19, and the fold is no launch: 58.4 -> 36 us a step (groups of 4, 128 channels at
// 56 x 56: 85 -> 47; 8 / stride 2 at 56 x 56: 86 -> 62; 32 at 7 x 7: 43 -> 34).  A third row ahead, and two chunks per workgroup so
// that it writes whole lines, were no faster.  Stores: streams_output and STREAM_GRAD in common.h.
#include "common.h"

namespace convbn {

namespace {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) void* lds_ptr_t;

constexpr unsigned INV = 1u << 30;   // row or column offset of nothing (reads zeros, stores are dropped); twice that still is
constexpr int CPX = 16;              // columns of a convolution wave
constexpr int WPX = 32;              // ... of a weight-gradient wave

__device__ __forceinline__ __amdgpu_buffer_rsrc_t g3_rsrc(const void* p, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ bf16x8 g3_load(__amdgpu_buffer_rsrc_t r, unsigned off) {
  return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
}
__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
// Workgroup ids are dealt round-robin over the 8 XCDs: consecutive logical numbers -- the chunks of the same pixels, which
// share cache lines, then neighbouring strips -- run on one XCD.
__device__ __forceinline__ int g3_logical(int id, int n) {
  const int per = n >> 3;
  return (n & 7) ? id : (id & 7) * per + (id >> 3);
}

struct G3Params {
  const bf16_t* a;      // the tensor with the halo: x, dZ (weight gradient: x)
  const bf16_t* y;      // weight gradient: dZ
  const bf16_t* w;      // forward: W [C][9][cg]; input gradient: w' [cg][9][C]
  bf16_t* out;
  float* part;          // weight gradient: [slices][C][9 cg]
  float* r_part;        // ... [slices][C] or null
  BnEpilogue bn;        // forward: the weight is unfolded (gamma == null: no BatchNorm, the bias b alone)
  int N, C, Ha, Wa, Ho, Wo, cg, lcg;
  int pa, pb;           // paddings of the window over a (input gradient, stride 1: of the rotated window)
  int u0, v0;           // stride 2, input gradient: first dZ row and column whose x positions a wave owns
  int R, nstrip, nseg, segw, items;   // items: strips x segments x images of a chunk
  int nchunk, nblk, bpc;              // chunks of 32 channels; workgroups in all and per chunk
};
struct G3Item { int n, h0, c0; };
__device__ __forceinline__ G3Item g3_item(const G3Params& p, int it) {
  const int seg = it % p.nseg, rest = it / p.nseg;
  return G3Item{rest / p.nstrip, rest % p.nstrip * p.R, seg * p.segw};
}

// The weight fragments of a chunk: lane row r = lane % 16 of fragment (t, o) is output channel (r / 4) 8 + o 4 + r % 4 -- so
// that a lane ends up with 8 consecutive channels of its pixel --, reduced channels 8 (lane / 16) ...  GRAD: from w', taps
// rotated if FLIP.  Every address is inside the weight; what is not in the channel's group is zeroed afterwards.
template <bool GRAD, bool FLIP>
__device__ __forceinline__ void g3_weights(const G3Params& p, int chunk, int lane, bf16x8 (&wf)[9][2]) {
  const int r = lane & 15, k0 = (lane >> 4) * 8;
  uint4 raw[9][2];
  if (!GRAD && p.cg == 4) {
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      const bf16_t* wr = p.w + (size_t)(chunk * 32 + (r >> 2) * 8 + o * 4 + (r & 3)) * 36;
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const uint2 v = *reinterpret_cast<const uint2*>(wr + t * 4);
        raw[t][o] = make_uint4(v.x, v.y, v.x, v.y);
      }
    }
  } else {
    const int step = GRAD ? p.C : p.cg;
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      const int ch = (r >> 2) * 8 + o * 4 + (r & 3);
      const bf16_t* wr = GRAD ? p.w + (size_t)(ch & (p.cg - 1)) * 9 * p.C + chunk * 32 + k0
                              : p.w + (size_t)(chunk * 32 + ch) * 9 * p.cg + (k0 & (p.cg - 1));
#pragma unroll
      for (int t = 0; t < 9; ++t) raw[t][o] = *reinterpret_cast<const uint4*>(wr + (FLIP ? 8 - t : t) * step);
    }
  }
#pragma unroll
  for (int o = 0; o < 2; ++o) {
    const int g = ((r >> 2) * 8 + o * 4 + (r & 3)) >> p.lcg;
    const bool lo = (k0 >> p.lcg) == g, hi = ((k0 + 4) >> p.lcg) == g;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const uint4 v = raw[t][o];
      wf[t][o] = __builtin_bit_cast(bf16x8, make_uint4(lo ? v.x : 0u, lo ? v.y : 0u, hi ? v.z : 0u, hi ? v.w : 0u));
    }
  }
}
// s and b' of the lane's 8 channels
__device__ __forceinline__ void g3_scale(const G3Params& p, int ch, float (&s)[8], float (&b)[8]) {
  if (!p.bn.gamma) {   // (an unscaled convolution)
#pragma unroll
    for (int e = 0; e < 8; ++e) { s[e] = 1.f; b[e] = p.bn.b ? p.bn.b[ch + e] : 0.f; }
    return;
  }
  const float* const bp = p.bn.b ? p.bn.b : p.bn.mean;
  float4 ga[2], va[2], me[2], be[2], bi[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    ga[h] = *reinterpret_cast<const float4*>(p.bn.gamma + ch + 4 * h);
    va[h] = *reinterpret_cast<const float4*>(p.bn.var + ch + 4 * h);
    me[h] = *reinterpret_cast<const float4*>(p.bn.mean + ch + 4 * h);
    be[h] = *reinterpret_cast<const float4*>(p.bn.beta + ch + 4 * h);
    bi[h] = *reinterpret_cast<const float4*>(bp + ch + 4 * h);
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    auto at = [&](const float4 (&v)[2]) { const float4 q = v[e >> 2]; return (e & 3) == 0 ? q.x : (e & 3) == 1 ? q.y : (e & 3) == 2 ? q.z : q.w; };
    s[e] = at(ga) / sqrtf(at(va) + p.bn.eps);
    b[e] = ((p.bn.b ? at(bi) : 0.f) - at(me)) * s[e] + at(be);
  }
}
// w' = s w as [cg][9][C] from the fragments: the workgroups of a chunk store a window position each
__device__ __forceinline__ void g3_emit_folded(const G3Params& p, int chunk, int wg, int lane, const bf16x8 (&wf)[9][2]) {
  const int r = lane & 15, k0 = (lane >> 4) * 8;
  bf16_t* const out = static_cast<bf16_t*>(p.bn.w_folded_out);
#pragma unroll
  for (int o = 0; o < 2; ++o) {
    const int chl = (r >> 2) * 8 + o * 4 + (r & 3), ch = chunk * 32 + chl;
    const float s = p.bn.gamma[ch] / sqrtf(p.bn.var[ch] + p.bn.eps);
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      if (wg != t % p.bpc) continue;
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if ((k0 + e) >> p.lcg == chl >> p.lcg)
          out[((size_t)((k0 + e) & (p.cg - 1)) * 9 + t) * p.C + ch] = (bf16_t)((float)wf[t][o][e] * s);
    }
  }
}

template <bool EPI, bool STREAM>
__device__ __forceinline__ void g3_store(__amdgpu_buffer_rsrc_t r, unsigned off, const f32x4 (&acc)[2], const float (&s)[8],
                                         const float (&b)[8]) {
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = EPI ? fmaf(acc[e >> 2][e & 3], s[e], b[e]) : acc[e >> 2][e & 3];
  const u32x4 t = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
  __builtin_amdgcn_raw_buffer_store_b128(t, r, (int)off, 0, STREAM ? 2 : 0);
}

// Stride 1 (GRAD: the input gradient, a = dZ with the rotated window) and the strided forward pass (S = 2).
template <int S, bool GRAD, bool STREAM>
__device__ __forceinline__ void g3_conv_body(const G3Params& p, const int block) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lb = g3_logical(block, p.nblk);
  const int chunk = lb % p.nchunk, wg = lb / p.nchunk;
  const int col = lane & 15, kq = lane >> 4;
  const unsigned px = (unsigned)p.C * 2u, arow = px * p.Wa, orow = px * p.Wo;
  const __amdgpu_buffer_rsrc_t ra = g3_rsrc(p.a, (size_t)p.N * p.Ha * arow), ro = g3_rsrc(p.out, (size_t)p.N * p.Ho * orow);
  const unsigned lane_ch = (unsigned)(chunk * 64 + kq * 16);
  bf16x8 wf[9][2];
  float s[8], b[8];
  g3_weights<GRAD, GRAD>(p, chunk, lane, wf);
  if constexpr (!GRAD) g3_scale(p, chunk * 32 + kq * 8, s, b);
  constexpr int D = S == 1 ? 2 : 1;            // rows (stride 2: pairs of rows) requested ahead
  constexpr int NR = S;                        // rows of a step
  for (int it = wg * 4 + wave; it < p.items; it += p.bpc * 4) {
    const G3Item im = g3_item(p, it);
    unsigned acol[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const int w = (im.c0 + col) * S + j - p.pb;
      acol[j] = col < p.segw && (unsigned)w < (unsigned)p.Wa ? (unsigned)w * px : INV;
    }
    const unsigned ocol = col < p.segw && im.c0 + col < p.Wo ? (unsigned)(im.c0 + col) * px + lane_ch : INV;
    const int rows = min(p.Ho - im.h0, p.R);
    // steps: stride 1, q = 0 .. rows + 1 brings input row h0 + q - pa; stride 2, q = 0 .. rows brings window rows 1 and 2 of
    // output row h0 + q - 1 (the second is row 0 of the next one)
    const int nq = S == 1 ? rows + 2 : rows + 1;
    int ha = S == 1 ? im.h0 - p.pa : (im.h0 - 1) * 2 + 1 - p.pa;
    const int hend = min(p.Ha, ha + nq * NR);
    unsigned aoff = ((unsigned)im.n * p.Ha + (unsigned)ha) * arow + lane_ch;
    unsigned ooff = ((unsigned)im.n * p.Ho + (unsigned)im.h0) * orow - (S == 1 ? 2u : 1u) * orow;
    bf16x8 fb[D][NR][3];
    auto fetch = [&](int slot) {   // (rows past the last one are nothing)
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        const unsigned r = (unsigned)ha < (unsigned)hend ? aoff : INV;
        ++ha;
        aoff += arow;
#pragma unroll
        for (int j = 0; j < 3; ++j) fb[slot][i][j] = g3_load(ra, r + acol[j]);
      }
    };
#pragma unroll
    for (int d = 0; d < D; ++d) fetch(d);
    f32x4 acc[3][2];
    constexpr int U = S == 1 ? 6 : 2;
    for (int q0 = 0; q0 < nq; q0 += U) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = q0 + u;
        if (q >= nq) break;
        bf16x8 cur[NR][3];
#pragma unroll
        for (int i = 0; i < NR; ++i)
#pragma unroll
          for (int j = 0; j < 3; ++j) cur[i][j] = fb[u % D][i][j];
        fetch(u % D);
        if constexpr (S == 1) {
#pragma unroll
          for (int o = 0; o < 2; ++o) acc[u % 3][o] = f32x4{0.f, 0.f, 0.f, 0.f};
          if (q == 0) {
#pragma unroll
            for (int o = 0; o < 2; ++o) acc[(u + 1) % 3][o] = acc[(u + 2) % 3][o] = f32x4{0.f, 0.f, 0.f, 0.f};
          }
#pragma unroll
          for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int i = 0; i < 3; ++i)   // window row i of output row q - i
#pragma unroll
              for (int o = 0; o < 2; ++o) acc[(u + 3 - i) % 3][o] = mfma(wf[i * 3 + j][o], cur[0][j], acc[(u + 3 - i) % 3][o]);
          const unsigned r = (unsigned)(q - 2) < (unsigned)rows ? ooff : INV;
          ooff += orow;
          g3_store<!GRAD, STREAM>(ro, r + ocol, acc[(u + 1) % 3], s, b);
        } else {
          if (q == 0) {
#pragma unroll
            for (int o = 0; o < 2; ++o) acc[u % 2][o] = f32x4{0.f, 0.f, 0.f, 0.f};
          }
#pragma unroll
          for (int o = 0; o < 2; ++o) acc[(u + 1) % 2][o] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int o = 0; o < 2; ++o) {
              acc[u % 2][o] = mfma(wf[3 + j][o], cur[0][j], acc[u % 2][o]);
              acc[(u + 1) % 2][o] = mfma(wf[j][o], cur[NR - 1][j], acc[(u + 1) % 2][o]);
              acc[u % 2][o] = mfma(wf[6 + j][o], cur[NR - 1][j], acc[u % 2][o]);
            }
          const unsigned r = (unsigned)(q - 1) < (unsigned)rows ? ooff : INV;
          ooff += orow;
          g3_store<!GRAD, STREAM>(ro, r + ocol, acc[u % 2], s, b);
        }
      }
    }
  }
  if constexpr (!GRAD) {   // (behind the rows: nobody waits for it)
    if (p.bn.w_folded_out && wave == 0) g3_emit_folded(p, chunk, wg, lane, wf);
  }
}
template <int S, bool GRAD, bool STREAM>
__global__ __launch_bounds__(256, 2) void g3_conv_kernel(G3Params p) {
  g3_conv_body<S, GRAD, STREAM>(p, blockIdx.x);
}

// Stride 2, input gradient.  In coordinates that count the padding (hh = h + ph), dZ row v reaches hh = 2v, 2v + 1, 2v + 2: a
// lane that owns dZ column u writes the dx columns 2u + 1 (window column 1 of u) and 2u + 2 (column 2 of u, 0 of u + 1), and
// a step the rows 2v + 1 and 2v + 2 likewise; u and v start at u0 and v0 (-1 with padding 0).
__global__ __launch_bounds__(256, 2) void g3_dgrad_s2_kernel(G3Params p) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lb = g3_logical(blockIdx.x, p.nblk);
  const int chunk = lb % p.nchunk, wg = lb / p.nchunk;
  const int col = lane & 15, kq = lane >> 4;
  const unsigned px = (unsigned)p.C * 2u, arow = px * p.Wa, orow = px * p.Wo;
  const __amdgpu_buffer_rsrc_t ra = g3_rsrc(p.a, (size_t)p.N * p.Ha * arow), ro = g3_rsrc(p.out, (size_t)p.N * p.Ho * orow);
  const unsigned lane_ch = (unsigned)(chunk * 64 + kq * 16);
  bf16x8 wf[9][2];
  g3_weights<true, false>(p, chunk, lane, wf);
  const float none[8] = {};
  for (int it = wg * 4 + wave; it < p.items; it += p.bpc * 4) {
    const G3Item im = g3_item(p, it);
    const int u = p.u0 + im.c0 + col, v0 = p.v0 + im.h0;
    unsigned acol[2], ocol[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      acol[k] = col < p.segw && (unsigned)(u + k) < (unsigned)p.Wa ? (unsigned)(u + k) * px + lane_ch : INV;
      const int w = 2 * u + 1 + k - p.pb;
      ocol[k] = col < p.segw && (unsigned)w < (unsigned)p.Wo ? (unsigned)w * px + lane_ch : INV;
    }
    const unsigned abase = (unsigned)im.n * p.Ha * arow, obase = (unsigned)im.n * p.Ho * orow;
    auto load_row = [&](int v, bool want, bf16x8 (&f)[2]) {
      const unsigned r = want && (unsigned)v < (unsigned)p.Ha ? abase + (unsigned)v * arow : INV;
#pragma unroll
      for (int k = 0; k < 2; ++k) f[k] = g3_load(ra, r + acol[k]);
    };
    bf16x8 f0[2], f1[2], nxt[2];   // dZ rows v, v + 1, v + 2
    load_row(v0, true, f0);
    load_row(v0 + 1, true, f1);
    load_row(v0 + 2, p.R > 1, nxt);
    for (int q = 0; q < p.R; ++q) {
      const int v = v0 + q;
      bf16x8 far[2];
      load_row(v + 3, q + 2 < p.R, far);
      f32x4 acc[2][2][2];   // [row][column][channel tile]
#pragma unroll
      for (int o = 0; o < 2; ++o) {
        const f32x4 z = {0.f, 0.f, 0.f, 0.f};
        acc[0][0][o] = mfma(wf[4][o], f0[0], z);
        acc[0][1][o] = mfma(wf[3][o], f0[1], mfma(wf[5][o], f0[0], z));
        acc[1][0][o] = mfma(wf[1][o], f1[0], mfma(wf[7][o], f0[0], z));
        acc[1][1][o] = mfma(wf[0][o], f1[1], mfma(wf[2][o], f1[0], mfma(wf[6][o], f0[1], mfma(wf[8][o], f0[0], z))));
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int h = 2 * v + 1 + i - p.pa;
        const unsigned r = (unsigned)h < (unsigned)p.Ho ? obase + (unsigned)h * orow : INV;
#pragma unroll
        for (int k = 0; k < 2; ++k) g3_store<false, STREAM_GRAD>(ro, r + ocol[k], acc[i][k], none, none);
      }
#pragma unroll
      for (int k = 0; k < 2; ++k) { f0[k] = f1[k]; f1[k] = nxt[k]; nxt[k] = far[k]; }
    }
  }
}

// ---- weight gradient
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bf16x8 g3_join(i32x2 a, i32x2 b) {
  const i32x4 v = {a[0], a[1], b[0], b[1]};
  return __builtin_bit_cast(bf16x8, v);
}
// Fragments (8 pixels of a channel per lane: two transposing reads, the second four pixels on) of a row's two 16-channel
// tiles, 32 bytes apart: of one window column (z), and of three, 64 bytes apart (x, pixels S apart).  Inline asm: the
// compiler would hold every LDS read until the copies in flight have landed.  The wait is in the same block: registers that a
// read still writes are nothing the compiler knows of.
__device__ __forceinline__ void g3_read_z(unsigned a, bf16x8 (&f)[2]) {
  i32x2 r[4];
  asm volatile("ds_read_b64_tr_b16 %0, %4\n\tds_read_b64_tr_b16 %1, %4 offset:256\n\t"
               "ds_read_b64_tr_b16 %2, %4 offset:32\n\tds_read_b64_tr_b16 %3, %4 offset:288\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]) : "v"(a) : "memory");
  f[0] = g3_join(r[0], r[1]);
  f[1] = g3_join(r[2], r[3]);
}
template <int S>
__device__ __forceinline__ void g3_read_x(unsigned a, bf16x8 (&f)[3][2]) {
  i32x2 r[12];
  asm volatile("ds_read_b64_tr_b16 %0, %12\n\tds_read_b64_tr_b16 %1, %12 offset:%13\n\t"
               "ds_read_b64_tr_b16 %2, %12 offset:32\n\tds_read_b64_tr_b16 %3, %12 offset:%13+32\n\t"
               "ds_read_b64_tr_b16 %4, %12 offset:64\n\tds_read_b64_tr_b16 %5, %12 offset:%13+64\n\t"
               "ds_read_b64_tr_b16 %6, %12 offset:96\n\tds_read_b64_tr_b16 %7, %12 offset:%13+96\n\t"
               "ds_read_b64_tr_b16 %8, %12 offset:128\n\tds_read_b64_tr_b16 %9, %12 offset:%13+128\n\t"
               "ds_read_b64_tr_b16 %10, %12 offset:160\n\tds_read_b64_tr_b16 %11, %12 offset:%13+160\n\t"
               "s_waitcnt lgkmcnt(0)"
               : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7]),
                 "=&v"(r[8]), "=&v"(r[9]), "=&v"(r[10]), "=&v"(r[11])
               : "v"(a), "n"(4 * S * 64) : "memory");
#pragma unroll
  for (int j = 0; j < 3; ++j)
#pragma unroll
    for (int k = 0; k < 2; ++k) f[j][k] = g3_join(r[(j * 2 + k) * 2], r[(j * 2 + k) * 2 + 1]);
}
template <int N> __device__ __forceinline__ void g3_wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

template <int S>
struct G3Wg {
  static constexpr int XPX = S == 1 ? 48 : 80;            // pixels of a staged x row (34 / 65 used), 16 a copy
  static constexpr int XROW = XPX * 64, ZROW = WPX * 64;
  static constexpr int STAGE = ZROW + S * XROW;
  static constexpr int NST = S == 1 ? 4 : 3;
  static constexpr int COPIES = WPX / 16 + S * (XPX / 16);   // of a step
  static constexpr int WAVE = NST * STAGE;
  static constexpr int LDS = 4 * WAVE;
};

// dw'[o][i][j][q] = sum over the pixels of dZ[pixel][o] X[pixel (i, j)][group(o) cg + q], r[o] = sum dZ.  A step brings a dZ row
// and the S x rows that end its windows; NT: pairs of 16-channel tiles (2: groups within a tile; 4: groups of 32).
// Zeros stand for what is outside, and an infinity times zero is no zero: products of rows that have no partner in the strip are
// skipped, and x pixels beside the segment's last windows are cleared where they would meet the zeros behind its dZ.  An
// infinite x then stays with the taps that touch it; an infinite dZ also reaches the taps whose column is in the padding.
template <int S, int NT>
__device__ __forceinline__ void g3_wgrad_body(const G3Params& p, const int block, unsigned char* smem) {
  using L = G3Wg<S>;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lb = g3_logical(block, p.nblk);
  const int chunk = lb % p.nchunk, wg = lb / p.nchunk;
  unsigned char* const ring = smem + wave * L::WAVE;
  const unsigned px = (unsigned)p.C * 2u, xrow = px * p.Wa, zrow = px * p.Wo;
  const __amdgpu_buffer_rsrc_t rx = g3_rsrc(p.a, (size_t)p.N * p.Ha * xrow), rz = g3_rsrc(p.y, (size_t)p.N * p.Ho * zrow);
  const int cpix = lane >> 2;                                        // copy: pixel of 16, 16-byte granule of its 64 bytes
  const unsigned cgr = (unsigned)(chunk * 64 + (lane & 3) * 16);
  // transposing read: group lane / 16 takes pixels 8 g .. 8 g + 7, the lane addresses pixel (lane % 16) / 4, quad lane % 4
  const int rpix = (lane >> 4) * 8 + ((lane & 15) >> 2);
  const unsigned ring_at = (unsigned)(size_t)(lds_ptr_t)ring;
  const unsigned zread = ring_at + rpix * 64 + (lane & 3) * 8, xread = ring_at + L::ZROW + rpix * S * 64 + (lane & 3) * 8;
  f32x4 acc[9][NT], racc[2];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int k = 0; k < NT; ++k) acc[t][k] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < 2; ++k) racc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
  const s16x8 one_bits = {0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80};
  const bf16x8 ones = __builtin_bit_cast(bf16x8, one_bits);

  for (int it = wg * 4 + wave; it < p.items; it += p.bpc * 4) {
    const G3Item im = g3_item(p, it);
    const int rows = min(p.Ho - im.h0, p.R), cols = min(p.Wo - im.c0, p.segw);
    unsigned xcol[L::XPX / 16], zcol[WPX / 16];
#pragma unroll
    for (int k = 0; k < L::XPX / 16; ++k) {
      const int c = k * 16 + cpix, w = im.c0 * S + c - p.pb;
      xcol[k] = c < (cols - 1) * S + 3 && (unsigned)w < (unsigned)p.Wa ? (unsigned)w * px + cgr : INV;
    }
#pragma unroll
    for (int k = 0; k < WPX / 16; ++k) {
      const int c = k * 16 + cpix;
      zcol[k] = c < cols ? (unsigned)(im.c0 + c) * px + cgr : INV;
    }
    // the lane's pixels (two a register) that have a dZ: what window columns below 3 - S read behind them is real x
    unsigned own[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const int left = cols - ((lane >> 4) * 8 + 2 * d);
      own[d] = left >= 2 ? 0xffffffffu : left == 1 ? 0xffffu : 0u;
    }
    // step q: dZ row h0 + q and the x rows S (h0 + q) + i - pa, stride 1: i = 0; stride 2: i = -1 and 0
    const int nq = S == 1 ? rows + 2 : rows + 1;
    int hx = im.h0 * S - p.pa - (S - 1), hq = hx, qf = 0;
    const int xend = min(p.Ha, hx + nq * S);
    unsigned xoff = ((unsigned)im.n * p.Ha + (unsigned)hx) * xrow, zoff = ((unsigned)im.n * p.Ho + (unsigned)im.h0) * zrow;
    unsigned fill = 0, read = 0;   // byte offsets of the stages that are filled and read next
    auto next = [](unsigned o) { return o + L::STAGE == (unsigned)L::WAVE ? 0u : o + L::STAGE; };
    auto fetch = [&]() {
      unsigned char* const st = ring + fill;
      fill = next(fill);
      const unsigned z = qf < rows ? zoff : INV;
      ++qf;
      zoff += zrow;
#pragma unroll
      for (int k = 0; k < WPX / 16; ++k) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rz, (lds_ptr_t)(st + k * 1024), 16, (int)(z + zcol[k]), 0, 0, 0);
        asm volatile("" ::: "memory");
      }
#pragma unroll
      for (int i = 0; i < S; ++i) {
        const unsigned x = (unsigned)hx < (unsigned)xend ? xoff : INV;
        ++hx;
        xoff += xrow;
#pragma unroll
        for (int k = 0; k < L::XPX / 16; ++k) {
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_ptr_t)(st + L::ZROW + i * L::XROW + k * 1024), 16, (int)(x + xcol[k]), 0, 0, 0);
          asm volatile("" ::: "memory");
        }
      }
    };
#pragma unroll
    for (int d = 0; d < L::NST - 1; ++d) fetch();
    bf16x8 zf[3][2];   // dZ rows q, q - 1, q - 2
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int k = 0; k < 2; ++k) zf[d][k] = bf16x8{};
    for (int q = 0; q < nq; ++q) {
      g3_wait_vm<L::COPIES * (L::NST - 2)>();   // this step's rows have landed (the later steps' may be in flight)
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        zf[2][k] = zf[1][k];
        zf[1][k] = zf[0][k];
      }
      bf16x8 xf[S][3][2];
      g3_read_z(zread + read, zf[0]);
#pragma unroll
      for (int i = 0; i < S; ++i) {
        g3_read_x<S>(xread + read + i * L::XROW, xf[i]);
#pragma unroll
        for (int j = 0; j < 3 - S; ++j)
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            const uint4 v = __builtin_bit_cast(uint4, xf[i][j][k]);
            xf[i][j][k] = __builtin_bit_cast(bf16x8, make_uint4(v.x & own[0], v.y & own[1], v.z & own[2], v.w & own[3]));
          }
      }
      read = next(read);
      fetch();   // (into the stage that the step before read: its multiplies have its operands)
#pragma unroll
      for (int k = 0; k < 2; ++k) racc[k] = mfma(ones, zf[0][k], racc[k]);   // (steps past the strip read zeros)
      // stride 1: x row q is window row i of dZ row q - i;  stride 2: the first is row 1 of dZ row q - 1, the second row 2 of it
      // and row 0 of dZ row q
      auto prods = [&](int tap_row, const bf16x8 (&x)[3][2], const bf16x8 (&z)[2]) {
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
          for (int k = 0; k < NT; ++k)
            acc[tap_row * 3 + j][k] = mfma(x[j][NT == 2 ? k : k >> 1], z[NT == 2 ? k : k & 1], acc[tap_row * 3 + j][k]);
      };
      const bool x0 = (unsigned)hq < (unsigned)p.Ha, x1 = (unsigned)(hq + S - 1) < (unsigned)p.Ha;   // the step's first, last x row
      hq += S;
      if (x1 && q < rows) prods(0, xf[S - 1], zf[0]);
      if (x0 && q >= 1 && q <= rows) prods(1, xf[0], zf[1]);
      if (x1 && (S == 1 ? q >= 2 : q >= 1)) prods(2, xf[S - 1], zf[S == 1 ? 2 : 1]);
    }
    g3_wait_vm<0>();   // the ring is refilled by the next strip
  }

  // ---- the four waves' sums, three taps at a time, through LDS; lane l of tile pair k: output channel (tile) l % 16, input
  // channels 4 (l / 16) .. + 3 of its tile
  const int K = 9 * p.cg, tid = threadIdx.x;
  float4* const red = reinterpret_cast<float4*>(smem);   // [wave][3 NT][64]
  __syncthreads();
#pragma unroll
  for (int t0 = 0; t0 < 9; t0 += 3) {
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int k = 0; k < NT; ++k)
        red[(wave * 3 * NT + t * NT + k) * 64 + lane] = __builtin_bit_cast(float4, acc[t0 + t][k]);
    __syncthreads();
    for (int e = tid; e < 3 * NT * 64; e += 256) {
      const int l = e & 63, k = (e >> 6) % NT, t = (e >> 6) / NT;
      float4 v = red[e];
#pragma unroll
      for (int w = 1; w < 4; ++w) {
        const float4 o = red[w * 3 * NT * 64 + e];
        v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w;
      }
      const int co = (NT == 2 ? k : k & 1) * 16 + (l & 15), ci = (NT == 2 ? k : k >> 1) * 16 + (l >> 4) * 4;
      if (ci >> p.lcg == co >> p.lcg)
        *reinterpret_cast<float4*>(p.part + ((size_t)wg * p.C + chunk * 32 + co) * K + (t0 + t) * p.cg + (ci & (p.cg - 1))) = v;
    }
    __syncthreads();
  }
  if (p.r_part) {
    float* const rr = reinterpret_cast<float*>(smem);
    if (lane < 16) { rr[wave * 32 + lane] = racc[0][0]; rr[wave * 32 + 16 + lane] = racc[1][0]; }   // (all rows are the sum)
    __syncthreads();
    if (tid < 32) p.r_part[(size_t)wg * p.C + chunk * 32 + tid] = (rr[tid] + rr[32 + tid]) + (rr[64 + tid] + rr[96 + tid]);
  }
}

template <int S, int NT>
__global__ __launch_bounds__(256, 2) void g3_wgrad_kernel(G3Params p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  g3_wgrad_body<S, NT>(p, blockIdx.x, smem);
}
// Both gradients of a stride-1 block: compute units that are done with the one take workgroups of the other.  (Stride 2: the
// weight gradient's ring leaves no room for a second workgroup.)
template <int NT>
__global__ __launch_bounds__(256, 2) void g3_pair_kernel(G3Params wg, G3Params dg) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  if ((int)blockIdx.x < wg.nblk) g3_wgrad_body<1, NT>(wg, blockIdx.x, smem);
  else g3_conv_body<1, true, STREAM_GRAD>(dg, blockIdx.x - wg.nblk);
}

// ---- host side
struct G3Plan { bool ok; int R, nstrip, nseg, segw, items, bpc; };
// `rows` x `cols` positions per image; `extra`: what a strip costs besides its rows; `wgs`: workgroups that the chip holds
G3Plan g3_plan(const Geom& g, int rows, int cols, int px, int extra, int wgs) {
  G3Plan p{};
  const int nchunk = g.Cin / 32;
  p.nseg = ceil_div(cols, px);
  p.segw = ceil_div(cols, p.nseg);
  int bpc = wgs / nchunk;
  if (bpc < 1) bpc = 1;
  long long best = -1;
  for (int ns = 1; ns <= rows; ++ns) {
    const int R = ceil_div(rows, ns);
    if (ceil_div(rows, R) != ns) continue;
    const long long items = (long long)g.N * ns * p.nseg;
    const long long cost = ((items + 4LL * bpc - 1) / (4LL * bpc)) * (R + extra);
    if (best < 0 || cost < best) { best = cost; p.R = R; }
  }
  p.nstrip = ceil_div(rows, p.R);
  p.items = g.N * p.nstrip * p.nseg;
  p.bpc = ceil_div(p.items, 4 * ceil_div(p.items, 4 * bpc));
  p.ok = true;
  return p;
}
int g3_first(int pad) { return pad == 0 ? -1 : 0; }   // stride 2: the first dZ row (column) that owns x rows
int g3_span(int in, int out, int pad) {               // ... and how many there are
  int last = (in - 1 + pad - 1) / 2;
  if (last < out - 1) last = out - 1;
  return last - g3_first(pad) + 1;
}
G3Plan g3_fprop_plan(const Geom& g) {
  return planned<G3Plan>(g, CONVBN_BF16, [&] { return g3_plan(g, g.Hout, g.Wout, CPX, g.sh == 1 ? 4 : 2, 512); });
}
G3Plan g3_dgrad_plan(const Geom& g) {
  return planned<G3Plan>(g, CONVBN_BF16, [&] {
    if (g.sh == 1) return g3_plan(g, g.Hin, g.Win, CPX, 4, 512);
    return g3_plan(g, g3_span(g.Hin, g.Hout, g.ph), g3_span(g.Win, g.Wout, g.pw), CPX, 2, 512);
  });
}
G3Plan g3_wgrad_plan(const Geom& g) {
  return planned<G3Plan>(g, CONVBN_BF16, [&] { return g3_plan(g, g.Hout, g.Wout, WPX, g.sh == 1 ? 4 : 3, g.sh == 1 ? 512 : 256); });
}
G3Params g3_params(const Geom& g, int groups, const G3Plan& pl) {
  G3Params p{};
  p.N = g.N; p.C = g.Cin;
  p.cg = g.Cin / groups;
  p.lcg = p.cg == 4 ? 2 : p.cg == 8 ? 3 : p.cg == 16 ? 4 : 5;
  p.R = pl.R; p.nstrip = pl.nstrip; p.nseg = pl.nseg; p.segw = pl.segw; p.items = pl.items;
  p.nchunk = g.Cin / 32;
  p.bpc = pl.bpc;
  p.nblk = p.nchunk * p.bpc;
  return p;
}

}  // namespace

bool g3_supported(const Geom& g, int groups, int dtype) {
  const int cg = g.Cin / groups;
  return dtype == CONVBN_BF16 && g.Cin == g.Cout && g.Cin % 32 == 0 && (cg == 4 || cg == 8 || cg == 16 || cg == 32) && g.kH == 3 &&
         g.kW == 3 && g.sh == g.sw && (g.sh == 1 || g.sh == 2) && g.ph <= 2 && g.pw <= 2 && (size_t)g.Min * g.Cin * 2 < INV &&
         (size_t)g.M * g.Cin * 2 < INV;
}
hipError_t launch_g3_fprop(const Geom& g, int groups, const void* x, const void* W, const BnEpilogue& bn, void* z, hipStream_t st) {
  const G3Plan pl = g3_fprop_plan(g);
  G3Params p = g3_params(g, groups, pl);
  p.a = (const bf16_t*)x; p.w = (const bf16_t*)W; p.out = (bf16_t*)z; p.bn = bn;
  p.Ha = g.Hin; p.Wa = g.Win; p.Ho = g.Hout; p.Wo = g.Wout; p.pa = g.ph; p.pb = g.pw;
  const bool stream = bn.gamma && streams_output((size_t)g.M * g.Cout * 2);   // (Eval's Y is read in the same call)
  if (g.sh == 1 && stream) hipLaunchKernelGGL((g3_conv_kernel<1, false, true>), dim3(p.nblk), dim3(256), 0, st, p);
  else if (g.sh == 1) hipLaunchKernelGGL((g3_conv_kernel<1, false, false>), dim3(p.nblk), dim3(256), 0, st, p);
  else if (stream) hipLaunchKernelGGL((g3_conv_kernel<2, false, true>), dim3(p.nblk), dim3(256), 0, st, p);
  else hipLaunchKernelGGL((g3_conv_kernel<2, false, false>), dim3(p.nblk), dim3(256), 0, st, p);
  return hipGetLastError();
}
namespace {
G3Params g3_dgrad_params(const Geom& g, int groups, const void* dz, const void* w_crsk, void* dx) {
  G3Params p = g3_params(g, groups, g3_dgrad_plan(g));
  p.a = (const bf16_t*)dz; p.w = (const bf16_t*)w_crsk; p.out = (bf16_t*)dx;
  p.Ha = g.Hout; p.Wa = g.Wout; p.Ho = g.Hin; p.Wo = g.Win;
  if (g.sh == 1) { p.pa = 2 - g.ph; p.pb = 2 - g.pw; }
  else { p.pa = g.ph; p.pb = g.pw; p.v0 = g3_first(g.ph); p.u0 = g3_first(g.pw); }
  return p;
}
G3Params g3_wgrad_params(const Geom& g, int groups, const void* x, const void* dz, float* part, float* r_part) {
  G3Params p = g3_params(g, groups, g3_wgrad_plan(g));
  p.a = (const bf16_t*)x; p.y = (const bf16_t*)dz; p.part = part; p.r_part = r_part;
  p.Ha = g.Hin; p.Wa = g.Win; p.Ho = g.Hout; p.Wo = g.Wout; p.pa = g.ph; p.pb = g.pw;
  return p;
}
}  // namespace
hipError_t launch_g3_dgrad(const Geom& g, int groups, const void* dz, const void* w_crsk, void* dx, hipStream_t st) {
  const G3Params p = g3_dgrad_params(g, groups, dz, w_crsk, dx);
  if (g.sh == 1) hipLaunchKernelGGL((g3_conv_kernel<1, true, STREAM_GRAD>), dim3(p.nblk), dim3(256), 0, st, p);
  else hipLaunchKernelGGL(g3_dgrad_s2_kernel, dim3(p.nblk), dim3(256), 0, st, p);
  return hipGetLastError();
}
int g3_wgrad_slices(const Geom& g) { return g3_wgrad_plan(g).bpc; }
#define G3_LAUNCH(KERNEL, LDS_BYTES, GRID, ...)                                                                          \
  do {                                                                                                                   \
    static LdsLimitOnce lds_once;                                                                                        \
    if (hipError_t e = set_lds_limit_once(lds_once, reinterpret_cast<const void*>(&KERNEL), LDS_BYTES); e != hipSuccess) \
      return e;                                                                                                          \
    hipLaunchKernelGGL((KERNEL), dim3(GRID), dim3(256), LDS_BYTES, st, __VA_ARGS__);                                     \
  } while (0)
hipError_t launch_g3_wgrad(const Geom& g, int groups, const void* x, const void* dz, float* part, float* r_part, hipStream_t st) {
  const G3Params p = g3_wgrad_params(g, groups, x, dz, part, r_part);
  constexpr int L1 = G3Wg<1>::LDS, L2 = G3Wg<2>::LDS;
  constexpr auto K12 = g3_wgrad_kernel<1, 2>, K14 = g3_wgrad_kernel<1, 4>, K22 = g3_wgrad_kernel<2, 2>, K24 = g3_wgrad_kernel<2, 4>;
  if (g.sh == 1) { if (p.cg == 32) G3_LAUNCH(*K14, L1, p.nblk, p); else G3_LAUNCH(*K12, L1, p.nblk, p); }
  else { if (p.cg == 32) G3_LAUNCH(*K24, L2, p.nblk, p); else G3_LAUNCH(*K22, L2, p.nblk, p); }
  return hipGetLastError();
}
bool g3_pair_supported(const Geom& g, int groups, int dtype) { return g3_supported(g, groups, dtype) && g.sh == 1; }
hipError_t launch_g3_pair(const Geom& g, int groups, const void* x, const void* dz, const void* w_crsk, void* dx, float* part,
                          float* r_part, hipStream_t st) {
  const G3Params w = g3_wgrad_params(g, groups, x, dz, part, r_part), d = g3_dgrad_params(g, groups, dz, w_crsk, dx);
  constexpr int L1 = G3Wg<1>::LDS;
  constexpr auto K2 = g3_pair_kernel<2>, K4 = g3_pair_kernel<4>;
  if (w.cg == 32) G3_LAUNCH(*K4, L1, w.nblk + d.nblk, w, d);
  else G3_LAUNCH(*K2, L1, w.nblk + d.nblk, w, d);
  return hipGetLastError();
}
#undef G3_LAUNCH

}  // namespace convbn
