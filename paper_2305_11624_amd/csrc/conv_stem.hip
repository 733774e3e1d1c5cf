// Convolutions of a network's first layer (Sec. 3.1's Y = w (*) X + b with at most four input
// channels, e.g. the 7x7 / stride-2 stem of a ResNet on RGB images), bf16 MFMA with fp32 accumulation.
//
// With 3 input channels the reduction index (tap, channel) has no 16-byte runs for the generic kernels to
// gather, and padding the channels to 8 makes them multiply and fetch mostly zeros.  Here the pixels are
// widened to 4 channels (8 bytes) on their way into LDS and the reduction index is ordered (window row i, window column
// j padded to 8, channel c padded to 4): the 8 consecutive reduction elements an MFMA lane needs -- two
// window columns x four channels -- are then 16 contiguous bytes of the input row, for every output pixel.
// So no im2col is ever materialised: the operand fragments are read straight from the raw input patch in
// LDS (output pixel wo, window columns j..j+1 -> patch bytes (wo sw + j) 8 ..), consecutive lanes 8 sw bytes
// apart.  The weights (Cout x kH x 8 x 4, zero-padded, packed by each workgroup for itself) stay resident in LDS; a workgroup
// is persistent and walks a run of tiles of 128 consecutive pixels of one output row: patch in (kH rows x (127 sw + 8) pixels),
// kH x 2 MFMA k-steps, s, b' and a ReLU in the epilogue, 16-byte stores out through LDS.  7-row windows on RGB images with rows of
// whole groups of four pixels and 33 to 64 output channels keep the weights in registers, store straight from the accumulators
// and hold the next patch in a second buffer.
#include "common.h"
#include "fold_tile.h"

#include <algorithm>

namespace convbn {

namespace {

constexpr int TPX = 128;            // output pixels per tile (32 per wave)
constexpr int KROW = 32;            // reduction elements per window row: 8 columns x 4 channels

struct StemParams {
  const bf16_t* x;      // X3: [N][H][W][3] (W % 4 == 0); else [N][H][W][4]
  const bf16_t* w;      // [Cout][kH][kW][Cin]
  const float* bias;    // [Cout] or null
  BnEpilogue bn;        // bn.gamma != null: the weight is unfolded, the epilogue applies s and b' (bias unused)
  int relu;
  bf16_t* z;            // [N][Ho][Wo][Cout]
  int N, H, W, Cin, Cout, kH, kW, sh, sw, ph, pw, Ho, Wo;
  int ntw, ntiles;      // tiles per output row, tiles in all
  int wpitch;           // LDS bytes per weight row: kH * 64 + 16
  int prow;             // LDS bytes per patch row: ((TPX - 1) sw + 8) * 8
  int pcols;            // pixels per patch row (X3: a multiple of 4, with up to 3 leading pixels of alignment)
};

// Fetches go through buffer descriptors of the rows that a tile needs (their byte offsets fit 30 bits, however large the image):
// what is outside is an offset beyond them and reads zeros, so that a fetch has no branch -- behind one, the compiler waited for
// each load on the spot: three to seven trips to memory in a row per tile (weight gradient, 7 x 7 on 224 x 224, 32 images: 46.3 ->
// 42.8 us).
constexpr unsigned NOWHERE = 1u << 30;
// `count` rows from row `row` of all images' on.  Rows that are not the image's, in front of the tensor even, are never read: their
// offsets are NOWHERE.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_rsrc(const bf16_t* base, long long row, int count, int row_elems) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(base) + row * row_elems, 0, count * row_elems * 2, 0x00020000);
}
__device__ __forceinline__ uint2 ld8(__amdgpu_buffer_rsrc_t r, unsigned off) {
  return __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
}
__device__ __forceinline__ uint4 ld16(__amdgpu_buffer_rsrc_t r, unsigned off) {
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
}

// A workgroup's tiles: a run of neighbours, which share input rows, and neighbouring runs on one XCD (workgroup ids are dealt
// round-robin over the 8 of them) with its L2.
struct TileRun { int first, end; };
__device__ __forceinline__ TileRun tile_run(int ntiles, int n = gridDim.x) {   // n: the workgroups that share them
  const int b = blockIdx.x, full = n & ~7;
  const int lb = b < full ? (b & 7) * (full >> 3) + (b >> 3) : b;
  return TileRun{(int)((long long)ntiles * lb / n), (int)((long long)ntiles * (lb + 1) / n)};
}

// pixels of a patch row (x3: up to 3 leading ones, whole groups of four)
constexpr int patch_cols(int sw, bool x3) { return x3 ? ((TPX - 1) * sw + 8 + 3 + 3) / 4 * 4 : (TPX - 1) * sw + 8; }

constexpr int ppt(bool x3) { return x3 ? 3 : 8; }   // most patch items a thread fetches per tile

// NCO: 32-channel fragments per workgroup (Cout = 32 NCO); KH: window rows (0 = run-time, any number); X3: the
// input has 3 channels and is fetched four pixels (24 contiguous bytes) at a time, else 4 channels, one pixel
// (8 bytes) at a time.
template <int NCO, int KH, bool X3>
__global__ __launch_bounds__(256) void stem_fprop_kernel(StemParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  float* biasl = reinterpret_cast<float*>(smem);                       // [128] b', [128] s (first 1024 bytes)
  unsigned char* wl = smem + 1024;                                     // [Cout][wpitch]
  unsigned char* patch = wl + 32 * NCO * p.wpitch;                     // [kH][prow]; reused to stage the output tile
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kb = lane >> 5, px = lane & 31;
  const int kH = KH > 0 ? KH : p.kH;

  // patch item e = tid + 256 k of a tile: (row i, pixel -- X3: group of four pixels -- q), the same for every tile
  constexpr int PPT = ppt(X3);
  constexpr int PXI = X3 ? 4 : 1;                 // pixels per item
  constexpr int NLD = X3 ? 3 : 1;                 // 8-byte loads per item
  const int icols = p.pcols / PXI;
  const int npatch = kH * icols;
  int pi[PPT], pq[PPT];
#pragma unroll
  for (int k = 0; k < PPT; ++k) {
    const int e = tid + 256 * k;
    pi[k] = e / icols;
    pq[k] = (e - pi[k] * icols) * PXI;
  }
  // first patch pixel of a tile: wo0 sw - pw, X3: rounded down to a multiple of four pixels
  auto patch_start = [&](int ws) {
    const int wbase = ws * TPX * p.sw - p.pw;
    return X3 ? (wbase >> 2) << 2 : wbase;
  };
  // fetch of a tile's patch into registers (zeros outside the image); the tile after the current one is
  // always in flight while the current one is multiplied
  uint2 pv[PPT][NLD];
  auto fetch = [&](int tile) {
    const int ws = tile % p.ntw;
    const int row = tile / p.ntw;
    const int ho = row % p.Ho, n = row / p.Ho;   // (a tile past the last one reads nothing)
    const int wstart = patch_start(ws);
    const int top = ho * p.sh - p.ph;
    const __amdgpu_buffer_rsrc_t xr = rows_rsrc(p.x, (long long)n * p.H + top, kH, p.W * (X3 ? 3 : 4));
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
      const int h = top + pi[k], w = wstart + pq[k];
      const bool ok = tid + 256 * k < npatch && tile < p.ntiles && (unsigned)h < (unsigned)p.H && (unsigned)w < (unsigned)p.W;
      const unsigned off = ok ? (unsigned)(pi[k] * p.W + w) * (X3 ? 6u : 8u) : NOWHERE;
#pragma unroll
      for (int j = 0; j < NLD; ++j) pv[k][j] = ld8(xr, off + 8 * j);
    }
  };
  // registers -> LDS, every pixel as 4 channels (X3: the 12 values of four pixels spread over 4 x 8 bytes)
  auto stash = [&](unsigned char* patch) {
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
      if (tid + 256 * k >= npatch) continue;
      unsigned char* dst = patch + pi[k] * p.prow + pq[k] * 8;
      if constexpr (X3) {
        const uint2 a = pv[k][0], b = pv[k][1], c = pv[k][2];
        *reinterpret_cast<uint4*>(dst) = make_uint4(a.x, a.y & 0xffffu, (a.y >> 16) | (b.x << 16), b.x >> 16);
        *reinterpret_cast<uint4*>(dst + 16) = make_uint4(b.y, c.x & 0xffffu, (c.x >> 16) | (c.y << 16), c.y >> 16);
      } else {
        *reinterpret_cast<uint2*>(dst) = pv[k][0];
      }
    }
  };
  const TileRun run = tile_run(p.ntiles);
  fetch(run.first);

  // ---- resident weights (behind the first patch's requests): 16-byte granules, two window columns of four channels, zeros
  // where the window or the channels end
  const int wrow_g = kH * KROW / 8;   // granules per weight row
  const int wtot = p.Cout * kH * p.kW * p.Cin;
  for (int e = tid; e < 32 * NCO * wrow_g; e += 256) {
    const int co = e / wrow_g, gq = e - co * wrow_g;
    const int i = gq >> 2, j0 = (gq & 3) * 2;
    const int at = ((co * kH + i) * p.kW + j0) * p.Cin;
    const bool c0 = co < p.Cout && j0 < p.kW, c1 = co < p.Cout && j0 + 1 < p.kW;
    unsigned d[4];
    if (p.Cin == 3 && at + 6 <= wtot) {   // the six values of the two columns, wherever they lie
      struct __attribute__((packed)) Six { unsigned a, b, c; };
      const Six r = *reinterpret_cast<const Six*>(p.w + at);
      d[0] = c0 ? r.a : 0u;
      d[1] = c0 ? r.b & 0xffffu : 0u;
      d[2] = c1 ? r.b >> 16 | r.c << 16 : 0u;
      d[3] = c1 ? r.c >> 16 : 0u;
    } else {
      unsigned v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const bool ok = (q < 4 ? c0 : c1) && (q & 3) < p.Cin;
        v[q] = ok ? reinterpret_cast<const unsigned short*>(p.w)[at + (q >> 2) * p.Cin + (q & 3)] : 0u;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) d[q] = v[2 * q] | v[2 * q + 1] << 16;
    }
    *reinterpret_cast<uint4*>(wl + co * p.wpitch + gq * 16) = make_uint4(d[0], d[1], d[2], d[3]);
  }
  if (tid < 32 * NCO) {
    float sc = 1.f, bb = 0.f;
    if (tid < p.Cout) bn_scale_bias(p.bn, p.bias, tid, &sc, &bb);
    biasl[tid] = bb;
    biasl[128 + tid] = sc;
  }
  if (p.bn.gamma && p.bn.w_folded_out) emit_folded_slice(p.bn, p.w, blockIdx.x, gridDim.x);   // w' for backward, on the side
  if constexpr (KH > 0) {
    // Known window height: the weight fragments stay in registers (read from LDS for every tile they were two thirds of its
    // traffic), which leaves room for two patches: a tile's successor is put in place while it is multiplied and stored, one
    // barrier a tile, and the outputs leave straight from the accumulators (the forward pass 25.9 -> 24.5 us).
    __syncthreads();
    const unsigned char* const wrow0 = wl + px * p.wpitch + kb * 16;
    bf16x8 wreg[2 * KH][NCO];
#pragma unroll
    for (int q = 0; q < 2 * KH; ++q)
#pragma unroll
      for (int f = 0; f < NCO; ++f) wreg[q][f] = *reinterpret_cast<const bf16x8*>(wrow0 + f * 32 * p.wpitch + q * 32);
    __syncthreads();   // the patches take the weights' place
    unsigned char* cur = wl;
    unsigned char* nxt = wl + KH * p.prow;
    stash(cur);
    fetch(run.first + 1);
    __syncthreads();
    for (int tile = run.first; tile < run.end; ++tile) {
      const int ws = tile % p.ntw;
      const int row = tile / p.ntw;
      const int ho = row % p.Ho, n = row / p.Ho;
      const int wo = ws * TPX + wave * 32 + px;
      f32x16 acc[NCO];
#pragma unroll
      for (int f = 0; f < NCO; ++f)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[f][e] = 0.f;
      const int lead = ws * TPX * p.sw - p.pw - patch_start(ws);
      const unsigned char* const prow0 = cur + ((wave * 32 + px) * p.sw + 2 * kb + lead) * 8;
#pragma unroll
      for (int i = 0; i < KH; ++i)
#pragma unroll
        for (int jh = 0; jh < 2; ++jh) {
          const unsigned char* bp = prow0 + i * p.prow + jh * 32;
          const uint2 b0 = *reinterpret_cast<const uint2*>(bp);
          const uint2 b1 = *reinterpret_cast<const uint2*>(bp + 8);
          const bf16x8 fb = __builtin_bit_cast(bf16x8, make_uint4(b0.x, b0.y, b1.x, b1.y));
#pragma unroll
          for (int f = 0; f < NCO; ++f) acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wreg[i * 2 + jh][f], fb, acc[f], 0, 0, 0);
        }
      // accumulator element e of lane l: channel 32 f + 8 (e / 4) + 4 (l / 32) + e % 4 of pixel l % 32; swapping the halves of
      // two registers gives every lane 8 channels of its pixel
      bf16_t* const zrow = p.z + (((size_t)n * p.Ho + ho) * p.Wo + wo) * p.Cout;
#pragma unroll
      for (int f = 0; f < NCO; ++f)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          unsigned pk[2][2];
#pragma unroll
          for (int qq = 0; qq < 2; ++qq) {
            const int q = 2 * j + qq, ch = 32 * f + 8 * q + 4 * kb;
            const float4 bb = *reinterpret_cast<const float4*>(biasl + ch), sc = *reinterpret_cast<const float4*>(biasl + 128 + ch);
            pk[qq][0] = pack_bf16x2(fmaf(acc[f][4 * q], sc.x, bb.x), fmaf(acc[f][4 * q + 1], sc.y, bb.y));
            pk[qq][1] = pack_bf16x2(fmaf(acc[f][4 * q + 2], sc.z, bb.z), fmaf(acc[f][4 * q + 3], sc.w, bb.w));
          }
          const auto lo = __builtin_amdgcn_permlane32_swap(pk[0][0], pk[1][0], false, false);
          const auto hi = __builtin_amdgcn_permlane32_swap(pk[0][1], pk[1][1], false, false);
          uint4 v = make_uint4(lo[0], hi[0], lo[1], hi[1]);
          if (p.relu) v = relu8(v);
          const int ch = 32 * f + (2 * j + kb) * 8;
          if (wo < p.Wo && ch < p.Cout) *reinterpret_cast<uint4*>(zrow + ch) = v;
        }
      stash(nxt);
      fetch(tile + 2);   // (behind the run's last: neighbours', dropped)
      __syncthreads();
      unsigned char* const t = cur;
      cur = nxt;
      nxt = t;
    }
    return;
  }

  for (int tile = run.first; tile < run.end; ++tile) {
    const int ws = tile % p.ntw;
    const int row = tile / p.ntw;
    const int ho = row % p.Ho, n = row / p.Ho;
    const int wo0 = ws * TPX;
    __syncthreads();   // the previous tile's staged output has been read
    stash(patch);
    fetch(tile + 1);   // (behind the run's last: the next run's first, dropped)
    __syncthreads();   // patch (and, first pass, weights and bias) visible

    f32x16 acc[NCO];
#pragma unroll
    for (int f = 0; f < NCO; ++f)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[f][e] = 0.f;
    // lane's pixel: wo0 + 32 wave + px; its window starts at patch pixel (32 wave + px) sw (+ the alignment pixels)
    const int lead = wo0 * p.sw - p.pw - patch_start(ws);
    const unsigned char* prow0 = patch + ((wave * 32 + px) * p.sw + 2 * kb + lead) * 8;
    const unsigned char* wrow0 = wl + px * p.wpitch + kb * 16;
    auto kstep = [&](int i, int jh) {   // window row i, columns 4 jh .. 4 jh + 3: lanes kb = 0 / 1 take two each
      const unsigned char* bp = prow0 + i * p.prow + jh * 32;
      const uint2 b0 = *reinterpret_cast<const uint2*>(bp);
      const uint2 b1 = *reinterpret_cast<const uint2*>(bp + 8);
      const bf16x8 fb = __builtin_bit_cast(bf16x8, make_uint4(b0.x, b0.y, b1.x, b1.y));
#pragma unroll
      for (int f = 0; f < NCO; ++f) {
        const bf16x8 fa = *reinterpret_cast<const bf16x8*>(wrow0 + f * 32 * p.wpitch + (i * 2 + jh) * 32);
        acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, fb, acc[f], 0, 0, 0);
      }
    };
    for (int i = 0; i < kH; ++i) { kstep(i, 0); kstep(i, 1); }
    __syncthreads();   // every wave is done with the patch: its memory now stages the output tile
    // ---- epilogue: accumulator element e of lane l is channel 8 (e / 4) + 4 (l / 32) + e % 4 of pixel l % 32.
    // Each wave rounds its 32 pixels x Cout channels into its own LDS block ([pixel][Cout], 16-byte granules
    // swizzled by pixel) and reads it back row-wise: every global store is 16 bytes per lane.
    constexpr int ROWB = 32 * NCO * 2;          // bytes per staged pixel row
    constexpr int GR = ROWB / 16;               // 16-byte granules per row
    unsigned char* st = patch + wave * 32 * ROWB;
    const int psw = (px >> 1) & (GR - 1);
#pragma unroll
    for (int f = 0; f < NCO; ++f)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int ch = f * 32 + q * 8 + kb * 4;
        const float4 bb = *reinterpret_cast<const float4*>(biasl + ch);
        const float4 sc = *reinterpret_cast<const float4*>(biasl + 128 + ch);
        const uint2 v = make_uint2(pack_bf16x2(fmaf(acc[f][q * 4 + 0], sc.x, bb.x), fmaf(acc[f][q * 4 + 1], sc.y, bb.y)),
                                   pack_bf16x2(fmaf(acc[f][q * 4 + 2], sc.z, bb.z), fmaf(acc[f][q * 4 + 3], sc.w, bb.w)));
        *reinterpret_cast<uint2*>(st + px * ROWB + (((ch >> 3) ^ psw) << 4) + ((ch & 7) << 1)) = v;
      }
    // (a wave reads only what it wrote itself: no workgroup barrier needed, the LDS counter orders it)
    constexpr int RPP = 64 / GR;                // pixel rows covered by one pass of the wave
#pragma unroll
    for (int pass = 0; pass < 32 / RPP; ++pass) {
      const int r = pass * RPP + lane / GR;
      const int g = (lane % GR) ^ ((r >> 1) & (GR - 1));
      uint4 v = *reinterpret_cast<const uint4*>(st + r * ROWB + ((lane % GR) << 4));
      if (p.relu) v = relu8(v);
      const int wo = wo0 + wave * 32 + r;
      const int ch = g * 8;
      if (wo < p.Wo && ch < p.Cout)
        *reinterpret_cast<uint4*>(p.z + (((size_t)n * p.Ho + ho) * p.Wo + wo) * p.Cout + ch) = v;
    }
  }
}

// ---- weight gradient of a first layer ------------------------------------------------------------------
// dw'[co][i][j][c] = sum over output pixels of dZ[pixel][co] X[pixel's window (i, j)][c]  and  r[co] = sum dZ
// (Sec. 3.2.1, App. B), with the same operand trick as the forward kernel: the reduced index is the pixel, so
// both MFMA operands are read with the transposing LDS load (ds_read_tr16_b64: a lane supplies the address of 8
// bytes -- here one padded input pixel (window column j, 4 channels) resp. 4 output channels of one pixel -- and
// receives 4 consecutive pixels of one row of the operand).  Rows of the left operand are the 32 (j, c) pairs of
// one window row, taken straight from the raw input patch: lane address = patch pixel (pixel sw + j).
// A persistent workgroup walks tiles of 128 pixels of one output row; wave w owns window rows w and w + 4 for
// all output channels and keeps their sums in registers over all its tiles; the partial sums of every workgroup
// go to memory once, as fp32 slices for the fold-back.
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ s16x4 read_tr(const unsigned char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p));
}
__device__ __forceinline__ bf16x8 join(s16x4 a, s16x4 b) {
  s16x8 v = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  return __builtin_bit_cast(bf16x8, v);
}

struct StemWgParams {
  const bf16_t* x;      // X3: [N][H][W][3] (W % 4 == 0); else [N][H][W][4]
  const bf16_t* dz;     // [N][Ho][Wo][Cout]
  float* part;          // [slices][Cout][kH kW Cin]
  float* r_part;        // [slices][Cout] or null
  int N, H, W, Cin, Cout, kH, kW, sh, sw, ph, pw, Ho, Wo;
  int ntw, ntiles, prow, pcols;
  int zpitch;           // LDS bytes per dZ pixel row: 2 Cout + 16
  int zt, buf, nbuf;    // LDS: offset of the dZ tile in a buffer, bytes of a buffer, buffers
};

// KH, SW: window rows and column stride at compile time (0: taken from the parameters): every operand is then an offset field
// of the reads, the eight steps of a tile are unrolled, and a row of ones behind the patch's (KH = 7) is wave 3's second: 33.2
// -> 23.5 us, the matrix pipe busy for a quarter of them.  Two workgroups share a compute unit, but for 128 output channels, whose
// 192 sums a lane would not all fit the registers then (32 images of 2 channels, 111 x 154, 4 x 4 / 2: a backward pass 152 us, so 110).
template <int NCO, bool X3, int KH, int SW>
__global__ __launch_bounds__(256, NCO == 4 ? 1 : 2) void stem_wgrad_kernel(StemWgParams p) {
  static_assert(KH == 0 || KH == 7, "seven window rows and the row of ones are two a wave");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  // two buffers (one, where two do not fit): patch [kH][prow], behind it at p.zt the dZ tile [TPX][zpitch]
  unsigned char* cur = smem;
  unsigned char* nxt = smem + (p.nbuf - 1) * p.buf;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kb = lane >> 5;
  const int eprime = (lane & 15) >> 2;                           // pixel (of 4) this lane addresses in a transposing read
  const int quad = ((lane >> 4) & 1) * 4 + (lane & 3);           // its 8-byte quad inside the 32-row operand block
  constexpr int PPT = ppt(X3), PXI = X3 ? 4 : 1, NLD = X3 ? 3 : 1;
  constexpr int NRW = 2;                                         // window rows per wave: w and w + 4 (kH <= 8)
  constexpr int ZG = 32 * NCO * 2 / 16;                          // 16-byte granules per dZ pixel row
  constexpr int ZPT = TPX * ZG / 256;                            // granules per thread and tile

  const int sw = SW > 0 ? SW : p.sw;
  const int prow = SW > 0 ? patch_cols(SW, X3) * 8 : p.prow, zpitch = KH > 0 ? 64 * NCO + 16 : p.zpitch;
  const int icols = p.pcols / PXI;
  const int npatch = p.kH * icols;
  int pi[PPT], pq[PPT];
#pragma unroll
  for (int k = 0; k < PPT; ++k) {
    const int e = tid + 256 * k;
    pi[k] = e / icols;
    pq[k] = (e - pi[k] * icols) * PXI;
  }
  auto patch_start = [&](int ws) {
    const int wbase = ws * TPX * sw - p.pw;
    return X3 ? (wbase >> 2) << 2 : wbase;
  };
  if constexpr (KH > 0)
    for (int e = tid; e < prow / 4; e += 256) {
      reinterpret_cast<unsigned*>(cur + KH * prow)[e] = 0x3f803f80u;
      reinterpret_cast<unsigned*>(nxt + KH * prow)[e] = 0x3f803f80u;
    }
  uint2 pv[PPT][NLD];
  uint4 zv[ZPT];
  auto fetch = [&](int tile) {
    const int ws = tile % p.ntw;
    const int row = tile / p.ntw;
    const int ho = row % p.Ho, n = row / p.Ho;   // (a tile past the last one reads nothing)
    const int wstart = patch_start(ws);
    const int top = ho * p.sh - p.ph;
    const __amdgpu_buffer_rsrc_t xr = rows_rsrc(p.x, (long long)n * p.H + top, p.kH, p.W * (X3 ? 3 : 4));
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
      const int h = top + pi[k], w = wstart + pq[k];
      const bool ok = tid + 256 * k < npatch && tile < p.ntiles && (unsigned)h < (unsigned)p.H && (unsigned)w < (unsigned)p.W;
      const unsigned off = ok ? (unsigned)(pi[k] * p.W + w) * (X3 ? 6u : 8u) : NOWHERE;
#pragma unroll
      for (int j = 0; j < NLD; ++j) pv[k][j] = ld8(xr, off + 8 * j);
    }
    const __amdgpu_buffer_rsrc_t zr = rows_rsrc(p.dz, row, 1, p.Wo * p.Cout);
    // dZ rows of the tile's pixels (zeros past the end of the output row: such pixels then add nothing)
#pragma unroll
    for (int k = 0; k < ZPT; ++k) {
      const int e = tid + 256 * k;
      const int px = e / ZG, gq = e - px * ZG;
      const int wo = ws * TPX + px;
      const bool ok = tile < p.ntiles && wo < p.Wo && gq * 8 < p.Cout;
      zv[k] = ld16(zr, ok ? ((unsigned)wo * p.Cout + gq * 8) * 2u : NOWHERE);
    }
  };
  auto stash = [&](unsigned char* patch) {
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
      if (tid + 256 * k >= npatch) continue;
      unsigned char* dst = patch + pi[k] * prow + pq[k] * 8;
      if constexpr (X3) {
        const uint2 a = pv[k][0], b = pv[k][1], c = pv[k][2];
        *reinterpret_cast<uint4*>(dst) = make_uint4(a.x, a.y & 0xffffu, (a.y >> 16) | (b.x << 16), b.x >> 16);
        *reinterpret_cast<uint4*>(dst + 16) = make_uint4(b.y, c.x & 0xffffu, (c.x >> 16) | (c.y << 16), c.y >> 16);
      } else {
        *reinterpret_cast<uint2*>(dst) = pv[k][0];
      }
    }
#pragma unroll
    for (int k = 0; k < ZPT; ++k) {
      const int e = tid + 256 * k;
      const int px = e / ZG, gq = e - px * ZG;
      *reinterpret_cast<uint4*>(patch + p.zt + px * zpitch + gq * 16) = zv[k];
    }
  };

  f32x16 acc[NRW][NCO];
#pragma unroll
  for (int t = 0; t < NRW; ++t)
#pragma unroll
    for (int f = 0; f < NCO; ++f)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[t][f][e] = 0.f;
  // The channel sums r are the product of the dZ fragments with ones, by wave 3, which has one window row fewer (of up to 7).
  // Read from the tile by the vector units they were 32 LDS reads a thread and tile.
  const s16x8 one_bits = {0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80};
  const bf16x8 ones = __builtin_bit_cast(bf16x8, one_bits);
  f32x16 racc[NCO];
#pragma unroll
  for (int f = 0; f < NCO; ++f)
#pragma unroll
    for (int e = 0; e < 16; ++e) racc[f][e] = 0.f;

  const TileRun run = tile_run(p.ntiles);
  fetch(run.first);
  stash(cur);
  fetch(run.first + 1);
  __syncthreads();
  for (int tile = run.first; tile < run.end; ++tile) {   // a tile's successor is put in place behind its products
    const int ws = tile % p.ntw;
    const int lead = ws * TPX * sw - p.pw - patch_start(ws);
    // lane-constant parts of the operand addresses
    const unsigned char* zl = cur + p.zt + (kb * 8 + eprime) * zpitch + (((lane >> 4) & 1) * 16 + (lane & 3) * 4) * 2;
    const unsigned char* xl = cur + wave * prow + (((kb * 8 + eprime) * sw + quad + lead) * 8);
    auto step = [&](int k) {
      bf16x8 zf[NCO];
#pragma unroll
      for (int f = 0; f < NCO; ++f)
        zf[f] = join(read_tr(zl + (k * 16) * zpitch + f * 64), read_tr(zl + (k * 16 + 4) * zpitch + f * 64));
#pragma unroll
      for (int t = 0; t < NRW; ++t) {
        if (KH == 0 && wave + 4 * t >= p.kH) break;
        const unsigned char* xr = xl + 4 * t * prow + (k * 16) * sw * 8;
        const bf16x8 xf = join(read_tr(xr), read_tr(xr + 4 * sw * 8));
#pragma unroll
        for (int f = 0; f < NCO; ++f) acc[t][f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf, zf[f], acc[t][f], 0, 0, 0);
      }
      if (KH == 0 && wave == 3) {
#pragma unroll
        for (int f = 0; f < NCO; ++f) racc[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, zf[f], racc[f], 0, 0, 0);
      }
    };
    if constexpr (KH > 0) {
#pragma unroll
      for (int k = 0; k < TPX / 16; ++k) step(k);
    } else {
      for (int k = 0; k < TPX / 16; ++k) step(k);
    }
    if (p.nbuf == 1) __syncthreads();   // every wave is done with the buffer
    stash(nxt);
    fetch(tile + 2);   // (behind the run's last: neighbours', dropped)
    __syncthreads();
    unsigned char* const t = cur;
    cur = nxt;
    nxt = t;
  }
  // ---- this workgroup's slice.  Accumulator element e of lane l: operand row 8 (e / 4) + 4 (l / 32) + e % 4 =
  // window column 2 (e / 4) + l / 32, channel e % 4; output channel f 32 + l % 32.  32 output channels at a time are gathered in
  // LDS and leave as whole lines (stored from the registers, 12 bytes
  // of a line each, the kernel took 42.8 us, like this 34.0).
  const int K = p.kH * p.kW * p.Cin;
  float* const rows = reinterpret_cast<float*>(smem);            // [32][K]
#pragma unroll
  for (int f = 0; f < NCO; ++f) {
    __syncthreads();   // every wave is done with the tiles, or with the channels before
#pragma unroll
    for (int t = 0; t < NRW; ++t) {
      const int i = wave + 4 * t;
      if (i >= p.kH) break;
      float* orow = rows + (lane & 31) * K + i * p.kW * p.Cin;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = 2 * q + kb;
        if (j >= p.kW) continue;
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (c < p.Cin) orow[j * p.Cin + c] = acc[t][f][q * 4 + c];
      }
    }
    __syncthreads();
    const int nco = min(32, p.Cout - f * 32);                    // (a multiple of 8: whole float4s)
    float4* const out = reinterpret_cast<float4*>(p.part + ((size_t)blockIdx.x * p.Cout + f * 32) * K);
    for (int e = tid; e < nco * K / 4; e += 256) out[e] = reinterpret_cast<const float4*>(rows)[e];
  }
  if (p.r_part && wave == 3 && kb == 0) {   // (every row of the product is the sum; column l % 32)
#pragma unroll
    for (int f = 0; f < NCO; ++f)
      if (f * 32 + lane < p.Cout) p.r_part[(size_t)blockIdx.x * p.Cout + f * 32 + lane] = KH > 0 ? acc[1][f][0] : racc[f][0];
  }
}

struct StemWgPlan { bool ok; bool x3; bool known; int nco; size_t lds; int grid; };
StemWgPlan stem_wg_work_out(const Geom& g, StemWgParams* pp) {
  StemWgPlan pl{false, false, false, 0, 0, 0};
  StemWgParams& p = *pp;
  p = StemWgParams{};
  if (g.kH > 8) return pl;   // two window rows per wave
  if ((size_t)g.Wout * g.Cout * 2 >= NOWHERE) return pl;
  p.N = g.N; p.H = g.Hin; p.W = g.Win; p.Cin = g.Cin; p.Cout = g.Cout; p.kH = g.kH; p.kW = g.kW;
  p.sh = g.sh; p.sw = g.sw; p.ph = g.ph; p.pw = g.pw; p.Ho = g.Hout; p.Wo = g.Wout;
  p.ntw = ceil_div(g.Wout, TPX);
  p.ntiles = g.N * g.Hout * p.ntw;
  const bool x3 = g.Cin == 3 && g.Win % 4 == 0;
  p.pcols = patch_cols(g.sw, x3);
  p.prow = p.pcols * 8;
  pl.nco = ceil_div(g.Cout, 32);
  if (pl.nco != 1 && pl.nco != 2 && pl.nco != 4) return pl;
  if (g.kH * (p.pcols / (x3 ? 4 : 1)) > 256 * ppt(x3)) return pl;
  p.zpitch = 32 * pl.nco * 2 + 16;
  pl.known = x3 && pl.nco == 2 && g.kH == 7 && g.sw == 2;   // the usual 7x7 / stride-2 RGB stem, 33 to 64 channels
  p.zt = (int)align_up((size_t)(g.kH + (pl.known ? 1 : 0)) * p.prow, 16);
  p.buf = p.zt + TPX * p.zpitch;
  p.nbuf = 2 * p.buf <= 80 * 1024 ? 2 : 1;   // (two workgroups share a compute unit's 160 KB)
  pl.lds = (size_t)p.nbuf * p.buf;
  // the sums of 32 output channels are gathered there at the end
  const size_t gather = (size_t)32 * g.K * 4;
  if (pl.lds < gather) pl.lds = gather;
  if (pl.lds > 80 * 1024) return pl;
  // two workgroups per CU (a lone one leaves the CU idle while it waits; 65 -> 48 us on the 7x7 stem); every
  // workgroup writes a full fp32 slice of dw', which the fold-back has to sum, so not more
  pl.grid = p.ntiles < 512 ? p.ntiles : 512;
  pl.x3 = x3;
  pl.ok = true;
  return pl;
}
StemWgPlan stem_wg_plan(const Geom& g, StemWgParams* pp) {
  struct Known { StemWgPlan pl; StemWgParams p; };
  const Known& k = planned<Known>(g, CONVBN_BF16, [&] {
    Known r;
    r.pl = stem_wg_work_out(g, &r.p);
    return r;
  });
  *pp = k.p;
  return k.pl;
}

// ---- input gradient of a first layer -------------------------------------------------------------------
// dX[h][w][c] = sum_{i,j,co} dZ[(h + ph - i) / sh][(w + pw - j) / sw][co] w'[co][i][j][c] over the taps for which the
// divisions are exact (Sec. 3.2.1).  With 3 input channels the result has almost no columns for a matrix product, so
// the sh x sw pixels of a block (a, b) = (h / sh, w / sw) and their (padded) 4 channels together form the 16 rows of
// one: every pixel of the block reads the same U x V neighbourhood of dZ -- rows a + Dh - u, columns b + Dw - v --
// only with a different subset of the taps, so   dX[block][(phase, c)] = sum_{u,v,co} Wt[(phase, c)][(u, v, co)]
// dZ[a + Dh - u][b + Dw - v][co],   Wt holding w' where phase (h % sh, w % sw) has a tap at (u, v) and zeros
// elsewhere (49 of 64 positions for 7x7 / stride 2).  That is a stride-1 convolution of dZ with a U x V window whose
// 16 output "channels" are un-shuffled to pixels (depth to space).  MFMA 16x16x32: rows = the 16 (phase, c)
// pairs, columns = 16 blocks, 32 output channels of one (u, v) per step; as in the forward kernel the column
// operand is read straight from the raw dZ patch in LDS (lane = block, 16 contiguous bytes = 8 channels) and the
// packed weight (16 x U V Cout) stays resident.  A lane ends up with the 4 channels of one dX pixel.
typedef float f32x4s __attribute__((ext_vector_type(4)));
constexpr int DG_PPT = 8;      // most 16-byte patch items a thread fetches per tile
constexpr int DG_NBT = 2;      // most 16-block groups a wave multiplies per tile

struct StemDgParams {
  const bf16_t* dz;     // [N][Ho][Wo][Cout]
  const bf16_t* w;      // w' as [Cin][kH][kW][Cout]
  bf16_t* dx;           // [N][H][W][Cin]
  int N, H, W, Cin, Cout, Ho, Wo, kH, kW, sh, sw, ph, pw;
  int U, V, Dh, Dw;     // block (a, b) reads dZ rows a + Dh - u (u < U), columns b + Dw - v (v < V)
  int KT;               // U V Cout
  int TBR, TBC;         // blocks per tile
  int nbr, nbc, ntiles; // tiles per image column / row, tiles in all
  int PR, PC, pitch;    // dZ patch rows (TBR + U - 1), columns (TBC + V - 1), bytes per pixel (2 Cout + 16)
  int wpitch;           // LDS bytes per weight row (2 KT + 16)
  int nbt;              // 16-block groups per tile
  int nbuf;             // patches in LDS
  unsigned mTBC, mPC;   // multipliers for n / TBC, n / PC (n < 65536)
  int nwg;              // the input gradient's workgroups, those behind them fold back
};

__device__ __forceinline__ int dg_div(int n, unsigned m, int d) { return d == 1 ? n : (int)__umulhi((unsigned)n, m); }

// UU, VV, KS: the dZ neighbourhood and Cout / 32 at compile time (0: taken from the parameters)
template <int UU, int VV, int KS, class Side>
__global__ __launch_bounds__(256, 2) void stem_dgrad_kernel(StemDgParams p, Side side) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  if constexpr (Side::BACK)
    if ((int)blockIdx.x >= p.nwg) {
      fold_back_side<256, ROW_ANY, 16, 1>(side, (int)blockIdx.x - p.nwg, smem);
      return;
    }
  unsigned char* wl = smem;                                         // [16][wpitch] (UU == 0)
  unsigned char* cur = UU > 0 ? smem : wl + 16 * p.wpitch;          // two patches (one, where two do not fit): [PR][PC][pitch]
  unsigned char* nxt = cur + (p.nbuf - 1) * p.PR * p.PC * p.pitch;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 15, kg = lane >> 4;                        // MFMA column (block) / row (phase, c) and 8-channel group

  // ---- patch items of this thread: granule gq (8 channels) of patch pixel (row, column), the same for every tile
  const int gpp = p.Cout / 8;
  const int nitems = p.PR * p.PC * gpp;
  int ipr[DG_PPT], ipc[DG_PPT];
#pragma unroll
  for (int k = 0; k < DG_PPT; ++k) {
    const int e = tid + 256 * k;
    const int pix = e / gpp;
    ipr[k] = dg_div(pix, p.mPC, p.PC);
    ipc[k] = (pix - ipr[k] * p.PC) | ((e - pix * gpp) << 16);
  }
  uint4 pv[DG_PPT];
  auto fetch = [&](int tile) {
    const int tr = tile % p.nbr;   // (down the columns: the rows that two tiles share come from the cache)
    const int t2 = tile / p.nbr;
    const int tc = t2 % p.nbc, n = t2 / p.nbc;   // (a tile past the last one reads nothing)
    // patch row r holds dZ row a0 + Dh - (U - 1) + r, column likewise
    const int h0 = tr * p.TBR + p.Dh - (p.U - 1), w0 = tc * p.TBC + p.Dw - (p.V - 1);
    const __amdgpu_buffer_rsrc_t zr = rows_rsrc(p.dz, (long long)n * p.Ho + h0, p.PR, p.Wo * p.Cout);
#pragma unroll
    for (int k = 0; k < DG_PPT; ++k) {
      const int h = h0 + ipr[k], w = w0 + (ipc[k] & 0xffff), gq = ipc[k] >> 16;
      const bool ok = tid + 256 * k < nitems && tile < p.ntiles && (unsigned)h < (unsigned)p.Ho && (unsigned)w < (unsigned)p.Wo;
      pv[k] = ld16(zr, ok ? ((unsigned)(ipr[k] * p.Wo + w) * p.Cout + gq * 8) * 2u : NOWHERE);
    }
  };
  auto stash = [&](unsigned char* patch) {
#pragma unroll
    for (int k = 0; k < DG_PPT; ++k)
      if (tid + 256 * k < nitems)
        *reinterpret_cast<uint4*>(patch + (ipr[k] * p.PC + (ipc[k] & 0xffff)) * p.pitch + (ipc[k] >> 16) * 16) = pv[k];
  };

  const int nph = p.sh * p.sw;                 // phases: rows 4 phase + c of the product
  const int ksteps = p.Cout / 32;
  const TileRun run = tile_run(p.ntiles, p.nwg);
  fetch(run.first);
  // ---- resident weight (behind the first patch's requests): Wt[(phase, c)][(u, v, co)], phase (qh, qw) reaching dZ row
  // a + dh(qh) - t through window row i0(qh) + sh t, i.e. u = Dh - dh(qh) + t; zeros where a phase has no tap and in the rows of
  // c >= Cin.  The element offset of w' that row r, position (u, v) reads, -1: none (strides 1 and 2: quotients are shifts):
  const int lh = p.sh - 1, lw = p.sw - 1;
  auto tap_at = [&](int r, int u, int v) {
    const int phase = r >> 2, c = r & 3, qh = phase >> lw, qw = phase & lw;
    const int th = u - (p.Dh - ((qh + p.ph) >> lh)), tw = v - (p.Dw - ((qw + p.pw) >> lw));
    const int i = ((qh + p.ph) & lh) + p.sh * th, j = ((qw + p.pw) & lw) + p.sw * tw;
    return phase < nph && c < p.Cin && th >= 0 && tw >= 0 && i < p.kH && j < p.kW ? ((c * p.kH + i) * p.kW + j) * p.Cout : -1;
  };
  // Known window: the fragments stay in registers, straight from w' (in LDS they were a third of its reads, which were what bound
  // the kernel, and 33 KB; 41.3 -> 33.3 us with the stores below).
  bf16x8 wreg[UU > 0 ? UU : 1][VV > 0 ? VV : 1][KS > 0 ? KS : 1];
  if constexpr (UU > 0) {
#pragma unroll
    for (int u = 0; u < UU; ++u)
#pragma unroll
      for (int v = 0; v < VV; ++v) {
        const int at = tap_at(col, u, v);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const uint4 t = *reinterpret_cast<const uint4*>(p.w + max(at, 0) + ks * 32 + kg * 8);
          wreg[u][v][ks] = __builtin_bit_cast(bf16x8, make_uint4(at >= 0 ? t.x : 0u, at >= 0 ? t.y : 0u, at >= 0 ? t.z : 0u, at >= 0 ? t.w : 0u));
        }
      }
  } else {
    const int cg = p.Cout / 8, UV = p.U * p.V;
    const int total = 16 * UV * cg;
    for (int e0 = tid; e0 < total; e0 += 4 * 256) {   // 16 bytes (8 output channels) at a time, four of them in flight
      uint4 v[4];
      int at[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int e = min(e0 + 256 * k, total - 1);
        const int pair = e / cg, r = pair / UV, uv = pair - r * UV, u = uv / p.V;
        at[k] = tap_at(r, u, uv - u * p.V);
        v[k] = *reinterpret_cast<const uint4*>(p.w + max(at[k], 0) + (e - pair * cg) * 8);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int e = e0 + 256 * k, r = e / (UV * cg), gq = e - r * UV * cg;
        if (e < total)
          *reinterpret_cast<uint4*>(wl + r * p.wpitch + gq * 16) =
              make_uint4(at[k] >= 0 ? v[k].x : 0u, at[k] >= 0 ? v[k].y : 0u, at[k] >= 0 ? v[k].z : 0u, at[k] >= 0 ? v[k].w : 0u);
      }
    }
  }
  stash(cur);
  fetch(run.first + 1);
  __syncthreads();   // patch (and the weight) visible
  for (int tile = run.first; tile < run.end; ++tile) {
    const int tr = tile % p.nbr;   // (down the columns: the rows that two tiles share come from the cache)
    const int t2 = tile / p.nbr;
    const int tc = t2 % p.nbc, n = t2 / p.nbc;
    // the wave's block groups: wave, wave + 4 (the lane's block: q = 16 group + col -> row ar, column bc of the tile)
    int ar[DG_NBT], bc[DG_NBT];
    bool live[DG_NBT];
    const unsigned char* bp[DG_NBT];
    f32x4s acc[DG_NBT];
#pragma unroll
    for (int t = 0; t < DG_NBT; ++t) {
      const int q = (wave + 4 * t) * 16 + col;
      live[t] = wave + 4 * t < p.nbt;
      const int a = dg_div(q, p.mTBC, p.TBC);
      ar[t] = a; bc[t] = q - a * p.TBC;
      const bool in = live[t] && a < p.TBR;
      // window origin of the block in the patch: its (u, v) = (0, 0) neighbour is patch pixel (ar + U - 1, bc + V - 1)
      bp[t] = cur + ((in ? a + p.U - 1 : p.U - 1) * p.PC + (in ? bc[t] + p.V - 1 : p.V - 1)) * p.pitch + kg * 16;
      acc[t] = f32x4s{0.f, 0.f, 0.f, 0.f};
    }
    const unsigned char* ap = wl + col * p.wpitch + kg * 16;
    auto step = [&](int u, int v, int ks, int nv, int cout2) {
      bf16x8 fa;
      if constexpr (UU > 0) fa = wreg[u][v][ks];
      else fa = *reinterpret_cast<const bf16x8*>(ap + (u * nv + v) * cout2 + ks * 64);
      const int boff = -(u * p.PC + v) * p.pitch + ks * 64;
#pragma unroll
      for (int t = 0; t < DG_NBT; ++t) {
        const bf16x8 fb = *reinterpret_cast<const bf16x8*>(bp[t] + boff);
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fb, acc[t], 0, 0, 0);
      }
    };
    if constexpr (UU > 0) {
#pragma unroll
      for (int u = 0; u < UU; ++u)
#pragma unroll
        for (int v = 0; v < VV; ++v)
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) step(u, v, ks, VV, KS * 64);
    } else {
      for (int u = 0; u < p.U; ++u)
        for (int v = 0; v < p.V; ++v)
          for (int ks = 0; ks < ksteps; ++ks) step(u, v, ks, p.V, p.Cout * 2);
    }
    // ---- lane (col, kg): block col of the group, product rows 4 kg .. 4 kg + 3 = phase kg, channels 0..3: one pixel, stored
    // as it is (neighbouring lanes write neighbouring bytes; gathering a tile's rows in LDS first cost a barrier and its reads)
#pragma unroll
    for (int t = 0; t < DG_NBT; ++t) {
      const int h = (tr * p.TBR + ar[t]) * p.sh + (kg >> lw), w = (tc * p.TBC + bc[t]) * p.sw + (kg & lw);
      if (!live[t] || ar[t] >= p.TBR || kg >= nph || h >= p.H || w >= p.W) continue;
      bf16_t* const o = p.dx + (((size_t)n * p.H + h) * p.W + w) * p.Cin;
      const unsigned lo = pack_bf16x2(acc[t][0], acc[t][1]), hi = pack_bf16x2(acc[t][2], acc[t][3]);
      if (p.Cin == 3) {
        struct __attribute__((packed)) Three { unsigned a; unsigned short b; };
        *reinterpret_cast<Three*>(o) = Three{lo, (unsigned short)hi};
      } else if (p.Cin == 4) {
        *reinterpret_cast<uint2*>(o) = make_uint2(lo, hi);
      } else {
        for (int c = 0; c < p.Cin; ++c) o[c] = from_f32<bf16_t>(acc[t][c]);
      }
    }
    if (p.nbuf == 1) __syncthreads();   // every wave is done with the patch
    stash(nxt);
    fetch(tile + 2);   // (behind the run's last: neighbours', dropped)
    __syncthreads();
    unsigned char* const t = cur;
    cur = nxt;
    nxt = t;
  }
}

struct StemDgPlan { bool ok; bool known; size_t lds; int grid, room; };   // room: workgroups that the chip holds at once
StemDgPlan stem_dg_work_out(const Geom& g, StemDgParams* pp) {
  StemDgPlan pl{false, false, 0, 0, 0};
  StemDgParams& p = *pp;
  p = StemDgParams{};
  if (g.sh > 2 || g.sw > 2 || g.Cout % 32 != 0 || g.Cout > 128) return pl;
  p.N = g.N; p.H = g.Hin; p.W = g.Win; p.Cin = g.Cin; p.Cout = g.Cout; p.Ho = g.Hout; p.Wo = g.Wout; p.sh = g.sh; p.sw = g.sw;
  p.kH = g.kH; p.kW = g.kW; p.ph = g.ph; p.pw = g.pw;
  // per phase q: first window row i0 = (q + pad) % s, its dZ row offset d = (q + pad) / s, taps T = ceil((k - i0) / s)
  auto span = [](int k, int s, int pad, int* D, int* U) {
    int dmax = 0;
    for (int q = 0; q < s; ++q) dmax = (q + pad) / s > dmax ? (q + pad) / s : dmax;
    int umax = 0;
    for (int q = 0; q < s; ++q) {
      const int i0 = (q + pad) % s;
      if (i0 >= k) continue;
      const int T = (k - i0 + s - 1) / s;
      const int u = dmax - (q + pad) / s + T;
      umax = u > umax ? u : umax;
    }
    *D = dmax; *U = umax;
  };
  span(g.kH, g.sh, g.ph, &p.Dh, &p.U);
  span(g.kW, g.sw, g.pw, &p.Dw, &p.V);
  if (p.U < 1 || p.V < 1) return pl;
  p.KT = p.U * p.V * g.Cout;
  p.wpitch = p.KT * 2 + 16;
  if ((size_t)16 * p.wpitch > 36 * 1024) return pl;
  p.pitch = g.Cout * 2 + 16;
  const int brows = ceil_div(g.Hin, g.sh), bcols = ceil_div(g.Win, g.sw);
  // tiles of 4 block rows x up to 32 block columns, the columns split evenly
  p.nbc = ceil_div(bcols, 32);
  p.TBC = ceil_div(bcols, p.nbc);
  p.TBR = brows < 4 ? brows : 4;
  p.nbr = ceil_div(brows, p.TBR);
  p.PR = p.TBR + p.U - 1; p.PC = p.TBC + p.V - 1;
  p.nbt = ceil_div(p.TBR * p.TBC, 16);
  if ((size_t)p.PR * g.Wout * g.Cout * 2 >= NOWHERE) return pl;
  if (p.nbt > 4 * DG_NBT || p.PR * p.PC * (g.Cout / 8) > 256 * DG_PPT) return pl;
  p.ntiles = g.N * p.nbr * p.nbc;
  p.mTBC = (unsigned)((1ull << 32) / (unsigned)p.TBC + 1);
  p.mPC = (unsigned)((1ull << 32) / (unsigned)p.PC + 1);
  pl.known = p.U == 4 && p.V == 4 && g.Cout == 64;   // the usual 7x7 / stride-2 stem with 64 channels: unrolled, weights in registers
  const size_t weight = pl.known ? 0 : (size_t)16 * p.wpitch, patch = (size_t)p.PR * p.PC * p.pitch;
  p.nbuf = weight + 2 * patch <= 80 * 1024 ? 2 : 1;
  pl.lds = weight + p.nbuf * patch;
  if (pl.lds > 80 * 1024) return pl;   // two workgroups per CU
  const int per_cu = (int)(160 * 1024 / pl.lds) < 2 ? 1 : 2;
  pl.room = 256 * (pl.known ? per_cu : std::min(4, (int)(160 * 1024 / pl.lds)));   // (250 or 120 registers a lane)
  pl.grid = p.ntiles < 256 * per_cu ? p.ntiles : 256 * per_cu;
  pl.ok = true;
  return pl;
}
StemDgPlan stem_dg_plan(const Geom& g, StemDgParams* pp) {
  struct Known { StemDgPlan pl; StemDgParams p; };
  const Known& k = planned<Known>(g, CONVBN_BF16, [&] {
    Known r;
    r.pl = stem_dg_work_out(g, &r.p);
    return r;
  });
  *pp = k.p;
  return k.pl;
}

bool stem_shape(const Geom& g, int dtype) {
  return dtype == CONVBN_BF16 && g.Cin <= 4 && g.kW <= 8 && g.kH <= 16 && g.Cout % 8 == 0 && g.Cout <= 128 && g.sw <= 4 &&
         (size_t)g.kH * g.Win * 8 < NOWHERE;
}

struct StemPlan { bool ok; bool x3; int nco; size_t lds; int grid; };
StemPlan stem_work_out(const Geom& g, StemParams* pp) {
  StemPlan pl{false, false, 0, 0, 0};
  StemParams& p = *pp;
  p = StemParams{};
  p.N = g.N; p.H = g.Hin; p.W = g.Win; p.Cin = g.Cin; p.Cout = g.Cout; p.kH = g.kH; p.kW = g.kW;
  p.sh = g.sh; p.sw = g.sw; p.ph = g.ph; p.pw = g.pw; p.Ho = g.Hout; p.Wo = g.Wout;
  p.ntw = ceil_div(g.Wout, TPX);
  p.ntiles = g.N * g.Hout * p.ntw;
  p.wpitch = g.kH * KROW * 2 + 16;
  const bool x3 = g.Cin == 3 && g.Win % 4 == 0;
  p.pcols = patch_cols(g.sw, x3);
  p.prow = p.pcols * 8;
  pl.nco = ceil_div(g.Cout, 32);
  if (pl.nco != 1 && pl.nco != 2 && pl.nco != 4) return pl;
  if (g.kH * (p.pcols / (x3 ? 4 : 1)) > 256 * ppt(x3)) return pl;   // the patch is fetched in at most ppt() rounds
  const size_t stage = (size_t)4 * 32 * 32 * pl.nco * 2;            // the output tile is staged over the patch
  const size_t patch = (size_t)g.kH * p.prow;
  pl.lds = 1024 + (size_t)32 * pl.nco * p.wpitch + (patch > stage ? patch : stage);
  if (pl.lds > 64 * 1024) return pl;   // two or more workgroups per CU hide each other's phases
  int per_cu = (int)(160 * 1024 / pl.lds) < 4 ? (int)(160 * 1024 / pl.lds) : 4;
  if (x3 && pl.nco == 2 && g.kH == 7) {   // (weights in registers, two patches)
    per_cu = 2;
    if (pl.lds < 1024 + 2 * patch) pl.lds = 1024 + 2 * patch;
  }
  pl.grid = p.ntiles < 256 * per_cu ? p.ntiles : 256 * per_cu;
  pl.x3 = x3;
  pl.ok = true;
  return pl;
}
StemPlan stem_plan(const Geom& g, StemParams* pp) {
  struct Known { StemPlan pl; StemParams p; };
  const Known& k = planned<Known>(g, CONVBN_BF16, [&] {
    Known r;
    r.pl = stem_work_out(g, &r.p);
    return r;
  });
  *pp = k.p;
  return k.pl;
}

}  // namespace

// 3-channel inputs whose rows are whole groups of four pixels, and 4-channel inputs, are read as they are; others
// need a copy widened to 4 channels ([N][H][W][4]) of this many bytes (0: none)
size_t stem_input_copy_bytes(const Geom& g) {
  return (g.Cin == 4 || (g.Cin == 3 && g.Win % 4 == 0)) ? 0 : (size_t)g.Min * 4 * 2;
}

bool stem_wgrad_supported(const Geom& g, int dtype) {
  if (!stem_shape(g, dtype)) return false;
  StemWgParams p;
  return stem_wg_plan(g, &p).ok;
}
int stem_wgrad_slices(const Geom& g) {
  StemWgParams p;
  return stem_wg_plan(g, &p).grid;
}
// x as for launch_fprop_stem; part [slices][Cout][K] and r_part [slices][Cout] (nullable): fp32 partial sums
hipError_t launch_wgrad_stem(const Geom& g, const void* x, const void* dz, float* part, float* r_part, hipStream_t st) {
  StemWgParams p;
  const StemWgPlan pl = stem_wg_plan(g, &p);
  if (!pl.ok) return hipErrorInvalidValue;
  p.x = (const bf16_t*)x; p.dz = (const bf16_t*)dz; p.part = part; p.r_part = r_part;
#define STEMWG(NC, X3V, KHV, SWV)                                                                                     \
  do {                                                                                                                \
    static LdsLimitOnce lds_once;                                                                                     \
    if (hipError_t e = set_lds_limit_once(lds_once, reinterpret_cast<const void*>(&stem_wgrad_kernel<NC, X3V, KHV, SWV>), 80 * 1024); \
        e != hipSuccess) return e;                                                                                    \
    hipLaunchKernelGGL((stem_wgrad_kernel<NC, X3V, KHV, SWV>), dim3(pl.grid), dim3(256), pl.lds, st, p);              \
  } while (0)
  if (pl.known) STEMWG(2, true, 7, 2);
  else if (pl.x3) { if (pl.nco == 1) STEMWG(1, true, 0, 0); else if (pl.nco == 2) STEMWG(2, true, 0, 0); else STEMWG(4, true, 0, 0); }
  else { if (pl.nco == 1) STEMWG(1, false, 0, 0); else if (pl.nco == 2) STEMWG(2, false, 0, 0); else STEMWG(4, false, 0, 0); }
#undef STEMWG
  return hipGetLastError();
}

bool stem_dgrad_supported(const Geom& g, int dtype) {
  if (!stem_shape(g, dtype)) return false;
  StemDgParams p;
  return stem_dg_plan(g, &p).ok;
}
// Whether the launch takes the fold-back along: only where both fit the chip at once.  The input gradient's workgroups are
// persistent, one behind a full round of them would start when they end (x[32,3,224,224], 7x7 / 2: 89.1 us a pass like that, 85.1
// with a launch of its own).
bool stem_dgrad_folds_back_aside(const Geom& g) {
  StemDgParams p;
  const StemDgPlan pl = stem_dg_plan(g, &p);
  return pl.ok && g.K >= 4 && pl.grid + fold_back_side_blocks(g.K, stem_wgrad_slices(g), g.Cout, 256) <= pl.room;
}
namespace {
template <int UU, int VV, int KS, class Side>
hipError_t launch_dgrad_inst(const StemDgParams& p, const StemDgPlan& pl, Side side, hipStream_t st) {
  static LdsLimitOnce lds_once;
  if (hipError_t e = set_lds_limit_once(lds_once, reinterpret_cast<const void*>(&stem_dgrad_kernel<UU, VV, KS, Side>), 80 * 1024);
      e != hipSuccess) return e;
  int nside = 0;
  size_t lds = pl.lds;
  if constexpr (Side::BACK) {
    nside = fold_back_side_blocks(side, 256);
    if (lds < (size_t)FOLD_BACK_SIDE_BYTES(256)) lds = FOLD_BACK_SIDE_BYTES(256);
  }
  hipLaunchKernelGGL((stem_dgrad_kernel<UU, VV, KS, Side>), dim3(pl.grid + nside), dim3(256), lds, st, p, side);
  return hipGetLastError();
}
}  // namespace
// w_crsk: w' as [Cin][kH][kW][Cout]
hipError_t launch_dgrad_stem(const Geom& g, const void* dz, const void* w_crsk, void* dx, hipStream_t st) {
  StemDgParams p;
  const StemDgPlan pl = stem_dg_plan(g, &p);
  if (!pl.ok) return hipErrorInvalidValue;
  p.dz = (const bf16_t*)dz; p.w = (const bf16_t*)w_crsk; p.dx = (bf16_t*)dx;
  p.nwg = pl.grid;
  if (g.fold_back) return pl.known ? launch_dgrad_inst<4, 4, 2>(p, pl, *g.fold_back, st) : launch_dgrad_inst<0, 0, 0>(p, pl, *g.fold_back, st);
  return pl.known ? launch_dgrad_inst<4, 4, 2>(p, pl, FoldSide{}, st) : launch_dgrad_inst<0, 0, 0>(p, pl, FoldSide{}, st);
}

bool stem_fprop_supported(const Geom& g, int dtype) {
  if (!stem_shape(g, dtype)) return false;
  StemParams p;
  return stem_plan(g, &p).ok;
}

// x: the input as it is, or its 4-channel copy where stem_input_copy_bytes() != 0; w: the (folded, or with bn the unfolded)
// weight in its own [Cout][kH][kW][Cin] order
hipError_t launch_fprop_stem(const Geom& g, const void* x, const void* w, const float* bias, void* z, int relu, hipStream_t st,
                             const BnEpilogue* bn) {
  StemParams p;
  const StemPlan pl = stem_plan(g, &p);
  if (!pl.ok) return hipErrorInvalidValue;
  if (bn) p.bn = *bn;
  p.relu = relu;
  p.x = (const bf16_t*)x; p.w = (const bf16_t*)w; p.bias = bias; p.z = (bf16_t*)z;
#define STEM(NC, KHV, X3V)                                                                                              \
  do {                                                                                                             \
    static LdsLimitOnce lds_once;                                                                                  \
    if (hipError_t e = set_lds_limit_once(lds_once, reinterpret_cast<const void*>(&stem_fprop_kernel<NC, KHV, X3V>), \
                                          64 * 1024); e != hipSuccess) return e;                                   \
    hipLaunchKernelGGL((stem_fprop_kernel<NC, KHV, X3V>), dim3(pl.grid), dim3(256), pl.lds, st, p);                \
  } while (0)
  if (pl.nco == 2 && g.kH == 7 && pl.x3) STEM(2, 7, true);   // the usual 7x7 RGB stem, 33 to 64 channels: rows unrolled
  else if (pl.x3) { if (pl.nco == 1) STEM(1, 0, true); else if (pl.nco == 2) STEM(2, 0, true); else STEM(4, 0, true); }
  else if (pl.nco == 1) STEM(1, 0, false);
  else if (pl.nco == 2) STEM(2, 0, false);
  else STEM(4, 0, false);
#undef STEM
  return hipGetLastError();
}

}  // namespace convbn
