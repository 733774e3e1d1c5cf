// Depthwise ConvBN block in Tune mode: one filter per channel (groups = channels), BatchNorm folded into
// the filter exactly as for the dense block (Sec. 3.3: the scale is per output channel, so
// w'[c] = s_c w[c], b' = (b - mu) s + beta), backward by Table 2's "Tune" row.
//
// A depthwise convolution has 2 k^2 FLOP per output element against 2-4 bytes of traffic: it is bound by
// memory, not by the matrix cores, so these are plain vector kernels: channels-last tensors, a thread owns
// VEC consecutive channels of one pixel (bf16: 8 channels = one 16-byte access, consecutive threads =
// consecutive channels), the k^2 window positions are re-read through the caches.
//   x, dx [N][H][W][C]   z, dz [N][Ho][Wo][C]   W, dW [C][kH][kW]   folded filter wf [kH kW][C] (tap-major)
#include "common.h"

#include <type_traits>

namespace convbn {

namespace {

template <typename T, int VEC> struct Vec;
template <> struct Vec<float, 1> {
  static __device__ __forceinline__ void load(const float* p, float (&v)[1]) { v[0] = *p; }
  static __device__ __forceinline__ void store(float* p, const float (&v)[1]) { *p = v[0]; }
};
template <> struct Vec<bf16_t, 1> {
  static __device__ __forceinline__ void load(const bf16_t* p, float (&v)[1]) { v[0] = (float)*p; }
  static __device__ __forceinline__ void store(bf16_t* p, const float (&v)[1]) { *p = (bf16_t)v[0]; }
};
template <> struct Vec<bf16_t, 8> {
  static __device__ __forceinline__ void load(const bf16_t* p, float (&v)[8]) {
    const uint4 t = *reinterpret_cast<const uint4*>(p);
    v[0] = bf16_lo(t.x); v[1] = bf16_hi(t.x); v[2] = bf16_lo(t.y); v[3] = bf16_hi(t.y);
    v[4] = bf16_lo(t.z); v[5] = bf16_hi(t.z); v[6] = bf16_lo(t.w); v[7] = bf16_hi(t.w);
  }
  static __device__ __forceinline__ void store(bf16_t* p, const float (&v)[8]) {
    *reinterpret_cast<uint4*>(p) = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                                              pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
  }
};

// wf[tap][c] = s_c W[c][tap], bfold[c] = (b - mu) s + beta.  gamma == nullptr: s = 1, b' = b.
template <typename T>
__global__ __launch_bounds__(256) void dw_fold_kernel(const T* __restrict__ W, const float* __restrict__ b,
                                                      const float* __restrict__ gamma, const float* __restrict__ beta,
                                                      const float* __restrict__ mean, const float* __restrict__ var,
                                                      float eps, int C, int taps, T* __restrict__ wf,
                                                      float* __restrict__ bfold) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= C) return;
  const float s = gamma ? gamma[c] / sqrtf(var[c] + eps) : 1.f;
  if (wf)
    for (int t = 0; t < taps; ++t) wf[(size_t)t * C + c] = from_f32<T>(to_f32(W[(size_t)c * taps + t]) * s);
  if (bfold) bfold[c] = gamma ? ((b ? b[c] : 0.f) - mean[c]) * s + beta[c] : (b ? b[c] : 0.f);
}

// Z[m][c] = b'[c] + sum_tap wf[tap][c] X[window position][c]
template <typename T, int VEC>
__global__ __launch_bounds__(256) void dw_fprop_kernel(const T* __restrict__ x, const T* __restrict__ wf,
                                                       const float* __restrict__ bias, T* __restrict__ z, Geom g) {
  const int cgs = g.Cin / VEC;
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (size_t)g.M * cgs) return;
  const int c = (int)(idx % cgs) * VEC;
  int m = (int)(idx / cgs);
  const int wo = m % g.Wout;
  m /= g.Wout;
  const int ho = m % g.Hout, n = m / g.Hout;
  float acc[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) acc[e] = bias ? bias[c + e] : 0.f;
  for (int i = 0; i < g.kH; ++i) {
    const int h = ho * g.sh + i - g.ph;
    if ((unsigned)h >= (unsigned)g.Hin) continue;
    for (int j = 0; j < g.kW; ++j) {
      const int w = wo * g.sw + j - g.pw;
      if ((unsigned)w >= (unsigned)g.Win) continue;
      float xv[VEC], wv[VEC];
      Vec<T, VEC>::load(x + (((size_t)n * g.Hin + h) * g.Win + w) * g.Cin + c, xv);
      Vec<T, VEC>::load(wf + (size_t)(i * g.kW + j) * g.Cin + c, wv);
#pragma unroll
      for (int e = 0; e < VEC; ++e) acc[e] += xv[e] * wv[e];
    }
  }
  Vec<T, VEC>::store(z + idx * VEC, acc);
}

// dX[m'][c] = sum_tap wf[tap][c] dZ[(h + ph - i)/sh, (w + pw - j)/sw][c] over the taps whose quotients are exact
template <typename T, int VEC>
__global__ __launch_bounds__(256) void dw_dgrad_kernel(const T* __restrict__ dz, const T* __restrict__ wf,
                                                       T* __restrict__ dx, Geom g) {
  const int cgs = g.Cin / VEC;
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (size_t)g.Min * cgs) return;
  const int c = (int)(idx % cgs) * VEC;
  int m = (int)(idx / cgs);
  const int w = m % g.Win;
  m /= g.Win;
  const int h = m % g.Hin, n = m / g.Hin;
  float acc[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
  for (int i = 0; i < g.kH; ++i) {
    const int hz = h + g.ph - i;
    if (hz < 0 || hz % g.sh != 0) continue;
    const int ho = hz / g.sh;
    if (ho >= g.Hout) continue;
    for (int j = 0; j < g.kW; ++j) {
      const int wz = w + g.pw - j;
      if (wz < 0 || wz % g.sw != 0) continue;
      const int wo = wz / g.sw;
      if (wo >= g.Wout) continue;
      float gv[VEC], wv[VEC];
      Vec<T, VEC>::load(dz + (((size_t)n * g.Hout + ho) * g.Wout + wo) * g.Cin + c, gv);
      Vec<T, VEC>::load(wf + (size_t)(i * g.kW + j) * g.Cin + c, wv);
#pragma unroll
      for (int e = 0; e < VEC; ++e) acc[e] += gv[e] * wv[e];
    }
  }
  Vec<T, VEC>::store(dx + idx * VEC, acc);
}

// ---- 3x3 windows, stride 1 or 2, any padding, bf16, C % 8 == 0 -------------------------------------------------
// A pass has to move its tensors once and multiply 9 times per element (18 with the weight gradient), so two things
// bound it: the bytes in flight, and the vector unit.  A thread owns 4 channels (8 bytes; consecutive threads =
// consecutive channels, then columns) of two neighbouring columns and slides down R rows: an input row is requested
// two steps (stride 2: one) before it is used, widened once, and multiplied into the three output rows that it
// reaches, which live in registers; the column overlap is re-read from the L1 (4 columns for 2 outputs).  Input gradient
// and weight gradient are one sweep -- dx and dw' both need dZ, and the pixel that owns a dx element owns its x too, so
// the halo is one tensor's --, and the filter is folded by the threads that use it: a forward pass is one launch, a
// backward pass two.  Before (a thread per four outputs of one column, all loads of its patch up front, each pass and
// the fold a launch of its own): 144 channels at 56 x 56, 32 images, 80.1 us a pass; now 38.2 (forward 14.4, backward 20.6,
// fold-back 4.8 in a trace that adds launches' ends; 144 MB).  4 x 2 and two steps ahead: three rows ahead, 256 threads a workgroup and 16-byte accesses were no
// faster; non-temporal loads cost the column overlap its L1 hits (54.6).  Stores: streams_output and STREAM_GRAD in common.h.
// Out-of-image loads and stores are offsets beyond the buffer, which read zeros and are dropped.
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
constexpr int DW_BLK = 512;              // threads of a workgroup
constexpr int DW_MAXQ = 64;              // channel quads of a workgroup (the others are its columns)
constexpr unsigned DW_INV = 1u << 30;    // row or column offset of nothing; twice that is still no valid offset

struct Dw3Params {
  const bf16_t* a;       // the tensor with the halo: x (forward), dZ (backward)
  const bf16_t* y;       // weight gradient: x
  bf16_t* out;           // z or dx
  const bf16_t* W;       // [C][9], or the folded filter [9][C] (tap_major)
  const float *b, *gamma, *beta, *mean, *var;   // gamma == null: s = 1; b: forward
  bf16_t* wf_out;        // forward: where the folded filter [9][C] is left, or null
  float* part;           // weight gradient: [C / 8][slices_all][10][8], row 9 the channel sums of dZ
  float eps;
  int tap_major;
  int N, C, Ha, Wa, Ho, Wo;     // images; a's and out's (and y's) planes
  int pa, pb;                   // a's row for output row o and window row i: o S + i - pa
  int u0, v0;                   // backward: the first column and row of the threads' domain (stride 1: of x, 2: of dZ)
  int R, nstrip, npair, cq, items, per_slice, slice0, slices_all;
  // A launch's offsets are 32 bits from the first rows that it touches: images of 1 GiB and more go in bands of strips.
  int strip0;                   // the launch's first strip
  int a_row0, o_row0;           // the rows that a, and out and y, point to
  unsigned a_bytes, o_bytes;    // how much of them a launch touches
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t dw_rsrc(const void* p, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ u32x2 dw_load(__amdgpu_buffer_rsrc_t r, unsigned off) {
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
}
template <bool STREAM>
__device__ __forceinline__ void dw_store(__amdgpu_buffer_rsrc_t r, unsigned off, const float (&v)[4]) {
  u32x2 t;
  t.x = pack_bf16x2(v[0], v[1]);
  t.y = pack_bf16x2(v[2], v[3]);
  __builtin_amdgcn_raw_buffer_store_b64(t, r, (int)off, 0, STREAM ? 2 : 0);
}
__device__ __forceinline__ void unpack4(u32x2 t, float (&v)[4]) {
  v[0] = bf16_lo(t.x); v[1] = bf16_hi(t.x); v[2] = bf16_lo(t.y); v[3] = bf16_hi(t.y);
}

// Workgroups are handed to the eight XCDs in turn: neighbouring slices, which share rows, go to one XCD and its L2.
__device__ __forceinline__ int dw_slice() {
  const int n = gridDim.y, b = blockIdx.y;
  return gridDim.x == 1 && n % 8 == 0 ? (b & 7) * (n >> 3) + (b >> 3) : b;
}

// The filter of a thread's 4 channels (s already in it) and, in forward (FWD), their b'.  Backward folds the w' that forward
// would have kept, rounded as that is.
template <bool FWD, bool ROT>
__device__ __forceinline__ void dw_filter(const Dw3Params& p, int c, float (&t)[9][4], float (&bb)[4]) {
  // (every load is issued before the first use; a vector that is not there is read from the filter, which is larger)
  const float* const any = reinterpret_cast<const float*>(p.W);
  const float4 ga = *reinterpret_cast<const float4*>((p.gamma ? p.gamma : any) + c);
  const float4 va = *reinterpret_cast<const float4*>((p.gamma ? p.var : any) + c);
  const float4 me = *reinterpret_cast<const float4*>((FWD && p.gamma ? p.mean : any) + c);
  const float4 be = *reinterpret_cast<const float4*>((FWD && p.gamma ? p.beta : any) + c);
  const float4 bi = *reinterpret_cast<const float4*>((FWD && p.b ? p.b : any) + c);
  const float gv[4] = {ga.x, ga.y, ga.z, ga.w}, vv[4] = {va.x, va.y, va.z, va.w}, mv[4] = {me.x, me.y, me.z, me.w};
  const float ev[4] = {be.x, be.y, be.z, be.w}, iv[4] = {bi.x, bi.y, bi.z, bi.w};
  float s[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    s[e] = p.gamma ? gv[e] / sqrtf(vv[e] + p.eps) : 1.f;
    const float b0 = p.b ? iv[e] : 0.f;
    bb[e] = !FWD ? 0.f : p.gamma ? (b0 - mv[e]) * s[e] + ev[e] : b0;
  }
  float w[9][4];
  if (!FWD && p.tap_major) {
#pragma unroll
    for (int q = 0; q < 9; ++q) unpack4(*reinterpret_cast<const u32x2*>(p.W + (size_t)q * p.C + c), w[q]);
  } else {
    unsigned raw[18];   // 36 consecutive values: element e * 9 + q is channel e, tap q
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const u32x2 v = *reinterpret_cast<const u32x2*>(p.W + (size_t)c * 9 + 4 * k);
      raw[2 * k] = v.x;
      raw[2 * k + 1] = v.y;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int q = 0; q < 9; ++q) {
        const int k = e * 9 + q;
        const float v = ((k & 1) ? bf16_hi(raw[k >> 1]) : bf16_lo(raw[k >> 1])) * s[e];
        w[q][e] = FWD ? v : (float)(bf16_t)v;
      }
  }
#pragma unroll
  for (int q = 0; q < 9; ++q)
#pragma unroll
    for (int e = 0; e < 4; ++e) t[q][e] = ROT ? w[8 - q][e] : w[q][e];
}
// w'[tap][c] = bf16(s w), a value per thread of the launch's first threads
__device__ __forceinline__ void dw_emit_folded(const Dw3Params& p) {
  if (!p.wf_out) return;
  const int nthr = gridDim.x * gridDim.y * DW_BLK;
  for (int j = (blockIdx.y * gridDim.x + blockIdx.x) * DW_BLK + threadIdx.x; j < 9 * p.C; j += nthr) {
    const int q = j / p.C, c = j - q * p.C;
    const float s = p.gamma ? p.gamma[c] / sqrtf(p.var[c] + p.eps) : 1.f;
    p.wf_out[j] = (bf16_t)((float)p.W[(size_t)c * 9 + q] * s);
  }
}

// Sums the weight-gradient accumulators of a workgroup's threads (thread = column lane * cq + quad) over its column lanes
// and writes them as one slice of `part`.  Five of the ten rows at a time: 40 KB of LDS.
__device__ __forceinline__ void dw_slice_sums(const Dw3Params& p, const float (&acc)[10][4], int L, float* red) {
  const int tid = threadIdx.x, ncol = p.cq * 4;
  const int slice = p.slice0 + dw_slice();
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 5; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) red[(q * 4 + e) * DW_BLK + tid] = acc[half * 5 + q][e];
    __syncthreads();
    for (int j = tid; j < 5 * ncol; j += DW_BLK) {
      const int q = j / ncol, col = j - q * ncol;
      const int c = (int)blockIdx.x * ncol + col;
      if (c >= p.C) continue;
      const float* src = red + (q * 4 + (col & 3)) * DW_BLK + (col >> 2);
      float v = 0.f;
      for (int l = 0; l < L; ++l) v += src[l * p.cq];
      p.part[(((size_t)(c >> 3) * p.slices_all + slice) * 10 + half * 5 + q) * 8 + (c & 7)] = v;
    }
  }
}

// Stride 1.  CONV: out[n][h][w] = b' + sum_{i,j} T[i][j] a[n][h + i - pa][w + j - pb], T the filter (backward: rotated).
// WG (a = dZ): dw'[8 - (i, j)] += y[n][h][w] a[n][h + i - pa][w + j - pb] over the owned (h, w), and the sums of a.
// Products with a position outside an image are skipped, not multiplied by zero: an infinite x or dZ at the border does
// not reach the taps that do not touch it.
// PAD1: pa = pb = 1, the sizes of a and out are the same.  Paddings above 2 put dZ rows and columns in front of (and behind) all
// that x meets: they count in the sums of a alone, and the domain starts with them, before the first row of x.
template <bool FWD, bool CONV, bool WG, bool PAD1, bool STREAM>
__global__ __launch_bounds__(DW_BLK, WG ? 2 : 4) void dw3_s1_kernel(Dw3Params p) {
  __shared__ float red[WG ? 20 * DW_BLK : 1];
  if (FWD) dw_emit_folded(p);
  const int pad_h = PAD1 ? 1 : p.pa, pad_w = PAD1 ? 1 : p.pb;
  constexpr bool AHEAD = !FWD && !PAD1;   // the domain may start before the first row of out
  const int L = DW_BLK / p.cq;
  const int tx = threadIdx.x % p.cq, lane = threadIdx.x / p.cq;
  const int c = ((int)blockIdx.x * p.cq + tx) * 4;
  const bool live = lane < L && c < p.C;
  const unsigned px = (unsigned)p.C * 2u, arow = px * p.Wa, orow = px * p.Wo;
  const __amdgpu_buffer_rsrc_t ra = dw_rsrc(p.a, p.a_bytes), ry = dw_rsrc(WG ? p.y : p.a, p.o_bytes);
  const __amdgpu_buffer_rsrc_t ro = dw_rsrc(p.out, p.o_bytes);
  float t[9][4], bb[4], wacc[10][4];
  if constexpr (WG) {
#pragma unroll
    for (int q = 0; q < 10; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) wacc[q][e] = 0.f;
  }
  const int slice = dw_slice(), it1 = min(p.items, (slice + 1) * p.per_slice);
  if (CONV && !WG && live) dw_filter<FWD, !FWD>(p, c, t, bb);
  bool first = true;
  if (live)
    for (int it = slice * p.per_slice + lane; it < it1; it += L) {
      const int pair = it % p.npair;
      const int rest = it / p.npair;
      const int strip = p.strip0 + rest % p.nstrip, n = rest / p.nstrip;
      const int w0 = pair * 2 + (AHEAD ? p.u0 : 0), h0 = strip * p.R + (AHEAD ? p.v0 : 0);
      unsigned acol[4], ocol[2];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int w = w0 + k - pad_w;
        acol[k] = (unsigned)w < (unsigned)p.Wa ? (unsigned)w * px : DW_INV;
      }
#pragma unroll
      for (int k = 0; k < 2; ++k) ocol[k] = (unsigned)(w0 + k) < (unsigned)p.Wo ? (unsigned)(w0 + k) * px : DW_INV;
      const bool has_l = acol[0] != DW_INV, has_r = acol[3] != DW_INV, two = ocol[1] != DW_INV;
      const unsigned abase = (unsigned)(n * p.Ha - p.a_row0) * arow + c * 2u, obase = (unsigned)(n * p.Ho - p.o_row0) * orow + c * 2u;
      // running offsets: the next row of a (with its index), of y and of out
      const int nq = p.R + 2, rows = max(min(p.Ho - h0, p.R), 0), hend = max(min(p.Ha, h0 - pad_h + nq), 0);
      const int row0 = AHEAD ? max(-h0, 0) : 0;   // the strip's first row that out has
      int ha = h0 - pad_h;
      unsigned aoff = abase + (unsigned)ha * arow, yoff = obase + (unsigned)h0 * orow, ooff = yoff - 2 * orow;
      u32x2 pa[2][4], py[2][2];
      auto fetch = [&](int q, int slot) {   // (unconditional: steps past the last one read nothing)
        const unsigned r = (unsigned)ha < (unsigned)hend ? aoff : DW_INV;
        ++ha;
        aoff += arow;
#pragma unroll
        for (int k = 0; k < 4; ++k) pa[slot][k] = dw_load(ra, r + acol[k]);
        if constexpr (WG) {
          const unsigned s = q >= row0 && q < rows ? yoff : DW_INV;
          yoff += orow;
#pragma unroll
          for (int k = 0; k < 2; ++k) py[slot][k] = dw_load(ry, s + ocol[k]);
        }
      };
      fetch(0, 0);
      fetch(1, 1);
      if (CONV && WG && first) dw_filter<FWD, !FWD>(p, c, t, bb);   // (behind the first rows' requests)
      first = false;
      float acc[3][2][4], yv[3][2][4], ye[3][2][4];   // ye: zero where the neighbouring column of a is outside
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int e = 0; e < 4; ++e) { acc[k][x][e] = 0.f; yv[k][x][e] = 0.f; ye[k][x][e] = 0.f; }
      for (int q0 = 0; q0 < nq; q0 += 6) {
#pragma unroll
        for (int u = 0; u < 6; ++u) {
          const int q = q0 + u;
          if (q >= nq) break;
          float av[4][4];
#pragma unroll
          for (int k = 0; k < 4; ++k) unpack4(pa[u & 1][k], av[k]);
          if constexpr (WG) {
#pragma unroll
            for (int k = 0; k < 2; ++k) unpack4(py[u & 1][k], yv[u % 3][k]);
            if constexpr (PAD1) {
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                ye[u % 3][0][e] = has_l ? yv[u % 3][0][e] : 0.f;
                ye[u % 3][1][e] = has_r ? yv[u % 3][1][e] : 0.f;
              }
            }
          }
          fetch(q + 2, u & 1);
          if constexpr (CONV) {
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
              for (int e = 0; e < 4; ++e) acc[u % 3][x][e] = bb[e];
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
              for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int x = 0; x < 2; ++x)
#pragma unroll
                  for (int e = 0; e < 4; ++e) acc[(u + 3 - i) % 3][x][e] += t[i * 3 + j][e] * av[x + j][e];
            const unsigned r = q - 2 >= row0 && q - 2 < rows ? ooff : DW_INV;   // the row that is complete now
            ooff += orow;
#pragma unroll
            for (int x = 0; x < 2; ++x) dw_store<STREAM>(ro, r + ocol[x], acc[(u + 1) % 3][x]);
          }
          if constexpr (WG) {
            if ((unsigned)(h0 + q - pad_h) < (unsigned)p.Ha) {
              if (q >= max(pad_h, 0) && q < max(pad_h, 0) + p.R) {   // a's owned pixels
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                  if constexpr (PAD1) wacc[9][e] += av[1][e] + av[2][e];
                  else wacc[9][e] += pad_w <= 0 ? av[0][e] + av[1][e] : pad_w == 1 ? av[1][e] + av[2][e] : av[2][e] + av[3][e];
                }
              }
#pragma unroll
              for (int i = 0; i < 3; ++i) {
                constexpr int T = 8;   // (a is swept with the rotated window)
                const float(&y)[2][4] = yv[(u + 3 - i) % 3];
                const float(&z)[2][4] = ye[(u + 3 - i) % 3];
                if (q >= i && q - i < p.R)   // (the others are the neighbouring strips' rows)
                  if (q - i >= row0 && q - i < rows) {
                    if constexpr (PAD1) {
#pragma unroll
                      for (int e = 0; e < 4; ++e) {
                        wacc[T - i * 3][e] += z[0][e] * av[0][e];
                        wacc[T - i * 3 - 1][e] += y[0][e] * av[1][e];
                      }
                      if (two) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                          wacc[T - i * 3 - 2][e] += y[0][e] * av[2][e] + z[1][e] * av[3][e];
                          wacc[T - i * 3][e] += y[1][e] * av[1][e];
                          wacc[T - i * 3 - 1][e] += y[1][e] * av[2][e];
                        }
                      }
                    } else {
#pragma unroll
                      for (int j = 0; j < 3; ++j)
#pragma unroll
                        for (int x = 0; x < 2; ++x)
                          if (ocol[x] != DW_INV && acol[x + j] != DW_INV) {
#pragma unroll
                            for (int e = 0; e < 4; ++e) wacc[T - i * 3 - j][e] += y[x][e] * av[x + j][e];
                          }
                    }
                  }
              }
            }
          }
        }
      }
    }
  if constexpr (WG) dw_slice_sums(p, wacc, L, red);
}

// Stride 2, forward: two neighbouring output columns (5 input columns); a step brings the two input rows that complete
// an output row, the second of which begins the next one.
template <bool STREAM>
__global__ __launch_bounds__(DW_BLK, 4) void dw3_s2_fprop_kernel(Dw3Params p) {
  dw_emit_folded(p);
  const int L = DW_BLK / p.cq;
  const int tx = threadIdx.x % p.cq, lane = threadIdx.x / p.cq;
  const int c = ((int)blockIdx.x * p.cq + tx) * 4;
  if (lane >= L || c >= p.C) return;
  const unsigned px = (unsigned)p.C * 2u, arow = px * p.Wa, orow = px * p.Wo;
  const __amdgpu_buffer_rsrc_t ra = dw_rsrc(p.a, p.a_bytes), ro = dw_rsrc(p.out, p.o_bytes);
  float t[9][4], bb[4];
  dw_filter<true, false>(p, c, t, bb);
  const int slice = dw_slice(), it1 = min(p.items, (slice + 1) * p.per_slice);
  for (int it = slice * p.per_slice + lane; it < it1; it += L) {
    const int pair = it % p.npair;
    const int rest = it / p.npair;
    const int strip = p.strip0 + rest % p.nstrip, n = rest / p.nstrip;
    const int w0 = pair * 2, h0 = strip * p.R;
    unsigned acol[5], ocol[2];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      const int w = w0 * 2 + k - p.pb;
      acol[k] = (unsigned)w < (unsigned)p.Wa ? (unsigned)w * px : DW_INV;
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) ocol[k] = w0 + k < p.Wo ? (unsigned)(w0 + k) * px : DW_INV;
    const unsigned abase = (unsigned)(n * p.Ha - p.a_row0) * arow + c * 2u, obase = (unsigned)(n * p.Ho - p.o_row0) * orow + c * 2u;
    u32x2 pa[2][5];
    auto fetch = [&](int q) {   // window rows 1 and 2 of output row h0 + q - 1
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int h = (h0 + q - 1) * 2 + 1 + i - p.pa;
        const unsigned r = q <= p.R && (unsigned)h < (unsigned)p.Ha ? abase + (unsigned)h * arow : DW_INV;
#pragma unroll
        for (int k = 0; k < 5; ++k) pa[i][k] = dw_load(ra, r + acol[k]);
      }
    };
    fetch(0);
    float acc[2][4];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[x][e] = 0.f;
    for (int q = 0; q <= p.R; ++q) {
      float av[2][5][4];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int k = 0; k < 5; ++k) unpack4(pa[i][k], av[i][k]);
      fetch(q + 1);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
          for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[x][e] += t[(i + 1) * 3 + j][e] * av[i][2 * x + j][e];
      const int o = h0 + q - 1;
      const unsigned r = q >= 1 && o < p.Ho ? obase + (unsigned)o * orow : DW_INV;
#pragma unroll
      for (int x = 0; x < 2; ++x) dw_store<STREAM>(ro, r + ocol[x], acc[x]);
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[x][e] = bb[e];
#pragma unroll
      for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[x][e] += t[j][e] * av[1][2 * x + j][e];
    }
  }
}

// Stride 2, backward.  In coordinates that count the padding (hh = h + ph), dZ row v reaches hh = 2v, 2v + 1, 2v + 2.  A
// thread that owns dZ columns u and u + 1 owns the x and dx columns 2u + 1 .. 2u + 4, which meet dZ columns u .. u + 2, and
// per step the rows 2v + 1 (window row 1 of dZ row v) and 2v + 2 (window row 2 of v, 0 of v + 1): with padding 1 nothing is
// computed twice and nothing lies outside.  u and v start at u0 and v0 (-1 with padding 0).
template <bool CONV, bool WG>
__global__ __launch_bounds__(DW_BLK, 2) void dw3_s2_bwd_kernel(Dw3Params p) {
  __shared__ float red[WG ? 20 * DW_BLK : 1];
  const int L = DW_BLK / p.cq;
  const int tx = threadIdx.x % p.cq, lane = threadIdx.x / p.cq;
  const int c = ((int)blockIdx.x * p.cq + tx) * 4;
  const bool live = lane < L && c < p.C;
  const unsigned px = (unsigned)p.C * 2u, arow = px * p.Wa, orow = px * p.Wo;
  const __amdgpu_buffer_rsrc_t ra = dw_rsrc(p.a, p.a_bytes), ry = dw_rsrc(WG ? p.y : p.a, p.o_bytes);
  const __amdgpu_buffer_rsrc_t ro = dw_rsrc(p.out, p.o_bytes);
  float t[9][4], bb[4], wacc[10][4];
  if (CONV && live) dw_filter<false, false>(p, c, t, bb);
  if constexpr (WG) {
#pragma unroll
    for (int q = 0; q < 10; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) wacc[q][e] = 0.f;
  }
  const int slice = dw_slice(), it1 = min(p.items, (slice + 1) * p.per_slice);
  if (live)
    for (int it = slice * p.per_slice + lane; it < it1; it += L) {
      const int pair = it % p.npair;
      const int rest = it / p.npair;
      const int strip = p.strip0 + rest % p.nstrip, n = rest / p.nstrip;
      const int u0 = p.u0 + pair * 2, v0 = p.v0 + strip * p.R;
      unsigned acol[3], ocol[4];
      bool inside = true;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const bool ok = (unsigned)(u0 + k) < (unsigned)p.Wa;
        acol[k] = ok ? (unsigned)(u0 + k) * px : DW_INV;
        inside &= ok;
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int w = 2 * u0 + 1 + k - p.pb;
        const bool ok = (unsigned)w < (unsigned)p.Wo;
        ocol[k] = ok ? (unsigned)w * px : DW_INV;
        inside &= ok;
      }
      const bool wave_inside = WG && __all(inside);
      const unsigned abase = (unsigned)(n * p.Ha - p.a_row0) * arow + c * 2u, obase = (unsigned)(n * p.Ho - p.o_row0) * orow + c * 2u;
      auto a_row = [&](int v) { return (unsigned)v < (unsigned)p.Ha ? abase + (unsigned)v * arow : DW_INV; };
      auto o_row = [&](int h) { return (unsigned)h < (unsigned)p.Ho ? obase + (unsigned)h * orow : DW_INV; };
      u32x2 pa[3], py[2][4];
      auto fetch = [&](int v) {   // dZ row v + 1 and the x rows of step v
        const bool step = v < v0 + p.R;
        const unsigned r = step ? a_row(v + 1) : DW_INV;
#pragma unroll
        for (int k = 0; k < 3; ++k) pa[k] = dw_load(ra, r + acol[k]);
        if constexpr (WG) {
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const unsigned s = step ? o_row(2 * v + 1 + i - p.pa) : DW_INV;
#pragma unroll
            for (int k = 0; k < 4; ++k) py[i][k] = dw_load(ry, s + ocol[k]);
          }
        }
      };
      float a0[3][4], a1[3][4];   // dZ rows v and v + 1
      {
        const unsigned r = a_row(v0);
        u32x2 f[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) f[k] = dw_load(ra, r + acol[k]);
        fetch(v0);
#pragma unroll
        for (int k = 0; k < 3; ++k) unpack4(f[k], a0[k]);
      }
      for (int q = 0; q < p.R; ++q) {
        const int v = v0 + q;
        float yv[2][4][4];
#pragma unroll
        for (int k = 0; k < 3; ++k) unpack4(pa[k], a1[k]);
        if constexpr (WG) {
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int k = 0; k < 4; ++k) unpack4(py[i][k], yv[i][k]);
        }
        fetch(v + 1);
        // column k of the four meets: k = 0: tap 1 of u;  1: tap 0 of u + 1, tap 2 of u;  2: tap 1 of u + 1;
        // 3: tap 0 of u + 2, tap 2 of u + 1
        if constexpr (CONV) {
          float acc[2][4][4];
#pragma unroll
          for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int m = k >> 1;
              if (k & 1) {
                acc[0][k][e] = t[3][e] * a0[m + 1][e] + t[5][e] * a0[m][e];
                acc[1][k][e] = t[0][e] * a1[m + 1][e] + t[2][e] * a1[m][e] + t[6][e] * a0[m + 1][e] + t[8][e] * a0[m][e];
              } else {
                acc[0][k][e] = t[4][e] * a0[m][e];
                acc[1][k][e] = t[1][e] * a1[m][e] + t[7][e] * a0[m][e];
              }
            }
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const unsigned r = o_row(2 * v + 1 + i - p.pa);
#pragma unroll
            for (int k = 0; k < 4; ++k) dw_store<STREAM_GRAD>(ro, r + ocol[k], acc[i][k]);
          }
        }
        if constexpr (WG) {
#pragma unroll
          for (int e = 0; e < 4; ++e) wacc[9][e] += a0[0][e] + a0[1][e];
          const bool z0 = (unsigned)v < (unsigned)p.Ha, z1 = (unsigned)(v + 1) < (unsigned)p.Ha;
          const bool r1 = (unsigned)(2 * v + 1 - p.pa) < (unsigned)p.Ho, r2 = (unsigned)(2 * v + 2 - p.pa) < (unsigned)p.Ho;
          if (wave_inside && __all(z0 && z1 && r1 && r2)) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const int m = k >> 1;
                if (k & 1) {
                  wacc[3][e] += yv[0][k][e] * a0[m + 1][e];
                  wacc[5][e] += yv[0][k][e] * a0[m][e];
                  wacc[0][e] += yv[1][k][e] * a1[m + 1][e];
                  wacc[2][e] += yv[1][k][e] * a1[m][e];
                  wacc[6][e] += yv[1][k][e] * a0[m + 1][e];
                  wacc[8][e] += yv[1][k][e] * a0[m][e];
                } else {
                  wacc[4][e] += yv[0][k][e] * a0[m][e];
                  wacc[1][e] += yv[1][k][e] * a1[m][e];
                  wacc[7][e] += yv[1][k][e] * a0[m][e];
                }
              }
          } else {
            auto prod = [&](float (&w)[4], bool ok, const float (&x)[4], unsigned xcol, const float (&a)[4], unsigned zcol) {
              if (ok && xcol != DW_INV && zcol != DW_INV) {
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] += x[e] * a[e];
              }
            };
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const int m = k >> 1;
              if (k & 1) {
                prod(wacc[3], r1 && z0, yv[0][k], ocol[k], a0[m + 1], acol[m + 1]);
                prod(wacc[5], r1 && z0, yv[0][k], ocol[k], a0[m], acol[m]);
                prod(wacc[0], r2 && z1, yv[1][k], ocol[k], a1[m + 1], acol[m + 1]);
                prod(wacc[2], r2 && z1, yv[1][k], ocol[k], a1[m], acol[m]);
                prod(wacc[6], r2 && z0, yv[1][k], ocol[k], a0[m + 1], acol[m + 1]);
                prod(wacc[8], r2 && z0, yv[1][k], ocol[k], a0[m], acol[m]);
              } else {
                prod(wacc[4], r1 && z0, yv[0][k], ocol[k], a0[m], acol[m]);
                prod(wacc[1], r2 && z1, yv[1][k], ocol[k], a1[m], acol[m]);
                prod(wacc[7], r2 && z0, yv[1][k], ocol[k], a0[m], acol[m]);
              }
            }
          }
        }
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
          for (int e = 0; e < 4; ++e) a0[k][e] = a1[k][e];
      }
    }
  if constexpr (WG) dw_slice_sums(p, wacc, L, red);
}

// Sums the slices of 8 channels (a workgroup's 320 bytes of a slice are contiguous) and folds back; gamma == null (Eval):
// dW = dw' only.
__global__ __launch_bounds__(1024) void dw3_fold_back_kernel(const float* __restrict__ part, int slices,
                                                             const bf16_t* __restrict__ W, const float* __restrict__ b,
                                                             const float* __restrict__ gamma, const float* __restrict__ mean,
                                                             const float* __restrict__ var, float eps,
                                                             bf16_t* __restrict__ dW, float* __restrict__ db,
                                                             float* __restrict__ dgamma, float* __restrict__ dbeta) {
  constexpr int LN = 51;   // slice lanes: 51 x 20 float4 of the 1024 threads
  __shared__ float4 red[LN * 20];
  __shared__ float mid[8][80];
  __shared__ float sums[80];
  const int tid = threadIdx.x;
  const int v4 = tid % 20, l = tid / 20;
  // (everything that is read is asked for at once) thread q * 8 + e: tap q of channel e, thread e: its vectors
  const int ch = blockIdx.x * 8 + (tid & 7);
  float w = 0.f, ga = 1.f, va = 1.f, mu = 0.f, bc = 0.f;
  if (tid < 72) w = (float)W[(size_t)ch * 9 + (tid >> 3)];
  if (tid < 72 && gamma) {
    ga = gamma[ch];
    va = var[ch];
    mu = mean[ch];
    if (b) bc = b[ch];
  }
  const float4* src = reinterpret_cast<const float4*>(part + (size_t)blockIdx.x * slices * 80);
  if (l < LN) {
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 6
    for (int s = l; s < slices; s += LN) {
      const float4 t = src[(size_t)s * 20 + v4];
      a.x += t.x; a.y += t.y; a.z += t.z; a.w += t.w;
    }
    red[l * 20 + v4] = a;
  }
  __syncthreads();
  const float* rf = reinterpret_cast<const float*>(red);
  if (tid < 640) {
    const int o = tid % 80, k = tid / 80;
    float v = 0.f;
#pragma unroll
    for (int j = 0; j < 7; ++j)
      if (k + 8 * j < LN) v += rf[(k + 8 * j) * 80 + o];
    mid[k][o] = v;
  }
  __syncthreads();
  if (tid < 80) {
    float v = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) v += mid[k][tid];
    sums[tid] = v;
  }
  __syncthreads();
  const float sd = gamma ? sqrtf(va + eps) : 1.f;
  const float sc = gamma ? ga / sd : 1.f;
  if (tid < 72) {
    const float dw = sums[tid];
    dW[(size_t)ch * 9 + (tid >> 3)] = (bf16_t)(sc * dw);
    mid[0][tid] = dw * w;
  }
  __syncthreads();
  if (tid >= 8 || !gamma) return;
  float dot = 0.f;
#pragma unroll
  for (int q = 0; q < 9; ++q) dot += mid[0][q * 8 + tid];
  const float r = sums[72 + tid];
  dgamma[ch] = (dot + r * (bc - mu)) / sd;
  dbeta[ch] = r;
  if (db) db[ch] = sc * r;
}

// ---- host side of these kernels
size_t dw3_row_bytes(const Geom& g) { return (size_t)(g.Win > g.Wout ? g.Win : g.Wout) * g.Cin * 2; }
bool dw3_shape(const Geom& g, int dtype) {   // an image fits a launch, or bands of a strip or two of it (eight rows) do
  const size_t rows = g.Hin > g.Hout ? g.Hin : g.Hout;
  return dtype == CONVBN_BF16 && g.Cin % 8 == 0 && g.kH == 3 && g.kW == 3 && g.sh == g.sw && (g.sh == 1 || g.sh == 2) &&
         (rows < 8 ? rows : 8) * dw3_row_bytes(g) < DW_INV;
}
struct Dw3Plan {
  int cq, nxb;               // channel quads of a workgroup, workgroups across the channels
  int imgs, band, launches;  // images and strips of a launch (all, or a band of one image's), launches
  int R, nstrip, npair, slices, per_slice;
};
// `waves`: per SIMD.  Rows per strip: as many as give every thread the same number of strips, a strip costing its rows
// and the ones it shares with its neighbours (`extra`).
Dw3Plan dw3_plan(const Geom& g, int rows, int cols, int extra, int waves) {
  Dw3Plan p;
  const int quads = g.Cin / 4;
  p.nxb = ceil_div(quads, DW_MAXQ);
  p.cq = ceil_div(quads, p.nxb);
  const int fit_rows = (int)((DW_INV - 1) / dw3_row_bytes(g));   // of the larger tensor, in one launch
  const int img_rows = g.Hin > g.Hout ? g.Hin : g.Hout;
  p.imgs = fit_rows / img_rows < g.N ? fit_rows / img_rows : g.N;
  const bool banded = p.imgs == 0;
  if (banded) p.imgs = 1;
  // a band of B strips touches at most sh B R + 4 rows of a tensor; bands are equally long but for the last
  const int most = banded ? (fit_rows - 4) / g.sh : rows;
  auto strips = [&](int ns, int R) { return banded ? ceil_div(ns, ceil_div(ns, most / R)) : ns; };   // of a launch
  p.npair = ceil_div(cols, 2);
  const int L = DW_BLK / p.cq;
  int want = 256 * waves / 2 / p.nxb;      // workgroups of eight waves that the chip holds
  if (want < 1) want = 1;
  long long best = -1;
  p.R = 1;
  for (int ns = 1; ns <= rows; ++ns) {
    const int R = ceil_div(rows, ns);
    if (ceil_div(rows, R) != ns || R > most) continue;
    const long long items = (long long)p.imgs * strips(ns, R) * p.npair;
    const long long rounds = (items + (long long)want * L - 1) / ((long long)want * L);
    const long long cost = ceil_div(ns, strips(ns, R)) * rounds * (R + extra);
    if (best < 0 || cost < best) { best = cost; p.R = R; }
  }
  p.nstrip = ceil_div(rows, p.R);
  p.band = strips(p.nstrip, p.R);
  p.launches = ceil_div(g.N, p.imgs) * ceil_div(p.nstrip, p.band);
  const int items = p.imgs * p.band * p.npair;
  const int rounds = ceil_div(items, want * L);
  p.per_slice = rounds * L;
  p.slices = ceil_div(items, p.per_slice);
  return p;
}
Dw3Plan dw3_fprop_plan(const Geom& g) {
  return planned<Dw3Plan>(g, 1, [&] { return dw3_plan(g, g.Hout, g.Wout, g.sh == 1 ? 4 : 2, 4); });
}
int dw3_first(int pad) { return pad == 0 ? -1 : 0; }   // stride 2: the first dZ row (column) that owns x rows
Dw3Plan dw3_bwd_plan(const Geom& g) {
  return planned<Dw3Plan>(g, 1, [&] {
    if (g.sh == 1)   // (what starts ahead of x ends behind it: paddings above 2 make dZ the larger)
      return dw3_plan(g, g.Hin > g.Hout ? g.Hin : g.Hout, g.Win > g.Wout ? g.Win : g.Wout, 4, 2);
    // x row Hin - 1 belongs to the step v with 2 v + 2 >= Hin - 1 + ph; every dZ row is some step's own
    auto span = [](int in, int out, int pad) {
      int last = (in - 1 + pad - 1) / 2;
      if (last < out - 1) last = out - 1;
      return last - dw3_first(pad) + 1;
    };
    return dw3_plan(g, span(g.Hin, g.Hout, g.ph), span(g.Win, g.Wout, g.pw), 2, 2);
  });
}
// One launch of a plan's: its images and strips.  a_lo .. a_hi, o_lo .. o_hi: the rows of the two planes that strips s0 .. s1 - 1
// touch, in terms of the domain's rows d0 = v0 + s0 R .. d1 = v0 + s1 R - 1 (clipped to the planes here).
struct Dw3Launch { int img0, N, strip0, nstrip, index; };
template <typename F>
hipError_t dw3_each_launch(const Dw3Plan& pl, const Geom& g, F&& launch) {
  int index = 0;
  for (int n = 0; n < g.N; n += pl.imgs)
    for (int s = 0; s < pl.nstrip; s += pl.band, ++index) {
      const hipError_t e = launch(Dw3Launch{n, g.N - n < pl.imgs ? g.N - n : pl.imgs, s,
                                            pl.nstrip - s < pl.band ? pl.nstrip - s : pl.band, index});
      if (e != hipSuccess) return e;
    }
  return hipSuccess;
}
Dw3Params dw3_params(const Dw3Plan& pl, const Geom& g, const Dw3Launch& l) {
  Dw3Params p{};
  p.eps = g.eps;
  p.N = l.N;
  p.C = g.Cin;
  p.R = pl.R; p.nstrip = l.nstrip; p.npair = pl.npair; p.cq = pl.cq;
  p.strip0 = l.strip0;
  p.items = l.N * l.nstrip * pl.npair;
  p.per_slice = pl.per_slice;
  p.slice0 = l.index * pl.slices;
  p.slices_all = pl.launches * pl.slices;
  return p;
}
// The planes' sizes are set: which rows the launch touches -- a: as x d + a_lo for the domain's first row d to as x d + a_hi for its
// last, out and y likewise with os, o_lo, o_hi -- and the tensors from there on.
void dw3_place(Dw3Params& p, const Dw3Plan& pl, const Dw3Launch& l, const void* a, const void* y, void* out, int as, int a_lo,
               int a_hi, int os, int o_lo, int o_hi) {
  const int d0 = p.v0 + l.strip0 * pl.R, d1 = p.v0 + (l.strip0 + l.nstrip) * pl.R - 1;
  auto clip = [](int v, int hi) { return v < 0 ? 0 : v > hi ? hi : v; };
  const bool whole = l.nstrip == pl.nstrip;
  p.a_row0 = whole ? 0 : clip(as * d0 + a_lo, p.Ha);
  p.o_row0 = whole ? 0 : clip(os * d0 + o_lo, p.Ho);
  const int a_end = whole ? p.Ha : clip(as * d1 + a_hi + 1, p.Ha), o_end = whole ? p.Ho : clip(os * d1 + o_hi + 1, p.Ho);
  const size_t arow = (size_t)p.Wa * p.C, orow = (size_t)p.Wo * p.C;   // elements
  p.a_bytes = (unsigned)(((size_t)(l.N - 1) * p.Ha + a_end - p.a_row0) * arow * 2);
  p.o_bytes = (unsigned)(((size_t)(l.N - 1) * p.Ho + o_end - p.o_row0) * orow * 2);
  p.a = static_cast<const bf16_t*>(a) + ((size_t)l.img0 * p.Ha + p.a_row0) * arow;
  const size_t o = ((size_t)l.img0 * p.Ho + p.o_row0) * orow;
  p.y = y ? static_cast<const bf16_t*>(y) + o : nullptr;
  p.out = out ? static_cast<bf16_t*>(out) + o : nullptr;
}

constexpr int WG_TAPS = 9;     // window positions a weight-gradient workgroup accumulates at once
constexpr int WG_CG = 32;      // channel groups per workgroup (x 8 pixel lanes = 256 threads)

// Partial sums over one slice of the output pixels (blockIdx.y) for WG_TAPS window positions starting at
// tap0 = WG_TAPS blockIdx.z:  part[slice][tap][c] = sum_m dZ[m][c] X[window position of m][c], and (first tap
// chunk only) r_part[slice][c] = sum_m dZ[m][c].  Thread -> channel group tid % 32, pixel lane tid / 32.
template <typename T, int VEC>
__global__ __launch_bounds__(256) void dw_wgrad_kernel(const T* __restrict__ x, const T* __restrict__ dz,
                                                       float* __restrict__ part, float* __restrict__ r_part, Geom g,
                                                       int px_per_slice) {
  __shared__ float red[8][WG_CG * VEC];
  const int cgs = g.Cin / VEC;
  const int tx = threadIdx.x % WG_CG, ty = threadIdx.x / WG_CG;
  const int cg = blockIdx.x * WG_CG + tx;
  const bool live = cg < cgs;
  const int c = cg * VEC;
  const int taps = g.kH * g.kW, tap0 = blockIdx.z * WG_TAPS;
  const int m0 = blockIdx.y * px_per_slice, m1 = min(g.M, m0 + px_per_slice);
  float acc[WG_TAPS][VEC], racc[VEC];
#pragma unroll
  for (int t = 0; t < WG_TAPS; ++t)
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[t][e] = 0.f;
#pragma unroll
  for (int e = 0; e < VEC; ++e) racc[e] = 0.f;
  if (live)
    for (int m = m0 + ty; m < m1; m += 8) {
      const int wo = m % g.Wout;
      const int q = m / g.Wout;
      const int ho = q % g.Hout, n = q / g.Hout;
      float gv[VEC];
      Vec<T, VEC>::load(dz + (size_t)m * g.Cin + c, gv);
#pragma unroll
      for (int e = 0; e < VEC; ++e) racc[e] += gv[e];
#pragma unroll
      for (int t = 0; t < WG_TAPS; ++t) {
        const int tap = tap0 + t;
        if (tap >= taps) break;
        const int i = tap / g.kW, j = tap - i * g.kW;
        const int h = ho * g.sh + i - g.ph, w = wo * g.sw + j - g.pw;
        if ((unsigned)h >= (unsigned)g.Hin || (unsigned)w >= (unsigned)g.Win) continue;
        float xv[VEC];
        Vec<T, VEC>::load(x + (((size_t)n * g.Hin + h) * g.Win + w) * g.Cin + c, xv);
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[t][e] += gv[e] * xv[e];
      }
    }
  // reduce the eight pixel lanes, one window position at a time (t == WG_TAPS: the channel sums)
  const int ncol = WG_CG * VEC;
#pragma unroll
  for (int t = 0; t <= WG_TAPS; ++t) {
    const int tap = tap0 + t;
    if (t < WG_TAPS && tap >= taps) continue;
    if (t == WG_TAPS && (blockIdx.z != 0 || !r_part)) continue;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < VEC; ++e) red[ty][tx * VEC + e] = t < WG_TAPS ? acc[t < WG_TAPS ? t : 0][e] : racc[e];
    __syncthreads();
    for (int col = threadIdx.x; col < ncol; col += 256) {
      const int cc = blockIdx.x * ncol + col;
      if (cc >= g.Cin) continue;
      float v = 0.f;
#pragma unroll
      for (int l = 0; l < 8; ++l) v += red[l][col];
      if (t < WG_TAPS) part[((size_t)blockIdx.y * taps + tap) * g.Cin + cc] = v;
      else r_part[(size_t)blockIdx.y * g.Cin + cc] = v;
    }
  }
}

// sums[row][c] = sum over slices of part[slice][row][c] (rows 0..taps-1) and of r_part[slice][c] (row taps).
// grid (ceil(C/16), taps + 1), thread -> channel tid % 16, slice lane tid / 16
__global__ __launch_bounds__(256) void dw_reduce_kernel(const float* __restrict__ part, const float* __restrict__ r_part,
                                                        int slices, int taps, int C, float* __restrict__ sums) {
  __shared__ float red[16][17];
  const int cl = threadIdx.x & 15, l = threadIdx.x >> 4;
  const int c = blockIdx.x * 16 + cl, row = blockIdx.y;
  float v = 0.f;
  if (c < C && (row < taps || r_part))
    for (int s = l; s < slices; s += 16)
      v += row < taps ? part[((size_t)s * taps + row) * C + c] : r_part[(size_t)s * C + c];
  red[l][cl] = v;
  __syncthreads();
  if (l != 0 || c >= C) return;
  v = 0.f;
#pragma unroll
  for (int k = 0; k < 16; ++k) v += red[k][cl];
  sums[(size_t)row * C + c] = v;
}

// dW[c][tap] = s dw', dgamma = (sum_tap dw' w + r (b - mu)) / sqrt(var + eps), dbeta = r, db = s r.
// gamma == nullptr (Eval path): dW = dw' only.
template <typename T>
__global__ __launch_bounds__(256) void dw_fold_back_kernel(const float* __restrict__ sums, const T* __restrict__ W,
                                                           const float* __restrict__ b, const float* __restrict__ gamma,
                                                           const float* __restrict__ mean, const float* __restrict__ var,
                                                           float eps, int C, int taps, T* __restrict__ dW,
                                                           float* __restrict__ db, float* __restrict__ dgamma,
                                                           float* __restrict__ dbeta) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= C) return;
  const float sd = gamma ? sqrtf(var[c] + eps) : 1.f;
  const float s = gamma ? gamma[c] / sd : 1.f;
  float dot = 0.f;
  for (int t = 0; t < taps; ++t) {
    const float dw = sums[(size_t)t * C + c];
    dW[(size_t)c * taps + t] = from_f32<T>(s * dw);
    dot += dw * to_f32(W[(size_t)c * taps + t]);
  }
  if (!gamma) return;
  const float r = sums[(size_t)taps * C + c];
  dgamma[c] = (dot + r * ((b ? b[c] : 0.f) - mean[c])) / sd;
  dbeta[c] = r;
  if (db) db[c] = s * r;
}

bool vec8(const Geom& g, int dtype) { return dtype == CONVBN_BF16 && g.Cin % 8 == 0; }

}  // namespace

hipError_t launch_dw_fold(const Geom& g, int dtype, const void* W, const float* b, const float* gamma,
                          const float* beta, const float* mean, const float* var, void* wf, float* bfold,
                          hipStream_t st) {
  const int C = g.Cin, taps = g.kH * g.kW;
  if (dtype == CONVBN_BF16)
    hipLaunchKernelGGL(dw_fold_kernel<bf16_t>, dim3(ceil_div(C, 256)), dim3(256), 0, st, (const bf16_t*)W, b, gamma,
                       beta, mean, var, g.eps, C, taps, (bf16_t*)wf, bfold);
  else
    hipLaunchKernelGGL(dw_fold_kernel<float>, dim3(ceil_div(C, 256)), dim3(256), 0, st, (const float*)W, b, gamma, beta,
                       mean, var, g.eps, C, taps, (float*)wf, bfold);
  return hipGetLastError();
}

hipError_t launch_dw_fprop(const Geom& g, int dtype, const void* x, const void* wf, const float* bias, void* z,
                           hipStream_t st) {
  const int vec = vec8(g, dtype) ? 8 : 1;
  const size_t total = (size_t)g.M * (g.Cin / vec);
  const dim3 grid((unsigned)((total + 255) / 256));
  if (vec == 8)
    hipLaunchKernelGGL((dw_fprop_kernel<bf16_t, 8>), grid, dim3(256), 0, st, (const bf16_t*)x, (const bf16_t*)wf, bias,
                       (bf16_t*)z, g);
  else if (dtype == CONVBN_BF16)
    hipLaunchKernelGGL((dw_fprop_kernel<bf16_t, 1>), grid, dim3(256), 0, st, (const bf16_t*)x, (const bf16_t*)wf, bias,
                       (bf16_t*)z, g);
  else
    hipLaunchKernelGGL((dw_fprop_kernel<float, 1>), grid, dim3(256), 0, st, (const float*)x, (const float*)wf, bias,
                       (float*)z, g);
  return hipGetLastError();
}

hipError_t launch_dw_dgrad(const Geom& g, int dtype, const void* dz, const void* wf, void* dx, hipStream_t st) {
  const int vec = vec8(g, dtype) ? 8 : 1;
  const size_t total = (size_t)g.Min * (g.Cin / vec);
  const dim3 grid((unsigned)((total + 255) / 256));
  if (vec == 8)
    hipLaunchKernelGGL((dw_dgrad_kernel<bf16_t, 8>), grid, dim3(256), 0, st, (const bf16_t*)dz, (const bf16_t*)wf,
                       (bf16_t*)dx, g);
  else if (dtype == CONVBN_BF16)
    hipLaunchKernelGGL((dw_dgrad_kernel<bf16_t, 1>), grid, dim3(256), 0, st, (const bf16_t*)dz, (const bf16_t*)wf,
                       (bf16_t*)dx, g);
  else
    hipLaunchKernelGGL((dw_dgrad_kernel<float, 1>), grid, dim3(256), 0, st, (const float*)dz, (const float*)wf,
                       (float*)dx, g);
  return hipGetLastError();
}

// pixel slices of the weight-gradient reduction: enough workgroups to fill the chip a few times over
int dw_wgrad_slices(const Geom& g, int dtype) {
  const int vec = vec8(g, dtype) ? 8 : 1;
  const int cblocks = ceil_div(g.Cin / vec, WG_CG) * ceil_div(g.kH * g.kW, WG_TAPS);
  int want = ceil_div(1024, cblocks);
  const int maxs = ceil_div(g.M, 64);
  if (want > maxs) want = maxs;
  if (want > 512) want = 512;
  if (want < 1) want = 1;
  return ceil_div(g.M, ceil_div(g.M, want));
}

hipError_t launch_dw_wgrad(const Geom& g, int dtype, const void* x, const void* dz, float* part, float* r_part,
                           hipStream_t st) {
  const int vec = vec8(g, dtype) ? 8 : 1;
  const int slices = dw_wgrad_slices(g, dtype);
  const int pps = ceil_div(g.M, slices);
  const dim3 grid(ceil_div(g.Cin / vec, WG_CG), slices, ceil_div(g.kH * g.kW, WG_TAPS));
  if (vec == 8)
    hipLaunchKernelGGL((dw_wgrad_kernel<bf16_t, 8>), grid, dim3(256), 0, st, (const bf16_t*)x, (const bf16_t*)dz, part,
                       r_part, g, pps);
  else if (dtype == CONVBN_BF16)
    hipLaunchKernelGGL((dw_wgrad_kernel<bf16_t, 1>), grid, dim3(256), 0, st, (const bf16_t*)x, (const bf16_t*)dz, part,
                       r_part, g, pps);
  else
    hipLaunchKernelGGL((dw_wgrad_kernel<float, 1>), grid, dim3(256), 0, st, (const float*)x, (const float*)dz, part,
                       r_part, g, pps);
  return hipGetLastError();
}

hipError_t launch_dw_fold_back(const Geom& g, int dtype, const float* part, const float* r_part, int slices,
                               float* sums, const void* W, const float* b, const float* gamma, const float* mean,
                               const float* var, void* dW, float* db, float* dgamma, float* dbeta, hipStream_t st) {
  const int C = g.Cin, taps = g.kH * g.kW;
  hipLaunchKernelGGL(dw_reduce_kernel, dim3(ceil_div(C, 16), taps + 1), dim3(256), 0, st, part, r_part, slices, taps, C,
                     sums);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (dtype == CONVBN_BF16)
    hipLaunchKernelGGL(dw_fold_back_kernel<bf16_t>, dim3(ceil_div(C, 256)), dim3(256), 0, st, sums, (const bf16_t*)W, b,
                       gamma, mean, var, g.eps, C, taps, (bf16_t*)dW, db, dgamma, dbeta);
  else
    hipLaunchKernelGGL(dw_fold_back_kernel<float>, dim3(ceil_div(C, 256)), dim3(256), 0, st, sums, (const float*)W, b,
                       gamma, mean, var, g.eps, C, taps, (float*)dW, db, dgamma, dbeta);
  return hipGetLastError();
}

// ---- the 3x3 kernels
bool dw3_supported(const Geom& g, int dtype) { return dw3_shape(g, dtype); }

size_t dw3_part_bytes(const Geom& g) {
  const Dw3Plan pl = dw3_bwd_plan(g);
  return (size_t)g.Cin * 10 * pl.slices * pl.launches * 4;
}

hipError_t launch_dw3_fprop(const Geom& g, const void* x, const void* W, const float* b, const float* gamma,
                            const float* beta, const float* mean, const float* var, void* z, void* w_folded,
                            hipStream_t st) {
  const Dw3Plan pl = dw3_fprop_plan(g);
  const bool stream = gamma && streams_output((size_t)g.M * g.Cout * 2);   // (Eval's Y is read in the same call)
  return dw3_each_launch(pl, g, [&](const Dw3Launch& l) {
    Dw3Params p = dw3_params(pl, g, l);
    p.W = (const bf16_t*)W; p.b = b; p.gamma = gamma; p.beta = beta; p.mean = mean; p.var = var;
    p.wf_out = l.index == 0 ? (bf16_t*)w_folded : nullptr;
    p.Ha = g.Hin; p.Wa = g.Win; p.Ho = g.Hout; p.Wo = g.Wout; p.pa = g.ph; p.pb = g.pw;
    // (stride 2 asks for a row more in front, which belongs to no output of the strip)
    dw3_place(p, pl, l, x, nullptr, z, g.sh, -p.pa - (g.sh - 1), 2 - p.pa, 1, 0, 0);
    const dim3 grid(pl.nxb, pl.slices);
    if (g.sh == 1 && stream) hipLaunchKernelGGL((dw3_s1_kernel<true, true, false, false, true>), grid, dim3(DW_BLK), 0, st, p);
    else if (g.sh == 1) hipLaunchKernelGGL((dw3_s1_kernel<true, true, false, false, false>), grid, dim3(DW_BLK), 0, st, p);
    else if (stream) hipLaunchKernelGGL(dw3_s2_fprop_kernel<true>, grid, dim3(DW_BLK), 0, st, p);
    else hipLaunchKernelGGL(dw3_s2_fprop_kernel<false>, grid, dim3(DW_BLK), 0, st, p);
    return hipGetLastError();
  });
}

hipError_t launch_dw3_bwd(const Geom& g, const void* x, const void* dz, const void* W, const void* w_folded,
                          const float* gamma, const float* var, void* dx, float* part, hipStream_t st) {
  const Dw3Plan pl = dw3_bwd_plan(g);
  return dw3_each_launch(pl, g, [&](const Dw3Launch& l) {
    Dw3Params p = dw3_params(pl, g, l);
    p.part = part;
    p.W = (const bf16_t*)(w_folded ? w_folded : W);
    p.tap_major = w_folded != nullptr;
    p.gamma = w_folded ? nullptr : gamma; p.var = var;
    p.Ha = g.Hout; p.Wa = g.Wout; p.Ho = g.Hin; p.Wo = g.Win;
    const dim3 grid(pl.nxb, pl.slices);
    if (g.sh == 1) {
      p.pa = 2 - g.ph; p.pb = 2 - g.pw;
      p.v0 = p.pa < 0 ? p.pa : 0; p.u0 = p.pb < 0 ? p.pb : 0;
      dw3_place(p, pl, l, dz, x, dx, 1, -p.pa, 2 - p.pa, 1, 0, 0);
      const bool pad1 = g.ph == 1 && g.pw == 1;
      if (dx && !part) hipLaunchKernelGGL((dw3_s1_kernel<false, true, false, false, STREAM_GRAD>), grid, dim3(DW_BLK), 0, st, p);
      else if (dx && pad1) hipLaunchKernelGGL((dw3_s1_kernel<false, true, true, true, STREAM_GRAD>), grid, dim3(DW_BLK), 0, st, p);
      else if (dx) hipLaunchKernelGGL((dw3_s1_kernel<false, true, true, false, STREAM_GRAD>), grid, dim3(DW_BLK), 0, st, p);
      else if (pad1) hipLaunchKernelGGL((dw3_s1_kernel<false, false, true, true, false>), grid, dim3(DW_BLK), 0, st, p);
      else hipLaunchKernelGGL((dw3_s1_kernel<false, false, true, false, false>), grid, dim3(DW_BLK), 0, st, p);
    } else {
      p.pa = g.ph; p.pb = g.pw; p.v0 = dw3_first(g.ph); p.u0 = dw3_first(g.pw);
      dw3_place(p, pl, l, dz, x, dx, 1, 0, 1, 2, 1 - p.pa, 2 - p.pa);
      if (dx && part) hipLaunchKernelGGL((dw3_s2_bwd_kernel<true, true>), grid, dim3(DW_BLK), 0, st, p);
      else if (dx) hipLaunchKernelGGL((dw3_s2_bwd_kernel<true, false>), grid, dim3(DW_BLK), 0, st, p);
      else hipLaunchKernelGGL((dw3_s2_bwd_kernel<false, true>), grid, dim3(DW_BLK), 0, st, p);
    }
    return hipGetLastError();
  });
}

hipError_t launch_dw3_fold_back(const Geom& g, const float* part, const void* W, const float* b, const float* gamma,
                                const float* mean, const float* var, void* dW, float* db, float* dgamma, float* dbeta,
                                hipStream_t st) {
  const Dw3Plan pl = dw3_bwd_plan(g);
  hipLaunchKernelGGL(dw3_fold_back_kernel, dim3(g.Cin / 8), dim3(1024), 0, st, part, pl.slices * pl.launches,
                     (const bf16_t*)W, b, gamma, mean, var, g.eps, (bf16_t*)dW, db, dgamma, dbeta);
  return hipGetLastError();
}

}  // namespace convbn
