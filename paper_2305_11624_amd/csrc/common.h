// Shared device helpers and the internal launch interface of libconvbn (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>

#include <mutex>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

#include "../../include/convbn.h"

namespace convbn {

typedef __bf16 bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16_t v) { return (float)v; }
template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float v) { return (bf16_t)v; }  // RNE

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t h) { return __uint_as_float(h << 16); }
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
// Round-to-nearest-even fp32 -> bf16 bit pattern (finite inputs; NaN stays NaN).
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
  bf16_t h = (bf16_t)f;
  return (uint32_t)__builtin_bit_cast(unsigned short, h);
}
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const f32x2 v = {lo, hi};   // one conversion for the pair (two, a shift and an or if they are rounded one by one)
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Geometry of one block, with the derived sizes the kernels index with.
struct Geom {
  int N, Cin, Hin, Win, Cout, kH, kW, sh, sw, ph, pw, Hout, Wout;
  int M;      // N*Hout*Wout   (output pixels)
  int Min;    // N*Hin*Win     (input pixels)
  int K;      // kH*kW*Cin     (reduction length of the forward conv)
  float eps;
  int act;    // the descriptor's CONVBN_ACT_* bits
  // What the convolution launched with this Geom does to its output on the way out (set per call by the host side,
  // not part of the problem): `post_add` (a tensor laid out like the output, or null) is added first, then ReLU, and /
  // or zero where `post_mask` (a tensor laid out like the output) is <= 0.
  int post_relu;
  const void* post_mask;
  const void* post_add;
  const struct FoldBackArgs* fold_back;   // an input gradient: the fold-back its launch takes along (fold_tile.h), or null
  const struct FoldBackTArgs* fold_back_t;   // ... a transposed block's (fold_back_t_tile.h; the window product)
  const void* add_out;   // the descriptor's addends (CONVBN_ACT_ADD_OUT / _IN), null where the bit is not set
  const void* add_in;
};

// What the fold-back of a block reads and writes (fold_tile.h): dW, dgamma, dbeta, db from the nsplit partial copies of dw' and
// the nrpart partial sums of dZ; identity: dW is the sum of the copies, nothing else is written.
struct FoldBackArgs {
  const float* part; const float* r_part; const void* W; const float* b; const float* gamma; const float* mean; const float* var;
  void* dW; float* db; float* dgamma; float* dbeta;
  float eps;
  int nsplit, nrpart, identity, Cout, K;
  int per;   // threads of a channel, where it rides in another launch
  static constexpr bool BACK = true;
};
struct FoldSide { static constexpr bool BACK = false; };   // (a launch that may fold on the side, from its BnEpilogue)

// The same on 8 packed bf16 values: max(., 0), and zero where the 8 packed bf16 values of m4 are <= 0.
__device__ __forceinline__ uint4 relu8(uint4 v) {
  unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const unsigned neg = ((w[i] >> 15) & 0x00010001u) * 0xffffu;   // 0xffff in every half whose sign bit is set
    w[i] &= ~neg;
  }
  return make_uint4(w[0], w[1], w[2], w[3]);
}
__device__ __forceinline__ uint4 mask8(uint4 v, uint4 m4) {
  unsigned w[4] = {v.x, v.y, v.z, v.w};
  const unsigned m[4] = {m4.x, m4.y, m4.z, m4.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const unsigned lo = __uint_as_float(m[i] << 16) > 0.f ? 0x0000ffffu : 0u;
    const unsigned hi = __uint_as_float(m[i] & 0xffff0000u) > 0.f ? 0xffff0000u : 0u;
    w[i] &= lo | hi;
  }
  return make_uint4(w[0], w[1], w[2], w[3]);
}
// v + a on 8 packed bf16 values each, added in fp32 and rounded once: what the element-wise sum of the two rounded
// tensors gives.
__device__ __forceinline__ uint4 add8(uint4 v, uint4 a4) {
  const unsigned w[4] = {v.x, v.y, v.z, v.w};
  const unsigned a[4] = {a4.x, a4.y, a4.z, a4.w};
  unsigned r[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    r[i] = pack_bf16x2(__uint_as_float(w[i] << 16) + __uint_as_float(a[i] << 16),
                       __uint_as_float(w[i] & 0xffff0000u) + __uint_as_float(a[i] & 0xffff0000u));
  return make_uint4(r[0], r[1], r[2], r[3]);
}
// ... about to be stored at element offset o of the output, the addend and the mask read on the spot.  (Requesting the mask values
// before the multiplies was measured on all four kernels that use this and changed nothing: what the mask costs them
// is its bytes, not the wait.)
__device__ __forceinline__ uint4 post_op8(uint4 v, int relu, const bf16_t* mask, const bf16_t* add, size_t o) {
  if (add) v = add8(v, *reinterpret_cast<const uint4*>(add + o));
  if (relu) v = relu8(v);
  if (mask) v = mask8(v, *reinterpret_cast<const uint4*>(mask + o));
  return v;
}

// Per-channel epilogue of a forward convolution that is given the UNFOLDED weight: Z = s (w (*) X) + b' with
// s = gamma / sqrt(var + eps) and b' = (b - mu) s + beta worked out by the kernel itself -- the same forward
// result as folding the weight first (Sec. 3.3), without materialising w'.  gamma == nullptr: not used.
struct BnEpilogue {
  const float* gamma;
  const float* beta;
  const float* mean;
  const float* var;
  const float* b;   // convolution bias or nullptr
  float eps;
  // Optional: the launch also leaves w' = s w as [Cin][taps][Cout] -- what Tune mode keeps for backward (Sec. 3.4.2)
  // -- every workgroup writing one slice of it, so that a forward pass that keeps w' is still a single launch.
  void* w_folded_out;
  int taps, Cin, Cout;
};

// s and b' of channel `ch` (no BatchNorm given: 1 and the bias), every load issued before the first use
__device__ __forceinline__ void bn_scale_bias(const BnEpilogue& bn, const float* bias, int ch, float* s, float* bb) {
  *s = 1.f;
  *bb = 0.f;
  if (bn.gamma) {
    const float ga = bn.gamma[ch], va = bn.var[ch], me = bn.mean[ch], be = bn.beta[ch], b = (bn.b ? bn.b : bn.mean)[ch];
    *s = ga / sqrtf(va + bn.eps);
    *bb = ((bn.b ? b : 0.f) - me) * *s + be;
  } else if (bias) {
    *bb = bias[ch];
  }
}

// Slice `wg` of `nwg` of w' = bf16(float(w) s), written in [Cin][taps][Cout] order (w is [Cout][taps][Cin]); the same
// values, bit for bit, as the fold kernel's.  Called by all threads of a workgroup.
__device__ __forceinline__ void emit_folded_slice(const BnEpilogue& bn, const bf16_t* __restrict__ w, int wg, int nwg) {
  bf16_t* out = static_cast<bf16_t*>(bn.w_folded_out);
  const int P = bn.Cout * bn.taps * bn.Cin;
  const int per = (P + nwg - 1) / nwg;
  const int end = min(P, (wg + 1) * per);
  for (int j = wg * per + (int)threadIdx.x; j < end; j += (int)blockDim.x) {
    const int co = j % bn.Cout;
    const int rest = j / bn.Cout;
    const int tap = rest % bn.taps, ci = rest / bn.taps;
    const float s = bn.gamma[co] / sqrtf(bn.var[co] + bn.eps);
    out[j] = (bf16_t)((float)w[((size_t)co * bn.taps + tap) * bn.Cin + ci] * s);
  }
}

// 16 bytes of a result past the caches (whole lines: 16-byte pieces of lines written at different times cost more)
__device__ __forceinline__ void store_result(void* p, uint4 v) {
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 t = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(t, static_cast<u32x4*>(p));
}

// Whether a depthwise or grouped block's forward output of that many bytes is stored past the caches.  The next block reads it
// at once, so what the line depends on is chains of blocks (pointwise, 3x3, pointwise; three or four in a row, forward):
//   MB   the 3x3 layers                          stored in the caches   past them
//   0.4  960 channels at 7 x 7, 4 images                         85.2        91.1 us
//   12.8 512 channels at 14 x 14, 64 images                     169.5       183.1
//   12.8 256 channels at 28 x 28, 32 images                     137.0       139.7
//   14.4 144 channels at 56 x 56, 16 images                    134.0       135.4
//   25.7 256 channels at 28 x 28, 64 images                     239.2       237.2
//   28.9 144 channels at 56 x 56, 32 images                     211.7       211.2
//   57.8 144 channels at 56 x 56, 64 images                     362.6       347.9
// 19.3 MB (96 channels at 112 x 112 / 2, 32 images): a chain of three takes 94 us either way, the block alone 21.6 and 18.4.
inline bool streams_output(size_t bytes) { return bytes >= ((size_t)16 << 20); }
// Their input gradients leave past the caches at every size.  A single block gains (inputs from memory: 144 channels at 56 x 56,
// 32 images, 52.8 -> 52.2 us a pass, 256 channels at 28 x 28 45.8 -> 44.5; inputs still in the last-level cache from the last
// time: 50.2 -> 42.4, 41.7 -> 41.0).  A step over the chains above takes within 1 % of the same up to 13 MB (64 images of 384
// channels at 14 x 14 311 -> 306, 32 of 1024 at 7 x 7 451.5 -> 455.3) and 0.5 - 2 % more above (57.8 MB: 931 -> 949).
constexpr bool STREAM_GRAD = true;

inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Raises a kernel's dynamic-LDS limit once per process -- also when several host threads launch it for the first
// time together -- and remembers the outcome.
struct LdsLimitOnce {
  std::once_flag once;
  hipError_t err = hipSuccess;
};
inline hipError_t set_lds_limit_once(LdsLimitOnce& s, const void* kernel, int bytes) {
  std::call_once(s.once, [&] { s.err = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes); });
  return s.err;
}
// The launch plan of a problem depends on its sizes alone, and a block call asks for it several times (is the shape
// taken, how much scratch, the launch itself): plans are worked out once per thread and problem and kept in a small
// direct-mapped table, compared by the whole key.  A step of the transposed block spent about 20 us of host time on
// planning, one of a deep 3x3 block about 15 us; a hit costs about 30 ns.
template <class Key, class Val>
class PlanTable {
 public:
  template <class F>
  const Val& get(const Key& k, F&& compute) {
    uint32_t h = 2166136261u;
    uint32_t w[(sizeof(Key) + 3) / 4] = {};
    memcpy(w, &k, sizeof(Key));
    for (uint32_t v : w) h = (h ^ v) * 16777619u;
    Slot& s = slots_[(h ^ (h >> 15)) % kSlots];
    if (!s.used || memcmp(&s.key, &k, sizeof(Key)) != 0) {
      s.val = compute();   // (first: a plan may look up plans of its own)
      memcpy(&s.key, &k, sizeof(Key));
      s.used = true;
    }
    return s.val;
  }

 private:
  static constexpr int kSlots = 64;
  struct Slot { bool used; Key key; Val val; };
  Slot slots_[kSlots] = {};
};
// ... of a block's problem: everything up to K in Geom, and the element type
struct GeomKey { int v[16]; int dtype; };
inline GeomKey geom_key(const Geom& g, int dtype) {
  static_assert(offsetof(Geom, K) == 15 * sizeof(int), "the sizes come first in Geom");
  GeomKey k;
  memcpy(k.v, &g, sizeof(k.v));
  k.dtype = dtype;
  return k;
}
template <class Val, class F>
const Val& planned(const Geom& g, int dtype, F&& compute) {   // one table per place of use (F is its own type there)
  static thread_local PlanTable<GeomKey, Val> table;
  return table.get(geom_key(g, dtype), compute);
}

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// ---- launchers (each enqueues on `st`, returns the hipError of the launch) ----

// fold.hip
// w_krsc / w_crsk / bfold may each be NULL (skipped).  identity != 0: s = 1, b' = b.
hipError_t launch_fold(const Geom& g, int dtype, const void* W, const float* b, const float* gamma,
                       const float* beta, const float* mean, const float* var, int identity,
                       void* w_krsc, void* w_crsk, float* bfold, hipStream_t st);
// Grouped fold: fold_group_item() writes one table entry (fold_group_item_bytes() bytes, host memory) for a
// bf16 block with K and Cout multiples of 8 (false otherwise) and returns its number of workgroups;
// launch_fold_group() runs a table that has been copied to device memory.
size_t fold_group_item_bytes();
bool fold_group_item(const Geom& g, int dtype, const void* W, const float* b, const float* gamma, const float* beta,
                     const float* mean, const float* var, int identity, void* w_krsc, void* w_crsk, float* bfold,
                     int first_block, void* item_out, int* blocks);
hipError_t launch_fold_group(const void* items_dev, int n, int grid_blocks, hipStream_t st);
// Sums `nsplit` fp32 partial copies of dJ/dw' ([nsplit][Cout][K]) and `nrpart` partial
// row-sum vectors ([nrpart][Cout]); writes dW, db, dgamma, dbeta (Table 2 "Tune").
// identity != 0 (Eval path): dW = sum of partials only, other outputs untouched.
hipError_t launch_fold_back(const Geom& g, int dtype, const float* dwf_part, int nsplit,
                            const float* r_part, int nrpart, const void* W, const float* b,
                            const float* gamma, const float* mean, const float* var, int identity,
                            void* dW, float* db, float* dgamma, float* dbeta, hipStream_t st);
// Grouped fold-back: fold_back_group_item() writes one table entry (host memory) for a bf16 block whose K is a
// multiple of 4 (false otherwise) and returns its number of workgroups; launch_fold_back_group() runs a table
// that has been copied to device memory.
size_t fold_back_group_item_bytes();
bool fold_back_group_item(const Geom& g, int dtype, const float* dwf_part, int nsplit, const float* r_part, int nrpart,
                          const void* W, const float* b, const float* gamma, const float* mean, const float* var,
                          void* dW, float* db, float* dgamma, float* dbeta, int first_block, void* item_out,
                          int* blocks);
hipError_t launch_fold_back_group(const void* items_dev, int n, int grid_blocks, hipStream_t st);
// fold_t.hip : fold / fold-back of the transposed block, weight [Ci][taps][Co] with the scale on co.
// w_same ([Ci][taps][Co]), w_swap ([Co][taps][Ci]) and bfold may each be NULL (skipped).  tap_major != 0:
// w_swap is [taps][Co][Ci] and bfold [taps][Co] (b' repeated for every tap) instead.  gamma == NULL: s = 1, b' = b.
hipError_t launch_fold_t(int dtype, int Ci, int Co, int taps, const void* W, const float* b, const float* gamma,
                         const float* beta, const float* mean, const float* var, float eps, int tap_major,
                         void* w_same, void* w_swap, float* bfold, hipStream_t st);
int fold_back_t_chunks(int Ci, int Co, int taps, int nsplit);   // rows of dot_part ([chunks][Co] fp32 scratch)
// dz [zrows.M][Co] gives r = sum dZ, through r_part ([colsum_parts(zrows)][Co] fp32 scratch).
// gamma == NULL (Eval path): dW = sum of the partial copies only; dz, the scratch and the other outputs are not touched.
// Its arguments where it rides in another launch (false: it cannot), and what then is left of it.
bool fold_back_t_side(int dtype, int Ci, int Co, int taps, const float* dwf_part, int nsplit, const Geom& zrows, const void* dz,
                      float* r_part, const void* W, const float* gamma, const float* var, float eps, float* dot_part, void* dW,
                      struct FoldBackTArgs* a);
hipError_t launch_fold_back_t_finish(int Ci, int Co, int taps, int nsplit, const Geom& zrows, const float* r_part, const float* b,
                                     const float* gamma, const float* mean, const float* var, float eps, const float* dot_part,
                                     float* db, float* dgamma, float* dbeta, hipStream_t st);
hipError_t launch_fold_back_t(int dtype, int Ci, int Co, int taps, const float* dwf_part, int nsplit,
                              const Geom& zrows, const void* dz, float* r_part, const void* W, const float* b,
                              const float* gamma, const float* mean, const float* var, float eps, float* dot_part, void* dW,
                              float* db, float* dgamma, float* dbeta, hipStream_t st);
int colsum_parts(const Geom& g);
hipError_t launch_colsum(const Geom& g, int dtype, const void* dz, float* r_part, hipStream_t st);
hipError_t launch_bn_affine_fwd(const Geom& g, int dtype, const void* y, const float* gamma,
                                const float* beta, const float* mean, const float* var, void* z,
                                hipStream_t st);
int bn_bwd_parts(const Geom& g);
hipError_t launch_bn_bwd(const Geom& g, int dtype, const void* dz, const void* y, const float* gamma,
                         const float* mean, const float* var, void* dy, float* part /*[parts][2][Cout]*/,
                         hipStream_t st);
hipError_t launch_bn_bwd_finalize(const Geom& g, const float* part, int parts, const float* gamma,
                                  const float* var, float* dgamma, float* dbeta, float* db,
                                  hipStream_t st);

// Copies a [rows][inner_in] matrix of `elem_bytes`-wide elements (2 or 4) into [rows][inner_out]:
// the first min(inner_in, inner_out) elements of every row, zeros behind them (fold.hip).
hipError_t launch_repitch(int elem_bytes, size_t rows, size_t inner_in, size_t inner_out, const void* src,
                          void* dst, hipStream_t st);

// aux_ops.hip : glue between blocks for the whole-backbone measurement
//   op: 0 relu (a), 1 relu backward (a = b > 0 ? a : 0), 2 a = relu(a + b), 3 a += b;  n % 8 == 0
hipError_t launch_eltwise(int op, int dtype, void* a, const void* b, const void* c, size_t n, hipStream_t st);
hipError_t launch_maxpool_fwd(int dtype, const void* x, void* y, unsigned char* idx, int N, int H, int W, int C,
                              hipStream_t st);
hipError_t launch_maxpool_bwd(int dtype, const void* dy, const unsigned char* idx, void* dx, int N, int H, int W,
                              int C, hipStream_t st);

// depthwise.hip : the depthwise block (groups = channels; g.Cin == g.Cout), plain vector kernels.
// wf is the folded filter in tap-major order [kH kW][C]; gamma == NULL means s = 1 (Eval comparison path).
hipError_t launch_dw_fold(const Geom& g, int dtype, const void* W, const float* b, const float* gamma,
                          const float* beta, const float* mean, const float* var, void* wf, float* bfold,
                          hipStream_t st);
hipError_t launch_dw_fprop(const Geom& g, int dtype, const void* x, const void* wf, const float* bias, void* z,
                           hipStream_t st);
hipError_t launch_dw_dgrad(const Geom& g, int dtype, const void* dz, const void* wf, void* dx, hipStream_t st);
int dw_wgrad_slices(const Geom& g, int dtype);
// part [slices][taps][C], r_part [slices][C] (nullable), sums [(taps + 1)][C]: fp32 scratch
hipError_t launch_dw_wgrad(const Geom& g, int dtype, const void* x, const void* dz, float* part, float* r_part,
                           hipStream_t st);
hipError_t launch_dw_fold_back(const Geom& g, int dtype, const float* part, const float* r_part, int slices,
                               float* sums, const void* W, const float* b, const float* gamma, const float* mean,
                               const float* var, void* dW, float* db, float* dgamma, float* dbeta, hipStream_t st);

// ... 3x3 windows with stride 1 or 2, bf16, channels multiples of 8: the filter is folded by the threads
// that use it (w is the unfolded [C][9] filter, gamma == null: s = 1), forward leaves w_folded [9][C] on the side (or
// null), and backward's two gradients are one launch (w_folded: what forward kept, or null; dx or part may be null; part:
// dw3_part_bytes()).
bool dw3_supported(const Geom& g, int dtype);
size_t dw3_part_bytes(const Geom& g);
hipError_t launch_dw3_fprop(const Geom& g, const void* x, const void* W, const float* b, const float* gamma,
                            const float* beta, const float* mean, const float* var, void* z, void* w_folded,
                            hipStream_t st);
hipError_t launch_dw3_bwd(const Geom& g, const void* x, const void* dz, const void* W, const void* w_folded,
                          const float* gamma, const float* var, void* dx, float* part, hipStream_t st);
hipError_t launch_dw3_fold_back(const Geom& g, const float* part, const void* W, const float* b, const float* gamma,
                                const float* mean, const float* var, void* dW, float* db, float* dgamma, float* dbeta,
                                hipStream_t st);

// conv_grouped.hip : the three contractions of a grouped block (groups divides g.Cin and g.Cout; cg = Cin / groups).
// w_krsc is [Cout][kH][kW][cg], w_crsk [cg][kH][kW][Cout]; part [slices][Cout][kH kW cg] fp32.  Where
// g_wgrad_makes_rsum() the weight-gradient launch also writes r_part [slices][Cout] (else it ignores it).
// bn != nullptr (g_fprop_scaled_supported): w_krsc is the UNFOLDED weight.
bool g_fprop_scaled_supported(const Geom& g, int groups, int dtype);
hipError_t launch_g_fprop(const Geom& g, int groups, int dtype, const void* x, const void* w_krsc, const float* bias,
                          void* z, hipStream_t st, const BnEpilogue* bn = nullptr);
hipError_t launch_g_dgrad(const Geom& g, int groups, int dtype, const void* dz, const void* w_crsk, void* dx,
                          hipStream_t st);
int g_wgrad_slices(const Geom& g, int groups, int dtype);
bool g_wgrad_makes_rsum(const Geom& g, int groups, int dtype);
hipError_t launch_g_wgrad(const Geom& g, int groups, int dtype, const void* x, const void* dz, float* part,
                          float* r_part, hipStream_t st);

// conv_grouped3.hip : the same for 3x3 windows, stride 1 or 2, groups of 4 to 32 channels (tensors under 1 GB).  W is the unfolded
// weight [Cout][kH][kW][cg] (bn: s, b' and where w' is left, or null); w_crsk as above; part [slices][Cout][kH kW cg], r_part
// [slices][Cout] or null.
bool g3_supported(const Geom& g, int groups, int dtype);
hipError_t launch_g3_fprop(const Geom& g, int groups, const void* x, const void* W, const BnEpilogue& bn, void* z, hipStream_t st);
hipError_t launch_g3_dgrad(const Geom& g, int groups, const void* dz, const void* w_crsk, void* dx, hipStream_t st);
int g3_wgrad_slices(const Geom& g);
hipError_t launch_g3_wgrad(const Geom& g, int groups, const void* x, const void* dz, float* part, float* r_part, hipStream_t st);
bool g3_pair_supported(const Geom& g, int groups, int dtype);   // both gradients as one launch
hipError_t launch_g3_pair(const Geom& g, int groups, const void* x, const void* dz, const void* w_crsk, void* dx, float* part,
                          float* r_part, hipStream_t st);

// conv_wave.hip : operands straight from memory into the matrix cores, the reduction split over a workgroup's waves.
// The fp32 path of a dense block (tensors under 2 GB): forward and input gradient (post-operation applied), weight
// gradient (fp32 copies [splits][Cout][K], r_part [splits][Cout] or null), and both gradients as one launch.
bool wave_f32_supported(const Geom& g, int dtype);
hipError_t launch_fprop_wave(const Geom& g, const void* x, const void* w_krsc, const float* bias, void* z, hipStream_t st,
                             const BnEpilogue* bn = nullptr);
hipError_t launch_dgrad_wave(const Geom& g, const void* dz, const void* w_crsk, const float* bias, void* dx,
                             hipStream_t st);
int wave_wgrad_splits(const Geom& g);
hipError_t launch_wgrad_wave(const Geom& g, const void* x, const void* dz, float* part, float* r_part, hipStream_t st);
hipError_t launch_pair_wave(const Geom& g, const void* x, const void* dz, const void* w_crsk, void* dx, float* part,
                            float* r_part, hipStream_t st);

// conv_direct.hip : one thread per output element, fp32 accumulation (any shape, both dtypes)
hipError_t launch_fprop_direct(const Geom& g, int dtype, const void* x, const void* w_krsc,
                               const float* bias, void* z, hipStream_t st);
hipError_t launch_dgrad_direct(const Geom& g, int dtype, const void* dz, const void* w_crsk,
                               const float* bias /*[Cin] or null*/, void* dx, hipStream_t st);
int wgrad_direct_splits(const Geom& g);
hipError_t launch_wgrad_direct(const Geom& g, int dtype, const void* x, const void* dz,
                               float* dwf_part /*[splits][Cout][K]*/, hipStream_t st);

// conv_stem.hip : forward convolution of a first layer (at most 4 input channels), bf16 MFMA, operands read
// straight from the raw input patch.  w is the weight as [Cout][kH][kW][Cin].
bool stem_fprop_supported(const Geom& g, int dtype);
bool stem_wgrad_supported(const Geom& g, int dtype);
int stem_wgrad_slices(const Geom& g);             // fp32 partial copies of dw' (and of r) the kernel writes
hipError_t launch_wgrad_stem(const Geom& g, const void* x, const void* dz, float* part, float* r_part, hipStream_t st);
bool stem_dgrad_supported(const Geom& g, int dtype);
bool stem_dgrad_folds_back_aside(const Geom& g);   // (where that and stem_wgrad_supported hold)
hipError_t launch_dgrad_stem(const Geom& g, const void* dz, const void* w_crsk, void* dx, hipStream_t st);
size_t stem_input_copy_bytes(const Geom& g);      // scratch for a 4-channel copy of the input (0: read as it is)
// bn != nullptr: w is the UNFOLDED weight and the epilogue applies s and b' (w' left on the side); relu: max(z, 0)
hipError_t launch_fprop_stem(const Geom& g, const void* x, const void* w, const float* bias, void* z, int relu, hipStream_t st,
                             const BnEpilogue* bn = nullptr);

// conv_igemm.hip : bf16 MFMA implicit GEMM with 64-bit addresses, for tensors of 2 GB and more (channels multiples of 8)
bool igemm_supported(const Geom& g, int dtype);
int wgrad_splits(const Geom& g);
hipError_t launch_fprop_igemm(const Geom& g, const void* x, const void* w_krsc, const float* bias,
                              void* z, hipStream_t st);
hipError_t launch_dgrad_igemm(const Geom& g, const void* dz, const void* w_crsk, const float* bias, void* dx,
                              hipStream_t st);
hipError_t launch_wgrad_igemm(const Geom& g, const void* x, const void* dz, float* dwf_part,
                              int nsplit, hipStream_t st);

// conv_tile.hip : bf16 MFMA convolution with the input window tile resident in LDS
// (every input element is fetched once per block and reused by all taps).
// conv_pw.hip: persistent weight-stationary kernel for 1x1 / stride-1 convolutions over long pixel ranges
// the tiled matrix product that takes the pointwise layers of the middle stages (conv_gm.hip); reached through the
// pw_* calls below
bool gm_supported(int M, int C, int R);
// Whether the product is one round, a workgroup per compute unit, that leaves too few of them for `aside` more.
bool gm_round_full(int M, int C, int R, int aside);
// sd != null: a strided pointwise layer -- the activation row of output pixel (n, ho, wo) is pixel (n, ho sh, wo sw) of an
// [N][Hs][Ws] tensor.
struct GmStride { int N, Ho, Wo, Hs, Ws, sh, sw; };
// conv_win.hip: the same product with any window and stride, channels multiples of 8 (tensors under 2 GB); the residue
// classes of a strided input gradient in one launch.  bn != nullptr: w_krsc is the UNFOLDED weight.
bool win_supported(const Geom& g, int dtype);
hipError_t launch_fprop_win(const Geom& g, const void* x, const void* w_krsc, const float* bias, void* z, hipStream_t st,
                            const BnEpilogue* bn = nullptr);
// Few pixels: the launches above and below on small tiles whose reduction the waves of a workgroup split (conv_ks_impl.h)
bool ks_fprop_taken(const Geom& g, int dtype);
bool ks_dgrad_taken(const Geom& g, int dtype);
hipError_t launch_dgrad_win(const Geom& g, const void* dz, const void* w_crsk, const float* bias, void* dx, hipStream_t st);
void win_describe(const Geom& g, bool fwd, char* text, size_t bytes);   // "win 128x64", "ks 32x32"
hipError_t launch_gm(int M, int C, int R, const void* act, const void* wgt, const float* bias, const BnEpilogue* bn,
                     void* out, int relu, const void* mask, const void* add, hipStream_t st, const GmStride* sd = nullptr,
                     bool grad = false,
                     const FoldBackArgs* fb = nullptr);   // grad: an input gradient
bool pw_fprop_supported(const Geom& g, int dtype);
bool pw_fprop_scaled_supported(const Geom& g, int dtype);     // ... with a BnEpilogue
bool pw_fprop_folds_aside(const Geom& g, int dtype);          // ... whose launch also leaves w_folded_out
bool pw_dgrad_supported(const Geom& g, int dtype);
hipError_t launch_fprop_pw(const Geom& g, const void* x, const void* w_krsc, const float* bias, void* z,
                           hipStream_t st, const BnEpilogue* bn = nullptr);
hipError_t launch_dgrad_pw(const Geom& g, const void* dz, const void* w_crsk, const float* bias, void* dx,
                           hipStream_t st);
// Forward of a transposed convolution whose stride equals its window (no padding), as one product with a
// depth-to-space store; g is the convolution the block is the adjoint of.  w_tap_major is [taps][g.Cin][g.Cout]
// (rows (tap, co)), bias_per_tap [taps][g.Cin] (the folded bias repeated per tap).
bool pw_tconv_supported(const Geom& g, int dtype);
hipError_t launch_tconv_pw(const Geom& g, const void* x, const void* w_tap_major, const float* bias_per_tap, void* z,
                           hipStream_t st);

// conv_st.hip : 3x3 / stride-1 convolutions of deep layers on 64-pixel x 128-channel tiles shared by eight waves
// (no split sums, no scratch).
bool st_fprop_supported(const Geom& g, int dtype);
bool st_dgrad_supported(const Geom& g, int dtype);
// bn != nullptr: w_krsc is the UNFOLDED weight and the epilogue applies the BatchNorm scale and folded bias itself
hipError_t launch_fprop_st(const Geom& g, const void* x, const void* w_krsc, const float* bias, void* z, hipStream_t st,
                           const BnEpilogue* bn = nullptr);
hipError_t launch_dgrad_st(const Geom& g, const void* dz, const void* w_crsk, const float* bias, void* dx, hipStream_t st);

// conv_rw.hip : 3x3 / stride-1 convolutions of shallow layers (64 -> 64 channels, long pixel streams): weight and
// window resident in LDS, one barrier per workgroup (no scratch).
bool rw_fprop_supported(const Geom& g, int dtype);
bool rw_dgrad_supported(const Geom& g, int dtype);
// bn != nullptr: w_krsc is the UNFOLDED weight and the epilogue applies the BatchNorm scale and folded bias itself
hipError_t launch_fprop_rw(const Geom& g, const void* x, const void* w_krsc, const float* bias, void* z, hipStream_t st,
                           const BnEpilogue* bn = nullptr);
hipError_t launch_dgrad_rw(const Geom& g, const void* dz, const void* w_crsk, const float* bias, void* dx, hipStream_t st);

bool tile_fprop_supported(const Geom& g, int dtype);
bool tile_fprop_scaled_supported(const Geom& g, int dtype);   // ... with a BnEpilogue
bool tile_dgrad_supported(const Geom& g, int dtype);
// Some problems split the reduced channels over several workgroups and need fp32 partial-output
// storage of this many bytes (0 otherwise), passed as `partials`.
size_t tile_fprop_partial_bytes(const Geom& g);
size_t tile_dgrad_partial_bytes(const Geom& g);
hipError_t launch_fprop_tile(const Geom& g, const void* x, const void* w_krsc, const float* bias,
                             void* z, float* partials, hipStream_t st, const BnEpilogue* bn = nullptr);
// The input-gradient launchers take an optional per-input-channel bias: a transposed convolution's forward
// pass is this kernel (Sec. 3.2.1), and its folded bias b' is added here.
hipError_t launch_dgrad_tile(const Geom& g, const void* dz, const void* w_crsk, const float* bias, void* dx,
                             float* partials, hipStream_t st);

// wgrad_win.hip : bf16 MFMA weight gradient of any window and stride (channels multiples of 8, tensors under 2 GB); also
// produces the per-channel sums r (one partial per split) when r_part != nullptr.
bool wgrad_win_supported(const Geom& g, int dtype);
int wgrad_win_splits(const Geom& g);
hipError_t launch_wgrad_win(const Geom& g, const void* x, const void* dz, float* dwf_part, float* r_part, hipStream_t st);

// win_pair.hip : the two above as one launch, for problems whose workgroups fit the chip together; win_pair_splits()
// (its tiles are its own: also more than wgrad_win_splits()) fp32 copies of dw' and of r.
bool win_pair_taken(const Geom& g, int dtype);
int win_pair_splits(const Geom& g);
void win_pair_describe(const Geom& g, char* text, size_t bytes);   // "ks 64x32 win 64x64": the tiles of either gradient
hipError_t launch_win_pair(const Geom& g, const void* x, const void* dz, const void* w_crsk, void* dx, float* dwf_part,
                           float* r_part, hipStream_t st);

// wgrad_sq.hip : bf16 MFMA weight gradient of 3x3 windows (any stride), one 32 x 32 channel pair x 9 taps per
// workgroup; same outputs as launch_wgrad_win (fp32 dw' copies [splits][Cout][taps][Cin], r_part [splits][Cout]).
bool wgrad_sq_supported(const Geom& g, int dtype);
int wgrad_sq_splits(const Geom& g);
hipError_t launch_wgrad_sq(const Geom& g, const void* x, const void* dz, float* dwf_part, float* r_part,
                           hipStream_t st);
// Input gradient and weight gradient (fp32 copies as launch_wgrad_sq writes them) of a block in one launch, where the
// resident-weight convolution takes the input gradient.
bool wgrad_dgrad_pair_supported(const Geom& g, int dtype);
hipError_t launch_wgrad_dgrad_pair(const Geom& g, const void* x, const void* dz, const void* w_crsk, void* dx,
                                   float* dwf_part, float* r_part, hipStream_t st);
// Weight gradient and fold-back in one launch, for problems whose pixels need no split (deep layers): writes dW,
// dgamma, dbeta and (b given) db directly; no fp32 copy of dw' is stored.  scratch: wgrad_sq_fused_scratch_bytes().
// w_folded_out (optional): the launch also leaves w' = s w there as [Cin][taps][Cout], for an input gradient that
// runs after it.
bool wgrad_sq_fused_supported(const Geom& g, int dtype);
float wgrad_sq_fused_us(const Geom& g);   // an estimate of that launch
size_t wgrad_sq_fused_scratch_bytes(const Geom& g);
hipError_t launch_wgrad_sq_fused(const Geom& g, const void* x, const void* dz, const void* W, const float* b,
                                 const float* gamma, const float* mean, const float* var, void* dW, float* db,
                                 float* dgamma, float* dbeta, void* scratch, void* w_folded_out, hipStream_t st);

}  // namespace convbn
