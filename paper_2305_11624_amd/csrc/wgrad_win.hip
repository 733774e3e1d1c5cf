// The window weight gradient as a launch of its own; its device code is in wgrad_win_impl.h.
#include "wgrad_win_impl.h"

namespace convbn {

using namespace wgw;

namespace {

constexpr int CUS = 256;   // a workgroup each (the ring fills the LDS)

// Slices of the pixels, about `workgroups` in all.  Every slice is an fp32 copy of dw': written here, read by the fold-back, and
// workspace that the caller holds.  So a slice has at least 128 pixels (two chunks) while the copies stay within 4 MB, else at
// least 256 (weight gradient and fold-back with slices of 128 and of 256 pixels: 256 -> 128 channels at 56 x 56, 4 images, 98 or 49
// copies of 0.13 MB 17.9 / 15.2 us; 512 -> 256 at 28 x 28, 4 images, 25 or 13 of 0.5 MB 16.9 / 14.9; 128 -> 512 at 28 x 28,
// 1 image, 7 or 4 of 0.26 MB 11.1 / 12.1), and the copies weigh no more than the inputs and 8 MB (3x3, 256 channels at 14 x 14,
// 8 images, 2.4 MB a copy: 4 copies 16.9 us, 1 copy 25.0).
constexpr size_t SHORT_SLICE_BYTES = (size_t)4 << 20;
void slice_up(WwParams& p, int workgroups) {
  int want = workgroups / (p.nta * p.ntb);
  const size_t copy = (size_t)p.Co * p.K * 4;
  const int few = (int)(SHORT_SLICE_BYTES / copy);
  int most = ceil_div(p.M, 128);
  if (most > few) most = ceil_div(p.M, 256) > few ? ceil_div(p.M, 256) : few;
  if (want > most) want = most;
  const int cap = (int)(((size_t)p.x_bytes + p.dz_bytes + ((size_t)8 << 20)) / copy);
  if (want > cap) want = cap;
  if (want < 1) want = 1;
  p.per = ceil_div(ceil_div(p.M, want), 128) * 128;
  p.slices = ceil_div(p.M, p.per);
}

// The tile: small ones have longer slices, hence fewer copies of dw' to write and to sum; large ones read less per multiply.
// The estimate: chunks of a workgroup's pixels, copies written at 4 TB/s (read, by the fold-back: 5 TB/s).  Weight gradient and
// fold-back, us, 128 x 128 and 64 x 64 tiles: 1024 -> 256 at 15 x 15, 11 images 16.1, 12.1; 3 x 3, 128 -> 128 at 28 x 28, 8 images
// 19.3, 15.5; 256 -> 1024 at 14 x 14, 32 images 21.0, 16.7; 3 x 3, 72 -> 136 at 27 x 33, 5 images 14.8, 12.0; a long range, transposed
// 4 x 4 / 2, 256 -> 128 at 28 x 28, 20 images, the pass: 84.7, 92.1.
WwPlan work_out_plan(const Geom& g, int workgroups) {
  WwPlan best{};
  WwParams q{};
  const size_t xb = (size_t)g.Min * g.Cin * 2, zb = (size_t)g.M * g.Cout * 2;
  if (g.Cin % 8 || g.Cout % 8 || xb >= OOB || zb >= OOB) return best;
  q.x_bytes = (unsigned)xb; q.dz_bytes = (unsigned)zb;
  q.Cin = g.Cin; q.Co = g.Cout; q.K = g.K; q.M = g.M; q.H = g.Hin; q.W = g.Win; q.Ho = g.Hout; q.Wo = g.Wout;
  q.kH = g.kH; q.kW = g.kW; q.sh = g.sh; q.sw = g.sw; q.ph = g.ph; q.pw = g.pw;
  for (int ta = 64; ta <= (g.Cout > 64 ? 128 : 64); ta += 64)
    for (int tb = 64; tb <= (g.K > 64 ? 128 : 64); tb += 64) {
      WwPlan pl{};
      pl.p = q;
      pl.ta = ta; pl.tb = tb;
      pl.p.nta = ceil_div(g.Cout, ta);
      pl.p.ntb = ceil_div(g.K, tb);
      slice_up(pl.p, workgroups);
      const int total = pl.p.nta * pl.p.ntb * pl.p.slices;
      const float copies = (float)pl.p.slices * g.Cout * g.K * 4.f * 1e-6f;   // MB
      const float chunk = ta == tb ? (ta == 64 ? 0.65f : 0.85f) : 0.5f;
      pl.us = 4.f + ceil_div(total, CUS) * ceil_div(pl.p.per, ta + tb == 128 ? 128 : 64) * chunk + copies * 0.25f;
      pl.fold_us = 3.f + copies * 0.2f;
      pl.ok = total <= workgroups || workgroups >= CUS;
      if (pl.ok && (!best.ok || pl.us + pl.fold_us < best.us + best.fold_us)) best = pl;
    }
  return best;
}
template <int TA, int TB>
__global__ __launch_bounds__(64 * NWAVES) void wgrad_win_kernel(WwParams p) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  body<TA, TB>(p, blockIdx.x, smem);
}

template <int TA, int TB>
hipError_t launch_inst(const WwParams& p, hipStream_t st) {
  static LdsLimitOnce lds_once;
  constexpr int lds = WwCfg<TA, TB>::LDS_BYTES;
  if (hipError_t e = set_lds_limit_once(lds_once, reinterpret_cast<const void*>(&wgrad_win_kernel<TA, TB>), lds); e != hipSuccess)
    return e;
  hipLaunchKernelGGL((wgrad_win_kernel<TA, TB>), dim3(ceil_div(p.nta * p.ntb * p.slices, 8) * 8), dim3(64 * NWAVES), lds, st, p);
  return hipGetLastError();
}

}  // namespace

const WwPlan& wgw::plan(const Geom& g) {
  return planned<WwPlan>(g, CONVBN_BF16, [&] { return work_out_plan(g, CUS); });
}
bool wgw::limited(const Geom& g, int workgroups, WwPlan* pl) {
  *pl = work_out_plan(g, workgroups);
  return pl->ok;
}

bool wgrad_win_supported(const Geom& g, int dtype) { return dtype == CONVBN_BF16 && plan(g).ok; }
int wgrad_win_splits(const Geom& g) { return plan(g).p.slices; }
hipError_t launch_wgrad_win(const Geom& g, const void* x, const void* dz, float* part, float* r_part, hipStream_t st) {
  const WwPlan& pl = plan(g);
  if (!pl.ok) return hipErrorInvalidValue;
  WwParams p = pl.p;
  p.x = (const bf16_t*)x; p.dz = (const bf16_t*)dz; p.part = part; p.r_part = r_part;
  if (pl.ta == 128) return pl.tb == 128 ? launch_inst<128, 128>(p, st) : launch_inst<128, 64>(p, st);
  return pl.tb == 128 ? launch_inst<64, 128>(p, st) : launch_inst<64, 64>(p, st);
}

}  // namespace convbn
