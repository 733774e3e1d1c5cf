// The window weight gradient as a launch of its own; its device code is in wgrad_win_impl.h.
#include "wgrad_win_impl.h"

namespace convbn {

using namespace wgw;

namespace {

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

WwPlan work_out_plan(const Geom& g) {
  WwPlan pl{};
  WwParams& p = pl.p;
  const size_t xb = (size_t)g.Min * g.Cin * 2, zb = (size_t)g.M * g.Cout * 2;
  if (g.Cin % 8 || g.Cout % 8 || xb >= OOB || zb >= OOB) return pl;
  p.x_bytes = (unsigned)xb; p.dz_bytes = (unsigned)zb;
  p.Cin = g.Cin; p.Co = g.Cout; p.K = g.K; p.M = g.M; p.H = g.Hin; p.W = g.Win; p.Ho = g.Hout; p.Wo = g.Wout;
  p.kH = g.kH; p.kW = g.kW; p.sh = g.sh; p.sw = g.sw; p.ph = g.ph; p.pw = g.pw;
  pl.ta = g.Cout > 64 ? 128 : 64;
  pl.tb = g.K > 64 ? 128 : 64;
  p.nta = ceil_div(g.Cout, pl.ta);
  p.ntb = ceil_div(g.K, pl.tb);
  slice_up(p, 256);   // one workgroup per compute unit (the ring fills its LDS), one round
  pl.ok = true;
  return pl;
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
  return planned<WwPlan>(g, CONVBN_BF16, [&] { return work_out_plan(g); });
}
WwParams wgw::limited(const Geom& g, int workgroups) {
  WwParams p = plan(g).p;
  slice_up(p, workgroups);
  return p;
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
