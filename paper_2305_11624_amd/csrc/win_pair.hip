// Both gradient passes of a small bf16 block in one launch: the window product's input gradient (conv_win_impl.h) and the
// window weight gradient (wgrad_win_impl.h).  They are independent, and alone each leaves most compute units idle and lasts
// as long as one workgroup's chain of copies (about 7 and 10 us for 256 -> 512 channels, 30 x 30 / 2, 6 images): together
// they take as long as the longer one.  A workgroup of either has a compute unit to itself (its ring fills the LDS), so
// this is for problems whose workgroups fit the chip together; the weight gradient's pixel slices are cut to that.
#include "conv_win_impl.h"
#include "wgrad_win_impl.h"

namespace convbn {

namespace {

constexpr int CUS = 256;

template <bool FLAT, int TA, int TB>
__global__ __launch_bounds__(512) void win_pair_kernel(wgw::WwParams w, win::WnParams d, int nw) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  if ((int)blockIdx.x < nw) wgw::body<TA, TB>(w, blockIdx.x, smem);
  else win::body<128, 64, 6, FLAT>(d, FoldSide{}, (int)blockIdx.x - nw, smem);
}

struct PairPlan { bool ok, flat; int ta, tb, nw; wgw::WwParams w; win::WnParams d; };
PairPlan work_out_plan(const Geom& g) {
  PairPlan pl{};
  const wgw::WwPlan& w = wgw::plan(g);
  if (!w.ok || !win::dgrad_params(g, &pl.d)) return pl;
  pl.flat = pl.d.C % win::CB != 0;
  if (pl.flat) win::lay_out<128, 64, true>(pl.d); else win::lay_out<128, 64, false>(pl.d);
  if (pl.d.nconv > CUS / 2) return pl;
  pl.ta = w.ta; pl.tb = w.tb;
  pl.w = wgw::limited(g, CUS - pl.d.nconv);
  const int total = pl.w.nta * pl.w.ntb * pl.w.slices;
  if (total + pl.d.nconv > CUS) return pl;
  pl.nw = ceil_div(total, 8) * 8;
  pl.ok = true;
  return pl;
}
const PairPlan& plan(const Geom& g) {
  return planned<PairPlan>(g, CONVBN_BF16, [&] { return work_out_plan(g); });
}

template <bool FLAT, int TA, int TB>
hipError_t launch_inst(const wgw::WwParams& w, const win::WnParams& d, int nw, hipStream_t st) {
  static LdsLimitOnce lds_once;
  constexpr int a = wgw::WwCfg<TA, TB>::LDS_BYTES, b = win::WnCfg<128, 64, 6>::LDS_BYTES, lds = a > b ? a : b;
  if (hipError_t e = set_lds_limit_once(lds_once, reinterpret_cast<const void*>(&win_pair_kernel<FLAT, TA, TB>), lds);
      e != hipSuccess) return e;
  hipLaunchKernelGGL((win_pair_kernel<FLAT, TA, TB>), dim3(nw + d.nconv), dim3(512), lds, st, w, d, nw);
  return hipGetLastError();
}

}  // namespace

bool win_pair_supported(const Geom& g, int dtype) { return dtype == CONVBN_BF16 && plan(g).ok; }
int win_pair_splits(const Geom& g) { return plan(g).w.slices; }
hipError_t launch_win_pair(const Geom& g, const void* x, const void* dz, const void* w_crsk, void* dx, float* part,
                           float* r_part, hipStream_t st) {
  const PairPlan& pl = plan(g);
  if (!pl.ok) return hipErrorInvalidValue;
  wgw::WwParams w = pl.w;
  win::WnParams d = pl.d;
  w.x = (const bf16_t*)x; w.dz = (const bf16_t*)dz; w.part = part; w.r_part = r_part;
  d.act = (const bf16_t*)dz; d.wgt = (const bf16_t*)w_crsk; d.out = (bf16_t*)dx;
  d.relu = g.post_relu; d.mask = (const bf16_t*)g.post_mask; d.add = (const bf16_t*)g.post_add;
#define PAIR_CASE(F_, TA_, TB_) if (pl.flat == F_ && pl.ta == TA_ && pl.tb == TB_) return launch_inst<F_, TA_, TB_>(w, d, pl.nw, st);
  PAIR_CASE(false, 128, 128) PAIR_CASE(false, 128, 64) PAIR_CASE(false, 64, 128) PAIR_CASE(false, 64, 64)
  PAIR_CASE(true, 128, 128) PAIR_CASE(true, 128, 64) PAIR_CASE(true, 64, 128) PAIR_CASE(true, 64, 64)
#undef PAIR_CASE
  return hipErrorInvalidValue;
}

}  // namespace convbn
