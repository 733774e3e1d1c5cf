// Both gradient passes of a small bf16 block in one launch: the wave-split input gradient (conv_ks_impl.h) and the
// window weight gradient (wgrad_win_impl.h).  They are independent, and alone each leaves most compute units idle and lasts
// as long as one workgroup's chain of copies: together they take as long as the longer one.  A workgroup of either has
// a compute unit to itself (the LDS), so this is for problems whose workgroups fit the chip together; the weight
// gradient's pixel slices are cut to that, and of the tiles of either those are taken whose longer chain is shortest.
#include "conv_ks_impl.h"
#include "wgrad_win_impl.h"

#include <stdio.h>

#include <algorithm>

namespace convbn {

namespace {

constexpr int CUS = 256;

// TM 128: the window product's 128 x 64 tiles (conv_win_impl.h; FLAT: as there), fewer workgroups where the wave-split ones would leave the weight
// gradient too few (256 -> 1024 at 14 x 14, 16 images, a pass: 21.6 us with them, 25.5 on two launches)
template <int TM, int TN, bool FLAT, int TA, int TB>
__global__ __launch_bounds__(512) void win_pair_kernel(wgw::WwParams w, win::WnParams d, int nw) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  if ((int)blockIdx.x < nw) wgw::body<TA, TB>(w, blockIdx.x, smem);
  else if constexpr (TM == 128) win::body<128, 64, 6, FLAT>(d, FoldSide{}, (int)blockIdx.x - nw, smem);
  else win::ks_body<TM, TN>(d, FoldSide{}, (int)blockIdx.x - nw, smem);
}

struct PairPlan { bool ok, flat; int tm, tn, ta, tb, nw, product; float us; wgw::WwParams w; win::WnParams d; };
template <int TM, int TN>
void consider(const Geom& g, PairPlan& best) {
  PairPlan pl{};
  if (!win::dgrad_params(g, &pl.d)) return;
  pl.flat = TM != 128 || pl.d.C % win::CB != 0;
  if (pl.flat) win::lay_out<TM, TN, true>(pl.d); else win::lay_out<TM, TN, false>(pl.d);
  int product = pl.d.nconv;   // (positions that no tap reaches: short workgroups, behind the others)
  for (int i = 0; i < pl.d.ncls; ++i)
    if (pl.d.c[i].nchunks == 0 && pl.d.c[i].first < product) product = pl.d.c[i].first;
  if (product >= CUS) return;
  wgw::WwPlan w{};
  if (!wgw::limited(g, CUS - (pl.d.nconv <= CUS / 2 ? pl.d.nconv : product), &w)) return;
  const int total = w.p.nta * w.p.ntb * w.p.slices;
  pl.nw = ceil_div(total, 8) * 8;
  if (pl.nw + product > CUS) return;
  float du = win::ks_us(TM, TN, pl.d);
  if (TM == 128) {   // (a chunk across tap borders takes half as long again)
    du = 0.f;
    for (int i = 0; i < pl.d.ncls; ++i)
      du = std::max(du, pl.flat ? 4.f + 0.45f * pl.d.c[i].nchunks : 4.5f + 0.3f * pl.d.c[i].nchunks);
  }
  pl.ok = true;
  pl.product = product;
  pl.tm = TM; pl.tn = TN; pl.ta = w.ta; pl.tb = w.tb; pl.w = w.p;
  pl.us = (du > w.us ? du : w.us) + w.fold_us;
  // Positions that no tap reaches make a second round where they do not fit the first (1 x 1 / 2, a pass: 88 -> 240 at 34 x 27, 13
  // images, 64 x 32 tiles and 280 workgroups 18.7 us, 128 x 64 and 184 16.0; 256 -> 512 at 22 x 22, 8 images 19.4, 17.5).
  if (pl.nw + pl.d.nconv > CUS) pl.us += 2.f;
  if (!best.ok || pl.us < best.us) best = pl;
}
PairPlan work_out_plan(const Geom& g) {
  PairPlan pl{};
  if (!wgw::plan(g).ok) return pl;
  consider<32, 32>(g, pl);
  consider<64, 32>(g, pl);
  consider<64, 64>(g, pl);
  consider<128, 64>(g, pl);
  return pl;
}
const PairPlan& plan(const Geom& g) {
  return planned<PairPlan>(g, CONVBN_BF16, [&] { return work_out_plan(g); });
}

template <int TM, int TN>
constexpr int dgrad_lds() {
  if constexpr (TM == 128) return win::WnCfg<128, 64, 6>::LDS_BYTES;
  else return win::KsCfg<TM, TN>::LDS_BYTES;
}
template <int TM, int TN, bool FLAT, int TA, int TB>
hipError_t launch_inst(const wgw::WwParams& w, const win::WnParams& d, int nw, hipStream_t st) {
  static LdsLimitOnce lds_once;
  constexpr int a = wgw::WwCfg<TA, TB>::LDS_BYTES, b = dgrad_lds<TM, TN>(), lds = a > b ? a : b;
  if (hipError_t e = set_lds_limit_once(lds_once, reinterpret_cast<const void*>(&win_pair_kernel<TM, TN, FLAT, TA, TB>), lds);
      e != hipSuccess) return e;
  hipLaunchKernelGGL((win_pair_kernel<TM, TN, FLAT, TA, TB>), dim3(nw + d.nconv), dim3(512), lds, st, w, d, nw);
  return hipGetLastError();
}

}  // namespace

// Against a launch each, the second of which takes the fold-back along, or, where the weight gradient of a deep layer comes with its
// fold-back in one launch, against that one and the input gradient; there a block that kept nothing pays for a fold as well, and a
// workgroup's chain of 128 x 64 tiles is long (hundreds of taps and channels).  The figures above are fitted to 186 shapes, each
// measured with tiles up to 64 x 64, with 128 x 64 and without the pair: on average the choice is 0.2 % slower than the best of the
// three.  A pass, us, one launch and two:
//   3 x 3, 256 -> 256 at 18 x 18, 1 image       22.2, 25.7     1 x 1, 256 -> 1024 at 14 x 14, 16 images        21.8, 25.7
//   1 x 1, 2048 -> 512 at 9 x 9, 3 images       22.1, 28.5     1 x 1 / 2, 128 -> 256 at 70 x 68, 3 images      14.8, 19.9
//   3 x 3, 72 -> 136 at 27 x 33, 5 images       21.3, 22.5     3 x 3, 256 -> 256 at 16 x 17, 17 images         49.1, 43.4
// and against the deep layers' launch: 3 x 3, 512 -> 512 at 7 x 7, 16 images 40.8, 42.6, with 128 x 64 tiles 24 images 54.1, 50.4,
// 36 images 54.4, 51.5; 640 -> 512 at 8 x 9, 4 images 40.9, 46.6.
bool win_pair_taken(const Geom& g, int dtype) {
  if (dtype != CONVBN_BF16 || !plan(g).ok) return false;
  const PairPlan& pl = plan(g);
  if (wgrad_sq_fused_supported(g, dtype)) return pl.tm < 128 && pl.us + 4.f <= wgrad_sq_fused_us(g) + win::ks_dgrad_us(g, false);
  const wgw::WwPlan& w = wgw::plan(g);
  const float d = win::ks_dgrad_us(g, true);
  return pl.us <= w.us + (d > w.fold_us ? d : w.fold_us) + 2.f;
}
int win_pair_splits(const Geom& g) { return plan(g).w.slices; }
void win_pair_describe(const Geom& g, char* text, size_t bytes) {
  const PairPlan& pl = plan(g);
  snprintf(text, bytes, "%s %dx%d win %dx%d", pl.tm == 128 ? "win" : "ks", pl.tm, pl.tn, pl.ta, pl.tb);
}
hipError_t launch_win_pair(const Geom& g, const void* x, const void* dz, const void* w_crsk, void* dx, float* part,
                           float* r_part, hipStream_t st) {
  const PairPlan& pl = plan(g);
  if (!pl.ok) return hipErrorInvalidValue;
  wgw::WwParams w = pl.w;
  win::WnParams d = pl.d;
  w.x = (const bf16_t*)x; w.dz = (const bf16_t*)dz; w.part = part; w.r_part = r_part;
  d.act = (const bf16_t*)dz; d.wgt = (const bf16_t*)w_crsk; d.out = (bf16_t*)dx;
  d.relu = g.post_relu; d.mask = (const bf16_t*)g.post_mask; d.add = (const bf16_t*)g.post_add;
#define PAIR_TILE(TM_, TN_, F_, TA_, TB_) \
  if (pl.tm == TM_ && pl.tn == TN_ && pl.flat == F_ && pl.ta == TA_ && pl.tb == TB_) return launch_inst<TM_, TN_, F_, TA_, TB_>(w, d, pl.nw, st);
#define PAIR_CASE(TM_, TN_, F_) \
  PAIR_TILE(TM_, TN_, F_, 64, 64) PAIR_TILE(TM_, TN_, F_, 128, 64) PAIR_TILE(TM_, TN_, F_, 64, 128) PAIR_TILE(TM_, TN_, F_, 128, 128)
  PAIR_CASE(32, 32, true) PAIR_CASE(64, 32, true) PAIR_CASE(64, 64, true) PAIR_CASE(128, 64, true) PAIR_CASE(128, 64, false)
#undef PAIR_CASE
#undef PAIR_TILE
  return hipErrorInvalidValue;
}

}  // namespace convbn
