// The window product as a launch of its own; its device code is in conv_win_impl.h.
#include "conv_ks_impl.h"

#include <stdio.h>

#include <algorithm>

namespace convbn {

using namespace win;

namespace {

constexpr int CUS = 256, KS_FEW = 6, KS_MANY = 48;
// The tile of the wave-split product: the smallest whose workgroups are one round (3 x 3, 512 -> 512: 32 x 32 8.9 us, 64 x 32 11.3,
// 64 x 64 14.3 where all three are; a second round takes as long as the first: 17.3), `aside` counted in: 256 tiles and eight
// workgroups that fold took 8.1 us (128 -> 512 at 31 x 31, 1 image), 128 x 64 tiles 5.4.  None where 64 x 64 tiles are more
// than that, or have fewer chunks than give six of the eight waves one (1 x 1, 88 -> 240 at 34 x 27 / 2, 13 images, forward: 5.0
// on 128 x 64 tiles, 5.7), or where the deep-layer kernel has the layer and its chain is long (`deep`; 512 -> 512 at 6 x 6, 46
// images, 72 chunks: 16.4 there, 17.7; 128 -> 128 at 28 x 28, 8 images, 18 chunks: 9.8 there, 8.3).
struct KsTile { int tm, tn; };   // tm == 0: not taken
KsTile ks_tile(int C, int R, int n, const int* M, const Window* cv, bool deep, int aside) {
  constexpr KsTile sizes[] = {{32, 32}, {64, 32}, {64, 64}};
  int chunks = 0;
  for (int i = 0; i < n; ++i) chunks = std::max(chunks, ceil_div(cv[i].kH * cv[i].kW * (C >> 3), CB / 8));
  for (const KsTile& t : sizes) {
    long long tiles = 0;
    for (int i = 0; i < n; ++i)
      if (cv[i].kH > 0) tiles += (long long)ceil_div(M[i], t.tm) * ceil_div(R, t.tn);
    if (tiles > CUS || (t.tm * t.tn > 32 * 32 && tiles + aside > CUS)) continue;   // (32 x 32: two workgroups a compute unit)
    return t.tm * t.tn < 64 * 64 || (chunks >= KS_FEW && (chunks <= KS_MANY || !deep)) ? t : KsTile{0, 0};
  }
  return {0, 0};
}
struct WnPlan { int tm, tn, nst; bool flat; bool ks = false; };
WnPlan win_plan(int C, int R, int n, const int* M, const Window* cv, bool deep, int aside) {
  auto tiles = [&](int tm, int tn) {   // those with a product to compute
    long long t = 0;
    for (int i = 0; i < n; ++i)
      if (cv[i].kH > 0) t += ceil_div(M[i], tm);
    return t * ceil_div(R, tn);
  };
  const bool flat = C % CB != 0;
  if (const KsTile t = ks_tile(C, R, n, M, cv, deep, aside); t.tm) return {t.tm, t.tn, 0, true, true};
  // the largest tile that still gives most compute units one (as in conv_gm.hip); a tile of 128 channels only where the
  // last one is more than half full
  const bool wide = R % 128 == 0 || R % 128 > 64;
  if (wide && !flat && tiles(256, 128) >= 160) return {256, 128, 3, false};
  // (four stages: 512 <- 256 x 16 taps at 14 x 14, 32 images, 34.7 us with three, 33.7; granules over tap borders have no use for it)
  if (wide && tiles(128, 128) >= 160) return {128, 128, flat ? 3 : 4, flat};
  return {128, 64, tiles(128, 64) > 256 ? 3 : 6, flat};
}

template <int TM, int TN, int NST, bool FLAT, class Side>
__global__ __launch_bounds__(64 * NWAVES, (WnCfg<TM, TN, NST>::WAVES_SIMD)) void conv_win_kernel(WnParams p, Side side) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  body<TM, TN, NST, FLAT>(p, side, blockIdx.x, smem);
}

template <int TM, int TN, int NST, bool FLAT, class Side>
hipError_t launch_inst(WnParams& p, Side side, hipStream_t st) {
  static LdsLimitOnce lds_once;
  constexpr int lds = WnCfg<TM, TN, NST>::LDS_BYTES;
  if (hipError_t e = set_lds_limit_once(lds_once, reinterpret_cast<const void*>(&conv_win_kernel<TM, TN, NST, FLAT, Side>), lds);
      e != hipSuccess) return e;
  lay_out<TM, TN, FLAT>(p);
  int nside;
  if constexpr (Side::BACK) nside = fold_back_side_blocks(side, 64 * NWAVES); else nside = fold_side_blocks(p.bn);
  hipLaunchKernelGGL((conv_win_kernel<TM, TN, NST, FLAT, Side>), dim3(p.nconv + nside), dim3(64 * NWAVES), lds, st, p, side);
  return hipGetLastError();
}

template <int TM, int TN, class Side>
__global__ __launch_bounds__(64 * NWAVES, (KsCfg<TM, TN>::WAVES_SIMD)) void conv_ks_kernel(WnParams p, Side side) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  ks_body<TM, TN>(p, side, blockIdx.x, smem);
}

template <int TM, int TN, class Side>
hipError_t launch_ks(WnParams& p, Side side, hipStream_t st) {
  static LdsLimitOnce lds_once;
  constexpr int lds = KsCfg<TM, TN>::LDS_BYTES;
  if (hipError_t e = set_lds_limit_once(lds_once, reinterpret_cast<const void*>(&conv_ks_kernel<TM, TN, Side>), lds); e != hipSuccess)
    return e;
  lay_out<TM, TN, true>(p);
  int nside;
  if constexpr (Side::BACK) nside = fold_back_side_blocks(side, 64 * NWAVES); else nside = fold_side_blocks(p.bn);
  hipLaunchKernelGGL((conv_ks_kernel<TM, TN, Side>), dim3(p.nconv + nside), dim3(64 * NWAVES), lds, st, p, side);
  return hipGetLastError();
}

// n problems that share the operands, in any order, as the parameters of a launch (no pointers)
WnParams make_params(int C, int R, int n, const int* M, const Window* cv, size_t act_bytes, size_t wgt_bytes) {
  WnParams p{};
  p.act_bytes = (unsigned)act_bytes; p.wgt_bytes = (unsigned)wgt_bytes;
  p.C = C; p.R = R; p.ncls = n;
  p.by_channel = wgt_bytes > act_bytes;
  int order[MAXC];   // most taps first
  for (int i = 0; i < n; ++i) {
    int j = i;
    for (; j > 0 && cv[order[j - 1]].kH * cv[order[j - 1]].kW < cv[i].kH * cv[i].kW; --j) order[j] = order[j - 1];
    order[j] = i;
  }
  for (int i = 0; i < n; ++i) {
    p.c[i].cv = cv[order[i]];
    p.c[i].M = M[order[i]];
  }
  return p;
}

hipError_t launch_win(int C, int R, int n, const int* M, const Window* cv, const void* act, size_t act_bytes, const void* wgt,
                      size_t wgt_bytes, const float* bias, const BnEpilogue* bn, void* out, int relu, const void* mask,
                      const void* add, hipStream_t st, bool deep, int aside, const FoldBackArgs* fb = nullptr,
                      const FoldBackTArgs* fbt = nullptr) {
  if (n < 1 || n > MAXC || C % 8 || R % 8 || act_bytes >= OOB || wgt_bytes >= OOB) return hipErrorInvalidValue;
  WnParams p = make_params(C, R, n, M, cv, act_bytes, wgt_bytes);
  p.act = (const bf16_t*)act; p.wgt = (const bf16_t*)wgt; p.bias = bias; p.out = (bf16_t*)out;
  if (bn) p.bn = *bn;
  p.relu = relu; p.mask = (const bf16_t*)mask; p.add = (const bf16_t*)add;
  const WnPlan pl = win_plan(C, R, n, M, cv, deep, aside);
#define WIN_CASE(TM_, TN_, NST_, F_) \
  if (!pl.ks && pl.tm == TM_ && pl.tn == TN_ && pl.nst == NST_ && pl.flat == F_) \
    return fb ? launch_inst<TM_, TN_, NST_, F_>(p, *fb, st) : fbt ? launch_inst<TM_, TN_, NST_, F_>(p, *fbt, st)                \
                                                                  : launch_inst<TM_, TN_, NST_, F_>(p, FoldSide{}, st);
  WIN_CASE(256, 128, 3, false) WIN_CASE(128, 128, 4, false) WIN_CASE(128, 64, 3, false) WIN_CASE(128, 64, 6, false)
  WIN_CASE(128, 128, 3, true) WIN_CASE(128, 64, 3, true) WIN_CASE(128, 64, 6, true)
#undef WIN_CASE
#define KS_CASE(TM_, TN_) \
  if (pl.ks && pl.tm == TM_ && pl.tn == TN_) \
    return fb ? launch_ks<TM_, TN_>(p, *fb, st) : fbt ? launch_ks<TM_, TN_>(p, *fbt, st) : launch_ks<TM_, TN_>(p, FoldSide{}, st);
  KS_CASE(32, 32) KS_CASE(64, 32) KS_CASE(64, 64)
#undef KS_CASE
  return hipErrorInvalidValue;
}

bool sizes_fit(const Geom& g, int dtype) {
  return dtype == CONVBN_BF16 && g.Cin % 8 == 0 && g.Cout % 8 == 0 && (size_t)g.Min * g.Cin * 2 < OOB &&
         (size_t)g.M * g.Cout * 2 < OOB && (size_t)g.Cout * g.K * 2 < OOB;
}

// The residue class (a, b) of input positions h = sh hq + a, w = sw wq + b of an input gradient (Sec. 3.2.1:
// dX = w'_rot (*) dZ) only receives the taps i = i0 + sh t with i0 = (a + ph) mod sh (columns alike), from
// dZ[hq + dh0 - t], dh0 = (a + ph - i0) / sh: a stride-1 window over dZ, taps in reverse.
void dgrad_class(const Geom& g, int a, int b, Window* cv, int* M) {
  const int Hq = 1 + (g.Hin - 1 - a) / g.sh, Wq = 1 + (g.Win - 1 - b) / g.sw;
  const int i0 = (a + g.ph) % g.sh, j0 = (b + g.pw) % g.sw;
  int kh = i0 < g.kH ? 1 + (g.kH - 1 - i0) / g.sh : 0;
  int kw = j0 < g.kW ? 1 + (g.kW - 1 - j0) / g.sw : 0;
  if (kh == 0 || kw == 0) { kh = 0; kw = 1; }   // no tap reaches these positions
  // (a stride may be larger than image and window: what it multiplies is formed where there is a second row or column)
  Window c{};
  c.kH = kh; c.kW = kw;
  c.cph = kh - 1 - (a + g.ph - i0) / g.sh; c.cpw = kw - 1 - (b + g.pw - j0) / g.sw;
  c.csh = c.csw = 1; c.aH = g.Hout; c.aW = g.Wout;
  c.a_n = g.Hout * g.Wout * g.Cout; c.a_h = g.Wout * g.Cout; c.a_w = g.Cout;
  c.oHo = Hq; c.oWo = Wq;
  c.wt_row = kh > 1 ? -g.sh * g.kW : 0; c.wt_col = kw > 1 ? -g.sw : 0;
  if (kh > 0) c.wt0 = i0 * g.kW + j0 - (kh - 1) * c.wt_row - (kw - 1) * c.wt_col;
  c.wrow = g.kH * g.kW * g.Cout;
  c.out_strided = g.sh > 1 || g.sw > 1;
  c.out_base = (a * g.Win + b) * g.Cin; c.out_n = g.Hin * g.Win * g.Cin;
  c.out_h = Hq > 1 ? g.sh * g.Win * g.Cin : 0; c.out_w = Wq > 1 ? g.sw * g.Cin : 0;
  *cv = c;
  *M = g.N * Hq * Wq;
}
Window fprop_window(const Geom& g) {
  Window c{};
  c.kH = g.kH; c.kW = g.kW; c.cph = g.ph; c.cpw = g.pw; c.csh = g.sh; c.csw = g.sw; c.aH = g.Hin; c.aW = g.Win;
  c.a_n = g.Hin * g.Win * g.Cin; c.a_h = g.Win * g.Cin; c.a_w = g.Cin;
  c.oHo = g.Hout; c.oWo = g.Wout;
  c.wt_row = g.kW; c.wt_col = 1; c.wrow = g.K;
  return c;
}
// Workgroups that fold behind a forward product: where w' is small enough to be kept (the call may decide otherwise)
int folds_aside(const Geom& g) { return g.K <= g.M ? ceil_div(ceil_div(g.K, 64) * ceil_div(g.Cout, 64), 2) : 0; }
// ... that fold back behind an input gradient (of the copies that a window weight gradient leaves; another kernel may have left others)
int folds_back_aside(const Geom& g) {
  return wgrad_win_supported(g, CONVBN_BF16) ? fold_back_side_blocks(g.K, wgrad_win_splits(g), g.Cout, 64 * NWAVES) : 0;
}
// residue classes that have positions, in rows and columns
int classes_h(const Geom& g) { return g.sh < g.Hin ? g.sh : g.Hin; }
int classes_w(const Geom& g) { return g.sw < g.Win ? g.sw : g.Win; }

}  // namespace

bool win::dgrad_params(const Geom& g, WnParams* p) {
  if (!sizes_fit(g, CONVBN_BF16) || classes_h(g) * classes_w(g) > MAXC) return false;
  Window c[MAXC];
  int M[MAXC], n = 0;
  for (int a = 0; a < classes_h(g); ++a)
    for (int b = 0; b < classes_w(g); ++b, ++n) dgrad_class(g, a, b, &c[n], &M[n]);
  *p = make_params(g.Cout, g.Cin, n, M, c, (size_t)g.M * g.Cout * 2, (size_t)g.Cout * g.K * 2);
  return true;
}

bool win_supported(const Geom& g, int dtype) { return sizes_fit(g, dtype); }
bool ks_fprop_taken(const Geom& g, int dtype) {
  if (!sizes_fit(g, dtype)) return false;
  const Window c = fprop_window(g);
  return ks_tile(g.Cin, g.Cout, 1, &g.M, &c, st_fprop_supported(g, dtype), folds_aside(g)).tm != 0;
}
namespace {
struct KsGrad { bool taken; float us, back_us; };
const KsGrad& ks_grad(const Geom& g) {
  return planned<KsGrad>(g, CONVBN_BF16, [&] {
    KsGrad r{};
    WnParams p;
    if (!dgrad_params(g, &p)) return r;
    Window c[MAXC];
    int M[MAXC];
    for (int i = 0; i < p.ncls; ++i) { c[i] = p.c[i].cv; M[i] = p.c[i].M; }
    const KsTile t = ks_tile(p.C, p.R, p.ncls, M, c, st_dgrad_supported(g, CONVBN_BF16), 0);
    if (t.tm == 0) {   // (another kernel's)
      for (int i = 0; i < p.ncls; ++i) r.us = std::max(r.us, 5.5f + 0.2f * ceil_div(c[i].kH * c[i].kW * p.C, CB));
      r.back_us = r.us;
      return r;
    }
    if (t.tm == 32) lay_out<32, 32, true>(p);
    else if (t.tn == 32) lay_out<64, 32, true>(p);
    else lay_out<64, 64, true>(p);
    r.taken = true;
    r.us = ks_us(t.tm, t.tn, p);
    // (where the compute units are full they start when its first workgroups are done: 3 x 3, 184 -> 208 at 22 x 48, 5 images, 249 tiles
    // and 52 that fold back 16.0 us; 32 x 32: two share a compute unit)
    r.back_us = t.tm > 32 && p.nconv + folds_back_aside(g) > CUS ? r.us + 4.f : r.us;
    return r;
  });
}
}  // namespace
bool ks_dgrad_taken(const Geom& g, int dtype) { return sizes_fit(g, dtype) && ks_grad(g).taken; }
float win::ks_dgrad_us(const Geom& g, bool back) { return back ? ks_grad(g).back_us : ks_grad(g).us; }

void win_describe(const Geom& g, bool fwd, char* text, size_t bytes) {
  Window c[MAXC];
  int M[MAXC], n = 1;
  if (fwd) {
    c[0] = fprop_window(g);
    M[0] = g.M;
  } else {   // (of more classes than a launch takes, those of the first)
    n = std::min(MAXC, classes_h(g) * classes_w(g));
    for (int i = 0; i < n; ++i) dgrad_class(g, i / classes_w(g), i % classes_w(g), &c[i], &M[i]);
  }
  const WnPlan pl = fwd ? win_plan(g.Cin, g.Cout, n, M, c, st_fprop_supported(g, CONVBN_BF16), folds_aside(g))
                        : win_plan(g.Cout, g.Cin, n, M, c, st_dgrad_supported(g, CONVBN_BF16), 0);
  snprintf(text, bytes, "%s %dx%d", pl.ks ? "ks" : "win", pl.tm, pl.tn);
}

hipError_t launch_fprop_win(const Geom& g, const void* x, const void* w_krsc, const float* bias, void* z, hipStream_t st,
                            const BnEpilogue* bn) {
  const Window c = fprop_window(g);
  return launch_win(g.Cin, g.Cout, 1, &g.M, &c, x, (size_t)g.Min * g.Cin * 2, w_krsc, (size_t)g.Cout * g.K * 2, bias, bn, z,
                    g.post_relu, g.post_mask, g.post_add, st, st_fprop_supported(g, CONVBN_BF16), folds_aside(g), nullptr, g.fold_back_t);
}
hipError_t launch_dgrad_win(const Geom& g, const void* dz, const void* w_crsk, const float* bias, void* dx, hipStream_t st) {
  Window c[MAXC];
  int M[MAXC], n = 0;
  const FoldBackArgs* fb = g.fold_back;
  auto flush = [&]() -> hipError_t {
    const int k = n;
    const FoldBackArgs* const f = fb;   // (along with the first launch)
    n = 0;
    fb = nullptr;
    return launch_win(g.Cout, g.Cin, k, M, c, dz, (size_t)g.M * g.Cout * 2, w_crsk, (size_t)g.Cout * g.K * 2, bias, nullptr, dx,
                      g.post_relu, g.post_mask, g.post_add, st, st_dgrad_supported(g, CONVBN_BF16), 0, f);
  };
  for (int a = 0; a < classes_h(g); ++a)
    for (int b = 0; b < classes_w(g); ++b) {
      dgrad_class(g, a, b, &c[n], &M[n]);
      if (++n == MAXC)
        if (hipError_t e = flush(); e != hipSuccess) return e;
    }
  return n > 0 ? flush() : hipSuccess;
}

}  // namespace convbn
