// The window product as a launch of its own; its device code is in conv_win_impl.h.
#include "conv_win_impl.h"

namespace convbn {

using namespace win;

namespace {

struct WnPlan { int tm, tn, nst; bool flat; };
WnPlan win_plan(int C, int R, int n, const int* M, const Window* cv) {
  auto tiles = [&](int tm, int tn) {   // those with a product to compute
    long long t = 0;
    for (int i = 0; i < n; ++i)
      if (cv[i].kH > 0) t += ceil_div(M[i], tm);
    return t * ceil_div(R, tn);
  };
  const bool flat = C % CB != 0;
  // the largest tile that still gives most compute units one (as in conv_gm.hip); a tile of 128 channels only where the
  // last one is more than half full
  const bool wide = R % 128 == 0 || R % 128 > 64;
  if (wide && !flat && tiles(256, 128) >= 160) return {256, 128, 3, false};
  if (wide && tiles(128, 128) >= 160) return {128, 128, 3, flat};
  return {128, 64, tiles(128, 64) > 256 ? 3 : 6, flat};
}

template <int TM, int TN, int NST, bool FLAT, class Side>
__global__ __launch_bounds__(64 * NWAVES) void conv_win_kernel(WnParams p, Side side) {
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
                      const void* add, hipStream_t st, const FoldBackArgs* fb = nullptr) {
  if (n < 1 || n > MAXC || C % 8 || R % 8 || act_bytes >= OOB || wgt_bytes >= OOB) return hipErrorInvalidValue;
  WnParams p = make_params(C, R, n, M, cv, act_bytes, wgt_bytes);
  p.act = (const bf16_t*)act; p.wgt = (const bf16_t*)wgt; p.bias = bias; p.out = (bf16_t*)out;
  if (bn) p.bn = *bn;
  p.relu = relu; p.mask = (const bf16_t*)mask; p.add = (const bf16_t*)add;
  const WnPlan pl = win_plan(C, R, n, M, cv);
#define WIN_CASE(TM_, TN_, NST_, F_) \
  if (pl.tm == TM_ && pl.tn == TN_ && pl.nst == NST_ && pl.flat == F_) \
    return fb ? launch_inst<TM_, TN_, NST_, F_>(p, *fb, st) : launch_inst<TM_, TN_, NST_, F_>(p, FoldSide{}, st);
  WIN_CASE(256, 128, 3, false) WIN_CASE(128, 128, 3, false) WIN_CASE(128, 64, 3, false) WIN_CASE(128, 64, 6, false)
  WIN_CASE(128, 128, 3, true) WIN_CASE(128, 64, 3, true) WIN_CASE(128, 64, 6, true)
#undef WIN_CASE
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

hipError_t launch_fprop_win(const Geom& g, const void* x, const void* w_krsc, const float* bias, void* z, hipStream_t st,
                            const BnEpilogue* bn) {
  Window c{};
  c.kH = g.kH; c.kW = g.kW; c.cph = g.ph; c.cpw = g.pw; c.csh = g.sh; c.csw = g.sw; c.aH = g.Hin; c.aW = g.Win;
  c.a_n = g.Hin * g.Win * g.Cin; c.a_h = g.Win * g.Cin; c.a_w = g.Cin;
  c.oHo = g.Hout; c.oWo = g.Wout;
  c.wt_row = g.kW; c.wt_col = 1; c.wrow = g.K;
  return launch_win(g.Cin, g.Cout, 1, &g.M, &c, x, (size_t)g.Min * g.Cin * 2, w_krsc, (size_t)g.Cout * g.K * 2, bias, bn, z,
                    g.post_relu, g.post_mask, g.post_add, st);
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
                      g.post_relu, g.post_mask, g.post_add, st, f);
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
