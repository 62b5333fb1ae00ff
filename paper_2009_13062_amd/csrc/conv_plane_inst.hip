// Instantiation of the pointwise convolution over planes of any size (conv_plane.h).
#include <algorithm>
#include <atomic>

#include "conv_plane.h"

namespace nf {

template <class Cfg>
__global__ __launch_bounds__(Cfg::kThreads, Cfg::kWPE) void conv_plane_kernel(ConvPlaneArgs a) {
  extern __shared__ __align__(1024) unsigned char smem_raw[];
  conv_plane_tile<Cfg>(a, (lds_u8_t*)smem_raw);
}

// Positions per tile: as many as the tile's columns and its chunks hold, in equal parts.  0: the shape does not fit.
template <class Cfg>
static int plane_step(const GemmArgs& a, int* cps) {
  const int P = a.cols, s = a.geom.stride;
  *cps = Cfg::kCpr;
  int most = Cfg::kBN;
  if (Cfg::kWhole) return P <= Cfg::kBN && a.ldb <= 8 * Cfg::kCpr ? (P + 7) / 8 * 8 : 0;
  if (s == 1) {
    const int slack = Cfg::kQuad ? (P % 8 ? 4 : 0) : 7;                     // elements in front of a channel's first
    if (P <= Cfg::kBN && P + slack <= 8 * Cfg::kCpr) return (P + 7) / 8 * 8;
    most = std::min(most, (8 * Cfg::kCpr - slack) / 8 * 8);
  } else {
    const int Wo = a.geom.Wo, Ho = P / Wo;
    *cps = (7 + (Wo - 1) * s + 1 + 7) / 8;
    // consecutive positions may start anywhere in an output row
    for (; most > 0; most -= 8)
      if (std::min((most - 1 + Wo - 1) / Wo + 1, Ho) * (long long)*cps <= Cfg::kCpr) break;
    if (most <= 0) return 0;
  }
  const int tiles = (P + most - 1) / most;
  return std::min(most, ((P + tiles - 1) / tiles + 7) / 8 * 8);
}

template <class Cfg>
static nf_status launch_plane(const GemmLaunch& L, hipStream_t s) {
  ConvPlaneArgs a;
  (GemmArgs&)a = L.a;
  a.step = plane_step<Cfg>(L.a, &a.cps);
  if (a.step <= 0 || a.K % Cfg::kBK || (Cfg::kQuad && (a.geom.stride != 1 || a.cols % 4))) return NF_EUNSUPPORTED;
  cw_divisor(a.cps, &a.rcp_cps, &a.one_cps);
  cw_divisor(a.geom.Wo, &a.rcp_wo, &a.one_wo);
  a.tiles_m = (a.rows + Cfg::kBM - 1) / Cfg::kBM;
  a.tiles_n = (a.cols + a.step - 1) / a.step;
  const long long total = (long long)a.tiles_m * a.tiles_n * a.nz0 * L.nz1;
  if (total <= 0 || total > 0x7fffffffLL) return NF_EUNSUPPORTED;
  auto kern = conv_plane_kernel<Cfg>;
  constexpr int kLds = Cfg::kLdsBytes;
  if (kLds > 64 * 1024) {
    static std::atomic<bool> opted_in{false};
    if (!opted_in.load(std::memory_order_acquire)) {
      if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kLds) != hipSuccess)
        return NF_ELAUNCH;
      opted_in.store(true, std::memory_order_release);
    }
  }
  nf_launch(kern, dim3((unsigned)total), dim3(Cfg::kThreads), kLds, s, a);
  return hipGetLastError() == hipSuccess ? NF_OK : NF_ELAUNCH;
}

//                                    FM FN WGM WGN BK CPR NS waves per SIMD, QUAD, WHOLE, AHEAD
using CfgPW64x64 = PlaneCfg<1, 1, 2, 2, 64, 7, 5, 2, false, true>;
using CfgPW128x64 = PlaneCfg<1, 1, 4, 2, 64, 7, 3, 4, false, true>;
using CfgPW64x224 = PlaneCfg<1, 1, 2, 7, 64, 25, 2, 4, true, true>;
using CfgPW64x224d = PlaneCfg<1, 1, 2, 7, 64, 25, 4, 2, true, true, true>;
using CfgPQ64x128 = PlaneCfg<1, 1, 2, 4, 64, 17, 3, 2, true, false, true>;
using CfgPQ128x128 = PlaneCfg<2, 1, 2, 4, 64, 17, 2, 2, true, false>;
using CfgPG32x64 = PlaneCfg<1, 1, 1, 2, 64, 9, 3, 1, false, false>;
using CfgPG128x64 = PlaneCfg<1, 1, 4, 2, 64, 21, 2, 4, false, false>;
using CfgPG128x64k32 = PlaneCfg<1, 1, 4, 2, 32, 28, 3, 4, false, false>;
using CfgPG128x128 = PlaneCfg<2, 1, 2, 4, 32, 36, 3, 4, false, false>;

// us of a launch: a + l per 64 of k; per 256 tiles (f of them) b per 64 of k, e, and r more with a residual; w per MB of weights; x per
// 64 of k and 256 tiles beyond the first.  Fitted to 1400 stride-1 problems (planes of 5 x 5 to 58 x 58, 64 ... 2048 channels, 1 ... 256
// images) and 900 strided ones, weights from HBM: mean error 3 to 8 %, of the loaders of pixel pairs 16 and 21 %.
struct PlaneCost { float a, l, b, e, r, w, x; };
constexpr PlaneCost kPlaneCost[kNumConvPlaneTiles] = {
    {3.02f, 0.440f, 0.020f, 0.94f, 0.05f, 0.036f, 0.313f}, {3.35f, 0.556f, 0.049f, 1.28f, 0.21f, 0.043f, 0.499f},
    {3.31f, 0.652f, 0.131f, 1.46f, 0.28f, 0.045f, 0.549f}, {3.88f, 0.539f, 0.057f, 1.61f, 0.42f, 0.082f, 0.797f},
    {3.23f, 0.463f, 0.020f, 1.40f, 0.27f, 0.041f, 0.435f}, {3.64f, 0.770f, 0.030f, 2.08f, 0.77f, 0.097f, 0.684f},
    {3.25f, 0.366f, 0.f, 0.51f, 0.05f, 0.015f, 0.183f}, {3.21f, 0.712f, 0.244f, 0.92f, 0.20f, 0.118f, 0.458f},
    {3.48f, 0.721f, 0.266f, 0.83f, 0.38f, 0.060f, 0.617f}, {4.29f, 0.827f, 0.353f, 1.11f, 0.51f, 0.037f, 0.770f}};
// the register-staged tiles on the same problems: [64 x 64, 128 x 128][k of whole pipeline rounds][planes of 4 k positions]
constexpr PlaneCost kPlaneRegCost[2][2][2] = {
    {{{4.11f, 0.696f, 0.f, 0.71f, 0.35f, 0.115f, 0.f},
      {3.30f, 0.633f, 0.f, 0.64f, 0.44f, 0.074f, 0.188f}},
     {{4.77f, 0.267f, 0.074f, 0.25f, 0.42f, 0.068f, 0.294f},
      {3.72f, 0.266f, 0.076f, 0.42f, 0.33f, 0.049f, 0.264f}}},
    {{{3.90f, 1.486f, 0.f, 2.66f, 0.65f, 0.f, 0.519f},
      {3.96f, 0.864f, 0.f, 2.48f, 1.20f, 0.046f, 0.875f}},
     {{5.07f, 0.107f, 0.794f, 2.05f, 0.58f, 0.006f, 0.f},
      {3.38f, 0.180f, 0.733f, 2.51f, 1.34f, 0.020f, 0.f}}}};
constexpr PlaneCost kPairCost[2] = {{5.24f, 0.457f, 0.f, 0.38f, 0.60f, 0.589f, 0.729f}, {5.86f, 0.637f, 0.426f, 3.25f, 0.89f, 0.f, 0.959f}};

static float plane_us(const PlaneCost& c, long long tiles, const GemmArgs& a) {
  const float k = (float)a.K / 64.0f, f = (float)tiles / 256.0f;
  const float mb = (float)a.nz0 * (float)a.rows * (float)a.K * 2e-6f;
  return c.a + (c.l + c.x * std::max(0.f, f - 1.f)) * k + f * (c.b * k + c.e + (a.R ? c.r : 0.f)) + c.w * mb;
}
template <class Cfg>
static void plane_try(int tile, float margin, const GemmLaunch& L, int* best, float* limit) {
  const GemmArgs& a = L.a;
  int cps;
  const int step = plane_step<Cfg>(a, &cps);
  if (step <= 0 || a.K % Cfg::kBK || (Cfg::kQuad && (a.geom.stride != 1 || a.cols % 4))) return;
  const long long tiles = (long long)((a.rows + Cfg::kBM - 1) / Cfg::kBM) * ((a.cols + step - 1) / step) * a.nz0 * L.nz1;
  const float us = plane_us(kPlaneCost[tile], tiles, a) / margin;
  if (us < *limit) { *best = tile; *limit = us; }
}

// The tile of conv_plane.h for a problem that would run in the register-staged tile `now`, or -1.
// Stride 1: where it is predicted 7 % faster, for the three tiles of many positions from 512 of k on 18 % (their slope is underestimated
// for some shapes).  Over the 1400 problems 7 % less time on average, seven slower by 4 to 9 %; 19 % less over 7 x 7 planes (32 models 512 ->
// 2048 24.8 -> 17.8 us), 14 x 14 256 -> 1024 16.6 -> 14.4, 50 x 50 64 -> 256 of 12 images 12.7 -> 10.1.
// (Over 7900 other problems of these ranges, even widths at stride 2 among them, 16 % less time, one in a hundred slower by more than 6 %: the
// models' error.)  Odd planes of more than 56 positions gain in the 32 x 64 tile only: the other gathering ones were a tenth slower.
// Strided, eight 2-byte loads per 16 bytes in the register-staged tile: always (3 models of 4 images 512 -> 1024 at 25 x 25 24.7 -> 13.0, 1024
// -> 2048 at 13 x 13 39.3 -> 18.7 us; 1.6 to 2.1 times as fast over every size).  Stride 2 over an even width, which has loaders of
// aligned pixel pairs: up to 24 wide where predicted 16 % faster, as those predictions are off by 16 % themselves (24 models 1024 -> 256 at
// 25 x 16 with a residual, predicted 13 % faster: 13.9 us in pairs, 19.8 here; 32 models 1024 -> 2048 at 14 x 14 46 -> 36 us; wider inputs are loaded
// whole for every second pixel: 32 models 256 -> 512 at 56 x 56 34 against 31, 6 models 256 -> 512 at 28 x 28 a tenth slower).
int pick_conv_plane(const GemmLaunch& L, int now, bool pairs) {
  const GemmArgs& a = L.a;
  const bool big = now == T128x128w8, one = a.geom.stride == 1;
  if (a.K % 64 || a.rows <= 32 || (pairs && a.geom.W > 24)) return -1;
  const long long tiles = (long long)((a.rows + kTileBM[now] - 1) / kTileBM[now]) * ((a.cols + kTileBN[now] - 1) / kTileBN[now]) * a.nz0 * L.nz1;
  int best = -1;
  float limit = one ? plane_us(kPlaneRegCost[big][a.K % (big ? 128 : 256) == 0][a.cols % 4 == 0], tiles, a)
                : pairs ? plane_us(kPairCost[big], tiles, a) : 3e38f;
  const float m = one ? 0.93f : 0.84f, wide = a.K >= 512 ? 0.82f : m;
  plane_try<CfgPW64x64>(PW64x64, m, L, &best, &limit);
  plane_try<CfgPW128x64>(PW128x64, m, L, &best, &limit);
  plane_try<CfgPG32x64>(PG32x64, m, L, &best, &limit);
  if (one) {
    plane_try<CfgPW64x224>(PW64x224, wide, L, &best, &limit);
    plane_try<CfgPW64x224d>(PW64x224d, wide, L, &best, &limit);
    if (a.K >= 128) plane_try<CfgPQ64x128>(PQ64x128, m, L, &best, &limit);
    plane_try<CfgPQ128x128>(PQ128x128, wide, L, &best, &limit);
  } else {
    plane_try<CfgPG128x64>(PG128x64, m, L, &best, &limit);
    plane_try<CfgPG128x64k32>(PG128x64k32, m, L, &best, &limit);
    plane_try<CfgPG128x128>(PG128x128, m, L, &best, &limit);
  }
  return best;
}

nf_status launch_conv_plane(int tile, const GemmLaunch& L, hipStream_t s) {
  const GemmArgs& a = L.a;
  // chunks of x, 32-bit byte offsets, division by Wo (cw_div: positions below 2^32 / Wo)
  if (a.rows <= 0 || a.lda % 8 || ((uintptr_t)a.A & 15) || ((uintptr_t)a.B & 15) || (long long)a.rows * a.K >= (1LL << 30) ||
      (long long)a.K * a.ldb >= (1LL << 30) || (long long)a.cols * a.geom.Wo >= (1LL << 32))
    return NF_EUNSUPPORTED;
  switch (tile) {
    case PW64x64: return launch_plane<CfgPW64x64>(L, s);
    case PW128x64: return launch_plane<CfgPW128x64>(L, s);
    case PW64x224: return launch_plane<CfgPW64x224>(L, s);
    case PW64x224d: return launch_plane<CfgPW64x224d>(L, s);
    case PQ64x128: return launch_plane<CfgPQ64x128>(L, s);
    case PQ128x128: return launch_plane<CfgPQ128x128>(L, s);
    case PG32x64: return launch_plane<CfgPG32x64>(L, s);
    case PG128x64: return launch_plane<CfgPG128x64>(L, s);
    case PG128x64k32: return launch_plane<CfgPG128x64k32>(L, s);
    case PG128x128: return launch_plane<CfgPG128x128>(L, s);
  }
  return NF_EUNSUPPORTED;
}

}  // namespace nf
