// Instantiation, tile choice and launch of the 3x3 kernels with wavefront-private pipelines (conv_wave.h).
#include <limits.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstring>

#include "conv_wave.h"
#include "gemm_launch.h"

namespace nf {

template <typename T, int NB, int KG, int NT>
static nf_status launch_kernel(long long total, int lds, const ConvWaveArgs<T>& a, hipStream_t s) {
  auto kern = conv_wave_kernel<T, NB, KG, NT>;
  if (lds > 64 * 1024) {
    static std::atomic<bool> opted_in{false};        // per kernel: idempotent, a benign race
    if (!opted_in.load(std::memory_order_acquire)) {
      if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) !=
          hipSuccess)
        return NF_ELAUNCH;
      opted_in.store(true, std::memory_order_release);
    }
  }
  nf_launch(kern, dim3((unsigned)total), dim3(KG * kWave), lds, s, a);
  return hipGetLastError() == hipSuccess ? NF_OK : NF_ELAUNCH;
}

// The tile with NB blocks of positions: patch, tasks per lane, LDS; nt == 0: it does not fit.
struct WaveTile { int tiles_n, PS, nt, lds; };
template <typename T>
static WaveTile wave_tile(const ConvWaveArgs<T>& a, int Ho, int NB, int KG) {
  constexpr int PX = ConvWaveType<T>::kPix, kMostTasks = sizeof(T) == 4 ? 24 : 15;      // a task is 4 or 8 registers
  WaveTile t{(a.HoWo + 32 * NB - 1) / (32 * NB), 0, 0, 0};
  // output rows that 32 NB consecutive positions can touch, the patch rows and image rows they need
  const int span = (int)std::min<long long>(Ho, 32 * NB % a.Wo == 0 ? 32 * NB / a.Wo : (32 * NB - 2 + a.Wo) / a.Wo + 1);
  const int PH = (span - 1) * a.stride + 3;
  const long long PS = (long long)PH * a.PW;
  if (PS >= 32768) return t;                                 // two 16-bit pixel slots share a register
  t.PS = (int)PS;
  t.lds = conv_wave_lds_bytes(NB, KG, t.PS);
  const long long npx = (long long)std::min(PH, a.H) * a.W;
  const long long nt = (2 * ((npx + PX - 1) / PX) + kWave - 1) / kWave;
  if (t.lds <= 160 * 1024 && nt <= kMostTasks) t.nt = (int)nt;
  return t;
}

template <typename T, int NB, int KG>
static nf_status launch_tile(const WaveTile& t, ConvWaveArgs<T>& a, int B, hipStream_t s) {
  a.tiles_m = (a.cog + 31) / 32;
  a.tiles_n = t.tiles_n;
  a.PS = t.PS;
  const long long total = (long long)a.tiles_m * a.tiles_n * a.nG * B;
  if (total <= 0 || total > 0x7fffffffLL) return NF_EUNSUPPORTED;
#define NF_CW(NT_) if (t.nt <= NT_) return launch_kernel<T, NB, KG, NT_>(total, t.lds, a, s)
  NF_CW(1); NF_CW(2); NF_CW(4); NF_CW(7); NF_CW(10); NF_CW(15);
  if constexpr (sizeof(T) == 4) { NF_CW(24); }
#undef NF_CW
  return NF_EUNSUPPORTED;
}

// Time of a tile (us) for choosing the number of blocks: launch, per round of workgroups the latency of one, and the rate at which a
// compute unit gets through the others of its round.  n: steps of a wavefront.  Fitted to every tile over 1265 bf16 and 1250
// float32 problems (8 ... 512 channels, planes of 7 x 7 to 100 x 100, either stride, 1 ... 128 images): predictions are off by 5 to
// 10 %, the tile chosen is 0.5 to 1 % behind the best one on average.
struct WaveCost { float launch, lat, lat_nb, lat_n, lat_n_nb, lat_n_nt, thr, thr_nb, thr_n, thr_n_nb; };
constexpr WaveCost kWaveCost[2][2] = {   // [float32][four wavefronts per tile]
    {{2.45f, 1.63f, 0.96f, 0.24f, 0.15f, 0.11f, 0.54f, 0.38f, 0.37f, 0.22f},
     {3.01f, 1.04f, 0.42f, 0.47f, 0.16f, 0.16f, 0.45f, 0.10f, 0.28f, 0.18f}},
    {{1.44f, 2.38f, 1.23f, 0.20f, 1.01f, 0.05f, 0.32f, 0.55f, 0.00f, 1.18f},
     {2.68f, 1.42f, 0.42f, 0.24f, 1.03f, 0.09f, 0.13f, 0.03f, 0.32f, 1.16f}}};

template <typename T>
static float wave_us(const ConvWaveArgs<T>& a, const WaveTile& t, int NB, int KG, int B) {
  constexpr bool kF32 = sizeof(T) == 4;
  const WaveCost& c = kWaveCost[kF32][KG == 4];
  const int n = (a.cig / (2 * ConvWaveType<T>::kEV) + KG - 1) / KG;
  const int nt = t.nt <= 1 ? 1 : t.nt <= 2 ? 2 : t.nt <= 4 ? 4 : t.nt <= 7 ? 7 : t.nt <= 10 ? 10 : t.nt <= 15 ? 15 : 24;
  const float W = (float)((double)((a.cog + 31) / 32) * t.tiles_n * a.nG * B * KG / 1024);      // workgroups of four wavefronts per compute unit
  const int occ = std::min(160 * 1024 / t.lds, conv_wave_occupancy(kF32, NB, KG, nt) * 4 / KG);
  const float rounds = ceilf(W * 4 / (KG * occ));
  return c.launch + rounds * (c.lat + c.lat_nb * NB + n * (c.lat_n + c.lat_n_nb * NB + c.lat_n_nt * nt)) +
         std::max(ceilf(W) - rounds, 0.f) * (c.thr + c.thr_nb * NB + n * (c.thr_n + c.thr_n_nb * NB));
}

// How many wavefronts share a tile, by the shape of ONE group (never by how many models or images there are: the order of the sum
// follows from it); 0 = another kernel.  A shape is taken where no number of images from 1 to 256 (float32: 1 to 48) is slower for it by more
// than a few percent.
//   bf16, groups of 32 k channels (conv_tap.h, which multiplies four wavefronts' worth of positions out of one block of 32 channels, is
//   the alternative): few positions and many channels, where that kernel waits; with many images it is ahead on larger planes, because
//   a 32-row tile reads a fragment from LDS for every multiplication.  Times against it at 1 / 32 / 256 images:
//     stride 1: 512 channels 7 x 7 0.41 / 0.74 / 0.75, 28 x 28 0.57 / 0.90 / 0.97; 256 channels 14 x 14 0.55 / 0.89 / 1.04, left out
//     17 x 17 0.53 / 1.03 / 1.18; 128 channels 11 x 11 0.67 / 0.80 / 1.02, left out 14 x 14 0.66 / 0.95 / 1.20; 64 channels 9 x 9 0.76 /
//     0.80 / 1.09, left out 14 x 14 0.75 / 0.83 / 1.43; 32 channels 5 x 5 0.90 / 0.91 / 0.90, left out 8 x 8, which then lost (1.0 / 1.10 / 1.28), now
//     0.89 / 0.90 / 0.93
//     stride 2: 512 channels 14 x 14 0.36 / 0.87 / 0.86, left out 18 x 18 0.37 / 1.08 / 1.44; 256 channels 8 x 8 0.56 / 0.74 / 0.64, 13 x 13
//     0.43 / 0.85 / 0.82, left out 10 x 10 0.53 / 0.91 / 1.11 and 14 x 14 0.44 / 0.87 / 1.01; 128 channels 8 x 8 0.69 / 0.72 / 0.85, left
//     out 9 x 9 0.66 / 0.84 / 1.39
//   (Over 7200 problems that are taken 32 % less time, 33 of them 4 to 12 % slower and one by a third, most with 64 images and more.)
//   and against the kernels that take groups of 16 (2 k + 1) channels (conv_patch.h, implicit GEMM): 16 channels on one wavefront
//   14 x 14 0.94 / 0.95 / 0.77, 28 x 28 0.98 / 0.78 / 0.55; 48 channels on four 13 x 13 0.66 / 0.63 / 0.86, stride 2 16 -> 8 0.73 / 0.70 / 0.69, left
//   out 14 x 14 0.73 / 0.69 / 1.15 and 36 -> 18 0.68 / 1.03 / 1.87.
//   Groups of 16 in pairs that conv_tap.h fuses: 32 groups at 8 x 8 0.77 / 0.89 / 0.83, stride 2 28 -> 14 0.70 / 0.87 / 0.81; left out 6 groups at
//   10 x 10 0.82 / 0.88 / 1.30.  Fewer than 32 outputs leave rows idle: 32 -> 16 6.7 against 8.2.
//   float32 (the gathered kernel of gemm_f32.h) at 1 / 12 / 48 images: stride 1 up to 64 x 64 positions 256 channels 14 x 14 0.55 / 0.60 /
//   0.99, 64 channels 64 x 64 0.59 / 0.91 / 0.91 (left out 72 x 72 0.65 / 1.00 / 1.08), 32 groups of 8 channels on one wavefront 28 x 28 0.70 /
//   0.43 / 0.40; left out 40 channels, five steps over four wavefronts, at 28 x 28 0.66 / 0.82 / 1.02 and 64 x 64 0.72 / 1.12 / 1.03.  Stride 2:
//   16 channels on one wavefront 28 x 28 0.92 / 0.71 / 0.62 (on four 0.88 / 1.25 / 1.21), left out 56 x 56 1.08 / 1.24 / 1.11; others on four
//   20 x 20 0.58 / 0.71 / 0.85, left out 128 channels 28 x 28 0.65 / 0.92 / 1.27.
static int wave_shares(bool f32, int cig, int cog, int g, long long HoWo, int stride) {
  if (f32) {
    if (stride > 1) return cig == 8 || (cig == 16 && HoWo > 64) ? HoWo <= 1600 : HoWo <= 400 ? 4 : 0;
    return cig == 8 || (cig == 16 && HoWo > 1200) ? 1 : HoWo <= (cig == 40 ? 400 : 4096) ? 4 : 0;
  }
  if (cig == 16) return g % 2 == 0 && cog <= 16 && HoWo > (stride > 1 ? 256 : 81) ? 0 : 1;
  if (cog < 32 && cig % 32 == 0) return 0;
  if (cig % 32) return HoWo <= (stride > 1 ? 64 : 169) ? 4 : 0;
  const int most = cig < 64 ? 25 : stride > 1 ? (cig < 384 ? 64 : 196) : cig < 128 ? 81 : cig < 256 ? 121 : cig < 384 ? 196 : cig < 512 ? 1300 : INT_MAX;
  return HoWo <= most || (stride > 1 && cig >= 256 && HoWo > 100 && HoWo <= 169) ? 4 : 0;
}

// The tile of a problem: wavefronts that share it and its blocks of positions; kg == 0: another kernel.
struct WaveChoice { int kg, nb; WaveTile tile; };
template <typename T>
static WaveChoice choose_wave(ConvWaveArgs<T>& a, int Ho, int B) {
  constexpr int EV = ConvWaveType<T>::kEV;
  const WaveChoice none{};
  const long long plane = (long long)a.H * a.W;
  if (a.cig % (2 * EV) != 0 || a.pad > 2 || a.W < 2 || Ho <= 0) return none;
  // 32-bit byte offsets inside one group's weights and inside one step's planes; exact divisions by Wo and W
  if ((long long)a.cog * a.cig * 9 * sizeof(T) >= (1LL << 31) || 2 * EV * plane * sizeof(T) >= (1LL << 31) ||
      (long long)a.HoWo * a.Wo >= (1LL << 32) || plane * a.W >= (1LL << 32)) return none;
  a.PW = std::max(a.W + a.pad, (a.Wo - 1) * a.stride + 3);
  WaveChoice c{wave_shares(sizeof(T) == 4, a.cig, a.cog, a.g, a.HoWo, a.stride), 0, {}};
  int forced = 0;
  if (const char* e = dev_getenv("NETFUSE_CW")) sscanf(e, "%d,%d", &c.kg, &forced);
  if (c.kg == 0) return none;
  float best_us = 0.f;
  for (int b : {1, 2, 3, 4, 5, 7}) {
    // one wavefront per tile: 3 and 5 blocks are not built, nor 7 in float32, where the registers of two chains leave room for one
    // wavefront per SIMD (32 groups of 8 channels at 28 x 28, 8 models: 31.6 us against 18.5 in two blocks)
    if (c.kg == 1 && (b == 3 || b == 5 || (b == 7 && sizeof(T) == 4))) continue;
    if (forced > 0 && b != forced) continue;
    const WaveTile t = wave_tile(a, Ho, b, c.kg);
    if (t.nt == 0) continue;
    const float us = wave_us(a, t, b, c.kg, B);
    if (c.nb == 0 || us < best_us) { c.nb = b; c.tile = t; best_us = us; }
  }
  return c.nb ? c : none;
}

template <typename T>
nf_status launch_conv_wave(ConvWaveArgs<T>& a, int Ho, int B, hipStream_t s) {
  const WaveChoice c = choose_wave(a, Ho, B);
  if (c.kg == 0 || ((uintptr_t)a.w & 15) != 0) return NF_EUNSUPPORTED;
  cw_divisor(a.W, &a.rcp_w, &a.one_w);
  cw_divisor(a.Wo, &a.rcp_wo, &a.one_wo);
#define NF_CWT(NB_, KG_) if (c.kg == KG_ && c.nb == NB_) return launch_tile<T, NB_, KG_>(c.tile, a, B, s)
  NF_CWT(1, 4); NF_CWT(2, 4); NF_CWT(3, 4); NF_CWT(4, 4); NF_CWT(5, 4); NF_CWT(7, 4);
  NF_CWT(1, 1); NF_CWT(2, 1); NF_CWT(4, 1);
  if constexpr (sizeof(T) == 2) { NF_CWT(7, 1); }
#undef NF_CWT
  return NF_EUNSUPPORTED;
}

template nf_status launch_conv_wave<bf16_t>(ConvWaveArgs<bf16_t>&, int, int, hipStream_t);
template nf_status launch_conv_wave<float>(ConvWaveArgs<float>&, int, int, hipStream_t);

template <typename T>
static int tile_of(int M, int B, int cig, int cog, int g, int H, int W, int stride, int pad) {
  ConvWaveArgs<T> a;
  memset(&a, 0, sizeof(a));
  const int Ho = (H + 2 * pad - 3) / stride + 1;
  a.cig = cig; a.cog = cog; a.g = g; a.nG = M * g; a.H = H; a.W = W; a.Wo = (W + 2 * pad - 3) / stride + 1;
  a.HoWo = Ho * a.Wo; a.stride = stride; a.pad = pad;
  const WaveChoice c = choose_wave(a, Ho, B);
  return 10 * c.kg + c.nb;
}

}  // namespace nf

// For the tests, which name the tile that a case is meant to run; not part of the interface.  10 x wavefronts + blocks of
// positions, 0 = another kernel.  Host only.
extern "C" int netfuse_conv_wave_tile(int f32, int M, int B, int cig, int cog, int g, int H, int W, int stride, int pad) {
  return f32 ? nf::tile_of<float>(M, B, cig, cog, g, H, W, stride, pad) : nf::tile_of<nf::bf16_t>(M, B, cig, cog, g, H, W, stride, pad);
}
