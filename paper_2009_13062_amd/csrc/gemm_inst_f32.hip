// Instantiation, tile choice and launch of the float32 matrix-pipe kernels (gemm_f32.h).
#include <atomic>

#include "gemm_f32.h"

namespace nf {

// 128-row tiles were tried as well and are never ahead (12 models, 512 x 3072 x 768: 377 us at 128 x 128, 308 at
// 128 x 64, 252 at 64 x 64): a compute unit with several tiles hides one workgroup's waits behind another's.
// CH chains (gemm_f32.h): 4 where dealing k out to four groups of wavefronts pays, else 2.  One model (us), 16-row tiles on
// two / four groups: 17 x 3072 x 768 23.6 / 22.0, 512 -> 512 at 7 x 7 62.2 / 52.0, 2048 -> 512 30.7 / 26.3, but 17 x 768 x 768
// 8.8 / 8.9 and 128 -> 128 at 28 x 28 (k = 1152) 20.1 / 19.8; four chains on one group cost it up to a tenth of its rate.
constexpr int kLongK = 1536;
template <int CH> using F64x64 = F32Cfg<64, 64, 2, 2, 32, 2, CH>;
template <int CH> using F64x64s = F32Cfg<64, 64, 2, 2, 32, 2, CH, 2>;
template <int CH> using F64x48s = F32Cfg<64, 48, 4, 1, 32, 2, CH, 2>;
template <int CH> using F32x64s = F32Cfg<32, 64, 2, 2, 32, 2, CH, 2>;
template <int CH> using F16x64s = F32Cfg<16, 64, 1, 4, 32, 2, CH, 2>;
using F32x64q = F32Cfg<32, 64, 2, 2, 32, 2, 4, 4>;
using F16x64q = F32Cfg<16, 64, 1, 4, 32, 2, 4, 4>;

enum { kF64x64, kF64x64s, kF64x48s, kF32x64s, kF32x64q, kF16x64s, kF16x64q, kNumF32Tiles };
constexpr int kBMs[kNumF32Tiles] = {64, 64, 64, 32, 32, 16, 16};
constexpr int kBNs[kNumF32Tiles] = {64, 64, 48, 64, 64, 64, 64};
constexpr int kGroups[kNumF32Tiles] = {1, 2, 2, 2, 4, 2, 4};
// Measured time per unit of tile area and k of the busiest compute unit, dense / gathered B, where a compute unit
// has one tile / several (then its workgroups fill each other's waits).  With one tile per unit the forms with k
// split over 2 or 4 groups of wavefronts are ahead of the plain ones (128 x 3072 x 768 at 8 models: 51 us against 64;
// 512 -> 512 at 7 x 7: 54 against 138); small tiles pay for gathering B once per row tile.
constexpr int kUnitCost[2][2][kNumF32Tiles] = {
    {{159, 142, 166, 170, 165, 176, 165}, {130, 142, 150, 143, 170, 176, 210}},
    {{220, 185, 0, 255, 230, 360, 320}, {173, 190, 0, 210, 250, 330, 340}}};

template <class Cfg, int KIND, bool AVEC>
static nf_status launch_kernel(GemmF32Args& a, long long total, hipStream_t s) {
  auto kern = gemm_f32_kernel<Cfg, KIND, AVEC>;
  if (Cfg::kLdsBytes > 64 * 1024) {
    static std::atomic<bool> opted_in{false};        // per kernel: idempotent, a benign race
    if (!opted_in.load(std::memory_order_acquire)) {
      if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                              Cfg::kLdsBytes) != hipSuccess)
        return NF_ELAUNCH;
      opted_in.store(true, std::memory_order_release);
    }
  }
  nf_launch(kern, dim3((unsigned)total), dim3(Cfg::kThreads), Cfg::kLdsBytes, s, a);
  return hipGetLastError() == hipSuccess ? NF_OK : NF_ELAUNCH;
}

template <class Cfg, int KIND>
static nf_status launch_cfg(GemmF32Args& a, long long problems, hipStream_t s) {
  a.tiles_m = (a.rows + Cfg::kBM - 1) / Cfg::kBM;
  a.tiles_n = (a.cols + Cfg::kBN - 1) / Cfg::kBN;
  const long long total = problems * a.tiles_m * a.tiles_n;
  if (total <= 0 || total > 0x7fffffffLL) return NF_EUNSUPPORTED;
  return a.K % 4 == 0 ? launch_kernel<Cfg, KIND, true>(a, total, s) : launch_kernel<Cfg, KIND, false>(a, total, s);
}

template <int CH>
static nf_status launch_tile(int tile, GemmF32Args& a, long long problems, bool gather, hipStream_t s) {
#define NF_F32(C) return gather ? launch_cfg<C, kF32Gather>(a, problems, s) : launch_cfg<C, kF32Dense>(a, problems, s)
  switch (tile) {
    case kF64x64: NF_F32(F64x64<CH>);
    case kF64x64s: NF_F32(F64x64s<CH>);
    case kF64x48s: return launch_cfg<F64x48s<CH>, kF32Dense>(a, problems, s);
    case kF32x64s: NF_F32(F32x64s<CH>);
    case kF16x64s: NF_F32(F16x64s<CH>);
  }
  if constexpr (CH == 4) {
    if (tile == kF32x64q) NF_F32(F32x64q);
    if (tile == kF16x64q) NF_F32(F16x64q);
  }
#undef NF_F32
  return NF_EUNSUPPORTED;
}

nf_status launch_gemm_f32(GemmF32Args& a, int nz1, bool gather, hipStream_t s) {
  const long long problems = (long long)a.nz0 * nz1;
  // a wide kernel over few channels (the image networks' stem)
  if (gather && a.khw > 31) return launch_cfg<F64x64<2>, kF32GatherWide>(a, problems, s);
  auto tiles = [&](int t) { return problems * ((a.rows + kBMs[t] - 1) / kBMs[t]) * ((a.cols + kBNs[t] - 1) / kBNs[t]); };
  const bool chains4 = a.K >= kLongK;
  int best = -1;
  long long best_cost = 0;
  for (int t = 0; t < kNumF32Tiles; ++t) {
    if (gather && t == kF64x48s) continue;
    if ((t == kF32x64q || t == kF16x64q) && !chains4) continue;
    const long long rounds = (tiles(t) + 255) / 256;
    // Up to 64 k a tile on one group walks 64 of them, one on two groups 128, half of them zeros; with several tiles per compute unit that is
    // time (us, without this factor / with it: 12 models of 1500 rows 50 -> 99 14.6 / 10.7, 18 of 1243 48 -> 258 31.9 / 19.7).  With one the two groups
    // are ahead all the same (5 x 3 images of 14 x 14, 31 -> 88 5.5 against 6.4), and with a few of 16 rows (7 x 2 of 30 x 30, 41 -> 34 7.1 against 7.7).
    const int walked = a.K <= 64 && kGroups[t] == 2 && rounds > (kBMs[t] == 16 ? 3 : 1) ? 2 : 1;
    const long long cost = rounds * kBMs[t] * kBNs[t] * kUnitCost[gather][rounds > 1][t] * walked;
    if (best < 0 || cost < best_cost) { best = t; best_cost = cost; }
  }
  return chains4 ? launch_tile<4>(best, a, problems, gather, s) : launch_tile<2>(best, a, problems, gather, s);
}

}  // namespace nf
