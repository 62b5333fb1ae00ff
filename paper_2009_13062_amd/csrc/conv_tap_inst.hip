// Instantiation and launch of the tap-major 3x3 convolution kernels (conv_tap.h, bf16).
#include <algorithm>
#include <atomic>
#include <cstdlib>

#include "conv_tap.h"
#include "gemm_launch.h"

namespace nf {

template <class Cfg, int VW, int NT, int KIND>
static nf_status launch_tap_kernel(long long total, int lds, const ConvTapArgs& a, hipStream_t s) {
  if constexpr (KIND == kTapRun && NT > 1)
    if (a.cig > kTapCB && a.run == 1) return launch_tap_kernel<Cfg, VW, NT, kTapTile>(total, lds, a, s);
  auto kern = conv_tap_kernel<Cfg, VW, NT, KIND>;
  if (lds > 64 * 1024) {
    static std::atomic<bool> opted_in{false};        // per kernel: idempotent, a benign race
    if (!opted_in.load(std::memory_order_acquire)) {
      if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                              160 * 1024) != hipSuccess)
        return NF_ELAUNCH;
      opted_in.store(true, std::memory_order_release);
    }
  }
  nf_launch(kern, dim3((unsigned)total), dim3(256), lds, s, a);
  return hipGetLastError() == hipSuccess ? NF_OK : NF_ELAUNCH;
}

static int fit_at_once(int lds, int most) { return std::max(1, std::min(160 * 1024 / 1280 / ((lds + 1279) / 1280), most)); }

int tile_run(long long groups, int tiles_n, int lds, int most, double alone, double start) {
  const int at_once = fit_at_once(lds, most);
  auto per_tile = [&](int run, long long j) { return start + run * std::max(alone, (double)j); };
  double best = 0;
  int pick = 1;
  for (int runs = 1, run; runs <= tiles_n; runs = run > 1 ? (tiles_n + run - 2) / (run - 1) : runs + 1) {
    run = (tiles_n + runs - 1) / runs;
    const long long wg = groups * runs, rounds = (wg - 1) / (256LL * at_once), rest = wg - rounds * 256 * at_once;
    const double t = rounds * per_tile(run, at_once) + per_tile(run, (rest + 255) / 256);
    if (runs == 1 || t <= best) { best = t; pick = run; }      // the shorter of two equals
  }
  return pick;
}

// Position tiles per workgroup (bm rows) of `groups` x tiles_n.
//   One block of 32 channels, whose weights stay in LDS: tile_run.  Over 4000 problems of 32 channels and of fused groups 0.1 % behind the
//   best run and 21 % less time than a tile per workgroup and an epilogue through LDS.
//   Two and three blocks: a run saves next to nothing of the start of a tile, and two workgroups that share a compute unit do not halve each
//   other's rate, so it pays only where it evens out the last round of one or two workgroups per compute unit.  Over 2000 problems 1.3 % ahead of
//   one tile each, 0.2 % behind the best run, 4 % slower at most (32 models, 64 channels at 56 x 56 22.4 us in tiles of their own, 20.2 in runs
//   of two; whole rounds as they are: 32 models, 8 images, 64 -> 128 at 28 x 28 58 us, 67 in runs of seven).
//   More: one tile.  The best run is 0.7 to 1.2 % ahead of it, and a wrong one far behind: 24 models, 256 channels at 20 x 20, 3 images 66 us in
//   tiles of their own, 108 in runs of two; 12 models of 256 at 64 x 64 80 and 99.
static int tap_run(int cig, int bm, long long groups, int tiles_n, int lds) {
  if (cig == kTapCB) return tile_run(groups, tiles_n, lds, 3);
  const int most = bm > 32 ? 2 : 3, at_once = fit_at_once(lds, most);
  if (cig > 3 * kTapCB || at_once > 2 || groups * tiles_n % (256 * at_once) == 0) return 1;
  return tile_run(groups, tiles_n, lds, most, 1.5, 0.1);
}

template <class Cfg, bool FUSED = false>
static nf_status launch_tap(const ConvPatchArgs& args, int B, hipStream_t s) {
  ConvTapArgs a;
  (ConvPatchArgs&)a = args;
  a.tiles_m = (a.cog + Cfg::kBM - 1) / Cfg::kBM;
  a.tiles_n = (a.HoWo + Cfg::kBN - 1) / Cfg::kBN;
  const long long groups = (long long)a.tiles_m * a.nG * B, tiles = groups * a.tiles_n;
  if (tiles <= 0 || tiles > 0x7fffffffLL || !cw_div_exact(a.HoWo, a.Wo)) return NF_EUNSUPPORTED;
  cw_divisor(a.Wo, &a.rcp_wo, &a.one_wo);
  a.PS = (a.PS + 7) / 8 * 8;
  // Pixels per chunk: the width with the fewest chunks per thread (a chunk is 8 loads and up to 32 staging registers),
  // the narrowest of those, which spreads the chunks over most threads.  Chunks start at any 2-byte address, so widths
  // need not be multiples of anything: 25 x 25 planes (12 groups of 128 channels) 47 -> 11.8 us and 13 x 13 -> 7 x 7
  // (512 channels) 189 -> 28.9 us against the implicit-GEMM kernel that took them when a chunk had to divide the width.
  int nt = 0;
  for (int vw = 8; vw >= 1; vw /= 2) {
    if (vw > a.W) continue;
    const int cpr = (a.W + vw - 1) / vw;
    const long long tasks = (long long)(kTapCB / 8) * (a.PS / a.PW) * cpr;     // patch tasks of the tallest tile
    const int n = (int)((tasks + 255) / 256);
    if (n <= (vw == 8 ? 2 : 3) && (nt == 0 || n <= nt)) { nt = n; a.VW = vw; a.cpr = cpr; }
  }
  const int lds = Cfg::lds_bytes(a.PS);
  if (lds > 160 * 1024) return NF_EUNSUPPORTED;
  a.run = tap_run(a.cig, Cfg::kBM, groups, a.tiles_n, lds);
  a.runs = (a.tiles_n + a.run - 1) / a.run;
  const long long total = groups * a.runs;
#define NF_TAP(VW_, NT_) return launch_tap_kernel<Cfg, VW_, NT_, FUSED ? kTapFused : kTapRun>(total, lds, a, s)
  if (nt > 0) switch (a.VW) {
    case 8: if (nt == 1) NF_TAP(8, 1); if (nt == 2) NF_TAP(8, 2); break;     // 32 staging registers per task
    case 4: if (nt == 1) NF_TAP(4, 1); if (nt == 2) NF_TAP(4, 2); if (nt == 3) NF_TAP(4, 3); break;
    case 2: if (nt == 1) NF_TAP(2, 1); if (nt == 2) NF_TAP(2, 2); if (nt == 3) NF_TAP(2, 3); break;
    case 1: if (nt == 1) NF_TAP(1, 1); if (nt == 2) NF_TAP(1, 2); if (nt == 3) NF_TAP(1, 3); break;
  }
#undef NF_TAP
  return NF_EUNSUPPORTED;
}

// 3x3, dilation 1, pad <= kLPad, (fused) groups of 32 k channels.  The caller has filled everything but the
// tiling.  NF_EUNSUPPORTED = take another kernel.
nf_status launch_conv_tap_3x3(ConvPatchArgs& a, int B, hipStream_t s) {
  if (a.cig % kTapCB != 0 || ((uintptr_t)a.x & 15) != 0) return NF_EUNSUPPORTED;
  if (a.S > 1) {
    // fused narrow groups: one 32-channel block, at most 32 rows; weight runs are read 16 or 8 bytes at a time
    if (a.cig != kTapCB || a.cog > 32 || a.cig_real * a.S != kTapCB || a.cog_real * a.S != a.cog) return NF_EUNSUPPORTED;
    if (((uintptr_t)a.w & (a.cig_real >= 8 ? 15 : 7)) != 0) return NF_EUNSUPPORTED;
    ConvPatchArgs f = a;
    if (a.stride == 1) {
      const int rows = a.PS / a.PW;
      f.PW = a.PW + ((a.Wo - a.PW) % 16 + 16) % 16;       // see below
      f.PS = rows * f.PW;
    }
    return launch_tap<ConvTapCfg<32, 1, 4, 2>, true>(f, B, s);
  }
  if (((uintptr_t)a.w & 15) != 0) return NF_EUNSUPPORTED;
  static const int forced_bm = [] { const char* e = dev_getenv("NETFUSE_TAP_BM"); return e ? atoi(e) : 0; }();
  const long long per_row_tile = (long long)((a.HoWo + 127) / 128) * a.nG * B;
  auto tiles = [&](int bm) { return per_row_tile * ((a.cog + bm - 1) / bm); };
  // measured on the 3x3 layers of ResNet-50 at 32 merged models: a taller row tile copies the input patch
  // less often, which pays from about 400 workgroups up; stride 2 (four times the patch per output) prefers
  // it earlier, unless most of the 128 positions of a tile are padding (7x7 outputs)
  int bm = 32;
  if (a.cog > 64 && a.stride > 1 && tiles(128) >= 200) bm = 128;
  else if (a.cog > 32 && (tiles(64) >= 400 || (a.stride > 1 && a.HoWo >= 128 && tiles(64) >= 256))) bm = 64;
  if (forced_bm == 32 || forced_bm == 64 || forced_bm == 128) bm = forced_bm;
  ConvPatchArgs c = a;                                  // the caller's copy stays intact for a fallback
  if (a.stride == 1) {
    // 16 consecutive lanes read 16 consecutive output positions; their pixels are consecutive within an
    // output row and PW - Wo + 1 apart across a row end.  With the 80-byte pixel pitch, 16 pixels whose
    // indices are distinct modulo 16 hit 16 distinct bank groups, so a row pitch congruent to Wo modulo
    // 16 keeps the reads conflict free across row ends (measured: a third of the LDS cycles on 14x14 images
    // were bank conflicts without it).
    const int rows = a.PS / a.PW;
    c.PW = a.PW + ((a.Wo - a.PW) % 16 + 16) % 16;
    c.PS = rows * c.PW;
  }
  // A patch that leaves no room for the weights of a tall tile runs in the next lower one, not in another kernel: the sum
  // has the same order in all three, and the number of models must not decide about it.
  nf_status st = NF_EUNSUPPORTED;
  if (bm == 128) st = launch_tap<ConvTapCfg<128, 2, 2, 1>>(c, B, s);
  if (st == NF_EUNSUPPORTED && bm >= 64) st = launch_tap<ConvTapCfg<64, 1, 4, 2>>(c, B, s);
  if (st == NF_EUNSUPPORTED) st = launch_tap<ConvTapCfg<32, 1, 4, 2>>(c, B, s);
  return st;
}

}  // namespace nf

// For the tests; not part of the interface.  Host only.
extern "C" int netfuse_div_exact(long long n, int d) { return nf::cw_div_exact(n, d); }
extern "C" int netfuse_conv_tap_run(int cig, int bm, long long groups, int tiles_n, int lds) { return nf::tap_run(cig, bm, groups, tiles_n, lds); }
