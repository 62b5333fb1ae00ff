// C ABI of the merged operators: argument validation on the host (before any HIP call), kernel
// selection by (storage type, shape class), launch with the model index folded into the grid.
#include <hip/hip_runtime.h>
#include <limits.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>

#include "../../include/netfuse.h"
#include "attention_f32.h"
#include "attention_kernels.h"
#include "conv_patch.h"
#include "conv_stem.h"
#include "conv_wave.h"
#include "gemm_launch.h"
#include "gemm_mfma.h"
#include "generic_kernels.h"
#include "nf_common.h"
#include "norm_kernels.h"
#include "probe_kernels.h"

using namespace nf;

namespace {

inline bool is_dtype(int dt) { return dt == NF_F32 || dt == NF_BF16; }
inline bool is_act(int a) { return a == NF_ACT_NONE || a == NF_ACT_RELU || a == NF_ACT_GELU; }
inline bool aligned(const void* p, size_t a) { return p == nullptr || ((uintptr_t)p % a) == 0; }

// product of non-negative ints, saturating at LLONG_MAX
inline long long prod(std::initializer_list<long long> v) {
  long long r = 1;
  for (long long x : v) {
    if (x < 0) return -1;
    if (x != 0 && r > LLONG_MAX / x) return LLONG_MAX;
    r *= x;
  }
  return r;
}
constexpr long long kMaxElems = (1LL << 62);     // element counts must stay below this
constexpr long long kMaxGrid = 0x7fffffffLL;

}  // namespace

namespace nf {
LaunchTiming& launch_timing() {
  static thread_local LaunchTiming t = {nullptr, nullptr};
  return t;
}
}  // namespace nf

namespace {

inline nf_status launched() { return hipGetLastError() == hipSuccess ? NF_OK : NF_ELAUNCH; }

inline unsigned grid_for(long long total, int per_block, long long cap = 1 << 20) {
  long long g = (total + per_block - 1) / per_block;
  if (g > cap) g = cap;
  if (g < 1) g = 1;
  return (unsigned)g;
}

nf_status launch_gemm_any(int bkind, int align_a, int tile, GemmLaunch& L, hipStream_t s) {
  switch (bkind) {
    case 8: return launch_gemm_bkind<8>(align_a, tile, L, s);
    case 24: return launch_gemm_bkind<24>(align_a, tile, L, s);
    case 22: return launch_gemm_bkind<22>(align_a, tile, L, s);
    case 21: return launch_gemm_bkind<21>(align_a, tile, L, s);
    case 27: return launch_gemm_bkind<27>(align_a, tile, L, s);
    case 2: return launch_gemm_bkind<2>(align_a, tile, L, s);
    case 1: return launch_gemm_bkind<1>(align_a, tile, L, s);
    case 0: return launch_gemm_bkind<0>(align_a, tile, L, s);
  }
  return NF_EUNSUPPORTED;
}

// Optional override for tile-shape sweeps: NETFUSE_TILE=<index into TileId>, read once.
int forced_tile() {
  static const int v = [] {
    const char* e = dev_getenv("NETFUSE_TILE");
    if (!e || !*e) return -1;
    const int t = atoi(e);
    return (t >= 0 && t < kNumTiles) ? t : -1;
  }();
  return v;
}

// Optional override for sweeps of the direct-to-LDS kernels: NETFUSE_DMA=<index into DmaTileId>, or -1
// to disable them.
int forced_dma() {
  static const int v = [] {
    const char* e = dev_getenv("NETFUSE_DMA");
    if (!e || !*e) return -2;
    const int t = atoi(e);
    return (t >= -1 && t < kNumDmaTiles) ? t : -2;
  }();
  return v;
}

// Direct-to-LDS kernel for a dense, fully aligned problem made of whole tiles, or -1.  With k a multiple of 64 from 256 up
// the ring tiles are compared with it and mostly taken (see netfuse_linear): there the 128 x 384 tile stays for full rounds of
// 128-row problems, the 128 x 288 tile for full rounds of 2304 columns; the others run for shorter and odd k.  *cost_out receives the
// cost of the choice in the model's unit (operand elements loaded by the busiest CU).
int pick_dma(int rows, int cols, int K, long long problems, long long* cost_out = nullptr) {
  const int f = forced_dma();
  if (f == -1) return -1;
  auto fits = [&](int t) { return rows % kDmaBM[t] == 0 && cols % kDmaBN[t] == 0 && K % kDmaBK[t] == 0; };
  if (f >= 0) return fits(f) ? f : -1;
  // Measured on MI355X: these kernels are bound by what ONE compute unit can pull through its vector
  // memory path (about 22 GB/s per CU at HBM latency, 3x that for L2 hits), not by the matrix pipe, so
  // the cost of a configuration is the operand bytes the busiest CU has to load: its share of the tiles
  // times (A tile + B tile).  Wide tiles re-read the activation rows less often; a tile count that is a
  // whole multiple of the 256 CUs leaves none of them idle.
  constexpr long long kCUs = 256;
  int best = -1;
  long long best_cost = 0;
  for (int t = 0; t < kNumDmaTiles; ++t) {
    if (!fits(t)) continue;
    if (t == D128x128k64s3w8 && !(rows == 128 && (K >= 2048 || fits(D128x384k32s4w12)))) continue;   // long-K / narrow layers only
    const long long tiles = problems * (rows / kDmaBM[t]) * (cols / kDmaBN[t]);
    const long long per_cu = (tiles + kCUs - 1) / kCUs;
    long long cost = per_cu * ((long long)kDmaBM[t] + kDmaBN[t]) * K;
    if (kDmaBK[t] == 64) cost -= cost / 16;               // whole 128-byte lines of A per k-step: slightly cheaper than k32
    if (best < 0 || cost < best_cost) { best = t; best_cost = cost; }
  }
  if (cost_out) *cost_out = best_cost;
  return best;
}

// pick_dma(), unless the register-staged 64x64 tile is expected to be faster (kPreferSmallTile).
// Few merged models leave most CUs without a whole-tile workgroup; the 64x64 register-staged tile
// with its deep load pipeline then spreads the operand stream over more of them.  Same cost model,
// with the measured handicap of that kernel per byte (encoder layer at 8 models: the K = 3072
// matmul 25.6 -> 14.6 us, the 768 x 768 one 12.6 -> 11.0 us; at 32 models nothing changes).
constexpr int kPreferSmallTile = -2;
int pick_dma_or_small(int N, int Nout, int K, long long M) {
  long long dma_cost = 0;
  const int d = pick_dma(N, Nout, K, M, &dma_cost);
  if (d < 0) return -1;
  const long long t64 = M * ((N + 63) / 64) * ((Nout + 63) / 64);
  const long long reg_cost = (t64 + 255) / 256 * 128 * K;
  if (forced_dma() == -2 && forced_tile() < 0 && K % 256 == 0 && reg_cost * 13 < dma_cost * 10) return kPreferSmallTile;
  return d;
}

// Streaming kernel (gemm_stream.h) for a problem that pick_dma() routed to direct-to-LDS tile d, or -1.
// Measured on MI355X, 32 models (us, register epilogue / LDS-staged epilogue of the same tile):
//   GELU epilogues, 128 rows: 768 -> 3072  37.8 / 39.4 (the only one of these that the ring tiles leave to it);
//   512 rows, three 256x256 tiles per workgroup through one pipeline: 105.6 / 119.1.  The barrier-free epilogue pays where the epilogue is VALU heavy; plain
//   bias / residual epilogues are as fast or faster through LDS (full-line stores), so they keep it --
//   except that 512-row problems whose 256x256 tiling leaves a quarter of the last round of workgroups
//   empty (768 -> 2304: 576 tiles) run as three 128x384 tiles per workgroup (82.7 / 88.4).
int pick_stream(int d, int N, int Nout, int K, long long M, int act, int* nsub) {
  *nsub = 1;
  if (d == D256x256k32s4) {
    const long long tiles = M * (N / 256) * (Nout / 256);
    if (act == NF_ACT_GELU) {
      if (tiles >= 3 * 256 && (Nout / 256) % 3 == 0) *nsub = 3;
      return S256x256k32;
    }
    if (tiles % 256 != 0 && N % 128 == 0 && Nout % 384 == 0 && (Nout / 384) % 3 == 0) {
      const long long t384 = M * (N / 128) * (Nout / 384);
      if (t384 % (3 * 256) == 0) { *nsub = 3; return S128x384k32; }
    }
    return -1;
  }
  if (d == D128x384k32s4w12 && act == NF_ACT_GELU) return S128x384k32;
  return -1;
}

// Developer override NETFUSE_STREAM="<StreamTileId>,<nsub>" (read at every call in builds with developer
// switches): force a streaming kernel and its number of column tiles per workgroup.
bool forced_stream(int* cfg, int* nsub) {
  const char* e = dev_getenv("NETFUSE_STREAM");
  if (!e || !*e) return false;
  return sscanf(e, "%d,%d", cfg, nsub) == 2 && *cfg >= 0 && *cfg < kNumStreamTiles && *nsub >= 1;
}

// Tile choice for the register-staged kernels.
int pick_tile(int rows, int cols, long long problems) {
  const int f = forced_tile();
  if (f >= 0) return f;
  auto tiles = [&](int t) {
    return problems * ((rows + kTileBM[t] - 1) / kTileBM[t]) * ((cols + kTileBN[t] - 1) / kTileBN[t]);
  };
  if (rows <= 32) return T32x128;
  // Measured over the pointwise layers of ResNet-50 / ResNeXt-50 at 16 and 32 merged models: the 8-wave
  // tile wins wherever it yields about a workgroup per CU (two when half of its columns are padding, as
  // on 7x7 images); below that, and for 64 rows, the 64x64 tile does.
  if (cols <= 64) return rows > 64 && tiles(T128x128w8) >= 512 ? T128x128w8 : T64x64;
  return rows > 64 && tiles(T128x128w8) >= 200 ? T128x128w8 : T64x64;
}

// Time model of the matmul kernels for choosing between them: 4 us of launch and ramp, plus per round of tiles over the
// 256 compute units b us per 768 of k and e us of prologue and epilogue.  Fitted to every kernel measured alone at
// hidden sizes 256, 768 and 1024 (the four matmuls of an encoder layer), 1 ... 32 models of 17 ... 1000 rows, weights
// cold: 252 row-major problems, mean error of a prediction 4 to 7 %.  (The whole-tile 128 x 288 kernel from full rounds at
// 768 and 1536 of k, 27 and 45 us: on 768 alone b came out too high and 1536 -> 2304 went to ring tiles that are a sixth slower.)
struct TileCost { int bm, bn; float b, e; };
float tile_us(const TileCost& t, int N, int Nout, int K, long long M) {
  const long long tiles = M * ((N + t.bm - 1) / t.bm) * ((Nout + t.bn - 1) / t.bn);
  return 4.0f + (float)((tiles + 255) / 256) * (t.b * (float)K / 768.0f + t.e);
}
constexpr TileCost kRegCost[kNumTiles] = {{64, 64, 3.77f, 0.48f}, {32, 128, 5.08f, 0.15f}, {128, 128, 6.69f, 3.04f}};
constexpr TileCost kDmaCost[kNumDmaTiles] = {{256, 256, 20.1f, 10.7f}, {128, 128, 9.4f, 4.3f}, {128, 128, 8.8f, 0.f},
                                             {128, 384, 13.8f, 18.1f}, {128, 288, 17.0f, 5.0f}, {128, 96, 8.0f, 2.0f}};
constexpr TileCost kRingCost[R256x256 + 1] = {{32, 32, 2.38f, 0.74f}, {64, 64, 3.61f, 0.43f}, {64, 128, 5.18f, 1.51f},
                                               {96, 128, 6.10f, 1.51f}, {96, 256, 9.95f, 2.07f}, {128, 128, 6.89f, 1.53f},
                                               {128, 256, 11.6f, 2.83f}, {128, 384, 16.2f, 4.24f}, {256, 256, 19.0f, 4.30f}};
// More than 128 rows, where row tiles share the weights: every ring tile, those between the powers of two too, by a model of its own.  Workgroups partly
// share a compute unit, so a us of launch, per 768 of k b us for every round begun and c us for every round's worth of tiles,
// e us of prologue and epilogue per round.  Fitted to every tile over 792 problems (an encoder layer's four matmuls at hidden
// sizes 256, 768 and 1024, 1 ... 32 models of 17 ... 1024 rows): mean error 5 to 10 %.  That error is a tenth of a tile, so the choice
// of the table above stands unless this model puts another tile kTallMargin below its own time for that choice: over 1632 problems
// of 129 ... 2048 rows 2.2 % off on average (24 models of 279 rows 4096 -> 1024 117 -> 74, 12 models 768 -> 2304 30.4 -> 22.6 us; 16 of 760
// rows 3072 -> 768 90 -> 61 us), one problem slower by 5 %; without the margin 1.9 %, and 55 slower by 4 to 20 % (32 models of 256
// rows 3072 -> 768 71 in place of 59 us).  Not at 256 of k, where a tile is over before its ring is full: 32 models of 384 rows
// 256 -> 768 took 12.8 to 17.3 us in 192 x 192 tiles, by where the operands lay, and 15.2 in 128 x 384.  With up to 128 rows the four
// tiles give nothing on average, and 16 models of 128 rows 1024 -> 3072 took 32 in place of 26 us.
constexpr float kTallMargin = 0.95f;
struct RingCost { int bm, bn; float a, b, e, c; };
float tile_us(const RingCost& t, int N, int Nout, int K, long long M) {
  const long long tiles = M * ((N + t.bm - 1) / t.bm) * ((Nout + t.bn - 1) / t.bn);
  const float n = (float)((tiles + 255) / 256), f = std::max(1.f, (float)tiles / 256), k = (float)K / 768.0f;
  return t.a + k * (t.b * n + t.c * f) + t.e * n;
}
constexpr RingCost kRingTallCost[kNumRingTiles] = {
    {32, 32, 4.05f, 1.45f, 0.61f, 1.26f},  {64, 64, 3.59f, 2.79f, 0.75f, 0.99f},  {64, 128, 1.27f, 3.79f, 3.81f, 1.48f},
    {96, 128, 1.47f, 4.92f, 3.95f, 0.98f}, {96, 256, 0.41f, 8.02f, 6.29f, 1.10f}, {128, 128, 1.03f, 5.24f, 4.74f, 1.22f},
    {128, 256, 0.f, 9.10f, 7.74f, 0.83f},  {128, 384, 0.f, 12.9f, 8.44f, 2.97f},  {256, 256, 0.f, 13.9f, 9.96f, 3.05f},
    {64, 256, 1.34f, 7.19f, 4.32f, 1.30f}, {160, 256, 0.f, 10.9f, 8.38f, 2.21f},  {192, 192, 0.f, 9.38f, 7.73f, 0.53f},
    {288, 128, 0.f, 8.98f, 7.48f, 1.08f}};
constexpr TileCost kRingPackedCost[kNumRingPackedTiles] = {{32, 32, 1.42f, 1.42f}, {64, 64, 3.35f, 1.60f}, {128, 64, 4.60f, 2.07f},
                                                           {128, 128, 7.14f, 2.69f}, {128, 256, 11.0f, 2.96f}, {256, 256, 18.6f, 4.12f}};

// The gemm_ring.h tile that is predicted to take less than `limit` us, or -1.
template <class Cost, int N_TILES>
int pick_ring(const Cost (&cost)[N_TILES], int N, int Nout, int K, long long M, float limit) {
  int best = -1;
  for (int t = 0; t < N_TILES; ++t) {
    const float us = tile_us(cost[t], N, Nout, K, M);
    if (us < limit) { best = t; limit = us; }
  }
  return best;
}

// The same for pointwise convolutions, whose k is short and whose planes may fill little of a tile: a + l us of latency per
// 64 of k, and per 256 tiles (padding included) b us per 64 of k and e us.  Fitted to every tile at planes of 2 x 4 to 72 x 72
// positions, 64 to 2048 channels, 1 to 256 images: 298 problems, mean error 7 to 11 %.
struct PointwiseCost { int bm, bn; float a, l, b, e; };
float pointwise_us(const PointwiseCost& t, int cog, int HoWo, int K, long long problems) {
  const long long tiles = problems * ((cog + t.bm - 1) / t.bm) * ((HoWo + t.bn - 1) / t.bn);
  const float k = (float)K / 64.0f;
  return t.a + t.l * k + (float)tiles / 256.0f * (t.b * k + t.e);
}
constexpr PointwiseCost kPointwiseCost[kNumRingConvTiles] = {{64, 64, 2.90f, 0.218f, 0.186f, 0.70f},
                                                             {64, 128, 3.12f, 0.273f, 0.255f, 1.40f},
                                                             {64, 256, 3.67f, 0.591f, 0.427f, 1.98f},
                                                             {128, 128, 3.41f, 0.486f, 0.458f, 1.94f},
                                                             {128, 256, 4.69f, 0.756f, 0.651f, 3.06f}};
constexpr PointwiseCost kPointwiseRegCost[2] = {{64, 64, 3.50f, 0.227f, 0.141f, 0.94f}, {128, 128, 3.25f, 0.315f, 0.518f, 2.46f}};

// The float32 matrix-pipe kernels address one problem's operands with 32-bit byte offsets.
bool f32_fits(long long a_elems, long long b_elems, int K) {
  return a_elems < (1LL << 29) && b_elems < (1LL << 29) && K < (1 << 24);
}
void f32_divisors(GemmF32Args& a) {
  auto rcp = [](int d, unsigned* r, unsigned* one) {
    *r = d == 1 ? 0u : (unsigned)(((1ULL << 32) + d - 1) / d);
    *one = d == 1 ? ~0u : 0u;
  };
  rcp(a.khw, &a.rcp_khw, &a.one_khw);
  rcp(a.KW, &a.rcp_kw, &a.one_kw);
}

// 3x3 through the wavefront-private pipelines of conv_wave.h, or NF_EUNSUPPORTED.
template <typename T>
nf_status conv_wave(const void* x, const void* w, const void* residual, void* y, const Epilogue& ep, int M, int B, int Cin, int Cout,
                    int g, int H, int W, int Ho, int Wo, int stride, int pad, hipStream_t s) {
  ConvWaveArgs<T> c;
  memset(&c, 0, sizeof(c));
  c.x = (const T*)x; c.w = (const T*)w; c.R = (const T*)residual; c.y = (T*)y;
  c.cig = Cin / g; c.cog = Cout / g; c.g = g; c.nG = M * g;
  c.H = H; c.W = W; c.Wo = Wo; c.HoWo = Ho * Wo; c.stride = stride; c.pad = pad;
  c.x_group = (long)c.cig * H * W; c.x_image = (long)M * Cin * H * W;
  c.y_group = (long)c.cog * c.HoWo; c.y_image = (long)M * Cout * c.HoWo;
  c.ep = ep;
  return launch_conv_wave(c, Ho, B, s);
}

// The register-staged tile of a convolution.  A gathered B operand (strided or k x k taps): its loads are the expensive part, so a few
// output positions are better served by tall tiles that gather them once per 128 output channels (measured).
int conv_reg_tile(int cog, int HoWo, long long problems, bool pointwise) {
  return !pointwise && forced_tile() < 0 && HoWo <= 64 && cog >= 256 ? (int)T128x128w8 : pick_tile(cog, HoWo, problems);
}

// Pointwise through the kernels of conv_plane.h where they are ahead of the register-staged tile `now`, or NF_EUNSUPPORTED.
nf_status conv_plane(const GemmLaunch& L, int H, int W, int Wo, int stride, int now, bool pairs, hipStream_t s) {
  GemmLaunch P = L;
  P.a.ldb = (long)H * W;
  P.a.geom.W = W; P.a.geom.Wo = Wo; P.a.geom.stride = stride;
  const int t = pick_conv_plane(P, now, pairs);
  return t < 0 ? NF_EUNSUPPORTED : launch_conv_plane(t, P, s);
}

// largest alignment (16, 8, 4 or 2 bytes) shared by a pointer and a row pitch / stride set
int common_align(std::initializer_list<const void*> ptrs, std::initializer_list<long long> elem_strides) {
  int al = 16;
  for (const void* p : ptrs)
    while (al > 2 && ((uintptr_t)p % al) != 0) al /= 2;
  for (long long st : elem_strides)
    while (al > 2 && ((st * 2) % al) != 0) al /= 2;
  return al;
}

}  // namespace

// ==========================================================================================
extern "C" {

nf_status netfuse_time_next_launch(void* start_event, void* stop_event) {
  LaunchTiming& t = launch_timing();
  t.start = (hipEvent_t)start_event;
  t.stop = (hipEvent_t)stop_event;
  return NF_OK;
}

nf_status netfuse_probe_mfma(void* sink, int iters, double* flops, void* stream) {
  if (!sink || iters <= 0 || !flops) return NF_EINVAL;
  if (!aligned(sink, 4)) return NF_EINVAL;
  const int wgs = 256;                                        // one workgroup of 16 wavefronts per compute unit
  *flops = (double)wgs * kProbeWaves * iters * 4 * kProbeFlopsPerMfma;
  nf_launch(probe_mfma_kernel, dim3(wgs), dim3(kProbeWaves * kWave), 0, (hipStream_t)stream, (float*)sink, iters, 0);
  return launched();
}

nf_status netfuse_probe_hbm_read(const void* src, long long bytes, void* sink, void* stream) {
  if (!src || !sink || bytes < 16 || bytes % 16) return NF_EINVAL;
  if (!aligned(src, 16) || !aligned(sink, 4)) return NF_EINVAL;
  const size_t chunks = (size_t)bytes / 16;
  const size_t per_wg = (size_t)256 * kProbeReadUnroll;
  size_t wgs = (chunks + per_wg - 1) / per_wg;
  if (wgs > 256 * 8) wgs = 256 * 8;                           // eight workgroups per compute unit, grid-stride beyond
  nf_launch(probe_hbm_read_kernel, dim3((unsigned)wgs), dim3(256), 0, (hipStream_t)stream, (const uint4*)src, chunks,
            (uint32_t*)sink, 0);
  return launched();
}

const char* netfuse_strerror(nf_status st) {
  switch (st) {
    case NF_OK: return "ok";
    case NF_EINVAL: return "invalid argument";
    case NF_EUNSUPPORTED: return "no kernel for these arguments";
    case NF_ELAUNCH: return "HIP launch failed";
  }
  return "unknown status";
}

nf_status netfuse_linear(const void* X, const void* W, const float* bias, const void* residual, void* Y,
                         int M, int N, int K, int Nout, nf_dtype dt, nf_act act, void* stream) {
  if (!X || !W || !Y) return NF_EINVAL;
  if (M <= 0 || N <= 0 || K <= 0 || Nout <= 0) return NF_EINVAL;
  if (!is_dtype(dt) || !is_act(act)) return NF_EINVAL;
  if (prod({M, N, K}) >= kMaxElems || prod({M, K, Nout}) >= kMaxElems || prod({M, N, Nout}) >= kMaxElems)
    return NF_EINVAL;
  const size_t esz = dt == NF_F32 ? 4 : 2;
  if (!aligned(X, esz) || !aligned(W, esz) || !aligned(Y, esz) || !aligned(residual, esz) || !aligned(bias, 4))
    return NF_EINVAL;
  hipStream_t s = (hipStream_t)stream;

  if (dt == NF_BF16) {
    const int al_a = common_align({X}, {K, (long long)N * K});
    const int al_b = common_align({W}, {Nout, (long long)K * Nout});
    // vector width of the B loader: its chunks must not straddle the end of a row
    int bkind = 1;
    if (al_b == 16 && Nout % 8 == 0) bkind = 8;
    int al = al_a;
    while (al > 2 && (K % (al / 2)) != 0) al /= 2;
    GemmLaunch L;
    memset(&L, 0, sizeof(L));
    GemmArgs& a = L.a;
    a.A = (const bf16_t*)X; a.B = (const bf16_t*)W; a.R = (const bf16_t*)residual; a.C = (bf16_t*)Y;
    a.B_end = a.B + (long long)M * K * Nout;
    a.lda = K; a.ldb = Nout; a.ldc = Nout;
    a.sA0 = (long)N * K; a.sB0 = (long)K * Nout; a.sC0 = (long)N * Nout;
    a.rows = N; a.cols = Nout; a.K = K; a.nz0 = M;
    L.nz1 = 1;
    a.ep.col_bias = bias; a.ep.col_vec_stride0 = Nout;
    a.ep.act = act; a.ep.act_before_residual = 1;
    a.ep.vec_store = Nout % 8 == 0 && aligned(Y, 16) && aligned(residual, 16)  ? 2
                     : Nout % 4 == 0 && aligned(Y, 8) && aligned(residual, 8) ? 1 : 0;
    if (bkind == 8 && al == 16) {
      int scfg, snsub;
      if (forced_stream(&scfg, &snsub)) {
        const nf_status st = launch_gemm_stream(scfg, snsub, L, s);
        if (st != NF_EUNSUPPORTED) return st;
      }
      const int d = pick_dma_or_small(N, Nout, K, M);
      if (forced_dma() == -2 && forced_tile() < 0 && ring_fits(Nout, K)) {
        // gemm_ring.h where its tiles are predicted to be faster, by more than the prediction is worth where a whole-tile
        // kernel is the alternative (a streaming kernel, 4 to 12 % faster, is priced as the whole-tile kernel of its tile).
        // Over the 252 problems this takes 11 % off on average, most for ragged rows: 12 models of 279 rows 31.9 -> 25.1
        // (768 -> 2304), 42.5 -> 33.7 (3072), 14.1 -> 12.2 (768), 36.0 -> 30.7 us (3072 -> 768); 1 model of 93 rows 3072 -> 768
        // 20 -> 16.1 us.
        const float now = tile_us(d >= 0 ? kDmaCost[d] : kRegCost[d == kPreferSmallTile ? T64x64 : pick_tile(N, Nout, M)], N, Nout, K, M);
        // With one row tile nothing shares the weights of a 128 x 384 tile, whole-tile or ring, and the model, fitted to both,
        // is too low for the ring one: 24, 32 and 48 models of 128 rows 768 -> 3072 32.2, 35.0, 59.4 us as before, 34.0, 36.5, 61.3 there.
        const float margin = d < 0 ? 1.0f : N == 128 && kDmaBN[d] == 384 ? 0.65f : 0.93f;
        int r = pick_ring(kRingCost, N, Nout, K, M, margin * now);
        if (N > 128 && K >= 512) {
          const int tall = pick_ring(kRingTallCost, N, Nout, K, M, r < 0 ? margin * now : kTallMargin * tile_us(kRingTallCost[r], N, Nout, K, M));
          if (tall >= 0) r = tall;
        }
        if (r >= 0) {
          const nf_status st = launch_gemm_ring(r, false, L, s);
          if (st != NF_EUNSUPPORTED) return st;
        }
      }
      if (d == kPreferSmallTile) return launch_gemm_any(bkind, al, T64x64, L, s);
      if (d >= 0) {
        const int sc = pick_stream(d, N, Nout, K, M, act, &snsub);
        if (sc >= 0) {
          const nf_status st = launch_gemm_stream(sc, snsub, L, s);
          if (st != NF_EUNSUPPORTED) return st;
        }
        return launch_gemm_dma(d, L, s);
      }
    }
    return launch_gemm_any(bkind, al, pick_tile(N, Nout, M), L, s);
  }
  // A few k over thousands of rows is mostly the matrix kernel's fixed cost per tile (8 models of 8192 rows, FMA / matrix kernel, us:
  // 2 -> 1 5.7 / 12.6, 16 -> 64 12.7 / 13.4, 32 -> 257 51 / 65); at 128 rows the matrix kernel is ahead (16 -> 16 7.8 / 4.3).
  if (!(K <= 32 && N >= 2048) && f32_fits(prod({N, K}), prod({K, Nout}), K)) {
    GemmF32Args a;
    memset(&a, 0, sizeof(a));
    a.A = (const float*)X; a.B = (const float*)W; a.R = (const float*)residual; a.C = (float*)Y;
    a.lda = K; a.ldb = Nout; a.ldc = Nout;
    a.sA0 = (long)N * K; a.sB0 = (long)K * Nout; a.sC0 = (long)N * Nout;
    a.a_bytes = (unsigned)(a.sA0 * 4); a.b_bytes = (unsigned)(a.sB0 * 4);
    a.rows = N; a.cols = Nout; a.K = K; a.nz0 = M;
    a.ep.col_bias = bias; a.ep.col_vec_stride0 = Nout;
    a.ep.act = act; a.ep.act_before_residual = 1;
    nf_status st = launch_gemm_split(a, s);
    if (st != NF_EUNSUPPORTED) return st;
    st = launch_gemm_f32(a, 1, false, s);
    if (st != NF_EUNSUPPORTED) return st;
  }
  const int tiles_m = (N + 63) / 64, tiles_n = (Nout + 63) / 64;
  const long long total = prod({tiles_m, tiles_n, M});
  if (total > kMaxGrid) return NF_EUNSUPPORTED;
  nf_launch(linear_generic_kernel<float>, dim3((unsigned)total), dim3(256), 0, s, (const float*)X,
                     (const float*)W, bias, (const float*)residual, (float*)Y, N, K, Nout, (int)act, tiles_m,
                     tiles_n);
  return launched();
}

// The fragment-packed kernel for (N, K, Nout) at M models: the tile width that needs the fewest rounds of
// workgroups over the 256 compute units, weighted by its width (a round streams width x K weights per unit);
// ties go to the wider tile.  -1 if no tile fits.
#ifndef NF_FRAG_HALF_TILES
#define NF_FRAG_HALF_TILES 1
#endif
static int pick_frag(int N, int Nout, int K, int M) {
  static const int forced = [] { const char* e = dev_getenv("NETFUSE_FRAG"); return e ? atoi(e) : -1; }();
  auto fits = [&](int t) { return N % kFragBM[t] == 0 && Nout % kFragBN[t] == 0 && K % kFragKUnit[t] == 0; };
  if (forced >= 0 && forced < kNumFragTiles && fits(forced)) return forced;
  auto tiles_of = [&](int t) { return (long long)M * (N / kFragBM[t]) * (Nout / kFragBN[t]); };
  auto best_of = [&](int lo, int hi) {
    int best = -1;
    long long best_cost = 0;
    for (int t = lo; t < hi; ++t) {
      if (!fits(t)) continue;
      const long long cost = (tiles_of(t) + 255) / 256 * kFragBN[t];
      if (best < 0 || cost < best_cost || (cost == best_cost && kFragBN[t] > kFragBN[best])) { best = t; best_cost = cost; }
    }
    return best;
  };
  // the 12- and 9-wavefront tiles wherever one of them divides the width, else the 128 / 256 column ones
  int pick = best_of(0, kNumFragMainTiles);
  if (pick < 0) pick = best_of(kNumFragMainTiles, kNumFragFullTiles);
  // With fewer models the 128-row tiles leave compute units idle or need a second, half empty round.  The
  // 64-row form of a width doubles the workgroups; the two row tiles of a column tile run side by side and share
  // its weights through L2, so a compute unit's weight stream costs about half as much as one of its own
  // (factor 0.45).  Only where that gives one round of more than 128 workgroups.  Measured at 16 models and 128
  // rows (us): 3072 -> 768 32.7 -> 24.5, 768 -> 768 12.8 -> 10.0 (96 columns), 768 -> 2304 24.4 -> 18.4 (288 against 96),
  // 768 -> 3072 29.2 -> 23.2 (384 against 96); forward 1.38 -> 1.15 ms.  At 8 models they lose against what runs now.
  if (NF_FRAG_HALF_TILES) {
    long long best_cost = pick < 0 ? -1 : 100 * ((tiles_of(pick) + 255) / 256 * kFragBN[pick]);
    for (int t = kNumFragFullTiles; t < kNumFragTiles; ++t) {
      if (!fits(t) || tiles_of(t) <= 128 || tiles_of(t) > 256) continue;
      const long long cost = 45LL * kFragBN[t];
      if (best_cost < 0 || cost < best_cost) { pick = t; best_cost = cost; }
    }
  }
  return pick;
}

// The 256 x 256 streaming kernel on packed weights (several column tiles per workgroup through one pipeline; gemm_stream.h).  It takes the
// shapes the 128-row fragment kernel has no tile for (output widths that are multiples of 256 but not of 96, 288 or 384, k that is no
// multiple of 128).  `preferred`: 256 x 256 tiles measured faster than the fragment kernel's, with a GELU epilogue and at least three of
// them per compute unit (without the GELU the fragment kernel is ahead: 75 against 88, 82 against 98, 32 against 39 us on the other
// three encoder shapes); for long k it is then gemm_ring.h's tile that runs (gelu_ring).  Returns the number of
// column tiles per workgroup, 0 = not applicable.
static int pick_packed_stream(int N, int Nout, int K, int M, int act, bool* preferred) {
  *preferred = false;
  if (N % 256 || Nout % 256 || K % 32) return 0;
  const int tn = Nout / 256;
  const long long tiles = (long long)M * (N / 256) * tn;
  // tiles a compute unit works through one after the other = rounds of workgroups x tiles per workgroup;
  // ties go to more tiles per workgroup (one launch ramp, epilogues under the next tile's loads)
  int best = 1;
  long long best_cost = 0;
  for (int n = 1; n <= tn; ++n) {
    if (tn % n) continue;
    const long long cost = ((tiles / n + 255) / 256) * n;
    if (n == 1 || cost <= best_cost) { best = n; best_cost = cost; }
  }
  *preferred = act == NF_ACT_GELU && tiles >= 3 * 256;
  return best;
}

// The 256 x 256 tile of gemm_ring.h (64 k per barrier) in the place of the streaming one (32), packed weights, GELU, three tiles per compute
// unit and more: from 512 of k up.  us: 32 models of 512 rows 768 -> 3072 106.3 -> 101.6, 1536 -> 3072 184 -> 168, 3072 -> 3072 327 -> 297;
// 64 of 256 rows 125 -> 111; 20 of 512 rows 4096 -> 5120 482 -> 445; 1 of 16384 rows 1024 -> 4096 173 -> 168.  Over 400 problems from 512
// up 10 % less time, 2 % more at most; over 340 from 256 to 448 3 % less and 8 % more at most, so these stay.
// Where a model has 2048 rows or more whose outputs lie a multiple of 4 KB apart, the ring tile's stores fall behind (8 models of 4096 rows
// 320 -> 2048 90 us streaming, 118; 768 -> 2048 135 and 169; 1024 of k 2 % less on average, 4 % more at most): from 1536 of k.
static bool gelu_ring(int N, int K, int Nout) { return K >= (N >= 2048 && Nout % 2048 == 0 ? 1536 : 512) && ring_fits(Nout, K); }

// For the tests; not part of the interface.  Host only.
int netfuse_packed_gelu_ring(int N, int K, int Nout) { return gelu_ring(N, K, Nout); }

int netfuse_linear_packed_supported(int M, int N, int K, int Nout, nf_dtype dt) {
  if (dt != NF_BF16 || M <= 0 || N <= 0 || K <= 0 || Nout <= 0) return 0;
  bool pref;
  const int f = pick_frag(N, Nout, K, M);
  if (f < 0) return pick_packed_stream(N, Nout, K, M, NF_ACT_NONE, &pref) > 0 ? 1 : 0;
  // With few models the fragment kernel's tiles leave most compute units idle.  netfuse_linear_packed then runs the tiles of gemm_ring.h that
  // split k over the wavefronts of a workgroup, which the row-major ones, one chain of k each, cannot: ahead where 32 x 32 tiles are
  // one round of workgroups (2 models of 128 rows 768 -> 768 7.0 -> 5.0 us, 3072 -> 768 15.8 -> 9.5, 4096 -> 1024 21.7 -> 12.0; 8 of 128 rows 256 -> 256
  // 4.4 -> 3.9; never behind over 40 such problems of hidden size 256 to 1024) and for long k over few rows (3 models of 128 rows 3072 -> 768 19.1
  // -> 16.6, 4096 -> 1024 25.7 -> 21.2; 8 to 21 % ahead over 18 problems of up to 768 rows in all).  Otherwise the answer is "no" below half a
  // workgroup per compute unit (3 models 768 -> 768 7.6 row-major against 7.7; one layer at 8 models 0.088 ms packed throughout, 0.074), although
  // netfuse_linear_packed itself still runs there and would be 7 to 17 % ahead for long k over more rows (8 models 3072 -> 768 19.7 row-major, 18.4; 12
  // models 4096 -> 1024 35.5 and 29.5).  The line at 128 tiles is older than the row-major ring tiles: of 480 problems answered "yes" they are
  // more than 5 % ahead for 129 (12 models of 384 rows 3072 -> 768 37.8 against 58.0 packed).
  const long long tiles = (long long)M * (N / kFragBM[f]) * (Nout / kFragBN[f]);
  if (tiles >= 128) return 1;
  return f < kNumFragFullTiles && ring_fits(Nout, K) && ((long long)M * (N / 32) * (Nout / 32) <= 256 || (K >= 2048 && (long long)M * N <= 768)) ? 1 : 0;
}

nf_status netfuse_linear_pack_weight(const void* W, void* Wp, int M, int K, int Nout, nf_dtype dt, void* stream) {
  if (!W || !Wp || W == Wp) return NF_EINVAL;
  if (M <= 0 || K <= 0 || Nout <= 0 || !is_dtype(dt)) return NF_EINVAL;
  if (K % 16 != 0 || Nout % 32 != 0) return NF_EINVAL;
  const long long total = prod({M, K, Nout});
  if (total >= kMaxElems) return NF_EINVAL;
  if (dt != NF_BF16) return NF_EUNSUPPORTED;
  if (!aligned(W, 2) || !aligned(Wp, 16)) return NF_EINVAL;
  return launch_pack_fragments((const bf16_t*)W, (bf16_t*)Wp, M, K, Nout, (hipStream_t)stream);
}

nf_status netfuse_linear_packed(const void* X, const void* Wp, const float* bias, const void* residual, void* Y,
                                int M, int N, int K, int Nout, nf_dtype dt, nf_act act, void* stream) {
  if (!X || !Wp || !Y) return NF_EINVAL;
  if (M <= 0 || N <= 0 || K <= 0 || Nout <= 0) return NF_EINVAL;
  if (!is_dtype(dt) || !is_act(act)) return NF_EINVAL;
  if (K % 16 != 0 || Nout % 32 != 0) return NF_EINVAL;
  if (prod({M, N, K}) >= kMaxElems || prod({M, K, Nout}) >= kMaxElems || prod({M, N, Nout}) >= kMaxElems)
    return NF_EINVAL;
  if (dt != NF_BF16) return NF_EUNSUPPORTED;
  if (!aligned(X, 2) || !aligned(Wp, 16) || !aligned(Y, 2) || !aligned(residual, 2) || !aligned(bias, 4))
    return NF_EINVAL;
  const int f = pick_frag(N, Nout, K, M);
  bool ps_preferred;
  const int ps = pick_packed_stream(N, Nout, K, M, act, &ps_preferred);
  if (f < 0 && ps <= 0) return NF_EUNSUPPORTED;
  GemmLaunch L;
  memset(&L, 0, sizeof(L));
  GemmArgs& a = L.a;
  a.A = (const bf16_t*)X; a.B = (const bf16_t*)Wp; a.R = (const bf16_t*)residual; a.C = (bf16_t*)Y;
  a.B_end = a.B + (long long)M * K * Nout;
  a.lda = K; a.ldb = 0; a.ldc = Nout;
  a.sA0 = (long)N * K; a.sB0 = (long)K * Nout; a.sC0 = (long)N * Nout;
  a.rows = N; a.cols = Nout; a.K = K; a.nz0 = M;
  L.nz1 = 1;
  a.ep.col_bias = bias; a.ep.col_vec_stride0 = Nout;
  a.ep.act = act; a.ep.act_before_residual = 1;
  if (ps > 0 && (ps_preferred || f < 0)) {
    if (ps_preferred && gelu_ring(N, K, Nout)) {
      const nf_status st = launch_gemm_ring(RP256x256, true, L, (hipStream_t)stream);
      if (st != NF_EUNSUPPORTED) return st;
    }
    a.ep.vec_store = 2;
    const nf_status st = launch_gemm_stream_packed(ps, L, (hipStream_t)stream);
    if (st != NF_EUNSUPPORTED || f < 0) return st;
  }
  // gemm_ring.h where its tiles are faster: few models (no tile of the fragment kernel fills the chip: 2 models of 128
  // rows 11.9 -> 5.6 us at 768 -> 768, 28.7 -> 10 us at 3072 -> 768), and widths that only the 128- and 256-column
  // tiles divide (hidden size 1024: 16 models of 128 rows 52.6 -> 30.2 us at 4096 -> 1024, 32 of 512 155.8 -> 121.7 us).
  // The 64-row tiles of the fragment kernel are ahead wherever they are chosen.
  if (f < kNumFragFullTiles && ring_fits(Nout, K)) {
    constexpr TileCost kFragCost[kNumFragFullTiles] = {{128, 96, 5.40f, 2.65f}, {128, 288, 16.2f, 0.f}, {128, 384, 16.7f, 2.44f},
                                                       {128, 128, 7.85f, 1.69f}, {128, 256, 11.8f, 2.52f}};
    const int r = pick_ring(kRingPackedCost, N, Nout, K, M, 0.93f * tile_us(kFragCost[f], N, Nout, K, M));
    if (r >= 0) {
      const nf_status st = launch_gemm_ring(r, true, L, (hipStream_t)stream);
      if (st != NF_EUNSUPPORTED) return st;
    }
  }
  return launch_gemm_frag(f, L, (hipStream_t)stream);
}

nf_status netfuse_linear_ragged(const void* X, const void* W, const float* bias, void* Y, int M, int N, int K,
                                const int* nout, nf_dtype dt, nf_act act, void* stream) {
  if (!X || !W || !Y || !nout) return NF_EINVAL;
  if (M <= 0 || N <= 0 || K <= 0) return NF_EINVAL;
  if (!is_dtype(dt) || !is_act(act)) return NF_EINVAL;
  const size_t esz = dt == NF_F32 ? 4 : 2;
  if (!aligned(X, esz) || !aligned(W, esz) || !aligned(Y, esz) || !aligned(bias, 4)) return NF_EINVAL;
  if (prod({M, N, K}) >= kMaxElems) return NF_EINVAL;
  // rows per workgroup: as many as there are, up to 8
  const int R = N >= 5 ? 8 : N >= 3 ? 4 : N;
  long long cols = 0, tiles = 0;
  for (int m = 0; m < M; ++m) {
    if (nout[m] <= 0) return NF_EINVAL;
    cols += nout[m];
    tiles += (long long)((N + R - 1) / R) * ((nout[m] + 63) / 64);
    if (cols > INT_MAX || tiles > kMaxGrid) return NF_EINVAL;
  }
  if (prod({cols, K}) >= kMaxElems || prod({cols, N}) >= kMaxElems) return NF_EINVAL;
  if (M > kRaggedMaxModels) return NF_EUNSUPPORTED;
  RaggedTable tab;
  tab.tile_start[0] = 0; tab.col_start[0] = 0;
  for (int m = 0; m < M; ++m) {
    tab.tile_start[m + 1] = tab.tile_start[m] + ((N + R - 1) / R) * ((nout[m] + 63) / 64);
    tab.col_start[m + 1] = tab.col_start[m] + nout[m];
  }
  for (int m = M + 1; m <= kRaggedMaxModels; ++m) { tab.tile_start[m] = tab.tile_start[M]; tab.col_start[m] = tab.col_start[M]; }
  hipStream_t s = (hipStream_t)stream;
  // 16 wavefronts share k where a model's rows leave compute units idle, 4 where there are plenty of workgroups or too little
  // k to share.  bf16, 4 models x 4096 rows (us, 4 / 16 wavefronts): 8 -> 1000 72 / 250, 128 -> 256 80 / 130, 768 -> 2 14 / 46; 8
  // models x 64 rows: 64 -> 64 and 256 -> 64 a quarter and two thirds slower with 4.
  const bool wide = K > 32 && N < 1024;
#define NF_RAGGED(T, R_, NW)                                                                                         \
  nf_launch((linear_ragged_kernel<T, R_, NW>), dim3((unsigned)tiles), dim3(NW * kWave), 0, s, (const T*)X, (const T*)W, \
            bias, (T*)Y, M, N, K, (int)act, tab)
#define NF_RAGGED_W(T, R_) if (wide) NF_RAGGED(T, R_, 16); else NF_RAGGED(T, R_, 4)
#define NF_RAGGED_R(T) \
  if (R == 1) { NF_RAGGED_W(T, 1); } else if (R == 2) { NF_RAGGED_W(T, 2); } else if (R == 4) { NF_RAGGED_W(T, 4); } else { NF_RAGGED_W(T, 8); }
  if (dt == NF_F32) { NF_RAGGED_R(float) } else { NF_RAGGED_R(bf16_t) }
#undef NF_RAGGED_W
#undef NF_RAGGED_R
#undef NF_RAGGED
  return launched();
}

nf_status netfuse_conv2d(const void* x, const void* w, const float* bias, const float* scale, const float* shift,
                         const void* residual, void* y, int M, int B, int Cin, int Cout, int g, int H, int W,
                         int KH, int KW, int stride, int pad, int dilation, nf_dtype dt, nf_act act,
                         void* stream) {
  if (!x || !w || !y) return NF_EINVAL;
  if (M <= 0 || B <= 0 || Cin <= 0 || Cout <= 0 || g <= 0 || H <= 0 || W <= 0 || KH <= 0 || KW <= 0)
    return NF_EINVAL;
  if (stride <= 0 || pad < 0 || dilation <= 0) return NF_EINVAL;
  if (Cin % g != 0 || Cout % g != 0) return NF_EINVAL;
  if ((scale == nullptr) != (shift == nullptr)) return NF_EINVAL;
  if (!is_dtype(dt) || !is_act(act)) return NF_EINVAL;
  const long long eh = (long long)H + 2LL * pad - (long long)dilation * (KH - 1) - 1;
  const long long ew = (long long)W + 2LL * pad - (long long)dilation * (KW - 1) - 1;
  if (eh < 0 || ew < 0) return NF_EINVAL;
  const long long Ho = eh / stride + 1, Wo = ew / stride + 1;
  const int cig = Cin / g, cog = Cout / g;
  const long long Ctot_in = (long long)M * Cin, Ctot_out = (long long)M * Cout;
  if (Ctot_in > INT_MAX || Ctot_out > INT_MAX || Ho * Wo > INT_MAX || (long long)H * W > INT_MAX ||
      prod({cig, KH, KW}) > INT_MAX || (long long)H + 2LL * pad > INT_MAX || (long long)W + 2LL * pad > INT_MAX)
    return NF_EINVAL;
  const long long n_in = prod({B, Ctot_in, H, W}), n_out = prod({B, Ctot_out, Ho, Wo});
  const long long n_w = prod({Ctot_out, cig, KH, KW});
  if (n_in >= kMaxElems || n_out >= kMaxElems || n_w >= kMaxElems) return NF_EINVAL;
  const size_t esz = dt == NF_F32 ? 4 : 2;
  if (!aligned(x, esz) || !aligned(w, esz) || !aligned(y, esz) || !aligned(residual, esz) || !aligned(bias, 4) ||
      !aligned(scale, 4) || !aligned(shift, 4))
    return NF_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  const int HoWo = (int)(Ho * Wo);
  const int Kdim = cig * KH * KW;

  static const bool no_mfma_conv = dev_getenv("NETFUSE_CONV_GENERIC") != nullptr;
  if (dt == NF_BF16 && !no_mfma_conv) {
    GemmLaunch L;
    memset(&L, 0, sizeof(L));
    GemmArgs& a = L.a;
    a.A = (const bf16_t*)w; a.B = (const bf16_t*)x; a.R = (const bf16_t*)residual; a.C = (bf16_t*)y;
    a.B_end = a.B + (long long)B * Ctot_in * H * W;
    a.lda = Kdim; a.ldc = HoWo;
    a.sA0 = (long)cog * Kdim; a.sA1 = 0;
    a.sB0 = (long)cig * H * W; a.sB1 = (long)Ctot_in * H * W;
    a.sC0 = (long)cog * HoWo; a.sC1 = (long)Ctot_out * HoWo;
    a.rows = cog; a.cols = HoWo; a.K = Kdim; a.nz0 = M * g;
    L.nz1 = B;
    L.weights_are_a = 1;
    a.ep.row_bias = bias; a.ep.row_scale = scale; a.ep.row_shift = shift;
    a.ep.row_vec_stride0 = cog; a.ep.row_vec_stride1 = 0;
    a.ep.act = act; a.ep.act_before_residual = 0;
    a.ep.vec_store = HoWo % 8 == 0 && aligned(y, 16) && aligned(residual, 16)  ? 2
                     : HoWo % 4 == 0 && aligned(y, 8) && aligned(residual, 8) ? 1
                     : HoWo <= 64 && ((long long)cog * HoWo) % 8 == 0 && aligned(y, 16) && aligned(residual, 16) ? 3 : 0;
    int al = common_align({w}, {Kdim});
    while (al > 2 && (Kdim % (al / 2)) != 0) al /= 2;
    const long long problems = (long long)M * g * B;
    const bool pointwise = KH == 1 && KW == 1 && stride == 1 && pad == 0;
    int tile = conv_reg_tile(cog, HoWo, problems, pointwise);
    if (pointwise) {
      // a 1x1 convolution is a matrix product over the channel dimension with the H*W positions as
      // columns (the converse of Section 3.1's remark that a matmul is a 1x1 convolution)
      a.ldb = (long)H * W;
      const int al_b = common_align({x}, {(long long)H * W});
      int bkind = 1;
      if (al_b == 16 && HoWo % 8 == 0) bkind = 8;
      if (bkind == 8 && al == 16 && cog > 32 && Kdim % 64 == 0 && forced_tile() < 0) {
        // gemm_ring.h with the widest tile that still gives 400 workgroups (two or three run on a compute unit).  Measured
        // against the register-staged tiles (us): 32 models 64 -> 64 at 56 x 56 11.8 -> 8.4, 64 -> 256 23.9 -> 19.2,
        // 128 -> 512 at 28 x 28 16.2 -> 13.7, 512 -> 128 11.3 -> 10.0; 2 models 512 -> 128 6.5 -> 5.8; 4 models of 4 images
        // 512 -> 2048 at 8 x 8 11.1 -> 9.5.
        auto tiles = [&](int bm, int bn) { return problems * ((cog + bm - 1) / bm) * ((HoWo + bn - 1) / bn); };
        auto us = [&](const PointwiseCost& c) { return pointwise_us(c, cog, HoWo, Kdim, problems); };
        int t = RC64x64;
        if (cog >= 128 && tiles(128, 256) >= 400) t = RC128x256;
        else if (cog >= 128 && tiles(128, 128) >= 400) t = RC128x128;
        else if (cog < 128 && tiles(64, 256) >= 400) t = RC64x256;
        else if (HoWo > 64 && tiles(64, 128) >= 200) t = RC64x128;
        // Such a tile may be mostly padding: 512 -> 2048 at 8 x 8, 32 models of 8 images 154 us in 128 x 256 tiles, 83 in 64 x 64.
        // Another one where the time model says so by 5 %; on planes of up to 64 positions, where the deep load pipeline of
        // the register-staged 64 x 64 tile counts, that one too (32 models 2048 -> 512 at 4 x 4: 16.3 against 14.1).
        float best = 0.95f * us(kPointwiseCost[t]);
        int pick = t;
        for (int i = 0; i < kNumRingConvTiles; ++i)
          if (us(kPointwiseCost[i]) < best) { pick = i; best = us(kPointwiseCost[i]); }
        if (HoWo <= 64 && us(kPointwiseRegCost[tile == T128x128w8]) < us(kPointwiseCost[pick]))
          return launch_gemm_any(bkind, al, tile, L, s);
        const nf_status st = launch_conv_ring(pick, L, s);
        if (st != NF_EUNSUPPORTED) return st;
      }
      if (bkind == 1 && forced_tile() < 0) {
        const nf_status st = conv_plane(L, H, W, (int)Wo, stride, tile, false, s);
        if (st != NF_EUNSUPPORTED) return st;
      }
      return launch_gemm_any(bkind, al, tile, L, s);
    }
    static const bool no_patch = dev_getenv("NETFUSE_NO_PATCH") != nullptr;
    if (!no_patch && KH == 7 && KW == 7 && stride == 2 && pad == 3 && dilation == 1 && cig == 3 && W % 8 == 0 &&
        aligned(x, 16)) {
      // the ResNet stem: a few input channels under a wide kernel (conv_stem.h)
      const int PWs = (std::max(8 + W, 2 * ((int)Wo - 1) + 12) + 7) / 8 * 8;     // copied columns and gathered segments fit
      const int span_s = (int)std::min<long long>(Ho, (126 + Wo) / Wo + 1);      // output rows one 128-position tile can touch
      const int PHs = (span_s - 1) * 2 + 7;
      ConvStemArgs c;
      memset(&c, 0, sizeof(c));
      c.x = (const bf16_t*)x; c.w = (const bf16_t*)w; c.R = (const bf16_t*)residual; c.y = (bf16_t*)y;
      c.cog = cog; c.nG = M * g; c.H = H; c.W = W; c.Ho = (int)Ho; c.Wo = (int)Wo; c.HoWo = HoWo;
      c.PW = PWs; c.PS = PHs * PWs; c.cpr = W / 8;
      c.x_group = (long)cig * H * W; c.x_image = (long)Ctot_in * H * W;
      c.y_group = (long)cog * HoWo; c.y_image = (long)Ctot_out * HoWo;
      c.ep = a.ep;
      c.ep.row_vec_stride0 = cog;
      const nf_status st = launch_conv_stem(c, B, s);
      if (st != NF_EUNSUPPORTED) return st;
    }
    if (KH == 3 && KW == 3 && dilation == 1) {
      const nf_status st = conv_wave<bf16_t>(x, w, residual, y, a.ep, M, B, Cin, Cout, g, H, W, (int)Ho, (int)Wo, stride, pad, s);
      if (st != NF_EUNSUPPORTED) return st;
    }
    // patch geometry (conv_patch.h): image column ix sits at patch column ix + 8; rows are copied in
    // chunks of VW pixels; a 128-position tile touches at most `span` output rows
    const int VW = W % 8 == 0 ? 8 : (W % 4 == 0 ? 4 : (W % 2 == 0 ? 2 : 1));
    const int maxcol = std::max(kLPad + W - 1, ((int)Wo - 1) * stride + KW - 1 - pad + kLPad);
    const int PWp = (maxcol + 1 + 7) / 8 * 8;
    const int span = (int)std::min<long long>(Ho, (126 + Wo) / Wo + 1);
    const int PHmax = (span - 1) * stride + KH;
    // narrow groups: fuse S = 32 / cig consecutive groups OF ONE MODEL into one 32-channel block
    // (block-diagonal weights).  The zero blocks are still multiplied with the neighbouring groups'
    // activations, and 0 * NaN = NaN, so a fused block never spans two models (g % S == 0): a non-finite
    // value in one model's input cannot reach another model's output.
    int S = 1;
    if (cig < 32 && 32 % cig == 0 && cig % 4 == 0 && (long long)(32 / cig) * cog <= 32 && g % (32 / cig) == 0 &&
        aligned(w, 8))
      S = 32 / cig;
    const int cig_e = S * cig, cog_e = S * cog;               // channels of the (fused) group a workgroup handles
    const long long patch_tasks = (long long)std::min(cig_e, 16) * PHmax * (W / VW);   // chunk copies per channel block
    // Both kernels below hold offsets inside a block of up to 32 planes, conv_tap.h also inside its up to 128 weight rows, in an int.
    const bool offsets_fit = 32LL * H * W <= INT_MAX && 128LL * 9 * cig_e <= INT_MAX;
    const bool patch_ok = offsets_fit && KH == 3 && KW == 3 && dilation == 1 && pad <= kLPad && aligned(x, 16) &&
                          ((S == 1 && cig % 16 == 0 && aligned(w, 16) && patch_tasks <= 12 * 256) ||
                           (S > 1 && 2 * patch_tasks <= 12 * 256));
    // the tap-major kernel (conv_tap.h) checks its own task and LDS bounds
    static const bool no_tap = dev_getenv("NETFUSE_NO_TAP") != nullptr;
    const bool tap_ok = !no_tap && offsets_fit && KH == 3 && KW == 3 && dilation == 1 && pad <= kLPad && cig_e % 32 == 0;
    if (!no_patch && (patch_ok || tap_ok)) {
      // k x k: MFMA operands from an LDS copy of the zero-padded input patch (conv_tap.h, conv_patch.h)
      ConvPatchArgs c;
      memset(&c, 0, sizeof(c));
      c.x = (const bf16_t*)x; c.w = (const bf16_t*)w; c.R = (const bf16_t*)residual; c.y = (bf16_t*)y;
      c.cig = cig_e; c.cog = cog_e; c.nG = M * g / S; c.S = S; c.cig_real = cig; c.cog_real = cog;
      c.H = H; c.W = W; c.Ho = (int)Ho; c.Wo = (int)Wo; c.HoWo = HoWo;
      c.stride = stride; c.pad = pad;
      c.PW = PWp; c.VW = VW; c.cpr = W / VW;
      c.PS = PHmax * PWp;               // padded per kernel configuration at launch
      c.x_group = (long)cig_e * H * W; c.x_image = (long)Ctot_in * H * W;
      c.y_group = (long)cog_e * HoWo; c.y_image = (long)Ctot_out * HoWo;
      c.ep = a.ep;
      c.ep.row_vec_stride0 = cog_e;
      if (tap_ok) {
        const nf_status st = launch_conv_tap_3x3(c, B, s);
        if (st != NF_EUNSUPPORTED) return st;
      }
      if (patch_ok) {
        const nf_status st = launch_conv_patch_3x3(c, B, s);
        if (st != NF_EUNSUPPORTED) return st;           // else: the implicit-GEMM kernel below takes any shape
      }
    }
    a.geom.H = H; a.geom.W = W; a.geom.KH = KH; a.geom.KW = KW; a.geom.Wo = (int)Wo;
    a.geom.stride = stride; a.geom.pad = pad; a.geom.dil = dilation;
    int bkind = 0;
    if (KH == 1 && KW == 1 && pad == 0) {
      // projection shortcuts; stride 2 over an even width is read as aligned pixel pairs where the shape allows
      bkind = 2;
      const long long plane = (long long)H * W;
      if (stride == 2 && W == 2 * Wo) {
        if (Wo % 4 == 0 && plane % 8 == 0 && aligned(x, 16)) bkind = 24;
        else if (Wo % 2 == 0 && plane % 4 == 0 && aligned(x, 8)) bkind = 22;
        else if (Wo == 7 && Ho <= 8 && plane % 4 == 0 && aligned(x, 8)) bkind = 27;
        else if (aligned(x, 4)) bkind = 21;
      }
      if (forced_tile() < 0) {
        const nf_status st = conv_plane(L, H, W, (int)Wo, stride, tile, bkind != 2, s);
        if (st != NF_EUNSUPPORTED) return st;
      }
      if (bkind == 2 && forced_tile() < 0) {
        // What comes here: operands that are not 16-byte aligned, k that is no multiple of 64, up to 32 outputs per group, rows too wide
        // for the chunks of a tile.  (The times below are of aligned operands, which conv_plane.h now takes.)
        // Eight 2-byte loads per 16 bytes of activations weigh more than a compute unit or two left idle: from 160 tiles of 128 x 128
        // up (3 models of 4 images 512 -> 1024 at 25 x 25: 37.8 us in 64 x 64 tiles, 29.0), but not where they fill a few
        // compute units only (2 models of one image 1024 -> 2048 at 13 x 13: 33.4 us in 32 of them, 26.5 in 64 x 64).
        const long long t128 = problems * ((cog + 127) / 128) * ((HoWo + 127) / 128);
        if (cog > 64 && HoWo > 64 && t128 >= 160) tile = T128x128w8;
        else if (HoWo <= 64 && tile == T128x128w8 && t128 < 64) tile = T64x64;
        // The deep pipeline holds twice the registers: one 128 x 128 tile per compute unit.  One k-step in flight and two tiles where
        // there is a second one to cover the wait, from 257 tiles on, or where k is over before the loader's offsets have paid.  One
        // step against deep over 1933 problems (64 ... 1024 channels, planes of 3 x 3 to 71 x 71, 1 ... 256 images), by tiles: up to 256 1.12
        // to 1.30; 257 ... 768 0.91 (up to 64 positions), 0.96 (more, k up to 256) and 1.0 (longer k; 0.90 for 8 models 1024 -> 2048 at
        // 33 x 33, 1.06 for 3 models of 4 images 512 -> 2048 at 25 x 25); beyond 0.87, 0.90 and 0.95.
        L.one_step = tile == T128x128w8 && (Kdim <= 64 || t128 > 256);
      }
    }
    return launch_gemm_any(bkind, al, tile, L, s);
  }

  // float32: the matrix-pipe kernels, except for narrow groups.  Its lowest tile is 16 rows x 64 positions with k padded to
  // 64 or 128, so a group of a few products per position costs it as much as one of 16 x 64; the direct kernel (one
  // thread per output) pays for what there is, but walks k alone: 0.15 to 0.3 us per k where the chip is not full.
  // Hence a limit on the products per position, by the taps that the other kernel has to look up per tile, and one on k
  // where a model has few groups.  Direct / matrix (us): depthwise 3x3 of 1024 channels at 14 x 14 5 / 50, 16 -> 1
  // channels per group 29 / 64, 4 -> 8 38 / 47, 8 -> 8 81 / 47; 7x7 depthwise 10 / 63, 2 -> 8 79 / 83; pointwise 8 -> 8
  // 23 / 25, 16 -> 8 38 / 25; one model with one group at 56 x 56: 8 -> 1 13 / 7, 16 -> 1 24 / 8.
  // Pointwise layers over planes that are no multiple of 4 positions: from 8 channels of k up the matrix kernel is ahead beyond 64 products (direct / matrix,
  // 32 models: 16 -> 13 in 64 groups over 15 x 15 132 / 59), below it depends on the number of models (one: 1 -> 64 channels in one group 0.6 to 0.7 of its
  // time, 64 groups in 32: 1.5 to 1.9), as up to 64 products.  Over 1619 odd problems of 1 to 64 groups and 1 to 32 models the form picked takes 13 % longer
  // than the better one on average (45 % at the line of the k x k layers, 4 % at that of the even planes, which is up to 1.8 times behind with few models).
  const bool f32_pointwise = KH == 1 && KW == 1 && stride == 1 && pad == 0;
  const long long f32_products = (long long)cog * Kdim;     // per position
  const bool f32_narrow = f32_pointwise && HoWo % 4 != 0 ? f32_products <= (Kdim < 8 ? 230 : 64)
                          : f32_pointwise                ? f32_products <= 64 && (g >= 64 || Kdim <= 16)
                                                         : f32_products <= 220 + 10LL * KH * KW && (g >= 64 || Kdim <= 72);
  if (dt == NF_F32 && KH * KW < 64 && !f32_narrow && f32_fits((long long)cog * Kdim, prod({cig, H, W}), Kdim)) {
    GemmF32Args a;
    memset(&a, 0, sizeof(a));
    a.A = (const float*)w; a.B = (const float*)x; a.R = (const float*)residual; a.C = (float*)y;
    a.lda = Kdim; a.ldb = (long)H * W; a.ldc = HoWo;
    a.sA0 = (long)cog * Kdim;
    a.sB0 = (long)cig * H * W; a.sB1 = (long)Ctot_in * H * W;
    a.sC0 = (long)cog * HoWo; a.sC1 = (long)Ctot_out * HoWo;
    a.a_bytes = (unsigned)(a.sA0 * 4); a.b_bytes = (unsigned)(a.sB0 * 4);
    a.rows = cog; a.cols = HoWo; a.K = Kdim; a.nz0 = M * g;
    a.ep.row_bias = bias; a.ep.row_scale = scale; a.ep.row_shift = shift; a.ep.row_vec_stride0 = cog;
    a.ep.act = act;
    a.H = H; a.W = W; a.KW = KW; a.khw = KH * KW; a.Wo = (int)Wo; a.stride = stride; a.pad = pad; a.dil = dilation;
    f32_divisors(a);
    if (KH == 3 && KW == 3 && dilation == 1) {
      const nf_status st = conv_wave<float>(x, w, residual, y, a.ep, M, B, Cin, Cout, g, H, W, (int)Ho, (int)Wo, stride, pad, s);
      if (st != NF_EUNSUPPORTED) return st;
    }
    const nf_status st = launch_gemm_f32(a, B, !f32_pointwise, s);
    if (st != NF_EUNSUPPORTED) return st;               // more tiles than a grid holds: the direct kernel strides over any number
  }

  ConvGeom geo;
  geo.B = B; geo.Ctot_in = (int)Ctot_in; geo.Ctot_out = (int)Ctot_out; geo.cig = cig; geo.cog = cog;
  geo.H = H; geo.W = W; geo.KH = KH; geo.KW = KW; geo.Ho = (int)Ho; geo.Wo = (int)Wo;
  geo.stride = stride; geo.pad = pad; geo.dil = dilation;
  const unsigned grid = grid_for(n_out, 256);
  if (dt == NF_F32)
    nf_launch(conv2d_generic_kernel<float>, dim3(grid), dim3(256), 0, s, (const float*)x,
                       (const float*)w, bias, scale, shift, (const float*)residual, (float*)y, geo, (int)act,
                       (size_t)n_out);
  else
    nf_launch(conv2d_generic_kernel<bf16_t>, dim3(grid), dim3(256), 0, s, (const bf16_t*)x,
                       (const bf16_t*)w, bias, scale, shift, (const bf16_t*)residual, (bf16_t*)y, geo, (int)act,
                       (size_t)n_out);
  return launched();
}

// For the tests, which name the tile of conv_plane.h that a case is meant to run; not part of the interface.  16-byte aligned operands; -1 =
// another kernel.  Host only.
int netfuse_conv_plane_tile(int M, int B, int cig, int cog, int g, int H, int W, int stride, int residual) {
  GemmLaunch L;
  memset(&L, 0, sizeof(L));
  const int Ho = (H - 1) / stride + 1, Wo = (W - 1) / stride + 1;
  L.a.rows = cog; L.a.cols = Ho * Wo; L.a.K = cig; L.a.nz0 = M * g; L.nz1 = B;
  L.a.R = residual ? (const bf16_t*)&L : nullptr;
  L.a.ldb = (long)H * W;
  L.a.geom.W = W; L.a.geom.Wo = Wo; L.a.geom.stride = stride;
  if (stride == 1 && L.a.cols % 8 == 0) return -1;
  return pick_conv_plane(L, conv_reg_tile(cog, L.a.cols, (long long)M * g * B, stride == 1), stride == 2 && W == 2 * Wo);
}

nf_status netfuse_layernorm(const void* x, const void* residual, const float* gamma, const float* beta, void* y,
                            int M, int rows, int H, float eps, nf_merge_dim layout, nf_dtype dt, void* stream) {
  if (!x || !gamma || !beta || !y) return NF_EINVAL;
  if (M <= 0 || rows <= 0 || H <= 0) return NF_EINVAL;
  if (!(eps >= 0.f)) return NF_EINVAL;
  if (layout != NF_MERGE_BATCH && layout != NF_MERGE_CHANNEL) return NF_EINVAL;
  if (!is_dtype(dt)) return NF_EINVAL;
  if (prod({M, rows, H}) >= kMaxElems) return NF_EINVAL;
  const size_t esz = dt == NF_F32 ? 4 : 2;
  if (!aligned(x, esz) || !aligned(y, esz) || !aligned(residual, esz) || !aligned(gamma, 4) || !aligned(beta, 4))
    return NF_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  const long long nrows = (long long)M * rows;
  const long long blocks = (nrows + 3) / 4;
  if (blocks > kMaxGrid) return NF_EUNSUPPORTED;
  const size_t va = 4 * esz;
  const bool vec = H % 4 == 0 && aligned(x, va) && aligned(y, va) && aligned(residual, va);
  const int ch = layout == NF_MERGE_CHANNEL;
  // rows that fit in registers: two per wavefront (they share the model's gamma and beta) of up to 512 features once there
  // are enough rows to keep every CU busy that way.  16384 rows of bf16 (us, one / two): 256 features 6.8 / 5.9, 512 8.2 /
  // 8.1, 768 10.4 / 10.7, with a residual 14.8 / 15.3; 4096 rows of 768 3.9 / 4.7.
  if (vec && H <= kWave * 4 * 4) {
    const int R = nrows >= 16384 && H <= 512 && rows % 2 == 0 ? 2 : 1, nit = (H + 255) / 256;
    const long long blocks_r = (nrows / R + 3) / 4;
#define NF_LNR(T, N, R_)                                                                                  \
  nf_launch((layernorm_rows_kernel<T, N, R_>), dim3((unsigned)blocks_r), dim3(256), 0, s,                  \
                     (const T*)x, (const T*)residual, gamma, beta, (T*)y, M, rows, H, eps, ch)
#define NF_LNR_T(T)                                                   \
  switch (nit) {                                                      \
    case 1: if (R == 2) NF_LNR(T, 1, 2); else NF_LNR(T, 1, 1); break; \
    case 2: if (R == 2) NF_LNR(T, 2, 2); else NF_LNR(T, 2, 1); break; \
    case 3: NF_LNR(T, 3, 1); break;                                   \
    default: NF_LNR(T, 4, 1); break;                                  \
  }
    if (dt == NF_F32) { NF_LNR_T(float) } else { NF_LNR_T(bf16_t) }
#undef NF_LNR_T
#undef NF_LNR
    return launched();
  }
#define NF_LN(T, VEC, MAXIT)                                                                             \
  nf_launch((layernorm_kernel<T, VEC, MAXIT>), dim3((unsigned)blocks), dim3(256), 0, s,         \
                     (const T*)x, (const T*)residual, gamma, beta, (T*)y, M, rows, H, eps, ch)
  if (dt == NF_F32) {
    if (vec) NF_LN(float, 4, 4); else NF_LN(float, 1, 8);
  } else {
    if (vec) NF_LN(bf16_t, 4, 4); else NF_LN(bf16_t, 1, 8);
  }
#undef NF_LN
  return launched();
}

nf_status netfuse_batchnorm(const void* x, const float* gamma, const float* beta, const float* mean,
                            const float* var, const void* residual, void* y, int M, int B, int C, int HW,
                            float eps, nf_dtype dt, nf_act act, void* stream) {
  if (!x || !gamma || !beta || !mean || !var || !y) return NF_EINVAL;
  if (M <= 0 || B <= 0 || C <= 0 || HW <= 0) return NF_EINVAL;
  if (!(eps >= 0.f)) return NF_EINVAL;
  if (!is_dtype(dt) || !is_act(act)) return NF_EINVAL;
  const long long Ctot = (long long)M * C;
  if (Ctot > INT_MAX || prod({B, Ctot, HW}) >= kMaxElems) return NF_EINVAL;
  const size_t esz = dt == NF_F32 ? 4 : 2;
  if (!aligned(x, esz) || !aligned(y, esz) || !aligned(residual, esz) || !aligned(gamma, 4) ||
      !aligned(beta, 4) || !aligned(mean, 4) || !aligned(var, 4))
    return NF_EINVAL;
  const long long rowsbc = (long long)B * Ctot;
  if (rowsbc > kMaxGrid) return NF_EUNSUPPORTED;
  hipStream_t s = (hipStream_t)stream;
  const long long n_el = prod({B, Ctot, HW});
  const int per = 16 / (int)esz;
  if (n_el % per == 0 && aligned(x, 16) && aligned(y, 16) && aligned(residual, 16) && n_el / per / 256 < kMaxGrid) {
    const long long chunks = n_el / per;
    const unsigned grid = (unsigned)((chunks + 255) / 256);
    if (dt == NF_F32)
      nf_launch(batchnorm_flat_kernel<float>, dim3(grid), dim3(256), 0, s, (const float*)x, gamma, beta, mean, var,
                (const float*)residual, (float*)y, (int)Ctot, HW, eps, (int)act, (size_t)chunks);
    else
      nf_launch(batchnorm_flat_kernel<bf16_t>, dim3(grid), dim3(256), 0, s, (const bf16_t*)x, gamma, beta, mean, var,
                (const bf16_t*)residual, (bf16_t*)y, (int)Ctot, HW, eps, (int)act, (size_t)chunks);
    return launched();
  }
  const unsigned gy = (unsigned)((HW + 1023) / 1024 > 64 ? 64 : (HW + 1023) / 1024);
  if (dt == NF_F32)
    nf_launch(batchnorm_kernel<float>, dim3((unsigned)rowsbc, gy), dim3(256), 0, s, (const float*)x,
                       gamma, beta, mean, var, (const float*)residual, (float*)y, (int)Ctot, HW, eps, (int)act);
  else
    nf_launch(batchnorm_kernel<bf16_t>, dim3((unsigned)rowsbc, gy), dim3(256), 0, s, (const bf16_t*)x,
                       gamma, beta, mean, var, (const bf16_t*)residual, (bf16_t*)y, (int)Ctot, HW, eps, (int)act);
  return launched();
}

nf_status netfuse_bn_fold(const float* gamma, const float* beta, const float* mean, const float* var, float* scale,
                          float* shift, int n, float eps, void* stream) {
  if (!gamma || !beta || !mean || !var || !scale || !shift) return NF_EINVAL;
  if (n <= 0 || !(eps >= 0.f)) return NF_EINVAL;
  if (!aligned(gamma, 4) || !aligned(beta, 4) || !aligned(mean, 4) || !aligned(var, 4) || !aligned(scale, 4) ||
      !aligned(shift, 4))
    return NF_EINVAL;
  nf_launch(bn_fold_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream, gamma,
                     beta, mean, var, scale, shift, n, eps);
  return launched();
}

nf_status netfuse_attention(const void* Q, const void* K, const void* V, const float* mask, void* O, int M, int B,
                            int S, int heads, int d, long stride_m, long stride_row, float scale, nf_dtype dt,
                            void* stream) {
  if (!Q || !K || !V || !O) return NF_EINVAL;
  if (M <= 0 || B <= 0 || S <= 0 || heads <= 0 || d <= 0) return NF_EINVAL;
  if (!is_dtype(dt) || !(scale == scale)) return NF_EINVAL;
  const long long hd = (long long)heads * d;
  if (hd > INT_MAX) return NF_EINVAL;
  if (stride_row < hd) return NF_EINVAL;                              // heads of one row are side by side
  if (prod({B, S}) > INT_MAX / 2) return NF_EINVAL;
  if (stride_m < 0 || (M > 1 && stride_m < (long long)(B * (long long)S - 1) * stride_row + hd)) return NF_EINVAL;
  if (prod({M, B, S, hd}) >= kMaxElems || prod({M, stride_m}) >= kMaxElems) return NF_EINVAL;
  const size_t esz = dt == NF_F32 ? 4 : 2;
  if (!aligned(Q, esz) || !aligned(K, esz) || !aligned(V, esz) || !aligned(O, esz) || !aligned(mask, 4))
    return NF_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  AttnArgs a;
  a.Q = Q; a.K = K; a.V = V; a.mask = mask; a.O = O;
  a.M = M; a.B = B; a.S = S; a.heads = heads; a.d = d;
  a.stride_m = stride_m; a.stride_row = stride_row; a.scale = scale;

  if (dt == NF_BF16 && d == kAttnD && stride_row % 8 == 0 && stride_m % 8 == 0 && aligned(Q, 16) &&
      aligned(K, 16) && aligned(V, 16) && aligned(O, 8)) {
    const int qblocks = (S + 127) / 128;
    const long long total = prod({M, B, heads, qblocks});
    if (total > kMaxGrid) return NF_EUNSUPPORTED;
    if (mask) nf_launch(attention_mfma_d64_kernel<true>, dim3((unsigned)total), dim3(256), 0, s, a, qblocks);
    else nf_launch(attention_mfma_d64_kernel<false>, dim3((unsigned)total), dim3(256), 0, s, a, qblocks);
    return launched();
  }
  const long long head_elems = (long long)(S - 1) * stride_row + d;         // one head's rows, first to last element
  // Up to 8 tokens the wavefront-per-query kernel below: of 64 features the two are level between 5 and 6 (us, that kernel / this one, 32 models x 8
  // sequences x 12 heads: 1 token 4.4 / 18.0, 4 11.3 / 17.2, 5 15.0 / 17.4, 6 20.0 / 17.4, 8 26.7 / 17.5; one model, 1 sequence: 3.3 / 4.5, 3.8 / 4.1, 3.9 / 3.8,
  // 4.1 / 3.8, 4.4 / 3.9), other head sizes have no form of 16 queries and pay for 32 (32 features: 8 tokens 14.8 / 15.6, 9 15.6 / 15.6).
  if (dt == NF_F32 && S > 8 && d % 4 == 0 && d <= 128 && head_elems < (1LL << 29)) {
    // Query groups and key shares, by the sequence length alone: the shares decide the order of the sums, and a model's bits do not depend on
    // what is merged with it.  Where 16 or 32 rows are all there are, wavefronts without queries take keys instead (us, 4 groups x 1 share / 2 x 2 /
    // 1 x 4: 12 models x 8 sequences of 10 tokens 18.3 / 12.5 / 9.3, 32 x 8 of 16 39.3 / 26.7 / 19.6, of 32 41 / 28.7 / 33.8, one of 16 5.9 / 4.6 / 4.0).  Above that
    // shares gain in small grids and lose in full ones (128 tokens, 2 models 9.4 / 6.8 / 5.5, 12 x 8 58 / 64 / 76; 40 tokens, 12 x 8 20.2 / 21.9 / 20.9).
    const int groups = S > 32 ? 4 : S > 16 || d <= 32 || d > 64 ? 2 : 1;
    const int qblocks = (S + 16 * groups - 1) / (16 * groups);
    const long long total = prod({M, B, heads, qblocks});
    if (total > kMaxGrid) return NF_EUNSUPPORTED;
    const unsigned bytes = (unsigned)(head_elems * 4);
#define NF_ATT(NB, KB, QG, KS) nf_launch((attention_f32_kernel<NB, KB, QG, KS>), dim3((unsigned)total), dim3(256), 0, s, a, qblocks, bytes)
    if (d <= 32) {
      if (groups == 4) NF_ATT(2, 64, 4, 1); else NF_ATT(2, 64, 2, 2);
    } else if (d <= 64) {
      if (groups == 4) NF_ATT(4, 64, 4, 1); else if (groups == 2) NF_ATT(4, 64, 2, 2); else NF_ATT(4, 64, 1, 4);
    } else {
      if (groups == 4) NF_ATT(8, 32, 4, 1); else NF_ATT(8, 32, 2, 2);
    }
#undef NF_ATT
    return launched();
  }
  if (d > 256) return NF_EUNSUPPORTED;
  const long long waves = prod({M, B, heads, S});
  const long long blocks = (waves + 3) / 4;
  if (blocks > kMaxGrid) return NF_EUNSUPPORTED;
  const int dpl = (d + 63) / 64;
#define NF_ATT(T, DPL) \
  nf_launch((attention_generic_kernel<T, DPL>), dim3((unsigned)blocks), dim3(256), 0, s, a)
  if (dt == NF_F32) {
    if (dpl == 1) NF_ATT(float, 1); else if (dpl == 2) NF_ATT(float, 2); else NF_ATT(float, 4);
  } else {
    if (dpl == 1) NF_ATT(bf16_t, 1); else if (dpl == 2) NF_ATT(bf16_t, 2); else NF_ATT(bf16_t, 4);
  }
#undef NF_ATT
  return launched();
}

nf_status netfuse_attention_relpos(const void* Q, const void* K, const void* V, const void* Kr, const float* bias_w,
                                   const float* bias_r, const float* mask, void* O, int M, int B, int S, int heads,
                                   int d, long stride_m, long stride_row, float scale, nf_dtype dt, void* stream) {
  if (!Q || !K || !V || !Kr || !O) return NF_EINVAL;
  if (M <= 0 || B <= 0 || S <= 0 || heads <= 0 || d <= 0) return NF_EINVAL;
  if (!is_dtype(dt) || !(scale == scale)) return NF_EINVAL;
  const long long hd = (long long)heads * d;
  if (hd > INT_MAX || stride_row < hd) return NF_EINVAL;
  if (prod({B, S}) > INT_MAX / 2) return NF_EINVAL;
  if (stride_m < 0 || (M > 1 && stride_m < (long long)(B * (long long)S - 1) * stride_row + hd)) return NF_EINVAL;
  if (prod({M, B, S, hd}) >= kMaxElems || prod({M, stride_m}) >= kMaxElems || prod({M, 2, S, hd}) >= kMaxElems)
    return NF_EINVAL;
  const size_t esz = dt == NF_F32 ? 4 : 2;
  if (!aligned(Q, esz) || !aligned(K, esz) || !aligned(V, esz) || !aligned(Kr, esz) || !aligned(O, esz) ||
      !aligned(mask, 4) || !aligned(bias_w, 4) || !aligned(bias_r, 4))
    return NF_EINVAL;
  if (d > 256) return NF_EUNSUPPORTED;
  const long long waves = prod({M, B, heads, S});
  const long long blocks = (waves + 3) / 4;
  if (blocks > kMaxGrid) return NF_EUNSUPPORTED;
  AttnRelArgs ra;
  AttnArgs& a = ra.a;
  a.Q = Q; a.K = K; a.V = V; a.mask = mask; a.O = O;
  a.M = M; a.B = B; a.S = S; a.heads = heads; a.d = d;
  a.stride_m = stride_m; a.stride_row = stride_row; a.scale = scale;
  ra.Kr = Kr; ra.bias_w = bias_w; ra.bias_r = bias_r;
  hipStream_t s = (hipStream_t)stream;
  if (dt == NF_BF16 && d == kAttnD && stride_row % 8 == 0 && stride_m % 8 == 0 && aligned(Q, 16) && aligned(K, 16) &&
      aligned(V, 16) && aligned(Kr, 16) && aligned(O, 8) && S <= (1 << 24)) {
    const int qblocks = (S + 127) / 128;
    const long long total = prod({M, B, heads, qblocks});
    if (total > kMaxGrid) return NF_EUNSUPPORTED;
    static std::atomic<bool> opted_in{false};          // 68 KB of LDS: one opt-in per process (idempotent)
    if (!opted_in.load(std::memory_order_acquire)) {
      if (hipFuncSetAttribute(reinterpret_cast<const void*>(attention_relpos_mfma_d64_kernel),
                              hipFuncAttributeMaxDynamicSharedMemorySize, kRelLdsBytes) != hipSuccess)
        return NF_ELAUNCH;
      opted_in.store(true, std::memory_order_release);
    }
    nf_launch(attention_relpos_mfma_d64_kernel, dim3((unsigned)total), dim3(256), kRelLdsBytes, s, ra, qblocks);
    return launched();
  }
  const int dpl = (d + 63) / 64;
#define NF_ATTR(T, DPL) nf_launch((attention_relpos_kernel<T, DPL>), dim3((unsigned)blocks), dim3(256), 0, s, ra)
  if (dt == NF_F32) {
    if (dpl == 1) NF_ATTR(float, 1); else if (dpl == 2) NF_ATTR(float, 2); else NF_ATTR(float, 4);
  } else {
    if (dpl == 1) NF_ATTR(bf16_t, 1); else if (dpl == 2) NF_ATTR(bf16_t, 2); else NF_ATTR(bf16_t, 4);
  }
#undef NF_ATTR
  return launched();
}

nf_status netfuse_maxpool2d(const void* x, void* y, int B, int Ctot, int H, int W, int k, int stride, int pad,
                            nf_dtype dt, void* stream) {
  if (!x || !y) return NF_EINVAL;
  if (B <= 0 || Ctot <= 0 || H <= 0 || W <= 0 || k <= 0 || stride <= 0 || pad < 0) return NF_EINVAL;
  if (pad >= k || !is_dtype(dt)) return NF_EINVAL;
  if ((long long)H + 2LL * pad < k || (long long)W + 2LL * pad < k) return NF_EINVAL;
  const int Ho = (H + 2 * pad - k) / stride + 1, Wo = (W + 2 * pad - k) / stride + 1;
  const long long n_in = prod({B, Ctot, H, W}), n_out = prod({B, Ctot, Ho, Wo});
  if (n_in >= kMaxElems || n_out >= kMaxElems) return NF_EINVAL;
  const size_t esz = dt == NF_F32 ? 4 : 2;
  if (!aligned(x, esz) || !aligned(y, esz)) return NF_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  if (dt == NF_BF16 && k == 3 && stride == 2 && pad == 1 && W % 8 == 0 && aligned(x, 16) && aligned(y, 8)) {
    // Wo = W / 2 is a multiple of 4: four outputs of one or two rows per thread from 16-byte loads
    const int rows = W <= 32 || Ho == 1 ? 1 : 2;
    const long long total = n_out / Wo / Ho * ((Ho + rows - 1) / rows) * (Wo / 4);
    const unsigned grid = grid_for(total, 256);
#define NF_POOL(kernel, I) nf_launch((kernel<I>), dim3(grid), dim3(256), 0, s, (const bf16_t*)x, (bf16_t*)y, H, W, Ho, Wo, (I)total)
    if (total + 256LL * grid < (1LL << 32)) {                // the loop's index does not wrap either
      if (rows == 1) NF_POOL(maxpool3x3s2_bf16_row_kernel, uint32_t); else NF_POOL(maxpool3x3s2_bf16_kernel, uint32_t);
    } else {
      if (rows == 1) NF_POOL(maxpool3x3s2_bf16_row_kernel, size_t); else NF_POOL(maxpool3x3s2_bf16_kernel, size_t);
    }
#undef NF_POOL
    return launched();
  }
  // Any other width from 8 columns, and float32.  Below 2^14 outputs, and in planes of one row, the launch is the time and the kernel for any
  // window is level or ahead (us, it and this one: 64 planes of 12 x 12 in float32 2.85 and 2.90, of 31 x 31 2.95 and 2.95, 4 of 1 x 4000 2.18 and
  // 2.41; 4096 of 9 x 9 in bf16 3.14 and 2.92, of 14 x 14 3.56 and 2.81).  The limits on H and W: a row or column past the edge is a 32-bit number too.
  if (k == 3 && stride == 2 && pad == 1 && W >= 8 && Ho > 1 && n_out > (1 << 14) && H < (1 << 30) && W < (1 << 30)) {
    const int nbx = (Wo + 3) / 4, nby = (Ho + 1) / 2;
    const long long total = n_out / Wo / Ho * nby * nbx;
    const unsigned grid = grid_for(total, 256);
    const bool small = total + 256LL * grid < (1LL << 32);
#define NF_POOL(T, I) nf_launch((maxpool3x3s2_any_kernel<T, I>), dim3(grid), dim3(256), 0, s, (const T*)x, (T*)y, H, W, Ho, Wo, nbx, nby, (I)total)
    if (dt == NF_F32) { if (small) NF_POOL(float, uint32_t); else NF_POOL(float, size_t); }
    else { if (small) NF_POOL(bf16_t, uint32_t); else NF_POOL(bf16_t, size_t); }
#undef NF_POOL
    return launched();
  }
  const unsigned grid = grid_for(n_out, 256);
  if (dt == NF_F32)
    nf_launch(maxpool2d_kernel<float>, dim3(grid), dim3(256), 0, s, (const float*)x, (float*)y, H, W, Ho,
                       Wo, k, stride, pad, (size_t)n_out);
  else
    nf_launch(maxpool2d_kernel<bf16_t>, dim3(grid), dim3(256), 0, s, (const bf16_t*)x, (bf16_t*)y, H, W,
                       Ho, Wo, k, stride, pad, (size_t)n_out);
  return launched();
}

nf_status netfuse_avgpool_global(const void* x, void* y, int B, int Ctot, int HW, nf_dtype dt, void* stream) {
  if (!x || !y) return NF_EINVAL;
  if (B <= 0 || Ctot <= 0 || HW <= 0 || !is_dtype(dt)) return NF_EINVAL;
  if (prod({B, Ctot, HW}) >= kMaxElems) return NF_EINVAL;
  const size_t esz = dt == NF_F32 ? 4 : 2;
  if (!aligned(x, esz) || !aligned(y, esz)) return NF_EINVAL;
  const long long nchan = (long long)B * Ctot;
  const long long blocks = (nchan + 3) / 4;
  if (blocks > kMaxGrid) return NF_EUNSUPPORTED;
  hipStream_t s = (hipStream_t)stream;
  if (HW <= 64) {
    const unsigned blocks16 = (unsigned)((nchan + 15) / 16);
    if (dt == NF_F32)
      nf_launch(avgpool_global_small_kernel<float>, dim3(blocks16), dim3(256), 0, s, (const float*)x,
                         (float*)y, (size_t)nchan, HW);
    else
      nf_launch(avgpool_global_small_kernel<bf16_t>, dim3(blocks16), dim3(256), 0, s, (const bf16_t*)x,
                         (bf16_t*)y, (size_t)nchan, HW);
    return launched();
  }
  if (dt == NF_F32)
    nf_launch(avgpool_global_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, s, (const float*)x,
                       (float*)y, (size_t)nchan, HW);
  else
    nf_launch(avgpool_global_kernel<bf16_t>, dim3((unsigned)blocks), dim3(256), 0, s, (const bf16_t*)x,
                       (bf16_t*)y, (size_t)nchan, HW);
  return launched();
}

nf_status netfuse_merge_transpose(const void* src, void* dst, int M, int rows, int H, int to_channel, nf_dtype dt,
                                  void* stream) {
  if (!src || !dst || src == dst) return NF_EINVAL;
  if (M <= 0 || rows <= 0 || H <= 0 || !is_dtype(dt)) return NF_EINVAL;
  const long long total = prod({M, rows, H});
  if (total >= kMaxElems) return NF_EINVAL;
  const size_t esz = dt == NF_F32 ? 4 : 2;
  if (!aligned(src, esz) || !aligned(dst, esz)) return NF_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  // rows of H elements move as whole 16-byte vectors when they are made of them: the same index map over
  // H * esz / 16 vectors per row
  if (((size_t)H * esz) % 16 == 0 && aligned(src, 16) && aligned(dst, 16)) {
    const int Hv = (int)((size_t)H * esz / 16);
    const long long total_v = prod({M, rows, Hv});
    nf_launch(merge_transpose_kernel<uint4>, dim3(grid_for(total_v, 256)), dim3(256), 0, s, (const uint4*)src, (uint4*)dst,
              M, rows, Hv, to_channel != 0, (size_t)total_v);
    return launched();
  }
  const unsigned grid = grid_for(total, 256);
  if (dt == NF_F32)
    nf_launch(merge_transpose_kernel<float>, dim3(grid), dim3(256), 0, s, (const float*)src, (float*)dst,
                       M, rows, H, to_channel != 0, (size_t)total);
  else
    nf_launch(merge_transpose_kernel<bf16_t>, dim3(grid), dim3(256), 0, s, (const bf16_t*)src,
                       (bf16_t*)dst, M, rows, H, to_channel != 0, (size_t)total);
  return launched();
}

}  // extern "C"
