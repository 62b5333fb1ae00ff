// Instantiation, tile choice and launch of the float32 kernels on bf16 matrix instructions (gemm_split.h).
#include "gemm_split.h"

namespace nf {

enum { kS64x64, kS64x48, kS64x32, kS32x64, kS32x32, kS16x64, kS16x32, kNumSplitTiles };
constexpr int kSplitBM[kNumSplitTiles] = {64, 64, 64, 32, 32, 16, 16};
constexpr int kSplitBN[kNumSplitTiles] = {64, 48, 32, 64, 32, 64, 32};
// Time model of a tile (us): latency a + l per 768 of k; per 256 tiles p + q per 768 of k; per round of tiles over the 256 compute units
// begun s per 768 of k + r.  Fitted to every tile over 260 problems (an encoder's matmuls at hidden sizes 256 to 1024, 4 ... 1500 rows, and
// 64 to 2048 rows times 16 to 4500 columns, 1 ... 32 models); over 316 others, 1 ... 2048 rows, the mean error of a prediction is 5 to 8 % and the tile it picks
// 0.5 % behind the best.
constexpr float kSplitCost[kNumSplitTiles][6] = {   // a, l, p, q, s, r
    {3.91f, 1.69f, 0.508f, 2.22f, 6.08f, 1.67f},
    {3.5f, 1.73f, 0.229f, 2.22f, 4.78f, 1.76f},
    {3.09f, 1.58f, 0.235f, 1.41f, 4.02f, 1.44f},
    {2.55f, 2.89f, 0.0475f, 2.54f, 2.29f, 1.49f},
    {2.78f, 2.33f, 0.f, 1.94f, 1.34f, 0.872f},
    {2.29f, 2.62f, 0.f, 2.43f, 1.08f, 1.08f},
    {2.87f, 1.25f, 0.f, 1.26f, 1.14f, 0.468f}};

template <class Cfg, bool TAIL>
static nf_status launch_kernel(GemmF32Args& a, long long total, hipStream_t s) {
  static_assert(Cfg::kLdsBytes <= 64 * 1024, "no opt-in");
  nf_launch(gemm_split_kernel<Cfg, TAIL>, dim3((unsigned)total), dim3(Cfg::kThreads), Cfg::kLdsBytes, s, a);
  return hipGetLastError() == hipSuccess ? NF_OK : NF_ELAUNCH;
}

template <class Cfg>
static nf_status launch_split(GemmF32Args& a, long long problems, hipStream_t s) {
  a.tiles_m = (a.rows + Cfg::kBM - 1) / Cfg::kBM;
  a.tiles_n = (a.cols + Cfg::kBN - 1) / Cfg::kBN;
  const long long total = problems * a.tiles_m * a.tiles_n;
  if (total <= 0 || total > 0x7fffffffLL) return NF_EUNSUPPORTED;
  return a.K % 32 == 0 ? launch_kernel<Cfg, false>(a, total, s) : launch_kernel<Cfg, true>(a, total, s);
}

// Whether a problem of this shape is this kernel's.  By the shape of one problem alone: its sums round differently from gemm_f32.h's, and a
// model's bits must not depend on how many are merged with it.  Few k over a large output is mostly the meeting of the chains in LDS, and at 64 of k
// gemm_f32.h walks no padding (us, gemm_f32.h / here: 13 models of 1913 rows 64 -> 69 10.4 / 12.9, 7 of 512 rows 64 -> 1496 18.2 / 22.2, 2 of 421 rows
// 64 -> 92 4.2 / 3.5; from 68 to 124 of k this is 6 to 18 % ahead up to 2^18 outputs, 3 to 13 % above; 4 of 2048 rows 128 -> 1296 41.0 / 41.0).  Of 511 drawn problems of 64 to 128 of k none is more than 5 % behind (13 with the line of 68 for 64 too), and 1.7 % more time than
// the better kernel on average.  Over 316 others (an encoder's matmuls at hidden sizes 256 to 1024; 64 to 4096 of k, 1 ... 2048 rows times 16 to 4500
// columns; 1 ... 32 models) 15 % less time, k from 1024 up 19 %; 9 are 5 to 11 % behind, of 3 to 36 rows over many models (13 of 4 rows 3072 -> 768
// 23.4 / 26.8, but one of 7 rows 4096 -> 1024 26.9 / 18.2).
// Matmuls only.  Pointwise convolutions gained one by one before the multiplication by 2^24 (8 models 2048 -> 512 over 7 x 7 26 / 17, 512 -> 256 over 28 x 28
// 22.5 / 18.9), but these multiplications draw more power than float32 ones and the clock of the whole chip follows: an image network of 8 models with
// its pointwise layers here takes 1191 us a pass in the steady state, 1152 without, at 2304 and 2403 MHz, its 3 x 3 layers and stem 4 % longer
// and most of the pointwise layers too.
bool split_takes(int rows, int cols, int K) {
  const long long out = (long long)rows * cols;
  return K % 4 == 0 && K >= 64 && (K >= 256 || out <= (K >= 128 ? 1 << 21 : K > 64 ? 1 << 18 : 1 << 16));
}

nf_status launch_gemm_split(GemmF32Args& a, hipStream_t s) {
  const long long problems = a.nz0;
  // byte offsets of the steps that are loaded past the end stay below 2^32, those of A's rows below 2^31
  if (!split_takes(a.rows, a.cols, a.K) || ((long long)a.K + 512) * a.ldb * 4 + 4096 >= (1LL << 32) ||
      (long long)a.rows * a.lda * 4 + 4096 >= (1LL << 31))
    return NF_EUNSUPPORTED;
  const float k = (float)a.K / 768.0f;
  int best = -1;
  float best_us = 0.f;
  for (int t = 0; t < kNumSplitTiles; ++t) {
    const long long tiles = problems * ((a.rows + kSplitBM[t] - 1) / kSplitBM[t]) * ((a.cols + kSplitBN[t] - 1) / kSplitBN[t]);
    const float f = (float)tiles / 256.0f, r = (float)((tiles + 255) / 256);
    const float* c = kSplitCost[t];
    const float us = c[0] + c[1] * k + f * (c[2] + c[3] * k) + r * (c[4] * k + c[5]);
    if (best < 0 || us < best_us) { best = t; best_us = us; }
  }
  switch (best) {
    case kS64x64: return launch_split<SplitCfg<4, 4, 1>>(a, problems, s);
    case kS64x48: return launch_split<SplitCfg<4, 3, 2>>(a, problems, s);
    case kS64x32: return launch_split<SplitCfg<4, 2, 1>>(a, problems, s);
    case kS32x64: return launch_split<SplitCfg<2, 4, 1>>(a, problems, s);
    case kS32x32: return launch_split<SplitCfg<2, 2, 2>>(a, problems, s);
    case kS16x64: return launch_split<SplitCfg<1, 4, 2>>(a, problems, s);
    case kS16x32: return launch_split<SplitCfg<1, 2, 2>>(a, problems, s);
  }
  return NF_EUNSUPPORTED;
}

// For the tests, which compare either side of the rule; not part of the interface.  Host only.
extern "C" int netfuse_f32_split_takes(int rows, int cols, int K) { return split_takes(rows, cols, K); }

}  // namespace nf
