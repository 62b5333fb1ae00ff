// Merged 7x7 / stride 2 / pad 3 convolution over a few input channels (the ResNet / ResNeXt stem;
// Section 3.1 "Convolution": M models = M groups of CIN input channels each), bf16, as an implicit
// GEMM with the input patch in LDS.
//
//   C[co][p] = sum_{ci,ky,kx} w[co][ci][ky][kx] * xpad[ci][2 oy + ky][2 ox + kx],   p = oy*Wo + ox
//
// With so few channels the k dimension is ordered for the B (activation) side: the 8 k-slots that one
// lane feeds into an MFMA step are ONE patch row segment, slot j = tap kx = j - 1 of row (ci, ky) (slot 0
// carries a zero weight).  Image column ix lives at patch column ix + 8, so the segment of output
// column ox starts at patch column 2 ox + 4: 16 contiguous bytes at a 4-byte aligned LDS address, read
// as dwords instead of eight 2-byte gathers.  The two lane halves take rows 2 s and 2 s + 1 of the
// CIN * 7 (ci, ky) rows in step s.  The weights are scattered into that order when they are copied to LDS.
//
// One workgroup = up to 64 output channels (32 where no more are left over from whole sixty-fours: half the wavefronts had no
// channels otherwise) and a run of tiles of 128 positions of one (image, model), as many as tile_run says.  The weights
// go through LDS once and then stay in registers (44), so a tile is its patch, one LDS segment per
// multiplication, and stores out of registers; the next tile's patch is on its way meanwhile and changes LDS buffers at the
// tile's only barrier.
// What bounds it: the patch reads and the issue of instructions.  With one tile per workgroup, the weights scattered into LDS
// for each and an epilogue through LDS -> this way, us: 32 models at 224 x 224 (51 MB of output) 34.5 -> 26.3, 2
// models of 32 channels at 384 x 384 8.8 -> 7.8; over 6500 problems 18 % less time.
#pragma once
#include "conv_plane.h"

namespace nf {

struct ConvStemArgs {
  const bf16_t* x; const bf16_t* w; const bf16_t* R; bf16_t* y;
  int cog, nG, H, W, Ho, Wo, HoWo;
  int PW, PS;                 // patch row pitch and plane pitch (elements, multiples of 8)
  int cpr;                    // 8-pixel chunks per image row (W / 8)
  int tiles_m, tiles_n, run, runs;           // tiles per workgroup, workgroups per (image, model, channels)
  unsigned rcp_wo, one_wo, rcp_cpr, one_cpr; // division by Wo and cpr (cw_div)
  long x_group, x_image, y_group, y_image;   // element strides
  Epilogue ep;
};

template <int CIN, int BM>
struct ConvStemCfg {
  static constexpr int kKH = 7, kKW = 7, kStride = 2, kPad = 3, kColPad = 8;
  static_assert(BM == 64 || BM == 32, "two blocks of 32 channels or one");
  static constexpr int kBM = BM, kBN = 128, kThreads = 256;
  static constexpr int kWGN = 128 / BM, FN = BM / 32, WN = 32 * FN;    // wavefronts: 2 blocks of channels x 2 of 64 positions, or 4 of 32
  static constexpr int kRows = CIN * kKH;                 // (ci, ky) rows of the k dimension
  static constexpr int kSteps = (kRows + 1) / 2;          // MFMA steps of 16 k: two rows each
  static constexpr int kK = kSteps * 16;                  // padded k extent in LDS
  static constexpr int kAPitch = kK + 8;                  // elements; (pitch / 8) odd -> 16-byte slots rotate
  static_assert((kAPitch / 8) % 2 == 1, "A pitch must rotate bank groups");
  static constexpr int kAEls = kBM * kAPitch;
  static constexpr int lds_bytes(int PS) { return 2 * (2 * CIN * PS > kAEls ? 2 * CIN * PS : kAEls); }   // the patches take the weights' place
};

// NT: patch chunks per thread (the host checks the bound); up to 6 the registers allow three workgroups per compute unit
template <class Cfg, int CIN, int NT>
__global__ __launch_bounds__(256, NT > 6 ? 2 : 3) void conv_stem_kernel(ConvStemArgs a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  lds_bf16_t* const As = (lds_bf16_t*)smem_raw;
  lds_bf16_t* const Ps = As;                               // [buffer][channel][patch row][column]
  constexpr int FN = Cfg::FN, KHW = Cfg::kKH * Cfg::kKW, KW = Cfg::kKW;
  const int tid = threadIdx.x, lane = tid % kWave, wm = tid / kWave / Cfg::kWGN, wn = tid / kWave % Cfg::kWGN;
  const int half = lane / 32, l32 = lane % 32;

  unsigned id = xcd_remap(blockIdx.x, gridDim.x);
  const int tm = id % a.tiles_m;  id /= a.tiles_m;
  const int rn = id % a.runs;     id /= a.runs;
  const int G = id % a.nG;
  const int b = id / a.nG;
  const int row0 = tm * Cfg::kBM, rows_left = a.cog - row0;
  const int t0 = rn * a.run, t1 = min(t0 + a.run, a.tiles_n);
  const bf16_t* xg = a.x + (long)b * a.x_image + (long)G * a.x_group;
  const bf16_t* wg = a.w + ((long)G * a.cog + row0) * (CIN * KHW);

  // ---- this thread's chunks of a patch: 8 pixels, aligned on both sides
  const int PHM = a.PS / a.PW, nchunk = CIN * PHM * a.cpr;
  unsigned c_src[NT], c_at[NT];                                 // c_at: patch row << 16 | LDS element (below 40960, see lds_bytes)
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    const int t = tid + u * 256;
    const int row = (int)cw_div(t, a.rcp_cpr, a.one_cpr), ch = t - row * a.cpr;
    int ci = 0;
#pragma unroll
    for (int c = 1; c < CIN; ++c) ci += row >= c * PHM;
    c_src[u] = (unsigned)ci * (unsigned)(a.H * a.W) + ch * 8;
    c_at[u] = (row - ci * PHM) << 16 | (ci * a.PS + (row - ci * PHM) * a.PW + Cfg::kColPad + ch * 8);
  }
  auto first_row = [&](int tn) { return (int)cw_div(tn * Cfg::kBN, a.rcp_wo, a.one_wo); };
  uint4 pre[NT];
  auto fetch = [&](int tn) {
    const int iy0 = first_row(tn) * Cfg::kStride - Cfg::kPad;
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      const int iy = iy0 + (int)(c_at[u] >> 16);
      pre[u] = make_uint4(0u, 0u, 0u, 0u);
      if (tid + u * 256 < nchunk && (unsigned)iy < (unsigned)a.H) pre[u] = *reinterpret_cast<const uint4*>(xg + (c_src[u] + (long)iy * a.W));
    }
  };
  auto commit = [&](int buf) {
#pragma unroll
    for (int u = 0; u < NT; ++u)
      if (tid + u * 256 < nchunk) lds_store16(Ps + buf * CIN * a.PS + (c_at[u] & 0xffff), pre[u]);     // rows past the image: zeros
  };
  fetch(t0);

  // ---- weights: natural (co, ci, ky, kx) order in memory -> LDS column (ci*7 + ky)*8 + 1 + kx of row co, then registers.
  // Task = the 7 taps of one (co, ci, ky): contiguous in memory at element 7 * task (any 2-byte alignment),
  // contiguous in LDS behind the zero slot; one division per task.
  for (int c = tid; c < Cfg::kAEls / 8; c += 256) lds_store16(As + c * 8, make_uint4(0, 0, 0, 0));
  __syncthreads();
  {
    const int ntask = min(rows_left, Cfg::kBM) * Cfg::kRows;
    for (int task = tid; task < ntask; task += 256) {
      const int co = task / Cfg::kRows, r = task - co * Cfg::kRows;      // r = ci*7 + ky
      const bf16_t* src = wg + task * KW;
      lds_bf16_t* dst = As + co * Cfg::kAPitch + r * 8 + 1;
      bf16_t v[KW];
#pragma unroll
      for (int kx = 0; kx < KW; ++kx) v[kx] = src[kx];
#pragma unroll
      for (int kx = 0; kx < KW; ++kx) dst[kx] = v[kx];
    }
  }
  __syncthreads();
  bf16x8_t af[Cfg::kSteps];
#pragma unroll
  for (int s = 0; s < Cfg::kSteps; ++s) af[s] = *(const lds_bf16x8_t*)(As + (wm * 32 + l32) * Cfg::kAPitch + half * 8 + s * 16);
  __syncthreads();
  // the columns beside the image and slot 0 stay zero; a chunk of the image is written for every tile
  for (int c = tid; c < 2 * CIN * a.PS / 8; c += 256) lds_store16(Ps + c * 8, make_uint4(0, 0, 0, 0));
  __syncthreads();
  commit(0);
  __syncthreads();

  typedef __attribute__((address_space(3))) const uint32_t lds_cu32_t;
  const long rvo = (long)G * a.cog + row0;
  const long out0 = (long)b * a.y_image + (long)G * a.y_group + (long)row0 * a.HoWo;
  for (int tn = t0; tn < t1; ++tn) {
    const int buf = (tn - t0) & 1, p0 = tn * Cfg::kBN;
    if (tn + 1 < t1) fetch(tn + 1);
    // ---- per-lane gather bases: patch offsets of this lane's output positions (columns past the end are not stored)
    int pix[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int p = min(p0 + wn * Cfg::WN + j * 32 + l32, a.HoWo - 1);
      const int oy = (int)cw_div(p, a.rcp_wo, a.one_wo), ox = p - oy * a.Wo;
      pix[j] = buf * CIN * a.PS + (oy - first_row(tn)) * Cfg::kStride * a.PW + ox * Cfg::kStride + (Cfg::kColPad - Cfg::kPad - 1);
    }
    f32x16_t acc[1][FN];
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[0][j][r] = 0.f;
    int upper = half;                                        // taken up anew per tile, or the offsets below stay in 11 registers
    asm volatile("" : "+v"(upper));
#pragma unroll
    for (int s = 0; s < Cfg::kSteps; ++s) {
      // rows 2s (lower lane half) and 2s+1 (upper half); offsets are wave uniform, the choice is per lane
      constexpr int kRows = Cfg::kRows;
      const int r0 = 2 * s, r1 = 2 * s + 1 < kRows ? 2 * s + 1 : 2 * s;     // a missing last row re-reads row r0 (zero weights)
      const int off0 = (r0 / Cfg::kKH) * a.PS + (r0 % Cfg::kKH) * a.PW;
      const int off1 = (r1 / Cfg::kKH) * a.PS + (r1 % Cfg::kKH) * a.PW;
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        lds_cu32_t* src = (lds_cu32_t*)(Ps + pix[j] + (upper ? off1 : off0));  // even element index: 4-byte aligned
        uint32_t w0 = src[0], w1 = src[1], w2 = src[2], w3 = src[3];
        w0 &= 0xffff0000u;                                                   // slot 0 multiplies a zero weight: keep it finite
        if (2 * s + 1 >= kRows && upper) { w0 = 0; w1 = 0; w2 = 0; w3 = 0; }
        const uint4 v = make_uint4(w0, w1, w2, w3);
        acc[0][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, v), af[s], acc[0][j], 0, 0, 0);
      }
    }
    bf16_t* const C = a.y + out0 + p0;
    const bf16_t* const R = a.R ? a.R + out0 + p0 : nullptr;
    const int ncol = a.HoWo - p0;
    if (a.ep.act == NF_ACT_RELU) plane_epilogue<1, FN, NF_ACT_RELU>(acc, C, R, a.HoWo, a.ep, rvo, 32 * wm, wn * Cfg::WN, rows_left, ncol);
    else if (a.ep.act == NF_ACT_GELU) plane_epilogue<1, FN, NF_ACT_GELU>(acc, C, R, a.HoWo, a.ep, rvo, 32 * wm, wn * Cfg::WN, rows_left, ncol);
    else plane_epilogue<1, FN, NF_ACT_NONE>(acc, C, R, a.HoWo, a.ep, rvo, 32 * wm, wn * Cfg::WN, rows_left, ncol);
    if (tn + 1 < t1) commit(buf ^ 1);
    __syncthreads();
  }
}

}  // namespace nf
