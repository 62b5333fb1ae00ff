// Merged 3 x 3 convolution (grouped, groups = M*g: Appendix A Eq. 2) over groups of 32 k input channels,
// bf16, as an implicit GEMM that reads BOTH MFMA operands with one aligned 16-byte LDS read per fragment.
//
//   C[co][p] = sum_{ci,ky,kx} w[co][ci][ky][kx] * xpad[ci][oy*s + ky][ox*s + kx],   p = oy*Wo + ox
//
// The k dimension of a block of 32 input channels is ordered tap-major: MFMA step (tap, g) covers channels
// 16 g .. 16 g + 15 of the block at tap (ky, kx), lane half h taking channels 16 g + 8 h .. + 7.  Both LDS
// tiles are laid out for that order while they are filled:
//   * the input patch of the tile's 128 output positions is kept channel-innermost, pixel (py, px) at
//     (py*PW + px) * 80 bytes holding its 32 channels (the 16 bytes of padding make consecutive pixels
//     rotate over the 64 LDS banks), so the 8 channels a lane needs at a tap are 16 contiguous bytes at
//     pixel(position) + tap offset, the offset being uniform over the wavefront;
//   * the weight tile holds row co as [tap][channel], so the A fragment of step (tap, g) is 16 contiguous
//     bytes as well.
// The reordering happens in registers between the global loads and the LDS writes: a weight task takes the
// 72 contiguous elements w[co][8 o .. 8 o + 7][0..8] (nine 16-byte loads) and writes nine 16-byte vectors,
// one per tap; a patch task takes VW pixels of 8 channel planes (eight loads) and writes VW 16-byte
// vectors, one per pixel.  Byte permutes with compile-time selectors do the shuffling.
// (conv_patch.h keeps the planes apart in LDS and gathers each tap of each channel with a 2-byte read:
// eight LDS reads per fragment, which bounds its 3x3 layers on small images.)
//
// It runs where many positions share a block's weights (planes beyond 14 x 14, narrow groups in pairs); small planes and many
// channels are conv_wave.h's (the rule and both sides' times: conv_wave_inst.hip).
//
// The patch carries its zero padding: it is zeroed once, and every channel block overwrites only the
// in-image pixels and clears the rows past the image.  Image column ix lives at patch column ix + kLPad.
//
// One workgroup = one (image, group, BM output channels) and a RUN of 128-position tiles, one where a group has many blocks
// (tap_run in conv_tap_inst.hip).  While a block is multiplied the next one of the tile, or the first of the next tile, is in flight in
// registers, and the outputs leave from registers (conv_plane.h's epilogue): single-block tiles of their own paid for their
// addresses, their zero fill and an empty memory pipe every time, and read the same weights again.  Per layer, a tile per workgroup and an
// epilogue through LDS -> this: 16 models' fused groups of 4 channels at 56 x 56 19.1 -> 14.7 us, of 8 at stride 2 from 56 x 56 25.9 ->
// 16.0; over 6000 problems of 32 to 512 channels 9 % less time, over 9000 of fused groups 21 %.
// Behind: one in a hundred of the former by 6 to 20 %, odd planes with a residual, whose 16-byte pieces straddle lines (64
// channels at 33 x 33 10.5 -> 12.4 us; through LDS 13 x 13 and 25 x 25 lose a tenth instead).
// What bounds it: no one pipe.  LDS is active for 15 to 35 % of the clocks (a fragment of each operand per MFMA at FM = FN = 1; a tenth to a
// half of that bank conflicts), a quarter to a half of the issue slots are filled; the rest is a block's commit, loads and multiplications behind
// two barriers with one or two wavefronts per SIMD.
#pragma once
#include "conv_patch.h"
#include "conv_plane.h"

namespace nf {

constexpr int kTapCB = 32;          // input channels per block
constexpr int kTapPixPitch = 40;    // elements per patch pixel (32 channels + 8)

template <int BM, int WGM, int WGN, int MINW = 1>
struct ConvTapCfg {
  static_assert(WGM * WGN == 4, "4 wavefronts");
  static constexpr int kBM = BM, kBN = 128, kWGM = WGM, kWGN = WGN, kThreads = 256;
  static constexpr int WM = BM / WGM, WN = kBN / WGN, FM = WM / 32, FN = WN / 32;
  static_assert(WM % 32 == 0 && WN % 32 == 0, "wave tile is made of 32x32 MFMA blocks");
  static constexpr int kTaps = 9;
  static constexpr int kAPitch = kTaps * kTapCB + 8;     // elements; (pitch / 8) odd -> 16-byte slots rotate
  static_assert((kAPitch / 8) % 2 == 1, "A pitch must rotate bank groups");
  static constexpr int kABytes = BM * kAPitch * 2;
  static constexpr int kWTasks = BM * (kTapCB / 8);      // weight tasks per block: (row, channel octet)
  static constexpr int kWPer = (kWTasks + 255) / 256;
  static constexpr int kMinWaves = MINW;
  static constexpr int lds_bytes(int PS) { return kABytes + PS * kTapPixPitch * 2; }
};

struct ConvTapArgs : ConvPatchArgs {
  int run, runs;                             // position tiles per workgroup, workgroups per (image, group, row tile)
  unsigned rcp_wo, one_wo;                   // division by Wo (cw_div)
};

// VW: pixels per patch chunk (= a.VW <= W).  NT: patch tasks per thread (the host checks the bound).
// kTapFused: S > 1 narrow groups (4, 8 or 16 channels each) share the single 32-channel block: the weight tile
// is block diagonal (row r carries its own group's channels at channel offset (r / cog_real) * cig_real,
// zeros elsewhere), filled once; see conv_patch.h for why no product crosses a group.
// kTapTile: several blocks, one tile per workgroup; kTapRun: any blocks, any run.
enum ConvTapKind { kTapRun, kTapTile, kTapFused };
template <class Cfg, int VW, int NT, int KIND>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(Cfg::kMinWaves))) void conv_tap_kernel(ConvTapArgs a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  lds_bf16_t* As = (lds_bf16_t*)smem_raw;
  lds_bf16_t* Ps = As + Cfg::kBM * Cfg::kAPitch;
  constexpr int FM = Cfg::FM, FN = Cfg::FN, CB = kTapCB, PP = kTapPixPitch;
  constexpr bool FUSED = KIND == kTapFused, TILE = KIND == kTapTile;
  constexpr int kDw = VW >= 2 ? VW / 2 : 1;            // dwords per loaded chunk
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int wm = wave / Cfg::kWGN, wn = wave % Cfg::kWGN;
  const int half = lane / 32, l32 = lane % 32;

  unsigned id = xcd_remap(blockIdx.x, gridDim.x);
  const int tm = id % a.tiles_m;  id /= a.tiles_m;
  const int rn = id % a.runs;     id /= a.runs;
  const int G = id % a.nG;
  const int b = id / a.nG;
  const int row0 = tm * Cfg::kBM, rows_left = a.cog - row0;
  const int t0 = TILE ? rn : rn * a.run, t1 = TILE ? t0 + 1 : min(t0 + a.run, a.tiles_n);
  const bf16_t* xg = a.x + (long)b * a.x_image + (long)G * a.x_group;
  const bf16_t* wg = a.w + ((long)G * a.cog + row0) * a.cig * 9;
  // ---- geometry of a tile's patch
  auto out_row = [&](int p) { return (int)cw_div(p, a.rcp_wo, a.one_wo); };
  auto last_of = [&](int tn) { return min((tn + 1) * Cfg::kBN, a.HoWo) - 1; };

  // ---- this thread's share of a channel block.  Weight task = (row, channel octet); patch task = (channel
  // octet, patch row, chunk of VW pixels).  The geometry does not change from block to block.
  int w_off[Cfg::kWPer], w_dst[Cfg::kWPer];                 // w_dst < 0: no such task
#pragma unroll
  for (int t = 0; t < Cfg::kWPer; ++t) {
    const int task = tid + t * 256, r = task / (CB / 8), o = task % (CB / 8);
    const bool live = Cfg::kWTasks % 256 == 0 || task < Cfg::kWTasks;
    w_off[t] = (min(r, rows_left - 1) * a.cig + 8 * o) * 9;  // rows past the end re-read the last one; never stored
    w_dst[t] = live ? r * Cfg::kAPitch + 8 * o : -1;
  }
  // ---- software pipeline over channel blocks: the global loads of block s+1 are in flight in registers
  // while block s is multiplied out of LDS
  uint32_t wv[Cfg::kWPer][36];
  uint32_t pv[NT][8][kDw];
  const long plane = (long)a.H * a.W;
  auto prefetch_w = [&](int ci0) {
#pragma unroll
    for (int t = 0; t < Cfg::kWPer; ++t) {
      if (FUSED || w_dst[t] < 0) continue;
      const bf16_t* p = wg + w_off[t] + (long)ci0 * 9;
#pragma unroll
      for (int q = 0; q < 9; ++q) {
        const uint4 v = *reinterpret_cast<const uint4*>(p + q * 8);
        wv[t][4 * q] = v.x; wv[t][4 * q + 1] = v.y; wv[t][4 * q + 2] = v.z; wv[t][4 * q + 3] = v.w;
      }
    }
  };
  // The first block's weights are requested before anything else: the index arithmetic below (a handful of
  // integer divisions per lane) and the zero fill of the patch then run under their trip from HBM instead of in
  // front of it (measured: 2.8 us from the start of a workgroup to its first load otherwise).
  prefetch_w(0);

  const int a_off = (wm * Cfg::WM + l32) * Cfg::kAPitch + half * 8;
  // offsets of this thread's chunks from the patch's first image row, in the image and in LDS; the tallest patch's
  int g_off[NT], l_off[NT], c_py[NT];
  {
    const int PHM = a.PS / a.PW, ntasks = (CB / 8) * PHM * a.cpr;
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      const int task = tid + u * 256;
      const int rest = task / a.cpr;
      // the last chunk of a row is pulled back to end with it: it writes some pixels a second time, with the same values
      const int ix = min((task - rest * a.cpr) * VW, a.W - VW);
      const int o = rest / PHM, py = rest - o * PHM;
      c_py[u] = task < ntasks ? py : 1 << 29;                // no chunk: a row that no patch has
      g_off[u] = (8 * o * a.H + py) * a.W + ix;
      l_off[u] = (py * a.PW + kLPad + ix) * PP + 8 * o;
    }
  }
  // zero the whole patch once: the columns beside the image are never written again
  for (int c = tid; c < a.PS * PP / 8; c += 256) lds_store16(Ps + c * 8, make_uint4(0, 0, 0, 0));

  int ph_next = 0, iy_next = 0;                              // rows of the patch that is on its way, its first image row
  auto live_row = [&](int u) { return c_py[u] < ph_next && (unsigned)(iy_next + c_py[u]) < (unsigned)a.H; };
  auto prefetch_x = [&](int tn, int ci0) {
    const int oy0 = out_row(tn * Cfg::kBN);
    iy_next = oy0 * a.stride - a.pad;
    ph_next = (out_row(last_of(tn)) - oy0) * a.stride + 3;   // <= PS / PW
    const bf16_t* xc = xg + (long)ci0 * plane + (long)iy_next * a.W;
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      if (!live_row(u)) continue;
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const bf16_t* p = xc + g_off[u] + c * plane;
        // rows and chunks start at any 2-byte address
        if constexpr (VW == 8) {
          const uint4 v = load_at<uint4>(p);
          pv[u][c][0] = v.x; pv[u][c][1] = v.y; pv[u][c][2] = v.z; pv[u][c][3] = v.w;
        } else if constexpr (VW == 4) {
          const uint2 v = load_at<uint2>(p);
          pv[u][c][0] = v.x; pv[u][c][1] = v.y;
        } else if constexpr (VW == 2) {
          pv[u][c][0] = load_at<uint32_t>(p);
        } else {
          pv[u][c][0] = *p;
        }
      }
    }
  };
  // selectors of perm(hi, lo, sel): 16 bits of `lo` (its low or high half) below 16 bits of `hi`
  auto pick = [](int lo_half, int hi_half) -> uint32_t {
    return (lo_half ? 0x0302u : 0x0100u) | ((hi_half ? 0x0706u : 0x0504u) << 16);
  };
  // Neighbouring lanes write VW pixels apart, 5 VW bank groups of 16 bytes: of the 16 groups, 16 lanes meet 2 (VW = 8), 4 or 8.  Every
  // other run of 16 / VW lanes therefore writes the two pixels of a pair in the other order, 5 groups off,
  // and twice as many are met, for no instruction more.  us: 64 channels at 56 x 56, 32 models 22.1 -> 20.9, 8 models 8.7 -> 7.9;
  // 16 models' fused groups of 4 channels 16.0 -> 14.7, of 8 at stride 2 17.9 -> 16.0.  (Swapping the pairs of VW = 8 as well, for a select
  // per dword, gave nothing more.)
  const bool flip = VW >= 2 && (tid * VW / 16) % 2;
  const uint32_t sel_even = flip ? pick(1, 1) : pick(0, 0), sel_odd = flip ? pick(0, 0) : pick(1, 1);
  const int swap = flip ? PP : 0;
  auto commit = [&](bool first, bool weights) {
#pragma unroll
    for (int t = 0; t < Cfg::kWPer; ++t) {
      if (FUSED || !weights || w_dst[t] < 0) continue;
#pragma unroll
      for (int tap = 0; tap < 9; ++tap) {
        uint32_t o[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int e0 = 9 * (2 * q) + tap, e1 = 9 * (2 * q + 1) + tap;     // elements (channel 2q, tap), (channel 2q+1, tap)
          o[q] = __builtin_amdgcn_perm(wv[t][e1 / 2], wv[t][e0 / 2], pick(e0 % 2, e1 % 2));
        }
        lds_store16(As + w_dst[t] + tap * CB, make_uint4(o[0], o[1], o[2], o[3]));
      }
    }
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      if (!live_row(u)) {
        if (first && c_py[u] < ph_next)                        // rows past the image: zero for all of the tile's blocks
          for (int i = 0; i < VW; ++i) lds_store16(Ps + l_off[u] + i * PP, make_uint4(0, 0, 0, 0));
        continue;
      }
#pragma unroll
      for (int i = 0; i < VW; ++i) {
        uint32_t o[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
          o[q] = __builtin_amdgcn_perm(pv[u][2 * q + 1][i / 2], pv[u][2 * q][i / 2], i % 2 ? sel_odd : sel_even);
        lds_store16(Ps + (i % 2 ? l_off[u] - swap : l_off[u] + swap) + i * PP, make_uint4(o[0], o[1], o[2], o[3]));
      }
    }
  };

  prefetch_x(t0, 0);
  if constexpr (FUSED) {
    for (int c = tid; c < Cfg::kBM * Cfg::kAPitch / 8; c += 256) lds_store16(As + c * 8, make_uint4(0, 0, 0, 0));
    __syncthreads();
    // task = (row, run of cw = 8 or 4 channels of the row's group): 9*cw contiguous weights, written as one
    // vector of cw channels per tap
    const int cw = a.cig_real >= 8 ? 8 : 4, subs = a.cig_real / cw;
    const bf16_t* ws = a.w + (long)G * a.cog * a.cig_real * 9;       // fused group G: rows G*cog .. of the weight tensor
    for (int task = tid; task < a.cog * subs; task += 256) {
      const int r = task / subs, sub = task - r * subs;
      const bf16_t* p = ws + ((long)r * a.cig_real + sub * cw) * 9;
      lds_bf16_t* dst = As + r * Cfg::kAPitch + (r / a.cog_real) * a.cig_real + sub * cw;
      uint32_t d[36];
      if (cw == 8) {
#pragma unroll
        for (int q = 0; q < 9; ++q) {
          const uint4 v = *reinterpret_cast<const uint4*>(p + q * 8);
          d[4 * q] = v.x; d[4 * q + 1] = v.y; d[4 * q + 2] = v.z; d[4 * q + 3] = v.w;
        }
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
          uint32_t o[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int e0 = 9 * (2 * q) + tap, e1 = 9 * (2 * q + 1) + tap;
            o[q] = __builtin_amdgcn_perm(d[e1 / 2], d[e0 / 2], pick(e0 % 2, e1 % 2));
          }
          lds_store16(dst + tap * CB, make_uint4(o[0], o[1], o[2], o[3]));
        }
      } else {
#pragma unroll
        for (int q = 0; q < 9; ++q) {
          const uint2 v = *reinterpret_cast<const uint2*>(p + q * 4);
          d[2 * q] = v.x; d[2 * q + 1] = v.y;
        }
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
          uint32_t o[2];
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int e0 = 9 * (2 * q) + tap, e1 = 9 * (2 * q + 1) + tap;
            o[q] = __builtin_amdgcn_perm(d[e1 / 2], d[e0 / 2], pick(e0 % 2, e1 % 2));
          }
          lds_store8(dst + tap * CB, o[0], o[1]);
        }
      }
    }
  }
  const long out0 = (long)b * a.y_image + (long)G * a.y_group + (long)row0 * a.HoWo;
  const long rvo = (long)G * a.cog + row0;
  const bool one_block = !TILE && a.cig == CB;             // its weights stay in LDS for the whole run
  // Several blocks.  The compiler cannot tell that no load is on its way any more once a block has been written to LDS (rows past the image
  // skip their part of a commit) and waits for a block's weights in the middle of issuing its pixel loads, whose addresses it builds in
  // registers that it takes to be still waiting.  Two ways to tell it so:
  //   kTapTile: a wait after the commit, where there is nothing to wait for.  us: 32 models, 256 channels, 28 -> 14 at stride 2 31.4 -> 29.4, 128
  //   channels, 56 -> 28 26.8 -> 25.8; over 260 problems of two and three tasks per thread 3 to 5 % less time (6 % more once).  With one task per
  //   thread that form is behind by as much (96 channels at 24 x 24 and 32 x 32 a tenth).
  //   One task per thread, 64 rows, three blocks and more: a wait in front of the barrier.  24 models, 96 channels at 33 x 33 17.3 -> 15.6 us, 8 models of
  //   4 images, 128 at 28 x 28 5 %; two blocks up to 5 % the other way, 32 rows and stride 2 2 %.
  auto none_on_the_way = [] { __builtin_amdgcn_s_waitcnt(0x0f70); };     // vmcnt(0)
  const bool wait = !TILE && Cfg::kBM == 64 && NT == 1 && a.cig > 2 * CB;
  auto landed = [&] { if (wait) none_on_the_way(); };
  landed();
  __syncthreads();                                         // the zero fills are complete
  for (int tn = t0; tn < t1; ++tn) {
    const int p0 = tn * Cfg::kBN, p_last = last_of(tn), oy_first = out_row(p0);
    // ---- fragment addresses (elements): per-lane base + wave-uniform (tap, channel group) offset
    int b_off[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int p = min(p0 + wn * Cfg::WN + j * 32 + l32, p_last);     // clamp: columns past the end are discarded
      const int oy = out_row(p), ox = p - oy * a.Wo;
      b_off[j] = (((oy - oy_first) * a.stride) * a.PW + ox * a.stride + (kLPad - a.pad)) * PP + half * 8;
    }
    f32x16_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    for (int ci0 = 0; ci0 < a.cig; ci0 += CB) {
      commit(ci0 == 0, TILE || !one_block || tn == t0);
      __syncthreads();
      // the next block, or the next tile's first one, is on its way while this one is multiplied
      const bool last = ci0 + CB == a.cig;
      const int ci_next = last ? 0 : ci0 + CB;
      if constexpr (TILE) {
        if (!last) {
          none_on_the_way();
          prefetch_w(ci_next);
          prefetch_x(tn, ci_next);
        }
      } else if (!last || tn + 1 < t1) {
        if (!one_block) prefetch_w(ci_next);
        prefetch_x(last ? tn + 1 : tn, ci_next);
      }
#pragma unroll
      for (int tap = 0; tap < 9; ++tap) {
        const int tap_off = ((tap / 3) * a.PW + tap % 3) * PP;           // wave-uniform
#pragma unroll
        for (int g = 0; g < CB / 16; ++g) {
          bf16x8_t af[FM], bfr[FN];
#pragma unroll
          for (int i = 0; i < FM; ++i) af[i] = *(const lds_bf16x8_t*)(As + a_off + i * 32 * Cfg::kAPitch + tap * CB + g * 16);
#pragma unroll
          for (int j = 0; j < FN; ++j) bfr[j] = *(const lds_bf16x8_t*)(Ps + b_off[j] + tap_off + g * 16);
#pragma unroll
          for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[j], af[i], acc[i][j], 0, 0, 0);
        }
      }
      landed();
      __syncthreads();
    }
    bf16_t* const C = a.y + out0 + p0;
    const bf16_t* const R = a.R ? a.R + out0 + p0 : nullptr;
    const int rw = wm * Cfg::WM, cw = wn * Cfg::WN, ncol = a.HoWo - p0;
    if (a.ep.act == NF_ACT_RELU) plane_epilogue<FM, FN, NF_ACT_RELU>(acc, C, R, a.HoWo, a.ep, rvo, rw, cw, rows_left, ncol);
    else if (a.ep.act == NF_ACT_GELU) plane_epilogue<FM, FN, NF_ACT_GELU>(acc, C, R, a.HoWo, a.ep, rvo, rw, cw, rows_left, ncol);
    else plane_epilogue<FM, FN, NF_ACT_NONE>(acc, C, R, a.HoWo, a.ep, rvo, rw, cw, rows_left, ncol);
  }
}

}  // namespace nf
