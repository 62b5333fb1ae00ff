// Pointwise convolution (bf16) over planes of any size, stride 1 or more: the direct-to-LDS contraction of gemm_ring.h for input
// planes that start at any element.
//
//   C[co][p] = sum_ci w[co][ci] * x[ci][oy*s][ox*s],   p = oy*Wo + ox
//
// The BK planes of a stage are one run of memory that starts 16 bytes aligned (BK planes are a multiple of 16 bytes), the
// single ones are not.  Loads to LDS move aligned 16-byte chunks, so the misalignment, the same for channel k in every stage,
// goes into the LDS addresses of the fragment reads:
//   * WHOLE: the tile spans the plane.  The run is copied as it lies, every line of it once.
//   * else CPR aligned chunks per channel that cover the tile's positions; stride 1: one segment of them, otherwise one per
//     output row.
//   * QUAD (planes of 4 k positions, stride 1): groups of four positions stay 8-byte aligned and transposing reads serve them.
//     Otherwise every element of a fragment is a 2-byte read of its own, eight per lane and 16 k.
// Chunks past a stage's own bytes are fetched from its last one instead; they hold nothing that is read.
//
// What bounds it: one wavefront issues an instruction every four clocks or so, and the 2-byte form takes about a hundred per 32 x 32
// block and 64 k (0.4 us per stage where a SIMD has one wavefront, whatever the depth of the ring), so the tiles are those with the
// most wavefronts per byte of weights (in the layers of ResNet-50 they fill 70 to 85 % of the issue slots, the 128-position tile of two
// wavefronts per SIMD 40 %); beyond that the weights' way from HBM (67 MB in 128-byte pieces and nothing else: 14 us).
// Reading a fragment's 2-byte elements a stage ahead, four channels interleaved in LDS so that transposing reads meet no
// bank twice, and rings of 4 to 9 stages were not faster; an epilogue through LDS, which moves whole aligned chunks, was slower
// than 16 bytes per lane at any element (25 x 25 planes 128 -> 512 13.0 against 9.4 us).
// The sum is one ascending chain as in gemm_mfma.h, so the choice between them changes no bit.
#pragma once
#include "conv_wave.h"
#include "gemm_launch.h"
#include "gemm_ring.h"

namespace nf {

struct ConvPlaneArgs : GemmArgs {            // ldb: positions of an input plane; geom: W, Wo, stride
  int step;                                  // positions per tile, a multiple of 8
  int cps;                                   // chunks per segment
  unsigned rcp_cps, one_cps, rcp_wo, one_wo; // division by cps and Wo (cw_div)
};

typedef __attribute__((address_space(3))) const uint16_t lds_u16_t;

template <int FM_, int FN_, int WGM_, int WGN_, int BK_, int CPR_, int NS_, int WPE_, bool QUAD_, bool WHOLE_, bool AHEAD_ = false>
struct PlaneCfg {
  static constexpr int FM = FM_, FN = FN_, kWGM = WGM_, kWGN = WGN_, kBK = BK_, kCpr = CPR_, kNS = NS_;
  static constexpr int kWPE = WPE_;                                     // wavefronts per SIMD the registers are limited for
  static constexpr bool kQuad = QUAD_, kWhole = WHOLE_;
  static constexpr bool kAhead = AHEAD_;                                // all of a stage's fragments are read under the stage before
  static constexpr int WM = 32 * FM, WN = 32 * FN, kBM = WM * kWGM, kBN = WN * kWGN;
  static constexpr int kNW = kWGM * kWGN, kThreads = kNW * kWave;
  static constexpr int kARow = kBK * 2, kABytes = kBM * kARow, kBBytes = kBK * kCpr * 16, kStage = kABytes + kBBytes;
  static constexpr int kABlocks = kABytes / 1024, kBBlocks = kBBytes / 1024, kBlocks = kABlocks + kBBlocks;
  static_assert(kBBlocks * 1024 == kBBytes && kABlocks * 1024 == kABytes, "whole 1 KB loads");
  static constexpr int kMaxPer = (kBlocks + kNW - 1) / kNW, kRem = kBlocks % kNW;
  static_assert(kNS >= 2 && (kNS - 2) * kMaxPer < 64, "vmcnt has 6 bits");
  static constexpr int kLdsBytes = kNS * kStage;
  static_assert(kLdsBytes <= 160 * 1024, "LDS");
  static constexpr int kACpr = kBK / 8, kARpi = 64 / kACpr, kARowsPer256 = 256 / kARow;
  __device__ static __forceinline__ int swz_a(int row) { return (row / kARowsPer256) % kACpr; }
};

// act((acc + bias[row]) * scale[row] + shift[row] + residual) over rows that start at any element, 16 bytes per access
template <int FM, int FN, int ACT>
__device__ __forceinline__ void plane_epilogue(const f32x16_t (&acc)[FM][FN], bf16_t* C, const bf16_t* R, long ldc, const Epilogue& ep,
                                               long rvo, int row0, int col0, int rows, int cols) {
  const int lane = threadIdx.x % kWave, half = lane / 32, l32 = lane % 32;
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int row = row0 + 32 * i + l32;
    const long off = (long)row * ldc + col0 + half * 8;
    const int left = row < rows ? cols - col0 - half * 8 : 0;
    const long rv = rvo + min(row, rows - 1);
    const float bias = ep.row_bias ? ep.row_bias[rv] : 0.f;
    const float scale = ep.row_scale ? ep.row_scale[rv] : 1.f, shift = ep.row_scale ? ep.row_shift[rv] : 0.f;
    uint4 rr[2 * FN];
#pragma unroll
    for (int p = 0; p < 2 * FN; ++p) {
      rr[p] = make_uint4(0u, 0u, 0u, 0u);
      const int here = left - 16 * p;
      if (R && here >= 8) rr[p] = load_at<uint4>(R + off + 16 * p);
      else if (R && here > 0) {
        bf16_t t[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) t[e] = e < here ? R[off + 16 * p + e] : (bf16_t)0;
        __builtin_memcpy(&rr[p], t, 16);
      }
    }
#pragma unroll
    for (int p = 0; p < 2 * FN; ++p) {
      float v[8];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float v0 = fmaf(acc[i][p / 2][8 * (p % 2) + e] + bias, scale, shift);
        const float v1 = fmaf(acc[i][p / 2][8 * (p % 2) + 4 + e] + bias, scale, shift);
        const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v0), __float_as_uint(v1), false, false);
        v[e] = __uint_as_float(s[0]);
        v[4 + e] = __uint_as_float(s[1]);
      }
      const uint32_t w[4] = {rr[p].x, rr[p].y, rr[p].z, rr[p].w};
      uint32_t o[4];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        o[e] = pack_bf16x2(act_const<ACT>(v[2 * e] + __uint_as_float(w[e] << 16)),
                           act_const<ACT>(v[2 * e + 1] + __uint_as_float(w[e] & 0xffff0000u)));
      const int here = left - 16 * p;
      if (here >= 8) store_at(C + off + 16 * p, make_uint4(o[0], o[1], o[2], o[3]));
      else if (here > 0) {
#pragma unroll
        for (int e = 0; e < 7; ++e)
          if (e < here) C[off + 16 * p + e] = (bf16_t)(o[e / 2] >> (16 * (e % 2)));
      }
    }
  }
}

template <class Cfg>
__device__ __forceinline__ void conv_plane_tile(const ConvPlaneArgs& a, lds_u8_t* smem) {
  constexpr int FM = Cfg::FM, FN = Cfg::FN, NS = Cfg::kNS, BK = Cfg::kBK, NW = Cfg::kNW, CPR = Cfg::kCpr;
  unsigned id = xcd_remap(blockIdx.x, gridDim.x);
  // consecutive ids: row tiles of one column tile, the next column tile, the next problem
  const int tm = id % a.tiles_m;  id /= a.tiles_m;
  const int tn = id % a.tiles_n;  id /= a.tiles_n;
  const int z = id % a.nz0, z1 = id / a.nz0;
  const int row0 = tm * Cfg::kBM, p0 = tn * a.step;
  const int rows = a.rows, ncol = min(a.cols - p0, a.step);
  const int lane = threadIdx.x % kWave;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), wm = w / Cfg::kWGN, wn = w % Cfg::kWGN;
  const int half = lane / 32, l32 = lane % 32, l16 = lane % 16;
  const int plane = (int)a.ldb, s = a.geom.stride, Wo = a.geom.Wo;
  const bool one_row = s == 1;                               // positions are then the plane's own elements
  const int oy0 = one_row ? 0 : (int)cw_div(p0, a.rcp_wo, a.one_wo);
  // first element, inside a channel's plane, of the segment of output row oy0 + seg
  auto seg_start = [&](int seg) { return one_row ? p0 : (oy0 + seg) * s * a.geom.W; };

  // this lane's chunk of each of its wave's blocks: a byte offset from the stage's start
  unsigned voff[Cfg::kMaxPer];
#pragma unroll
  for (int t = 0; t < Cfg::kMaxPer; ++t) {
    const int blk = t * NW + w;
    if (blk < Cfg::kABlocks) {
      const int r = blk * Cfg::kARpi + lane / Cfg::kACpr;
      const int c = (lane % Cfg::kACpr) ^ Cfg::swz_a(r);
      voff[t] = (unsigned)((long)min(row0 + r, rows - 1) * a.lda + c * 8) * 2u;
    } else {
      const int f = (blk - Cfg::kABlocks) * 64 + lane;
      unsigned at = (unsigned)f * 8u;
      if constexpr (!Cfg::kWhole) {
        const int k = f / CPR, c = f % CPR, seg = one_row ? 0 : (int)cw_div(c, a.rcp_cps, a.one_cps);
        at = ((unsigned)(k * plane + seg_start(seg)) & ~7u) + (unsigned)(c - seg * a.cps) * 8u;
      }
      voff[t] = min(at, (unsigned)(BK * plane) - 8u) * 2u;
    }
  }
  const unsigned inc_a = BK * 2, inc_b = BK * (unsigned)plane * 2;
  unsigned pa = 0, pb = 0;
  const auto ra = lds_rsrc(a.A + z * a.sA0, (unsigned)((long)rows * a.lda * 2));
  const auto rb = lds_rsrc(a.B + z * a.sB0 + z1 * a.sB1, (unsigned)((long)a.K * plane * 2));
  const bool extra = Cfg::kRem == 0 || w < Cfg::kRem;
  auto issue_stage = [&](int slot) {
    lds_u8_t* stage = smem + slot * Cfg::kStage;
#pragma unroll
    for (int t = 0; t < Cfg::kMaxPer; ++t)
      if (t + 1 < Cfg::kMaxPer || extra) {
        if (t * NW + w < Cfg::kABlocks) __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, stage + (t * NW + w) * 1024, 16, voff[t], pa, 0, 0);
        else __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, stage + (t * NW + w) * 1024, 16, voff[t], pb, 0, 0);
      }
    pa += inc_a;
    pb += inc_b;
  };
  auto wait_landed = [&]() {
    if (extra) wait_vmcnt<(NS - 2) * Cfg::kMaxPer>(); else wait_vmcnt<(NS - 2) * (Cfg::kMaxPer - 1)>();
  };
  const int n = a.K / BK;
  for (int g = 0; g < NS - 1; ++g)
    if (g < n) issue_stage(g);                               // under their trip: where this lane reads its fragments

  int a_off[FM];
#pragma unroll
  for (int i = 0; i < FM; ++i) a_off[i] = (wm * Cfg::WM + i * 32 + l32) * Cfg::kARow;
  const int a_swz = Cfg::swz_a(l32);
  constexpr int kBReads = Cfg::kQuad ? 2 : 8;
  const int slice = Cfg::kWhole ? 32 * plane : 256 * CPR;    // bytes of 16 channels
  int b_off[FN][kBReads];
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    const int col = wn * Cfg::WN + j * 32;                   // columns past the tile's read its last ones and are not stored
    if constexpr (Cfg::kQuad) {
      const int nn = min(col + ((lane / 16) % 2) * 16 + (l16 % 4) * 4, ncol - 4);
#pragma unroll
      for (int hl = 0; hl < 2; ++hl) {
        const int k = 8 * half + l16 / 4 + 4 * hl;
        b_off[j][hl] = Cfg::kABytes + (Cfg::kWhole ? k * plane + nn : k * CPR * 8 + ((k * plane) & 7) + nn) * 2;
      }
    } else {
      const int p = p0 + min(col + l32, ncol - 1);
      const int oy = one_row ? 0 : (int)cw_div(p, a.rcp_wo, a.one_wo), seg = oy - oy0;
      const int x = one_row ? p - p0 : (p - oy * Wo) * s;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int k = 8 * half + e;
        if constexpr (Cfg::kWhole) b_off[j][e] = Cfg::kABytes + (k * plane + oy * s * a.geom.W + x) * 2;
        else b_off[j][e] = Cfg::kABytes + ((k * CPR + seg * a.cps) * 8 + ((k * plane + seg_start(seg)) & 7) + x) * 2;
      }
    }
  }

  f32x16_t acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // Fragments are double buffered, as in gemm_ring.h: by slices of 16 k, or by whole stages.
  constexpr int S = BK / 16, D = Cfg::kAhead ? S : 1;
  struct Frag {
    bf16x8_t a[FM];
    s16x4_t q[FN][Cfg::kQuad ? 2 : 1];
    uint16_t u[FN][Cfg::kQuad ? 1 : 8];
  } fr[2][D];
  auto read_slice = [&](Frag& f, int slot, int kk) {
    const lds_u8_t* stage = smem + slot * Cfg::kStage;
#pragma unroll
    for (int i = 0; i < FM; ++i) f.a[i] = *(const lds_bf16x8_t*)(stage + a_off[i] + (((2 * kk + half) ^ a_swz) * 16));
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      if constexpr (Cfg::kQuad) {
#pragma unroll
        for (int hl = 0; hl < 2; ++hl)
          f.q[j][hl] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(stage + b_off[j][hl] + kk * slice));
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) f.u[j][e] = *(lds_u16_t*)(stage + b_off[j][e] + kk * slice);
      }
    }
  };
  auto multiply = [&](const Frag& f) {
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      bf16x8_t b;
      if constexpr (Cfg::kQuad) {
        b = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(f.q[j][0], f.q[j][1], 0, 1, 2, 3, 4, 5, 6, 7));
      } else {
        uint32_t o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (uint32_t)f.u[j][2 * e] | (uint32_t)f.u[j][2 * e + 1] << 16;
        __builtin_memcpy(&b, o, 16);
      }
#pragma unroll
      for (int i = 0; i < FM; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, f.a[i], acc[i][j], 0, 0, 0);
    }
  };
  // A stage has landed (for this wave) once at most the loads of the NS - 2 younger stages in flight are pending.
  auto landed = [&](bool full) {
    if (full) wait_landed(); else wait_vmcnt<0>();
    wait_lgkmcnt0();                                         // and this wave's own reads of the stage before are done
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  int slot = 0;
  landed(NS - 2 < n);
#pragma unroll
  for (int kk = 0; kk < D; ++kk) read_slice(fr[0][kk], 0, kk);
  if (NS - 1 < n) issue_stage(NS - 1);
  // One stage.  more: another follows; full: NS - 2 stages beyond that one are in flight; issue: the slot is filled again.
  auto stage = [&](Frag (&cur)[D], Frag (&nxt)[D], bool more, bool full, bool issue) {
    const int next = slot + 1 == NS ? 0 : slot + 1;
    if constexpr (Cfg::kAhead) {
      if (more) {
        landed(full);
#pragma unroll
        for (int kk = 0; kk < S; ++kk) read_slice(nxt[kk], next, kk);
      } else {
        wait_lgkmcnt0();
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kk = 0; kk < S; ++kk) multiply(cur[kk]);
    } else {
#pragma unroll
      for (int kk = 0; kk + 1 < S; ++kk) {
        read_slice(fr[(kk + 1) & 1][0], slot, kk + 1);
        __builtin_amdgcn_sched_barrier(0);
        multiply(fr[kk & 1][0]);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (more) {
        landed(full);
        read_slice(fr[0][0], next, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      multiply(fr[(S - 1) & 1][0]);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (issue) issue_stage(slot);                            // every wave is past its reads of this slot
    slot = next;
  };
  int g = 0;
  for (; g + 1 + NS < n; g += 2) {
    stage(fr[0], fr[1], true, true, true);
    stage(fr[1], fr[0], true, true, true);
  }
  for (; g < n; g += 2) {
    stage(fr[0], fr[1], g + 1 < n, g + NS - 1 < n, g + NS < n);
    if (g + 1 < n) stage(fr[1], fr[0], g + 2 < n, g + NS < n, g + 1 + NS < n);
  }

  const long coff = z * a.sC0 + z1 * a.sC1 + p0;
  const int rw = row0 + wm * Cfg::WM, cw = wn * Cfg::WN;
  bf16_t* const C = a.C + coff;
  const bf16_t* const R = a.R ? a.R + coff : nullptr;
  const long rvo = z * a.ep.row_vec_stride0;
  if (a.ep.act == NF_ACT_RELU) plane_epilogue<FM, FN, NF_ACT_RELU>(acc, C, R, a.ldc, a.ep, rvo, rw, cw, rows, ncol);
  else if (a.ep.act == NF_ACT_GELU) plane_epilogue<FM, FN, NF_ACT_GELU>(acc, C, R, a.ldc, a.ep, rvo, rw, cw, rows, ncol);
  else plane_epilogue<FM, FN, NF_ACT_NONE>(acc, C, R, a.ldc, a.ep, rvo, rw, cw, rows, ncol);
}

}  // namespace nf
