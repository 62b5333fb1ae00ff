// Merged matmul (bf16) for any number of rows per model and any number of models: the direct-to-LDS contraction of
// gemm_dma.h with ragged tiles, a k split inside the workgroup, and a wide choice of tiles.
//
//   Y[z][i][j] = act(sum_k X[z][i][k] * W[z][k][j] + bias[z][j]) + residual[z][i][j]
//
// W row-major [K][Nout] (transposing LDS reads) or packed as operand fragments (PB, pack_kernels.h: every fragment is
// one direct-to-LDS load of 1 KB and one plain 16-byte LDS read).
//
// One workgroup per tile, NS - 1 stages in flight: a compute unit's time is the latency of its operand stream, so the
// rings are as deep as LDS allows (64 to 128 KB on their way) and the wavefronts many and small.
// KG > 1 (packed weights only): KG k-groups of WGM x WGN wavefronts share a tile, group q takes k-steps q, q + KG, ...
// through LDS stages of its own; the partial sums are added through LDS in ascending group order.  A wavefront
// that has its stages to itself needs no barrier in the loop: it waits for its own loads only.
// What bounds it: direct-to-LDS loads bring a compute unit about 45 bytes per ns here, half of what loads into registers
// bring the fragment kernel (gemm_frag.h), which therefore stays where its whole tiles fit.
//
// Ragged tiles: rows and column chunks outside the problem are fetched from the last valid one instead (no load is
// ever conditional) and never stored.
#pragma once
#include "gemm_stream.h"

namespace nf {

template <int FM_, int FN_, int WGM_, int WGN_, int KG_, int BK_, int NS_, int WPE_>
struct RingCfg {
  static constexpr int FM = FM_, FN = FN_, kWGM = WGM_, kWGN = WGN_, kKG = KG_, kBK = BK_, kNS = NS_;
  static constexpr int kWPE = WPE_;                                     // wavefronts per SIMD the registers are limited for
  static constexpr int WM = 32 * FM, WN = 32 * FN, kBM = WM * kWGM, kBN = WN * kWGN;
  static constexpr int kNW = kWGM * kWGN, kThreads = kNW * kKG * kWave;
  static_assert(kBK == 32 || kBK == 64, "A rows of 64 or 128 bytes per stage");
  static constexpr int kARow = kBK * 2, kBRow = kBN * 2;                // bytes per LDS row
  static constexpr int kABytes = kBM * kARow, kBBytes = kBK * kBRow, kStage = kABytes + kBBytes;
  static constexpr int kABlocks = kABytes / 1024, kBBlocks = kBBytes / 1024, kBlocks = kABlocks + kBBlocks;
  static constexpr int kMaxPer = (kBlocks + kNW - 1) / kNW, kRem = kBlocks % kNW;   // waves < kRem (or all) issue kMaxPer
  static_assert(kNS >= 2 && (kNS - 2) * kMaxPer < 64, "vmcnt has 6 bits");
  static constexpr int kLdsPipe = kKG * kNS * kStage;
  static constexpr int kLdsReduce = kKG > 1 ? kKG * kBM * kBN * 4 : 0;
  static constexpr int kLdsBytes = kLdsPipe > kLdsReduce ? kLdsPipe : kLdsReduce;
  static_assert(kLdsBytes <= 160 * 1024, "LDS");
  static constexpr int kACpr = kBK / 8, kARpi = 64 / kACpr, kARowsPer256 = 256 / kARow;
  static constexpr int kBCpr = kBN / 8;
  __device__ static __forceinline__ int swz_a(int row) { return (row / kARowsPer256) % kACpr; }
  // four consecutive k rows x 64 bytes, read together by 32 lanes of a transposing read, have to tile 256 bytes
  __device__ static __forceinline__ int swz_b(int krow) {
    if constexpr (kBRow % 256 == 0) return 4 * (krow % 4);
    else if constexpr (kBRow % 256 == 128) return 4 * (krow / 2 % 2);
    else return 0;
  }
};

// Epilogue of a convolution: act((acc + bias[row]) * scale[row] + shift[row] + residual), constants per output row.
template <int FM, int FN, int ACT>
__device__ __forceinline__ void conv_epilogue(const f32x16_t (&acc)[FM][FN], bf16_t* C, const bf16_t* R, long ldc, const Epilogue& ep,
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
    for (int p = 0; p < 2 * FN; ++p)
      rr[p] = R && 16 * p < left ? *reinterpret_cast<const uint4*>(R + off + 16 * p) : make_uint4(0u, 0u, 0u, 0u);
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
      if (16 * p < left) *reinterpret_cast<uint4*>(C + off + 16 * p) = make_uint4(o[0], o[1], o[2], o[3]);
    }
  }
}

// Partial sums of KG groups: every group leaves its accumulators in LDS ([group][wave][block][4-column group][lane],
// 16 bytes per lane), then group q finishes pieces q, q + KG, ... of its wave position's FM x FN x 2.
template <class Cfg, int ACT>
__device__ __forceinline__ void ring_reduce_epilogue(lds_f32_t* red, int w, int q, bf16_t* C, const bf16_t* R, long ldc,
                                                     const float* bias, int row0, int col0, int rows, int cols) {
  constexpr int kPieces = Cfg::FM * Cfg::FN * 2, kGroupFloats = Cfg::kNW * kPieces * 2 * kWave * 4;
  const int lane = threadIdx.x % kWave, half = lane / 32, l32 = lane % 32;
  for (int p = q; p < kPieces; p += Cfg::kKG) {
    const int i = p / 2 / Cfg::FN, j = p / 2 % Cfg::FN, qq = p % 2;
    const int cq = col0 + 32 * j + 16 * qq;
    float4 b0 = make_float4(0.f, 0.f, 0.f, 0.f), b1 = b0;
    if (bias) {
      if (cq + 8 <= cols) b0 = *reinterpret_cast<const float4*>(bias + cq + 4 * half);
      if (cq + 16 <= cols) b1 = *reinterpret_cast<const float4*>(bias + cq + 8 + 4 * half);
    }
    const lds_f32_t* src = red + ((w * kPieces + p) * 2 * kWave + lane) * 4;
    f32x4v_t s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
    for (int g = 0; g < Cfg::kKG; ++g) {
      s0 += *(const lds_f32x4_t*)(src + g * kGroupFloats);
      s1 += *(const lds_f32x4_t*)(src + g * kGroupFloats + kWave * 4);
    }
    const float a0[4] = {s0.x, s0.y, s0.z, s0.w}, a1[4] = {s1.x, s1.y, s1.z, s1.w};
    const int row = row0 + 32 * i + l32, c = cq + 8 * half;
    const bool ok = row < rows && c < cols;
    const long off = (long)row * ldc + c;
    const uint4 res = R && ok ? *reinterpret_cast<const uint4*>(R + off) : make_uint4(0u, 0u, 0u, 0u);
    const uint4 o = epi_piece<ACT>(a0, a1, b0, b1, res);
    if (ok) *reinterpret_cast<uint4*>(C + off) = o;
  }
}

// A, B: this problem's operands (B: row-major or packed); C, R, bias: this problem's output.  CONV: a pointwise
// convolution, A its weights, B its input planes, rvo the offset of its per-row constants.
template <class Cfg, bool PB, bool CONV>
__device__ __forceinline__ void gemm_ring_tile(const bf16_t* __restrict__ A, long lda, const bf16_t* __restrict__ B, long ldb, int K, lds_u8_t* smem,
                                               bf16_t* C, const bf16_t* R, long ldc, const float* bias, const Epilogue& ep, long rvo,
                                               int row0, int col0, int rows, int cols) {
  const int act = ep.act;
  constexpr int FM = Cfg::FM, FN = Cfg::FN, NS = Cfg::kNS, BK = Cfg::kBK, KG = Cfg::kKG, NW = Cfg::kNW;
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int q = wave / NW, w = wave % NW, wm = w / Cfg::kWGN, wn = w % Cfg::kWGN;
  const int half = lane / 32, l32 = lane % 32, l16 = lane % 16;
  lds_u8_t* const ring = smem + q * NS * Cfg::kStage;

  // this lane's chunk of each of its wave's blocks: a byte offset from the group's current k position (uniform)
  unsigned voff[Cfg::kMaxPer];
#pragma unroll
  for (int t = 0; t < Cfg::kMaxPer; ++t) {
    const int blk = t * NW + w;
    if (blk < Cfg::kABlocks) {
      const int r = blk * Cfg::kARpi + lane / Cfg::kACpr;
      const int c = (lane % Cfg::kACpr) ^ Cfg::swz_a(r);
      voff[t] = (unsigned)((long)min(row0 + r, rows - 1) * lda + c * 8) * 2u;
    } else if constexpr (PB) {
      const int bb = blk - Cfg::kABlocks, cb = min(col0 / 32 + bb / (BK / 16), cols / 32 - 1);
      voff[t] = (unsigned)(((long)cb * (K / 16) + bb % (BK / 16)) * 512 + lane * 8) * 2u;
    } else {
      const int flat = (blk - Cfg::kABlocks) * 64 + lane, kr = flat / Cfg::kBCpr;
      const int c = (flat % Cfg::kBCpr) ^ Cfg::swz_b(kr);
      voff[t] = (unsigned)((long)kr * ldb + min(col0 + c * 8, cols - 8)) * 2u;
    }
  }
  // k position of the next stage in A and B (bytes, uniform; an operand is smaller than 2 GB)
  const unsigned inc_a = KG * BK * 2, inc_b = PB ? KG * (BK / 16) * 1024 : KG * BK * (unsigned)ldb * 2;
  unsigned pa = (unsigned)q * BK * 2, pb = PB ? (unsigned)q * (BK / 16) * 1024 : (unsigned)q * BK * (unsigned)ldb * 2;
  // Loads through a buffer resource where a slice is more than one multiplication (see lds_rsrc): they let the multiplications of a
  // slice start while the next slice's reads are under way.
  constexpr bool kBuf = FM * FN > 1;
  const auto ra = lds_rsrc(A, (unsigned)((long)rows * lda * 2)), rb = lds_rsrc(B, (unsigned)((long)K * (PB ? cols : ldb) * 2));
  auto load = [&](bool weights, unsigned off, lds_u8_t* dst) {
    if constexpr (kBuf) {
      if (weights) __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, dst, 16, off, pb, 0, CONV ? 0 : kWeightCpol);
      else __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, dst, 16, off, pa, 0, 0);
    } else {
      if (weights) __builtin_amdgcn_global_load_lds((glb_u8_t*)((const char*)B + pb + off), dst, 16, 0, CONV ? 0 : kWeightCpol);
      else __builtin_amdgcn_global_load_lds((glb_u8_t*)((const char*)A + pa + off), dst, 16, 0, 0);
    }
  };
  const bool extra = Cfg::kRem == 0 || w < Cfg::kRem;
  auto issue_stage = [&](int slot) {
    lds_u8_t* stage = ring + slot * Cfg::kStage;
#pragma unroll
    for (int t = 0; t < Cfg::kMaxPer; ++t) {
      if (t + 1 < Cfg::kMaxPer || extra) {
        // activations keep the default cache policy, weights (read once per forward pass) are non-temporal
        load(t * NW + w >= Cfg::kABlocks, voff[t], stage + (t * NW + w) * 1024);
      }
    }
    pa += inc_a;
    pb += inc_b;
  };
  auto wait_landed = [&]() {
    if (extra) wait_vmcnt<(NS - 2) * Cfg::kMaxPer>(); else wait_vmcnt<(NS - 2) * (Cfg::kMaxPer - 1)>();
  };

  int a_off[FM], b_off[FN][PB ? 1 : 2];
#pragma unroll
  for (int i = 0; i < FM; ++i) a_off[i] = (wm * Cfg::WM + i * 32 + l32) * Cfg::kARow;
  const int a_swz = Cfg::swz_a(l32);
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    if constexpr (PB) {
      b_off[j][0] = Cfg::kABytes + (wn * FN + j) * (BK / 16) * 1024 + lane * 16;
    } else {
#pragma unroll
      for (int hl = 0; hl < 2; ++hl) {
        const int kr = 8 * half + l16 / 4 + 4 * hl;           // k rows advance by 16 per slice: same swizzle
        const int n = wn * Cfg::WN + j * 32 + ((lane / 16) % 2) * 16 + (l16 % 4) * 4;
        b_off[j][hl] = Cfg::kABytes + kr * Cfg::kBRow + (((n / 8) ^ Cfg::swz_b(kr)) * 16) + ((n / 4) % 2) * 8;
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

  const int nk = K / BK;
  const int n = (nk - q + KG - 1) / KG, nmax = (nk + KG - 1) / KG;     // steps of this group, of group 0
  for (int s = 0; s < NS - 1; ++s)
    if (s < n) issue_stage(s);
  // Fragments are double buffered: the LDS reads of the next 16-k slice are issued in front of the multiplications of the
  // current one, also across the stage boundary, so that the matrix pipe does not wait for them (lock-step wavefronts
  // that first read a whole stage and then multiplied it spent a third of the loop on the reads).
  constexpr int S = BK / 16;
  struct Frag { bf16x8_t a[FM], b[FN]; } fr[2];
  auto read_slice = [&](Frag& f, int slot, int kk) {
    const lds_u8_t* stage = ring + slot * Cfg::kStage;
#pragma unroll
    for (int i = 0; i < FM; ++i) f.a[i] = *(const lds_bf16x8_t*)(stage + a_off[i] + (((2 * kk + half) ^ a_swz) * 16));
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      if constexpr (PB) {
        f.b[j] = *(const lds_bf16x8_t*)(stage + b_off[j][0] + kk * 1024);
      } else {
        const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(stage + b_off[j][0] + kk * 16 * Cfg::kBRow));
        const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(stage + b_off[j][1] + kk * 16 * Cfg::kBRow));
        const s16x8_t both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        f.b[j] = __builtin_bit_cast(bf16x8_t, both);
      }
    }
  };
  auto multiply = [&](const Frag& f) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.b[j], f.a[i], acc[i][j], 0, 0, 0);
  };
  // stage g has landed (for this wave) once at most the loads of the younger stages in flight are pending
  auto landed = [&](int g) {
    if (g + NS - 2 < n) wait_landed(); else wait_vmcnt<0>();
    wait_lgkmcnt0();                                          // and this wave's own reads of the stage before are done
    if constexpr (NW > 1) __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  int slot = 0;
  landed(0);
  if (KG == 1 || n > 0) read_slice(fr[0], 0, 0);
  if (NS - 1 < n) issue_stage(NS - 1);
  for (int g = 0; g < nmax; ++g) {
    const bool live = KG == 1 || g < n;
    const int next = slot + 1 == NS ? 0 : slot + 1;
#pragma unroll
    for (int kk = 0; kk + 1 < S; ++kk) {
      if (live) {
        read_slice(fr[(kk + 1) & 1], slot, kk + 1);
        __builtin_amdgcn_sched_barrier(0);
        multiply(fr[kk & 1]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (g + 1 < nmax) {
      landed(g + 1);
      if (KG == 1 || g + 1 < n) read_slice(fr[0], next, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (live) multiply(fr[(S - 1) & 1]);
    __builtin_amdgcn_sched_barrier(0);
    if (g + NS < n) issue_stage(slot);                        // every wave is past its reads of this slot
    slot = next;
  }

  const int rw = row0 + wm * Cfg::WM, cw = col0 + wn * Cfg::WN;
  if constexpr (CONV) {
    static_assert(KG == 1, "no split k");
    if (act == NF_ACT_RELU) conv_epilogue<FM, FN, NF_ACT_RELU>(acc, C, R, ldc, ep, rvo, rw, cw, rows, cols);
    else if (act == NF_ACT_GELU) conv_epilogue<FM, FN, NF_ACT_GELU>(acc, C, R, ldc, ep, rvo, rw, cw, rows, cols);
    else conv_epilogue<FM, FN, NF_ACT_NONE>(acc, C, R, ldc, ep, rvo, rw, cw, rows, cols);
  } else if constexpr (KG == 1) {
    if (act == NF_ACT_GELU) reg_epilogue<FM, FN, NF_ACT_GELU>(acc, C, R, ldc, bias, rw, cw, rows, cols);
    else if (act == NF_ACT_RELU) reg_epilogue<FM, FN, NF_ACT_RELU>(acc, C, R, ldc, bias, rw, cw, rows, cols);
    else reg_epilogue<FM, FN, NF_ACT_NONE>(acc, C, R, ldc, bias, rw, cw, rows, cols);
  } else {
    __syncthreads();                                          // every group is done with the stages
    lds_f32_t* const red = (lds_f32_t*)smem;
    lds_f32_t* const dst = red + (((q * NW + w) * FM * FN) * 4 * kWave + lane) * 4;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
          *(lds_f32x4_t*)(dst + ((i * FN + j) * 4 + r4) * kWave * 4) =
              f32x4v_t{acc[i][j][4 * r4], acc[i][j][4 * r4 + 1], acc[i][j][4 * r4 + 2], acc[i][j][4 * r4 + 3]};
    __syncthreads();
    if (act == NF_ACT_GELU) ring_reduce_epilogue<Cfg, NF_ACT_GELU>(red, w, q, C, R, ldc, bias, rw, cw, rows, cols);
    else if (act == NF_ACT_RELU) ring_reduce_epilogue<Cfg, NF_ACT_RELU>(red, w, q, C, R, ldc, bias, rw, cw, rows, cols);
    else ring_reduce_epilogue<Cfg, NF_ACT_NONE>(red, w, q, C, R, ldc, bias, rw, cw, rows, cols);
  }
}

}  // namespace nf
