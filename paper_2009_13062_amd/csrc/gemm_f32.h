// float32 matrix-pipe contraction of the merged matmul and the merged convolution (float32 storage).
//
//   C[z][i][j] = sum_k A[z][i][k] * B[z][k][j]     fp32 products and sums, one fused epilogue
//
// The same reading of both operators as gemm_mfma.h (z = model, or model x group x image; A row-major with k
// contiguous; B k-major, for a convolution gathered from the input planes), on v_mfma_f32_16x16x4_f32.
//
// What bounds it: the fp32 matrix rate (256 flop per clock and compute unit, a sixteenth of bf16), so a k-step of
// a 64 x 64 tile takes 1024 clocks of matrix pipe for 16 KB of operands.  Operand traffic is therefore cheap, and
// the design spends it freely to take ANY shape: every global access is a buffer load whose resource covers
// exactly one problem's operand.  Whatever lies outside -- rows and columns of ragged tiles, k past the end, taps
// outside the image -- is given an offset outside that range and comes back as 0, so no load is ever conditional
// (the compiler then waits for one k-step at a time) and no problem can read another one's data.
//
// k order inside a 16-k slice: lane group g = lane / 16 takes k = 4 g .. 4 g + 3, and matrix instruction t uses
// element t of each group, so the A fragment of four instructions is ONE 16-byte LDS read.  B stays [k][j] as in
// memory, one 4-byte read per instruction; row pitches are congruent to 4 modulo 16 floats, which puts the four
// lane groups of either read on different LDS banks.  The product is computed transposed (the instruction's A
// operand is the B fragment) so that a lane ends up with 4 consecutive columns of one output row.
//
// D k-steps of loads are in flight in a ring of register slots while a double-buffered LDS stage is multiplied.
//
// One order of the sum for every tile: k-step n belongs to chain n mod CH, and the chains are added at the end, first
// those 2 apart, then the two sums.  Which tile runs depends on how many models (and images) are merged, and a model's
// bits must not, so CH follows from K alone; the tiles differ in how many groups of wavefronts the chains are dealt to.
//
// Measured (8 models, us; the plain FMA kernels -> this): pointwise 64 -> 256 at 56 x 56 460 -> 17.
// Matmuls of enough k are gemm_split.h's.  Of the convolutions it runs the pointwise ones, k x k but 3 x 3, and 3 x 3 over wide planes at
// stride 2 or groups that are no multiple of 8 channels; the other 3 x 3 ones are conv_wave.h's.  Narrow groups and few k over many rows stay with
// the FMA kernels (netfuse_api.hip).
//
// Rows of B of any length move 16 bytes at a time; those that are no multiple of 4 were gathered 4 bytes at a time (8 models, us: 2048 -> 512 over 7 x 7 27.6 ->
// 17.8, 512 -> 2048 with residual 20.7 -> 17.1, 256 -> 64 over 49 x 49 18.4 -> 13.0; 32 models of 384 rows 64 -> 1001 35 -> 30; 536 drawn problems: 27 % less
// time, none slower).
#pragma once
#include "gemm_launch.h"

namespace nf {

// KG groups of 4 wavefronts share a tile: group q takes k-steps q, q + KG, ... (chains q and, if there are more than
// KG, q + KG ...) through LDS stages of its own, and the partial sums meet in LDS at the end.  For tiles of which a
// compute unit gets only one (few models, small images): one wavefront per SIMD would wait out every load and LDS read.
template <int BM, int BN, int WGM, int WGN, int BK, int D, int CH, int KG = 1>
struct F32Cfg {
  static_assert(WGM * WGN == 4 && (CH == 2 || CH == 4) && CH % KG == 0, "4 wavefronts per group, whole chains");
  static constexpr int kBM = BM, kBN = BN, kWGM = WGM, kWGN = WGN, kBK = BK, kD = D, kKG = KG, kThreads = 256 * KG;
  static constexpr int kChains = CH / KG;                                           // accumulated by one wavefront
  static constexpr int kUnroll = D > kChains ? D : kChains;
  static constexpr int WM = BM / WGM, WN = BN / WGN, FM = WM / 16, FN = WN / 16;
  static_assert(WM % 16 == 0 && WN % 16 == 0 && BK % 16 == 0 && D % 2 == 0 && kUnroll % D == 0 && kUnroll % kChains == 0, "16 x 16 x 16 blocks, even ring");
  static constexpr int kPitchA = BK + 4, kPitchB = BN + 4;
  static constexpr int kStageA = BM * kPitchA, kStage = kStageA + BK * kPitchB;     // floats
  static constexpr int kLdsBytes = KG * 2 * kStage * 4;
  static_assert(kLdsBytes <= 160 * 1024 && (KG - 1) * BM * BN <= KG * 2 * kStage, "LDS");
  static_assert(BK == 32, "the chains are made of 32-k steps in every tile");
  static constexpr int kAChunks = BM * BK / 4, kAPer = (kAChunks + 255) / 256;
  static constexpr int kBChunks = BK * BN / 4, kBPer = (kBChunks + 255) / 256;
  static constexpr int kGPer = BK * BN / 256;                                       // gathered elements per thread
};

constexpr unsigned kF32Oob = 0x80000000u;   // a byte offset outside every operand
constexpr int kF32Dense = 0, kF32Gather = 1, kF32GatherWide = 2;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t f32_rsrc(const float* base, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ u32x4_t buf_load16(__amdgpu_buffer_rsrc_t r, unsigned off) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0);
}
__device__ __forceinline__ uint32_t buf_load4(__amdgpu_buffer_rsrc_t r, unsigned off) {
  return __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0);
}
// n / d, branch free; exact while n < 2^32 / d
__device__ __forceinline__ unsigned div_by(unsigned n, unsigned rcp, unsigned one) { return __umulhi(n, rcp) + (n & one); }

// KIND kF32Dense: B moves 4 columns at a time, at any 4-byte alignment; the columns past a row's end are the next row's first, or 0, and are
// not stored.  kF32Gather / kF32GatherWide: B through the convolution geometry,
// 4 bytes at a time, any shape, with at most 31 / 63 taps.  AVEC: K % 4 == 0, so A moves in whole 4-k chunks.
template <class Cfg, int KIND, bool AVEC>
__global__ __launch_bounds__(Cfg::kThreads, 2) void gemm_f32_kernel(GemmF32Args a) {   // 2: keeps the chains out of the
  // accumulation registers, where the compiler moves them about in the loop (4 % of a 64 x 64 tile's time)
  constexpr bool GATHER = KIND != kF32Dense;
  constexpr int BK = Cfg::kBK, D = Cfg::kD, FM = Cfg::FM, FN = Cfg::FN, BN = Cfg::kBN;
  constexpr int KG = Cfg::kKG;
  extern __shared__ __align__(16) float smem[];
  const int tid = threadIdx.x % 256, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int q = KG > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / 256) : 0;
  lds_f32_t* const lds = (lds_f32_t*)smem + q * 2 * Cfg::kStage;
  const int wm = wave / Cfg::kWGN, wn = wave % Cfg::kWGN;
  const int g = lane / 16, l16 = lane % 16;

  unsigned id = xcd_remap(blockIdx.x, gridDim.x);
  const int tm = id % a.tiles_m;  id /= a.tiles_m;
  const int tn = id % a.tiles_n;  id /= a.tiles_n;
  const int z0 = id % a.nz0, z1 = id / a.nz0;
  const int row0 = tm * Cfg::kBM, col0 = tn * BN;
  const __amdgpu_buffer_rsrc_t ra = f32_rsrc(a.A + z0 * a.sA0, a.a_bytes);
  const __amdgpu_buffer_rsrc_t rb = f32_rsrc(a.B + z0 * a.sB0 + z1 * a.sB1, a.b_bytes);

  // ---- A: chunk c = 4 consecutive k of one row
  unsigned a_base[Cfg::kAPer];
  int a_k[Cfg::kAPer];
#pragma unroll
  for (int t = 0; t < Cfg::kAPer; ++t) {
    const int c = tid + t * 256, r = row0 + c / (BK / 4);
    a_k[t] = c % (BK / 4) * 4;
    // a chunk of a row past the end never becomes valid: its k starts past K
    if (r >= a.rows || (Cfg::kAChunks % 256 != 0 && c >= Cfg::kAChunks)) a_k[t] += a.K;
    a_base[t] = (unsigned)(((long)r * a.lda + c % (BK / 4) * 4) * 4);
  }
  u32x4_t av[D][Cfg::kAPer];
  auto fetch_a = [&](int slot, int k0, int lo, int hi) {      // chunks lo .. hi - 1 of this thread
#pragma unroll
    for (int t = lo; t < hi; ++t) {
      const unsigned off = a_base[t] + (unsigned)k0 * 4u;
      if constexpr (AVEC) {
        av[slot][t] = buf_load16(ra, k0 + a_k[t] < a.K ? off : kF32Oob);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) av[slot][t][e] = buf_load4(ra, k0 + a_k[t] + e < a.K ? off + 4u * e : kF32Oob);
      }
    }
  };
  // ---- B, dense: chunk c = 4 consecutive columns of one k row
  unsigned b_base[GATHER ? 1 : Cfg::kBPer];
  int b_k[GATHER ? 1 : Cfg::kBPer];
  if constexpr (!GATHER) {
#pragma unroll
    for (int t = 0; t < Cfg::kBPer; ++t) {
      const int c = tid + t * 256, j = col0 + c % (BN / 4) * 4;
      b_k[t] = c / (BN / 4);
      b_base[t] = (unsigned)(((long)b_k[t] * a.ldb + j) * 4);
      if (j >= a.cols || (Cfg::kBChunks % 256 != 0 && c >= Cfg::kBChunks)) b_k[t] += a.K;
    }
  }
  u32x4_t bv[D][GATHER ? 1 : Cfg::kBPer];
  // ---- B, gathered: lane = output position, wavefront = k row, so that (channel, tap) of
  // a k is wave-uniform; each lane keeps which taps of its position lie OUTSIDE the image as bits, the last bit
  // (31 or 63, no tap) being set for the rows past the end of k.  An element then costs five vector instructions:
  // two broadcasts, the address, the bit as an all-ones word, and an `or` that throws the address out of range.
  constexpr int kNoTap = KIND == kF32GatherWide ? 63 : 31;
  unsigned p_off = 0, p_lo = ~0u, p_hi = ~0u;
  if constexpr (GATHER) {
    static_assert(BN == 64, "a wavefront of positions");
    const int p = col0 + lane;
    const int oy = p / a.Wo, ox = p - oy * a.Wo;
    const int iy0 = oy * a.stride - a.pad, ix0 = ox * a.stride - a.pad;
    p_off = (unsigned)(iy0 * a.W + ix0) * 4u;
    if (p < a.cols) {
      int ky = 0, kx = 0;
      for (int tap = 0; tap < a.khw; ++tap) {
        const int iy = iy0 + ky * a.dil, ix = ix0 + kx * a.dil;
        const unsigned in = iy >= 0 && iy < a.H && ix >= 0 && ix < a.W;
        if (tap < 32) p_lo ^= in << tap; else p_hi ^= in << (tap - 32);
        if (++kx == a.KW) { kx = 0; ++ky; }
      }
    }
  }
  uint32_t gv[D][GATHER ? Cfg::kGPer : 1];
  struct KSplit { int koff, bit; };
  auto split_k = [&](int k0) {                                // lane r splits k0 + r into (channel, tap) for everybody
    const unsigned k = (unsigned)(k0 + lane % BK);
    const unsigned ci = div_by(k, a.rcp_khw, a.one_khw), tap = k - ci * (unsigned)a.khw;
    const unsigned ky = div_by(tap, a.rcp_kw, a.one_kw), kx = tap - ky * (unsigned)a.KW;
    return KSplit{((int)ci * a.H * a.W + ((int)ky * a.W + (int)kx) * a.dil) * 4, k < (unsigned)a.K ? (int)tap : kNoTap};
  };
  auto fetch_b = [&](int slot, int k0, const KSplit& ks, int lo, int hi) {
    if constexpr (GATHER) {
#pragma unroll
      for (int e = lo; e < hi; ++e) {
        const int r = e * 4 + wave;
        const int b = __builtin_amdgcn_readlane(ks.bit, r);
        const unsigned word = KIND == kF32GatherWide && b >= 32 ? p_hi : p_lo;
        const unsigned out = (unsigned)__builtin_amdgcn_sbfe((int)word, (unsigned)b & 31u, 1u);
        gv[slot][e] = buf_load4(rb, (p_off + (unsigned)__builtin_amdgcn_readlane(ks.koff, r)) | out);
      }
    } else {
#pragma unroll
      for (int t = lo; t < hi; ++t)
        bv[slot][t] = buf_load16(rb, k0 + b_k[t] < a.K ? b_base[t] + (unsigned)k0 * (unsigned)a.ldb * 4u : kF32Oob);
    }
  };
  constexpr int kBPieces = GATHER ? Cfg::kGPer : Cfg::kBPer;
  auto commit_a = [&](int slot, int buf, int lo, int hi) {
    lds_f32_t* As = lds + buf * Cfg::kStage;
#pragma unroll
    for (int t = lo; t < hi; ++t) {
      const int c = tid + t * 256;
      if (Cfg::kAChunks % 256 == 0 || c < Cfg::kAChunks)
        *(lds_u32x4_t*)(As + c / (BK / 4) * Cfg::kPitchA + c % (BK / 4) * 4) = av[slot][t];
    }
  };
  auto commit_b = [&](int slot, int buf, int lo, int hi) {
    lds_f32_t* Bs = lds + buf * Cfg::kStage + Cfg::kStageA;
#pragma unroll
    for (int t = lo; t < hi; ++t) {
      if constexpr (GATHER) {
        Bs[(t * 4 + wave) * Cfg::kPitchB + lane] = __uint_as_float(gv[slot][t]);
      } else {
        const int c = tid + t * 256;
        if (Cfg::kBChunks % 256 == 0 || c < Cfg::kBChunks)
          *(lds_u32x4_t*)(Bs + c / (BN / 4) * Cfg::kPitchB + c % (BN / 4) * 4) = bv[slot][t];
      }
    }
  };

  constexpr int NC = Cfg::kChains;
  f32x4_t chain[NC][FM][FN];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) chain[c][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  f32x4_t (&acc)[FM][FN] = chain[0];
  const int a_off = (wm * Cfg::WM + l16) * Cfg::kPitchA + 4 * g;
  const int b_off = 4 * g * Cfg::kPitchB + wn * Cfg::WN + l16;
  // One k-step: stage i (LDS buffer `buf`) is multiplied, the loads of stage i + D go out into the slot that stage i
  // left, and stage i + 1 moves from its slot into the other buffer.  A step is BK / 4 groups of FM x FN matrix
  // instructions, and the other work is dealt out over the groups: issuing it takes the wavefront no longer than the
  // matrix pipe is busy with a group anyway.  The fragments of group n + 1 are read before group n is multiplied.
  auto step = [&](f32x4_t (&sum)[FM][FN], int buf, int slot, int k_fetch, int next_slot) {
    constexpr int G = BK / 4;
    const lds_f32_t* As = lds + buf * Cfg::kStage + a_off;
    const lds_f32_t* Bs = lds + buf * Cfg::kStage + Cfg::kStageA + b_off;
    f32x4v_t af[2][FM];
    float bf[2][FN];
    auto read_a = [&](int s) {
#pragma unroll
      for (int i = 0; i < FM; ++i) af[s & 1][i] = *(const lds_f32x4_t*)(As + i * 16 * Cfg::kPitchA + s * 16);
    };
    auto read_b = [&](int n) {
#pragma unroll
      for (int j = 0; j < FN; ++j) bf[n & 1][j] = Bs[(n / 4 * 16 + n % 4) * Cfg::kPitchB + j * 16];
    };
    read_a(0);
    read_b(0);
    KSplit ks{0, 0};
    if constexpr (GATHER) ks = split_k(k_fetch);
#pragma unroll
    for (int n = 0; n < G; ++n) {
      if (n + 1 < G) read_b(n + 1);
      if (n % 4 == 2 && n / 4 + 1 < BK / 16) read_a(n / 4 + 1);
      fetch_a(slot, k_fetch, n * Cfg::kAPer / G, (n + 1) * Cfg::kAPer / G);
      fetch_b(slot, k_fetch, ks, n * kBPieces / G, (n + 1) * kBPieces / G);
      if (n >= G / 2) {
        constexpr int H = G - G / 2;
        const int m = n - G / 2;
        commit_a(next_slot, buf ^ 1, m * Cfg::kAPer / H, (m + 1) * Cfg::kAPer / H);
        commit_b(next_slot, buf ^ 1, m * kBPieces / H, (m + 1) * kBPieces / H);
      }
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          sum[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(bf[n & 1][j], af[(n / 4) & 1][i][n % 4], sum[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // k-steps past the end load zeros and add nothing
  constexpr int U = Cfg::kUnroll;
  const int nst = ((a.K + BK * KG - 1) / (BK * KG) + U - 1) / U * U;
#pragma unroll
  for (int u = 0; u < D; ++u) {
    const int k0 = (u * KG + q) * BK;
    KSplit ks{0, 0};
    if constexpr (GATHER) ks = split_k(k0);
    fetch_a(u, k0, 0, Cfg::kAPer);
    fetch_b(u, k0, ks, 0, kBPieces);
    __builtin_amdgcn_sched_barrier(0);                       // slots are waited for in this order
  }
  commit_a(0, 0, 0, Cfg::kAPer);
  commit_b(0, 0, 0, kBPieces);
  __syncthreads();
  for (int i = 0; i < nst; i += U) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      step(chain[u % NC], u & 1, u % D, ((i + u + D) * KG + q) * BK, (u + 1) % D);
      __syncthreads();                                       // stage i + u + 1 is published, the buffer of stage i + u free
    }
  }
  auto add_to = [&](f32x4_t (&sum)[FM][FN], const f32x4_t (&other)[FM][FN]) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[i][j][e] += other[i][j][e];
  };
  if constexpr (NC == 4) { add_to(chain[0], chain[2]); add_to(chain[1], chain[3]); }
  if constexpr (NC >= 2) add_to(chain[0], chain[1]);
  if constexpr (KG > 1) {                                    // the stages are free: sums of groups 1 .. KG - 1 go there
    lds_f32_t* const part = (lds_f32_t*)smem + (wave * FM * FN * kWave + lane) * 4;
    constexpr int kGroup = 4 * FM * FN * kWave * 4;          // floats per group
    if (q > 0) {
#pragma unroll
      for (int i = 0; i < FM * FN; ++i)
        *(lds_f32x4_t*)(part + (q - 1) * kGroup + i * kWave * 4) = __builtin_bit_cast(f32x4v_t, acc[i / FN][i % FN]);
    }
    __syncthreads();
    if (q > 0) return;
#pragma unroll
    for (int i = 0; i < FM * FN; ++i) {
      f32x4v_t v[KG];
#pragma unroll
      for (int p = 1; p < KG; ++p) v[p] = *(const lds_f32x4_t*)(part + (p - 1) * kGroup + i * kWave * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (KG == 4) acc[i / FN][i % FN][e] = (acc[i / FN][i % FN][e] + v[2][e]) + (v[1][e] + v[3][e]);
        else acc[i / FN][i % FN][e] += v[1][e];
      }
    }
  }

  // ---- epilogue: lane = row l16 of a 16-row block, columns 4 g .. 4 g + 3 of a 16-column block
  const Epilogue& ep = a.ep;
  const long cz = z0 * a.sC0 + z1 * a.sC1;
  const float* cb = ep.col_bias ? ep.col_bias + z0 * ep.col_vec_stride0 : nullptr;
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int row = row0 + wm * Cfg::WM + i * 16 + l16;
    if (row >= a.rows) continue;
    const long rv = z0 * ep.row_vec_stride0 + row;
    const float rbias = ep.row_bias ? ep.row_bias[rv] : 0.f;
    const float rscale = ep.row_scale ? ep.row_scale[rv] : 1.f, rshift = ep.row_scale ? ep.row_shift[rv] : 0.f;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int col = col0 + wn * Cfg::WN + j * 16 + 4 * g;
      if (col >= a.cols) continue;
      const long o = cz + (long)row * a.ldc + col;
      f32x4_t v = acc[i][j];
      // 4 columns in one access, 4-byte aligned, but for the columns behind a row's last four (one by one, us:
      // pointwise 64 -> 256 with residual, 64 images at 49 x 49 182 -> 127; 32 models of 384 rows 64 -> 1001 52 -> 36).
      const bool whole = col + 4 <= a.cols;
      f32x4_t res = f32x4_t{0.f, 0.f, 0.f, 0.f}, bias = res;
      if (whole) {
        if (a.R) res = load_at<f32x4_t>(a.R + o);
      } else if (a.R) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (col + e < a.cols) res[e] = a.R[o + e];
      }
      if (cb) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (col + e < a.cols) bias[e] = cb[col + e];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float x = v[e] + rbias + bias[e];
        if (ep.row_scale) x = fmaf(x, rscale, rshift);
        v[e] = ep.act_before_residual ? apply_act(x, ep.act) + res[e] : apply_act(x + res[e], ep.act);
      }
      if (whole) {
        store_at(a.C + o, v);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (col + e < a.cols) a.C[o + e] = v[e];
      }
    }
  }
}

}  // namespace nf
