// float32 contraction on the bf16 matrix instructions: merged matmul, float32 storage.
//
//   C[z][i][j] = act(sum_k A[z][i][k] * B[z][k][j] + bias[z][j]) + R[z][i][j]
//
// A float32 is the sum of three bf16 numbers (24 bits of significand, 8 in each): x = x1 + x2 + x3 with x1 = bf16(x),
// x2 = bf16(x - x1), x3 = x - x1 - x2, every difference exact as long as the last bit of x3 is a bf16 number: bf16 has float32's exponents
// but ends at 2^-133 where float32 ends at 2^-149.  So both operands are multiplied by 2^24 first, which puts the last bit of ANY float32 at a normal
// bf16 number, and the sums by 2^-48 at the end.  Of the nine products of two such sums the six down to 2^-16 of the first are multiplied and
// summed in float32 on v_mfma_f32_16x16x32_bf16; the three left out come to 2^-28.2 of a product on average, at most 2^-24.2 (4 million drawn
// products).  Six bf16 instructions take 96 clocks for 16 x 16 x 32 products, the float32 ones (v_mfma_f32_16x16x4_f32) 256.  (bf16 splitting with
// six products: Henry, Tang, Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations", 2019.)
//
// A sum that is not finite (an operand that is not, or one of 2^104 and more, whose first part is infinite, or a sum of 2^80 and more on its way)
// is computed again from the operands themselves, on the float32 instructions: the wavefront that finishes it walks all of k once more for its 16
// rows.  8 models of 128 rows 3072 -> 768 with one row that holds an infinity 42 -> 82 us, with one in every row 86 (a walk of one lane per sum took 2260
// and 9370), 768 -> 2304 38 -> 64 and 73.
//
// A workgroup is four wavefronts, one per chain of k, that share nothing until their sums meet in LDS: no barrier couples them in the loop.
// B: a lane loads 8 rows of FN neighbouring columns straight into registers, where v_cvt_pk_bf16_f32 makes pairs along k of them, so nothing
// is transposed (column FN c + j of the tile is column c of block j).  A: 8 rows x 128 bytes per load, through LDS of the wavefront's own into
// the operand's layout: straight from memory a load touched 16 half lines, and that alone bounded the kernel (8 models of 128 rows
// 3072 -> 768: 41 us with loads and nothing else; per byte A cost 2.3 times what B did).  The splitting of a row block (6.5 instructions per
// element) is dealt out between the multiplications of the block before it: a lone wavefront issues a vector instruction every 6 clocks and
// both in one stretch each took 50 us there where this takes 38.  Loads are buffer loads of any 4-byte alignment whose resource covers
// one problem's operand: what lies past its end comes back as 0 (rows of k past the end, columns behind the last row).
//
// What bounds it: operands of 4 bytes from L2, 35 to 45 bytes per ns and compute unit, then issue slots.  Measured (8 models of 128 rows, us,
// gemm_f32.h -> this): 768 -> 2304 39.0 -> 32.5, 768 -> 768 15.8 -> 13.1, 768 -> 3072 43.7 -> 35.9, 3072 -> 768 49.4 -> 37.7; 12 models of 512 rows 768 ->
// 3072 230 -> 186, 3072 -> 768 239 -> 181; 1 model of 128 rows 3072 -> 768 21.5 -> 14.2.  The multiplication by 2^24 is 4 to 8 % of it (768 -> 2304 31.4 -> 33.0,
// 12 models of 512 rows 3072 -> 768 171 -> 181; without it the error is 3.5e-5 where an operand is 2^-120).
// Error against 64 bits (2-norm, K = 64, 768, 3072): 1.0e-7, 3.5e-7, 4.9e-7 -> 0.5e-7, 2.0e-7, 4.2e-7.
//
// Measured and dropped: stages of a 128 x 128 tile split once per workgroup and shared through LDS (1.3 us per 32 k: LDS traffic and the barrier,
// 203 us at 12 models of 512 rows 768 -> 3072, 259 with 3072 -> 768); eight chains of k in as many wavefronts (no change).
//
// One order of the sum for every tile: 32-k step n belongs to chain n mod 4, one chain per wavefront, and the chains are added
// in ascending order.
#pragma once
#include "gemm_dma.h"
#include "gemm_f32.h"

namespace nf {

template <int FM_, int FN_, int D_>
struct SplitCfg {
  static constexpr int FM = FM_, FN = FN_, D = D_;             // 16-row blocks, 16-column blocks, steps of loads in flight
  static constexpr int kBM = 16 * FM, kBN = 16 * FN, kKG = 4, kThreads = kKG * kWave, kBK = 32;
  static constexpr int kALoads = 2 * FM, kAStage = FM * 2048;   // 1 KB loads of a step's rows (8 rows x 128 bytes), bytes of a stage
  static constexpr int kLdsA = kKG * 2 * kAStage, kLdsSums = kKG * FM * FN * kWave * 16;
  static constexpr int kLdsBytes = kLdsA > kLdsSums ? kLdsA : kLdsSums;
  static_assert(D == 1 || D == 2, "one remainder step");
};

constexpr float kSplitScale = 0x1p24f, kSplitUnscale = 0x1p-48f, kSplitLargest = 3.402823466e38f;

// x, y (consecutive k) -> the three bf16 parts of 2^24 x, 2^24 y, packed in pairs
__device__ __forceinline__ void split3(float x, float y, uint32_t& p1, uint32_t& p2, uint32_t& p3) {
  x *= kSplitScale;
  y *= kSplitScale;
  p1 = pack_bf16x2(x, y);
  x -= __uint_as_float(p1 << 16);
  y -= __uint_as_float(p1 & 0xffff0000u);
  p2 = pack_bf16x2(x, y);
  x -= __uint_as_float(p2 << 16);
  y -= __uint_as_float(p2 & 0xffff0000u);
  p3 = pack_bf16x2(x, y);
}

struct SplitFrag { u32x4_t p[3]; };

template <int FN>
__device__ __forceinline__ void buf_load_cols(float (&v)[FN], __amdgpu_buffer_rsrc_t r, unsigned off) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
  static_assert(FN >= 2 && FN <= 4, "8, 12 or 16 bytes");
  if constexpr (FN == 4) {
    const u32x4_t t = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0);
#pragma unroll
    for (int j = 0; j < FN; ++j) v[j] = __uint_as_float(t[j]);
  } else if constexpr (FN == 3) {
    const u32x3 t = __builtin_amdgcn_raw_buffer_load_b96(r, (int)off, 0, 0);
#pragma unroll
    for (int j = 0; j < FN; ++j) v[j] = __uint_as_float(t[j]);
  } else {
    const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0);
#pragma unroll
    for (int j = 0; j < FN; ++j) v[j] = __uint_as_float(t[j]);
  }
}

// FN neighbouring columns of one output row: the residual that the epilogue reads, and the epilogue.
template <int FN>
struct SplitRow {
  typedef float vec_t __attribute__((ext_vector_type(FN)));
  vec_t res;
  long at;

  __device__ __forceinline__ void read(const GemmF32Args& a, int z, int row, int col) {
    at = z * a.sC0 + (long)row * a.ldc + col;
#pragma unroll
    for (int j = 0; j < FN; ++j) res[j] = 0.f;
    if (a.R) {
      if (col + FN <= a.cols) __builtin_memcpy(&res, a.R + at, sizeof(float) * FN);
      else
#pragma unroll
        for (int j = 0; j < FN; ++j)
          if (col + j < a.cols) res[j] = a.R[at + j];
    }
  }
  __device__ __forceinline__ void finish(const GemmF32Args& a, int col, const float (&v)[FN], const float (&bias)[FN]) const {
    vec_t out;
#pragma unroll
    for (int j = 0; j < FN; ++j) out[j] = apply_act(v[j] + bias[j], a.ep.act) + res[j];
    if (col + FN <= a.cols) __builtin_memcpy(a.C + at, &out, sizeof(float) * FN);
    else
#pragma unroll
      for (int j = 0; j < FN; ++j)
        if (col + j < a.cols) a.C[at + j] = out[j];
  }
};

// What lanes of a wavefront exchange through LDS: the hardware keeps a wavefront's LDS accesses in order, the compiler has to.
__device__ __forceinline__ void wave_lds_fence() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

// TAIL: K is no multiple of 32 (but of 4).
template <class Cfg, bool TAIL>
__global__ __launch_bounds__(Cfg::kThreads, 2) void gemm_split_kernel(GemmF32Args a) {
  constexpr int FM = Cfg::FM, FN = Cfg::FN, D = Cfg::D, KG = Cfg::kKG;
  extern __shared__ __align__(16) float smem[];
  const int lane = threadIdx.x % kWave, g = lane / 16, l16 = lane % 16;
  const int q = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);

  unsigned id = xcd_remap(blockIdx.x, gridDim.x);
  const int tm = id % a.tiles_m;  id /= a.tiles_m;
  const int tn = id % a.tiles_n;  id /= a.tiles_n;
  const int z = id;
  const int row0 = tm * Cfg::kBM, col0 = tn * Cfg::kBN;
  const __amdgpu_buffer_rsrc_t ra = f32_rsrc(a.A + z * a.sA0, a.a_bytes), rb = f32_rsrc(a.B + z * a.sB0, a.b_bytes);

  // A: load t is rows 8 t .. 8 t + 7, 128 bytes of each; through LDS of the wavefront's own, 16-byte chunks of a row exchanged by its
  // number, so that reads and writes meet every bank equally.  Rows past the end are the last one again.
  unsigned a_off[Cfg::kALoads];
#pragma unroll
  for (int t = 0; t < Cfg::kALoads; ++t) a_off[t] = (unsigned)(((long)min(row0 + 8 * t + lane / 8, a.rows - 1) * a.lda + lane % 8 * 4) * 4);
  lds_u8_t* const own_lds = (lds_u8_t*)smem + q * 2 * Cfg::kAStage;
  lds_u8_t* const a_to = own_lds + lane / 8 * 128;             // rows 8 t + lane / 8: exchanged by (row / 2) % 8 = 4 (t % 2) + lane / 16
  const int a_chunk = lane % 8;
  const lds_u8_t* const a_from = own_lds + l16 * 128;
  // columns past the end read what lies there (they are not stored)
  const unsigned pitch = (unsigned)a.ldb * 4u;
  const unsigned b_off = (unsigned)(8 * g) * pitch + (unsigned)(col0 + FN * l16) * 4u;

  u32x4_t ar[Cfg::kALoads];
  float bv[D][8][FN];
  auto load_a = [&](int k0) {
#pragma unroll
    for (int t = 0; t < Cfg::kALoads; ++t) {
      unsigned off = a_off[t] + (unsigned)k0 * 4u;
      if constexpr (TAIL) off = k0 + a_chunk * 4 < a.K ? off : kF32Oob;
      ar[t] = buf_load16(ra, off);
    }
  };
  auto write_a = [&](int stage) {
#pragma unroll
    for (int t = 0; t < Cfg::kALoads; ++t)
      *(lds_u32x4_t*)(a_to + stage * Cfg::kAStage + t * 1024 + ((a_chunk ^ (t % 2 * 4 + lane / 16)) * 16)) = ar[t];
  };
  auto load_b = [&](int slot, int k0) {
#pragma unroll
    for (int i = 0; i < 8; ++i) buf_load_cols<FN>(bv[slot][i], rb, b_off + (unsigned)(k0 + i) * pitch);
  };

  f32x4_t acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int nk = (a.K + 31) / 32, n = (nk - q + KG - 1) / KG;  // steps in all, of this wavefront
  auto k_of = [&](int s) { return (s * KG + q) * 32; };        // past the end: B comes back as 0 and is not used
  // Step s, u = s modulo 2: the rows of step s + 1 go to LDS and those of s + 2 are asked for, the columns of step s are split and
  // those of s + D asked for, and a row block at a time is read, split and multiplied.
  auto step = [&](int u, int s) {
    write_a(u ^ 1);
    load_a(k_of(s + 2));
    SplitFrag fb[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        uint32_t p1, p2, p3;
        split3(bv[u % D][2 * p][j], bv[u % D][2 * p + 1][j], p1, p2, p3);
        fb[j].p[0][p] = p1; fb[j].p[1][p] = p2; fb[j].p[2][p] = p3;
      }
    load_b(u % D, k_of(s + D));
    SplitFrag fa[2];
    f32x4v_t ax[2][2];
    auto read_a = [&](int i) {
#pragma unroll
      for (int c = 0; c < 2; ++c) ax[i % 2][c] = *(const lds_f32x4_t*)(a_from + u * Cfg::kAStage + i * 2048 + (((2 * g + c) ^ (l16 / 2)) * 16));
    };
    auto split_a = [&](int i) {
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          uint32_t p1, p2, p3;
          split3(ax[i % 2][c][2 * h], ax[i % 2][c][2 * h + 1], p1, p2, p3);
          fa[i % 2].p[0][2 * c + h] = p1; fa[i % 2].p[1][2 * c + h] = p2; fa[i % 2].p[2][2 * c + h] = p3;
        }
    };
    read_a(0);
    split_a(0);
    if (FM > 1) read_a(1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      constexpr int kPa[6] = {2, 0, 1, 1, 0, 0}, kPb[6] = {0, 2, 1, 0, 1, 0};      // smallest products first
      if (i + 2 < FM) read_a(i + 2);
#pragma unroll
      for (int t = 0; t < 6; ++t)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, fa[i % 2].p[kPa[t]]),
                                                              __builtin_bit_cast(bf16x8_t, fb[j].p[kPb[t]]), acc[i][j], 0, 0, 0);
      if (i + 1 < FM) split_a(i + 1);
#pragma unroll
      for (int t = 0; t < 6 * FN; ++t) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        if (i + 1 < FM) __builtin_amdgcn_sched_group_barrier(0x2, (52 + 6 * FN - 1) / (6 * FN), 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    wave_lds_fence();                                          // the next step's writes are behind this step's reads
  };
  load_a(k_of(0));
#pragma unroll
  for (int d = 0; d < D; ++d) load_b(d, k_of(d));
  write_a(0);
  load_a(k_of(1));
  wave_lds_fence();
  int s = 0;
  for (; s + 2 <= n; s += 2) {
    step(0, s);
    step(1, s + 1);
  }
  if (s < n) step(0, s);
  __syncthreads();                                             // the sums go where the stages were

  // Every wavefront leaves its sums in LDS ([chain][block][lane]) and finishes a quarter of the rows, whose residuals and constants are
  // on their way meanwhile.
  const int col = col0 + FN * l16;
  auto block_of = [&](int u) { return FM == 4 ? q : (q * FM + u) / 4; };        // of this wavefront's FM rows per lane
  auto row_of = [&](int u) { return 4 * g + (FM == 4 ? u : (q * FM + u) % 4); };
  SplitRow<FN> rows[FM];
  float bias[FN];
  const float* const cb = a.ep.col_bias ? a.ep.col_bias + z * a.ep.col_vec_stride0 : nullptr;
#pragma unroll
  for (int j = 0; j < FN; ++j) bias[j] = cb && col + j < a.cols ? cb[col + j] : 0.f;
#pragma unroll
  for (int u = 0; u < FM; ++u) {
    const int row = row0 + 16 * block_of(u) + row_of(u);
    if (row < a.rows && col < a.cols) rows[u].read(a, z, row, col);
  }
  lds_f32_t* const part = (lds_f32_t*)smem + lane * 4;
  constexpr int kChain = FM * FN * kWave * 4;
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
      *(lds_f32x4_t*)(part + q * kChain + (i * FN + j) * kWave * 4) = __builtin_bit_cast(f32x4v_t, acc[i][j]);
  __syncthreads();

  float sum[FM][FN];
  bool again = false;                                          // a sum that is infinite or NaN
  f32x4v_t own[FM == 4 ? FN : 1];
  if constexpr (FM == 4)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      f32x4v_t c[KG];
#pragma unroll
      for (int p = 0; p < KG; ++p) c[p] = *(const lds_f32x4_t*)(part + p * kChain + (q * FN + j) * kWave * 4);
      own[j] = ((c[0] + c[1]) + c[2]) + c[3];
    }
#pragma unroll
  for (int u = 0; u < FM; ++u)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      if constexpr (FM == 4) {
        sum[u][j] = own[j][u];
      } else {
        const lds_f32_t* src = part + (block_of(u) * FN + j) * kWave * 4 + row_of(u) - 4 * g;
        sum[u][j] = ((src[0] + src[kChain]) + src[2 * kChain]) + src[3 * kChain];
      }
      again |= !(fabsf(sum[u][j]) <= kSplitLargest) && row0 + 16 * block_of(u) + row_of(u) < a.rows && col + j < a.cols;
    }
  if (__any(again)) {
    // The 16 rows of which this wavefront finishes some once more, from the operands themselves, 16 k in ascending order at a time; in the block, too, the
    // sums of column c of block j are lane c's, so the values replaced are those that are not finite and no others.
    f32x4_t whole[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) whole[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const unsigned again_a = (unsigned)(((long)min(row0 + 16 * block_of(0) + l16, a.rows - 1) * a.lda + 4 * g) * 4);
    const unsigned again_b = (unsigned)(4 * g) * pitch + (unsigned)col * 4u;
    constexpr int kDeep = FN == 2 ? 3 : 2;                     // registers: no more than the loop above
    u32x4_t x[2][kDeep];
    float w[2][kDeep][4][FN];
    auto fetch = [&](int slot, int k0) {                       // past the end of k both operands are 0
#pragma unroll
      for (int i = 0; i < kDeep; ++i) {
        x[slot][i] = buf_load16(ra, k0 + 16 * i + 4 * g < a.K ? again_a + (unsigned)(k0 + 16 * i) * 4u : kF32Oob);
#pragma unroll
        for (int t = 0; t < 4; ++t) buf_load_cols<FN>(w[slot][i][t], rb, again_b + (unsigned)(k0 + 16 * i + t) * pitch);
      }
    };
    auto multiply = [&](int slot) {
#pragma unroll
      for (int i = 0; i < kDeep; ++i)
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int j = 0; j < FN; ++j)
            whole[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(x[slot][i][t]), w[slot][i][t][j], whole[j], 0, 0, 0);
    };
    fetch(0, 0);
    for (int k0 = 0; k0 < a.K; k0 += 32 * kDeep) {
      fetch(1, k0 + 16 * kDeep);
      __builtin_amdgcn_sched_barrier(0);
      multiply(0);
      fetch(0, k0 + 32 * kDeep);
      __builtin_amdgcn_sched_barrier(0);
      multiply(1);
    }
#pragma unroll
    for (int u = 0; u < FM; ++u)
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        float v = whole[j][0];
#pragma unroll
        for (int r = 1; r < 4; ++r) v = row_of(u) - 4 * g == r ? whole[j][r] : v;
        sum[u][j] = fabsf(sum[u][j]) <= kSplitLargest ? sum[u][j] * kSplitUnscale : v;
      }
  } else {
#pragma unroll
    for (int u = 0; u < FM; ++u)
#pragma unroll
      for (int j = 0; j < FN; ++j) sum[u][j] *= kSplitUnscale;
  }
#pragma unroll
  for (int u = 0; u < FM; ++u)
    if (row0 + 16 * block_of(u) + row_of(u) < a.rows && col < a.cols) rows[u].finish(a, col, sum[u], bias);
}

}  // namespace nf
