// float32 merged attention on the matrix pipe (v_mfma_f32_16x16x4_f32), head sizes up to 128 that are multiples of 4.
//
// Workgroup = QG groups of 16 query rows of one (model, sequence, head) times KS shares of the keys, a wavefront each; the keys pass KB at
// a time through one LDS stage, the next stage's loads being in flight in registers meanwhile, and a share is KB / KS of every stage.  Scores
// are computed transposed, S^T = K Q^T, with the k order of gemm_f32.h (lane group g = lane / 16 takes features 4 g .. + 3 of a
// 16-feature slice): a lane then holds 4 keys of ONE query per 16-key block, which is already the B operand of O^T = V^T P^T with key
// 4 g + t in instruction t.  Block i of V^T is features i, NB + i, 2 NB + i ..., so a lane reads NB neighbouring ones at once and ends up
// with 4 NB neighbouring outputs.  Loads are buffer loads over one head's rows; keys past the sequence and features past d come back as 0.
//
// Scores, mask and maximum stay in natural units, weights come from expf: in log2 units (one fma and v_exp_f32 per key, 10 to 15 % faster: 12 models of 512 tokens
// 96 against 111) scale and mask were rounded once more, which with a mask of ordinary numbers raised the error against 64 bits by up to 15 % (12 tokens
// 1.12e-7 -> 1.32e-7, 128 2.75e-7 -> 3.03e-7), weights below 2^-126 became 0, and scores past 2^31 gave NaN: the rounded maximum lay 2^7 and more beside
// the largest score.
//
// Bound by latency where the chip is not full, by the matrix pipe where it is (12 models x 512 tokens: 55 % of its 157 TFLOP/s).
// Measured (12 heads of 64, us; with bounds and mask looked up per key and V read 4 bytes at a time -> this): 2 models of 128 tokens
// 10.6 -> 9.4, 8 11.2 -> 10.3, 12 x 8 sequences 59 -> 58, 12 of 300 with a mask 50 -> 46, 12 of 512 117 -> 111, with a mask 124 -> 111.  Error against 64
// bits (2-norm): 64 tokens 2.87e-7 -> 2.85e-7, 128 3.35e-7 -> 3.32e-7, 512 5.04e-7 -> 4.99e-7; with a mask 2.08e-7 -> 2.04e-7, 2.80e-7 -> 2.75e-7, 4.90e-7 -> 4.72e-7.
#pragma once
#include "attention_kernels.h"
#include "gemm_f32.h"

namespace nf {

template <int NB, int KB, int QG, int KS>       // NB 16-feature blocks per head, KB keys per stage; wavefronts: QG query groups x KS shares of a stage
__global__ __launch_bounds__(QG * KS * kWave) void attention_f32_kernel(AttnArgs a, int qblocks, unsigned head_bytes) {
  constexpr int D = NB * 16, kPitch = D + 4;    // pitch congruent to 4 modulo 16: both reads spread over the LDS banks
  constexpr int kThreads = QG * KS * kWave;
  constexpr int kPer = KB * D / 4 / kThreads;   // 16-byte chunks per thread and tensor
  constexpr int kOwn = KB / 16 / KS;            // 16-key blocks of a stage per wavefront
  constexpr int kOut = NB / KS;                 // 4-feature pieces that a lane finishes
  static_assert(KB * D / 4 % kThreads == 0 && KB % (16 * KS) == 0 && NB % KS == 0, "whole chunks, blocks and pieces");
  constexpr int kStage = 2 * KB * kPitch, kShares = KS > 1 ? kThreads * (4 * NB + 2) : 0;
  __shared__ __align__(16) float smem[kStage > kShares ? kStage : kShares];
  __shared__ __align__(16) float mask_smem[KB];
  lds_f32_t* const Ks = (lds_f32_t*)smem;
  lds_f32_t* const Vs = Ks + KB * kPitch;
  lds_f32_t* const Ms = (lds_f32_t*)mask_smem;  // the key mask of a stage
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int g = lane / 16, l16 = lane % 16;
  const int share = wave / QG, key0 = share * kOwn * 16;       // of a stage
  unsigned id = xcd_remap(blockIdx.x, gridDim.x);
  const int qb = id % qblocks;  id /= qblocks;
  const int h = id % a.heads;   id /= a.heads;
  const int b = id % a.B;
  const int m = id / a.B;
  const long head_off = (long)m * a.stride_m + ((long)b * a.S) * a.stride_row + (long)h * a.d;
  const __amdgpu_buffer_rsrc_t rq = f32_rsrc((const float*)a.Q + head_off, head_bytes);
  const __amdgpu_buffer_rsrc_t rk = f32_rsrc((const float*)a.K + head_off, head_bytes);
  const __amdgpu_buffer_rsrc_t rv = f32_rsrc((const float*)a.V + head_off, head_bytes);
  const float* mk = a.mask ? a.mask + ((long)m * a.B + b) * a.S : nullptr;

  const int q = (qb * QG + wave % QG) * 16 + l16;
  f32x4_t qf[NB];
#pragma unroll
  for (int s = 0; s < NB; ++s) {
    const int f = 16 * s + 4 * g;
    qf[s] = __builtin_bit_cast(f32x4_t, buf_load16(rq, q < a.S && f < a.d ? (unsigned)(((long)q * a.stride_row + f) * 4) : kF32Oob));
  }

  u32x4_t kreg[kPer], vreg[kPer];
  float mreg = 0.f;
  auto fetch = [&](int j0) {
    if (mk) mreg = tid < KB && j0 + tid < a.S ? mk[j0 + tid] : 0.f;
#pragma unroll
    for (int t = 0; t < kPer; ++t) {
      const int c = tid + t * kThreads, key = j0 + c / (D / 4), f = c % (D / 4) * 4;
      const unsigned off = key < a.S && f < a.d ? (unsigned)(((long)key * a.stride_row + f) * 4) : kF32Oob;
      kreg[t] = buf_load16(rk, off);
      vreg[t] = buf_load16(rv, off);
    }
  };
  auto commit = [&]() {
    if (mk && tid < KB) Ms[tid] = mreg;
#pragma unroll
    for (int t = 0; t < kPer; ++t) {
      const int c = tid + t * kThreads, o = c / (D / 4) * kPitch + c % (D / 4) * 4;
      *(lds_u32x4_t*)(Ks + o) = kreg[t];
      *(lds_u32x4_t*)(Vs + o) = vreg[t];
    }
  };

  f32x4_t o_acc[NB];                            // element r of block i: feature NB (4 g + r) + i of query l16
#pragma unroll
  for (int i = 0; i < NB; ++i) o_acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float mrun = kLowest, lrun = 0.f;            // lrun: this lane's partial sum
  fetch(0);
  for (int j0 = 0; j0 < a.S; j0 += KB) {
    commit();
    if (j0 + KB < a.S) fetch(j0 + KB);
    __syncthreads();
    f32x4_t sc[kOwn];
#pragma unroll
    for (int kb = 0; kb < kOwn; ++kb) sc[kb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NB; ++s) {
      f32x4v_t kf[kOwn];
#pragma unroll
      for (int kb = 0; kb < kOwn; ++kb) kf[kb] = *(const lds_f32x4_t*)(Ks + (key0 + kb * 16 + l16) * kPitch + 16 * s + 4 * g);
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int kb = 0; kb < kOwn; ++kb) sc[kb] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[kb][t], qf[s][t], sc[kb], 0, 0, 0);
    }
    // element r of block kb: key j0 + key0 + 16 kb + 4 g + r of query l16
#pragma unroll
    for (int kb = 0; kb < kOwn; ++kb) {
      f32x4v_t mv = {0.f, 0.f, 0.f, 0.f};
      if (mk) mv = *(const lds_f32x4_t*)(Ms + key0 + kb * 16 + 4 * g);
#pragma unroll
      for (int r = 0; r < 4; ++r) sc[kb][r] = fmaf(sc[kb][r], a.scale, mv[r]);
    }
    if (j0 + KB > a.S) {                        // uniform: only the last stage has keys past the end
#pragma unroll
      for (int kb = 0; kb < kOwn; ++kb)
#pragma unroll
        for (int r = 0; r < 4; ++r) sc[kb][r] = j0 + key0 + kb * 16 + 4 * g + r < a.S ? sc[kb][r] : -INFINITY;   // weight 0 under any scale and mask
    }
    float mloc = kLowest;
#pragma unroll
    for (int kb = 0; kb < kOwn; ++kb)
#pragma unroll
      for (int r = 0; r < 4; ++r) mloc = fmaxf(mloc, sc[kb][r]);
    mloc = across_halves(across_rows(mloc, MaxOp{}), MaxOp{});
    const float mnew = fmaxf(mrun, mloc), corr = expf(mrun - mnew);
    mrun = mnew;
    lrun *= corr;
#pragma unroll
    for (int kb = 0; kb < kOwn; ++kb) {
#pragma unroll
      for (int r = 0; r < 4; ++r) sc[kb][r] = expf(sc[kb][r] - mnew);
      lrun += (sc[kb][0] + sc[kb][1]) + (sc[kb][2] + sc[kb][3]);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) o_acc[i][r] *= corr;
#pragma unroll
    for (int kb = 0; kb < kOwn; ++kb)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const lds_f32_t* vr = Vs + (key0 + kb * 16 + 4 * g + t) * kPitch + NB * l16;
        float v[NB];
        if constexpr (NB == 2) {
          v[0] = vr[0];
          v[1] = vr[1];
        } else {
#pragma unroll
          for (int i = 0; i < NB; i += 4) {
            const f32x4v_t w = *(const lds_f32x4_t*)(vr + i);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[i + e] = w[e];
          }
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) o_acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[i], sc[kb][t], o_acc[i], 0, 0, 0);
      }
    __syncthreads();                            // the stage is free
  }
  lrun = across_halves(across_rows(lrun, AddOp{}), AddOp{});
  // Feature 4 NB g + e of this lane's query is o_acc[e % NB][e / NB]; share s finishes pieces s kOut ... of four.
  f32x4v_t out[kOut];
  if constexpr (KS == 1) {
#pragma unroll
    for (int u = 0; u < kOut; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) out[u][r] = o_acc[(4 * u + r) % NB][(4 * u + r) / NB];
  } else {
    lds_f32_t* const max_of = Ks + kThreads * 4 * NB;
    lds_f32_t* const sum_of = max_of + kThreads;
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      f32x4v_t v;
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = o_acc[(4 * u + r) % NB][(4 * u + r) / NB];
      *(lds_f32x4_t*)(Ks + (u * kThreads + tid) * 4) = v;
    }
    max_of[tid] = mrun;
    sum_of[tid] = lrun;
    __syncthreads();
    const int first = tid % (QG * kWave);       // this lane in share 0
    float c[KS], top = kLowest;
#pragma unroll
    for (int s = 0; s < KS; ++s) top = fmaxf(top, max_of[first + s * QG * kWave]);
    lrun = 0.f;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      c[s] = expf(max_of[first + s * QG * kWave] - top);
      lrun = fmaf(sum_of[first + s * QG * kWave], c[s], lrun);
    }
#pragma unroll
    for (int u = 0; u < kOut; ++u) {
      out[u] = f32x4v_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const f32x4v_t v = *(const lds_f32x4_t*)(Ks + ((share * kOut + u) * kThreads + first + s * QG * kWave) * 4);
#pragma unroll
        for (int r = 0; r < 4; ++r) out[u][r] = fmaf(v[r], c[s], out[u][r]);
      }
    }
  }
  if (q >= a.S) return;
  float* Op = (float*)a.O + (((long)m * a.B + b) * a.S + q) * ((long)a.heads * a.d) + (long)h * a.d;
#pragma unroll
  for (int u = 0; u < kOut; ++u) {
    const int f = 4 * (NB * g + share * kOut + u);             // d is a multiple of 4: whole pieces only
    if (f < a.d) {
      f32x4v_t v;
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = out[u][r] / lrun;
      __builtin_memcpy(Op + f, &v, sizeof(v));
    }
  }
}

}  // namespace nf
