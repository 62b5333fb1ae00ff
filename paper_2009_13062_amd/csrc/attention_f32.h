// float32 merged attention on the matrix pipe (v_mfma_f32_16x16x4_f32), head sizes up to 128 that are multiples of 4.
//
// Workgroup = 4 wavefronts = 64 query rows of one (model, sequence, head); a wavefront owns 16 of them and walks the
// keys KB at a time through one LDS stage, the next block's loads being in flight in registers meanwhile.  Scores are
// computed transposed, S^T = K Q^T, with the k order of gemm_f32.h (lane group g = lane / 16 takes features 4 g .. + 3
// of a 16-feature slice): a lane then holds 4 keys of ONE query per 16-key block, which is already the B operand of
// O^T = V^T P^T with key 4 g + t in instruction t.  Loads are buffer loads over one head's rows; keys past the
// sequence and features past d come back as 0.
//
// Bound by latency at the sizes it is used at (8 models x 12 heads x 128 tokens: 192 workgroups, 3.4 us of matrix
// pipe each); the wavefront-per-query kernel it replaces there reads every key row once per query.
#pragma once
#include "attention_kernels.h"
#include "gemm_f32.h"

namespace nf {

constexpr int kAttnF32Queries = 64;

template <int NB, int KB>                       // NB 16-feature blocks per head, KB keys per stage
__global__ __launch_bounds__(256) void attention_f32_kernel(AttnArgs a, int qblocks, unsigned head_bytes) {
  constexpr int D = NB * 16, kPitch = D + 4;    // pitch congruent to 4 modulo 16: both reads spread over the LDS banks
  constexpr int kPer = KB * D / 4 / 256;        // 16-byte chunks per thread and tensor
  static_assert(KB * D / 4 % 256 == 0 && KB % 16 == 0, "whole chunks per thread");
  __shared__ __align__(16) float smem[2 * KB * kPitch];
  lds_f32_t* const Ks = (lds_f32_t*)smem;
  lds_f32_t* const Vs = Ks + KB * kPitch;
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int g = lane / 16, l16 = lane % 16;
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

  const int q = qb * kAttnF32Queries + wave * 16 + l16;
  f32x4_t qf[NB];
#pragma unroll
  for (int s = 0; s < NB; ++s) {
    const int f = 16 * s + 4 * g;
    qf[s] = __builtin_bit_cast(f32x4_t, buf_load16(rq, q < a.S && f < a.d ? (unsigned)(((long)q * a.stride_row + f) * 4) : kF32Oob));
  }

  u32x4_t kreg[kPer], vreg[kPer];
  auto fetch = [&](int j0) {
#pragma unroll
    for (int t = 0; t < kPer; ++t) {
      const int c = tid + t * 256, key = j0 + c / (D / 4), f = c % (D / 4) * 4;
      const unsigned off = key < a.S && f < a.d ? (unsigned)(((long)key * a.stride_row + f) * 4) : kF32Oob;
      kreg[t] = buf_load16(rk, off);
      vreg[t] = buf_load16(rv, off);
    }
  };
  auto commit = [&]() {
#pragma unroll
    for (int t = 0; t < kPer; ++t) {
      const int c = tid + t * 256, o = c / (D / 4) * kPitch + c % (D / 4) * 4;
      *(lds_u32x4_t*)(Ks + o) = kreg[t];
      *(lds_u32x4_t*)(Vs + o) = vreg[t];
    }
  };

  f32x4_t o_acc[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) o_acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float mrun = kLowest, lrun = 0.f;            // lrun: this lane's partial sum
  fetch(0);
  for (int j0 = 0; j0 < a.S; j0 += KB) {
    commit();
    if (j0 + KB < a.S) fetch(j0 + KB);
    __syncthreads();
    f32x4_t sc[KB / 16];
#pragma unroll
    for (int kb = 0; kb < KB / 16; ++kb) sc[kb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NB; ++s) {
      f32x4v_t kf[KB / 16];
#pragma unroll
      for (int kb = 0; kb < KB / 16; ++kb) kf[kb] = *(const lds_f32x4_t*)(Ks + (kb * 16 + l16) * kPitch + 16 * s + 4 * g);
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int kb = 0; kb < KB / 16; ++kb) sc[kb] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[kb][t], qf[s][t], sc[kb], 0, 0, 0);
    }
    // element r of block kb: key j0 + 16 kb + 4 g + r of query l16
    float mloc = kLowest;
#pragma unroll
    for (int kb = 0; kb < KB / 16; ++kb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int key = j0 + kb * 16 + 4 * g + r;
        sc[kb][r] = key < a.S ? sc[kb][r] * a.scale + (mk ? mk[key] : 0.f) : kLowest;
        mloc = fmaxf(mloc, sc[kb][r]);
      }
    mloc = across_halves(across_rows(mloc, MaxOp{}), MaxOp{});
    const float mnew = fmaxf(mrun, mloc), corr = expf(mrun - mnew);
    mrun = mnew;
    lrun *= corr;
#pragma unroll
    for (int kb = 0; kb < KB / 16; ++kb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float p = j0 + kb * 16 + 4 * g + r < a.S ? expf(sc[kb][r] - mnew) : 0.f;
        sc[kb][r] = p;
        lrun += p;
      }
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) o_acc[i][r] *= corr;
#pragma unroll
    for (int kb = 0; kb < KB / 16; ++kb)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const lds_f32_t* vr = Vs + (kb * 16 + 4 * g + t) * kPitch + l16;
#pragma unroll
        for (int i = 0; i < NB; ++i) o_acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(vr[16 * i], sc[kb][t], o_acc[i], 0, 0, 0);
      }
    __syncthreads();                            // the stage is free
  }
  lrun = across_halves(across_rows(lrun, AddOp{}), AddOp{});
  if (q >= a.S) return;
  float* Op = (float*)a.O + (((long)m * a.B + b) * a.S + q) * ((long)a.heads * a.d) + (long)h * a.d;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int f = 16 * i + 4 * g;               // d is a multiple of 4: whole pieces only
    if (f < a.d) {
#pragma unroll
      for (int r = 0; r < 4; ++r) Op[f + r] = o_acc[i][r] / lrun;
    }
  }
}

}  // namespace nf
