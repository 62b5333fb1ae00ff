// Instantiation of the ragged, k-split direct-to-LDS matmul kernels (gemm_ring.h).
#include <atomic>

#include "gemm_launch.h"
#include "gemm_ring.h"

namespace nf {

template <class Cfg, bool PB, bool CONV>
__global__ __launch_bounds__(Cfg::kThreads, Cfg::kWPE) void gemm_ring_kernel(GemmArgs a) {
  extern __shared__ __align__(1024) unsigned char smem_raw[];
  unsigned id = xcd_remap(blockIdx.x, gridDim.x);
  // consecutive ids: row tiles of one column panel, then the next panel, then the next problem
  const int tm = id % a.tiles_m;  id /= a.tiles_m;
  const int tn = id % a.tiles_n;  id /= a.tiles_n;
  const int z = id % a.nz0, z1 = id / a.nz0;
  const long coff = z * a.sC0 + z1 * a.sC1;
  const float* bias = a.ep.col_bias ? a.ep.col_bias + z * a.ep.col_vec_stride0 : nullptr;
  gemm_ring_tile<Cfg, PB, CONV>(a.A + z * a.sA0, a.lda, a.B + z * a.sB0 + z1 * a.sB1, a.ldb, a.K, (lds_u8_t*)smem_raw,
                                a.C + coff, a.R ? a.R + coff : nullptr, a.ldc, bias, a.ep, z * a.ep.row_vec_stride0,
                                tm * Cfg::kBM, tn * Cfg::kBN, a.rows, a.cols);
}

template <class Cfg, bool PB, bool CONV = false>
static nf_status launch_ring(GemmLaunch& L, hipStream_t s) {
  GemmArgs& a = L.a;
  a.tiles_m = (a.rows + Cfg::kBM - 1) / Cfg::kBM;
  a.tiles_n = (a.cols + Cfg::kBN - 1) / Cfg::kBN;
  const long long total = (long long)a.tiles_m * a.tiles_n * a.nz0 * L.nz1;
  if (total <= 0 || total > 0x7fffffffLL) return NF_EUNSUPPORTED;
  auto kern = gemm_ring_kernel<Cfg, PB, CONV>;
  constexpr int kLds = Cfg::kLdsBytes;
  if (kLds > 64 * 1024) {
    static std::atomic<bool> opted_in{false};
    if (!opted_in.load(std::memory_order_acquire)) {
      if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kLds) !=
          hipSuccess)
        return NF_ELAUNCH;
      opted_in.store(true, std::memory_order_release);
    }
  }
  nf_launch(kern, dim3((unsigned)total), dim3(Cfg::kThreads), kLds, s, a);
  return hipGetLastError() == hipSuccess ? NF_OK : NF_ELAUNCH;
}

// Row-major weights: k is summed in one ascending chain, as by every other bf16 kernel behind netfuse_linear (float32 has an
// order of its own, gemm_f32.h), so that a model's result does not depend on how many models are merged with it.  Small wave tiles (a 32 x 32 block per
// wavefront) with deep rings: 2 to 16 wavefronts share the loads and leave their latency to each other.
//                             FM FN WGM WGN KG BK NS waves per SIMD
static nf_status launch_ring_tile(int tile, GemmLaunch& L, hipStream_t s) {
  switch (tile) {
    case R32x32: return launch_ring<RingCfg<1, 1, 1, 1, 1, 64, 9, 1>, false>(L, s);
    case R64x64: return launch_ring<RingCfg<1, 1, 2, 2, 1, 64, 5, 2>, false>(L, s);
    case R64x128: return launch_ring<RingCfg<1, 1, 2, 4, 1, 64, 6, 2>, false>(L, s);
    case R96x128: return launch_ring<RingCfg<1, 1, 3, 4, 1, 64, 5, 3>, false>(L, s);
    case R96x256: return launch_ring<RingCfg<3, 1, 1, 8, 1, 64, 3, 2>, false>(L, s);
    case R128x128: return launch_ring<RingCfg<1, 1, 4, 4, 1, 64, 4, 4>, false>(L, s);
    case R128x256: return launch_ring<RingCfg<2, 2, 2, 4, 1, 64, 3, 2>, false>(L, s);
    case R128x384: return launch_ring<RingCfg<2, 3, 2, 4, 1, 32, 4, 2>, false>(L, s);
    case R256x256: return launch_ring<RingCfg<4, 2, 2, 4, 1, 64, 2, 2>, false>(L, s);
    case R64x256: return launch_ring<RingCfg<2, 1, 1, 8, 1, 64, 3, 2>, false>(L, s);
    // heights between the powers of two, a column of row blocks per wavefront: five multiplications per slice of 16 k for seven LDS reads
    // (five of rows, two transposing ones of the weights), in the other two three for five; a single block takes three for one
    case R160x256: return launch_ring<RingCfg<5, 1, 1, 8, 1, 32, 5, 2>, false>(L, s);
    case R192x192: return launch_ring<RingCfg<3, 1, 2, 6, 1, 64, 3, 3>, false>(L, s);
    case R288x128: return launch_ring<RingCfg<3, 1, 3, 4, 1, 64, 3, 3>, false>(L, s);
  }
  return NF_EUNSUPPORTED;
}
static nf_status launch_ring_packed_tile(int tile, GemmLaunch& L, hipStream_t s) {
  switch (tile) {
    case RP32x32: return launch_ring<RingCfg<1, 1, 1, 1, 8, 64, 2, 2>, true>(L, s);
    case RP64x64: return launch_ring<RingCfg<2, 2, 1, 1, 4, 64, 2, 1>, true>(L, s);
    case RP128x64: return launch_ring<RingCfg<2, 2, 2, 1, 2, 64, 3, 1>, true>(L, s);
    case RP128x128: return launch_ring<RingCfg<2, 2, 2, 2, 2, 32, 3, 2>, true>(L, s);
    case RP128x256: return launch_ring<RingCfg<2, 2, 2, 4, 1, 64, 3, 2>, true>(L, s);
    case RP256x256: return launch_ring<RingCfg<4, 2, 2, 4, 1, 64, 2, 2>, true>(L, s);
  }
  return NF_EUNSUPPORTED;
}

// Pointwise convolutions: short k (64 ... 2048 channels), so a tile is mostly prologue and epilogue; two or more workgroups
// per compute unit run them under each other's loads.
static nf_status launch_ring_conv_tile(int tile, GemmLaunch& L, hipStream_t s) {
  switch (tile) {
    case RC64x64: return launch_ring<RingCfg<1, 1, 2, 2, 1, 64, 3, 2>, false, true>(L, s);
    case RC64x128: return launch_ring<RingCfg<1, 1, 2, 4, 1, 64, 3, 2>, false, true>(L, s);
    case RC64x256: return launch_ring<RingCfg<1, 2, 2, 4, 1, 32, 3, 4>, false, true>(L, s);
    case RC128x128: return launch_ring<RingCfg<2, 1, 2, 4, 1, 64, 2, 4>, false, true>(L, s);
    case RC128x256: return launch_ring<RingCfg<2, 2, 2, 4, 1, 32, 3, 2>, false, true>(L, s);
  }
  return NF_EUNSUPPORTED;
}

static bool ring_aligned(const GemmArgs& a) {
  return a.rows > 0 && a.lda % 8 == 0 && a.ldb % 8 == 0 && a.ldc % 8 == 0 && ((uintptr_t)a.A & 15) == 0 &&
         ((uintptr_t)a.B & 15) == 0 && ((uintptr_t)a.C & 15) == 0 && ((uintptr_t)a.R & 15) == 0 &&
         (long long)a.rows * a.K < (1LL << 30) && (long long)a.K * a.cols < (1LL << 30);   // 32-bit byte offsets
}

nf_status launch_gemm_ring(int tile, bool packed, GemmLaunch& L, hipStream_t s) {
  const GemmArgs& a = L.a;
  if (!ring_fits(a.cols, a.K) || (packed && a.cols % 32) || L.nz1 != 1 || !ring_aligned(a)) return NF_EUNSUPPORTED;
  if (((uintptr_t)a.ep.col_bias & 15) || a.ep.col_vec_stride0 % 4) return NF_EUNSUPPORTED;
  return packed ? launch_ring_packed_tile(tile, L, s) : launch_ring_tile(tile, L, s);
}

nf_status launch_conv_ring(int tile, GemmLaunch& L, hipStream_t s) {
  const GemmArgs& a = L.a;
  if (a.cols % 8 || a.K % 64 || !ring_aligned(a)) return NF_EUNSUPPORTED;
  return launch_ring_conv_tile(tile, L, s);
}

}  // namespace nf
