// Merged 3 x 3 convolution (grouped, groups = M*g: Appendix A Eq. 2), bf16 and float32: every wavefront runs a pipeline
// of its own, with no workgroup barrier between its first load and the sum of the wavefronts' parts.
//
//   C[co][p] = sum_{ci,ky,kx} w[co][ci][ky][kx] * xpad[ci][oy*s + ky][ox*s + kx],   p = oy*Wo + ox
//
// One workgroup = 32 output channels x 32 NB consecutive positions of one (image, group); its KG = 4 wavefronts split the INPUT
// CHANNELS (KG = 1, a workgroup of one wavefront, where there are too few to split).  A step of a wavefront is 32 bytes of
// channels (16 bf16 or 8 float32), wavefront q taking steps q, q + KG, ...; lane half h owns 16 bytes of them (kEV channels):
//   * weights: the 288 contiguous bytes w[co][channels of the step][0..8] of 32 rows are requested a step ahead in whole
//     runs, 16 bytes per lane, and change lanes through 9 KB of LDS of the wavefront's own, untouched.  A lane reads its row's
//     144 bytes of its half back with nine 16-byte reads: all nine taps of its channels.  float32 multiplies the
//     registers as they are (element 9 c + tap), bf16 regroups them by tap with byte permutes.  Rows of an odd octet
//     store their halves exchanged, which puts the 16 lanes of a read on distinct banks.  (Direct-to-LDS loads beside
//     loads into registers would make the compiler wait for all of either kind: it counts them apart.)
//   * input: a task loads one dword of kEV channel planes (two bf16 pixels, one float32 pixel) a step ahead and leaves one
//     16-byte vector per pixel in the wavefront's own LDS patch, [half][pixel][16 bytes].  The patch carries its zero padding,
//     so the fragment of any tap is one 16-byte read at pixel(position) + a uniform offset, conflict free over consecutive
//     pixels.
//   * multiplication: bf16 one 32x32x16 instruction per tap and block, float32 four 32x32x2 (one per channel of the
//     vector).  Transposed as everywhere here: a lane ends up with 4 consecutive positions of one output channel.
// The partial sums meet in LDS and are added pairwise in one order, so a result does not depend on NB.  A float32 wavefront that
// has a tile to itself keeps two chains (even and odd channels of a vector): with one its sums were rounded 1.35 (8 and 16
// channels, random signs) to 1.7 times (one sign) as far off as the two chains of gemm_f32.h, which it stands in for.
//
// Why: at 14 x 14 and 7 x 7 a workgroup that shares one channel block between its wavefronts (conv_tap.h) has nothing
// to multiply while the next block arrives and is shuffled into LDS between two barriers (matrix pipe 15 to 20 % busy);
// the gathered float32 kernel (gemm_f32.h) loads every operand element nine times, 4 bytes at a time.
// What bounds it: float32 the matrix pipe (a step of 2 blocks takes 1.9 us of it and 2.6 us in all); bf16 the trip of a step's
// operands from memory, of which a wavefront has one step under way: a form with two or four steps in flight was not faster
// (7 x 7: 31.9 / 32.3 / 37 us), nor one that writes the next step to a second LDS stage under the current step's
// multiplications (34.2; it leaves room for one workgroup per compute unit instead of two or three).
// Measured (us, before -> now; float32 8 models: the gathered kernel, bf16: conv_tap.h):
//   float32 256 -> 256 at 14 x 14 42.5 -> 28.5, 512 at 7 x 7 58.3 -> 31.1, 128 at 28 x 28 37.3 -> 27.3, 64 at 56 x 56 35.1 -> 26.4,
//   512 at 14 x 14 stride 2 59.0 -> 34.1; bf16 32 models 512 at 7 x 7 42.3 -> 32.4 (151 MB of weights: 4.7 TB/s), 512 at 14 x 14
//   stride 2 48.6 -> 35.9, 256 at 14 x 14 22.1 -> 19.5; 3 models of 4 images 512 at 7 x 7 26.0 -> 13.8, 256 at 13 x 13 16.3 -> 12.8.
#pragma once
#include <type_traits>

#include "gemm_dma.h"

namespace nf {

template <typename T>
struct ConvWaveArgs {
  const T* x; const T* w; const T* R; T* y;
  int cig, cog, g, nG, H, W, Wo, HoWo, stride, pad;     // g groups per model, nG of all models
  int PW, PS;                                // patch pixels per row and in all (the tallest tile)
  int tiles_m, tiles_n;
  unsigned rcp_w, one_w, rcp_wo, one_wo;     // division by W and Wo (div_by)
  long x_group, x_image, y_group, y_image;   // element strides
  Epilogue ep;
};

constexpr int kWaveStage = 32 * 288;         // bytes of one step's weights

template <typename T> struct ConvWaveType;
template <> struct ConvWaveType<bf16_t> { static constexpr int kEV = 8, kPix = 2; };
template <> struct ConvWaveType<float> { static constexpr int kEV = 4, kPix = 1; };

// per wavefront: a step's operands, later a partial sum
inline int conv_wave_lds_bytes(int NB, int KG, int PS) {
  const int pipe = kWaveStage + 32 * PS, part = 32 * (32 * NB + 4) * 4;
  return KG * (pipe > part ? pipe : part);
}

typedef uint32_t cw_u32x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) cw_u32x4_t lds_cw_u32x4_t;
typedef __attribute__((address_space(1))) const cw_u32x4_t glb_cw_u32x4_t;
struct __attribute__((packed, aligned(2))) AnyU32 { uint32_t v; };
static_assert(alignof(AnyU32) == 2);
typedef __attribute__((address_space(1))) const AnyU32 glb_any_u32_t;

// Lanes of one wavefront exchange values through LDS: the hardware keeps a wavefront's LDS accesses in order, this keeps the compiler
// from moving one side's accesses past the other's.  No instruction.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
}

// n / d, branch free (cw_divisor, cw_div_exact in gemm_launch.h); exact at least while n < 2^32 / d
__device__ __forceinline__ unsigned cw_div(unsigned n, unsigned rcp, unsigned one) { return __umulhi(n, rcp) + (n & one); }

// The fragments of tap + ahead are read in front of the instructions of a tap: enough of them to cover an LDS read.
constexpr int conv_wave_ahead(bool f32, int NB) { return f32 || NB >= 6 ? 1 : NB >= 3 ? 2 : NB == 2 ? 3 : 5; }
// Chains of a wavefront's sum: two for float32 where no other wavefront shares the tile.
constexpr int conv_wave_chains(bool f32, int KG) { return f32 && KG == 1 ? 2 : 1; }
// Wavefronts per SIMD that the registers leave room for: two where that takes no more than a few of them away.
constexpr int conv_wave_occupancy(bool f32, int NB, int KG, int NT) {
  return 122 + 16 * NB * conv_wave_chains(f32, KG) + NT * (f32 ? 6 : 10) + 4 * NB * (conv_wave_ahead(f32, NB) + 1) <= 280 ? 2 : 1;
}

// NB: blocks of 32 positions.  KG: wavefronts that share a tile's channels.  NT: input tasks per lane and step (the host
// checks the bound).
template <typename T, int NB, int KG, int NT>
__global__ __launch_bounds__(KG * kWave, conv_wave_occupancy(sizeof(T) == 4, NB, KG, NT)) void conv_wave_kernel(ConvWaveArgs<T> a) {
  constexpr int EV = ConvWaveType<T>::kEV, PX = ConvWaveType<T>::kPix, CB = 2 * EV;
  constexpr bool F32 = sizeof(T) == 4;
  extern __shared__ __align__(1024) unsigned char smem_raw[];
  const int lane = threadIdx.x % kWave, half = lane / 32, l32 = lane % 32;
  const int q = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  lds_u8_t* const Ws = (lds_u8_t*)smem_raw + q * (kWaveStage + 32 * a.PS);
  lds_u8_t* const Ps = Ws + kWaveStage;

  unsigned id = xcd_remap(blockIdx.x, gridDim.x);
  const int tm = id % a.tiles_m;  id /= a.tiles_m;
  const int tn = id % a.tiles_n;  id /= a.tiles_n;
  const int G = id % a.nG, b = id / a.nG;
  const int row0 = tm * 32, p0 = tn * 32 * NB;
  const int rows_left = a.cog - row0, cols_left = min(a.HoWo - p0, 32 * NB);
  const int steps = a.cig / CB, n = steps > q ? (steps - q + KG - 1) / KG : 0;

  // ---- weights of a step: LDS slot s = 18 r + jj of 16 bytes holds piece j of row r
  unsigned w_off[9];
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    const int s = i * 64 + lane, r = s / 18, jj = s - 18 * r;
    const int j = (r & 8) ? (jj >= 9 ? jj - 9 : jj + 9) : jj;
    w_off[i] = (unsigned)(min(r, rows_left - 1) * a.cig * 9) * (unsigned)sizeof(T) + j * 16;   // rows past the end: the last one, never stored
  }
  // Running pointers and offsets are hidden from the compiler's loop analysis, which would turn every load's address into a
  // 64-bit vector register pair of its own; this way it is a scalar base plus a 32-bit offset.
  auto here = [](unsigned off) { asm volatile("" : "+v"(off)); return off; };
  const glb_u8_t* wp = (const glb_u8_t*)(a.w + ((long)G * a.cog + row0) * a.cig * 9) + q * 288;
  cw_u32x4_t wr[9];
  auto load_w = [&]() {
    asm volatile("" : "+s"(wp));
#pragma unroll
    for (int i = 0; i < 9; ++i) wr[i] = *(glb_cw_u32x4_t*)(wp + here(w_off[i]));
    wp += KG * 288;
  };
  if (n > 0) load_w();                                       // before the index arithmetic, which runs under their trip
  __builtin_amdgcn_sched_barrier(0);

  // ---- geometry of the tile's patch: image rows a0 .. a1 - 1 are one contiguous run of pixels in every plane
  const int p_last = p0 + cols_left - 1;
  const int oy_first = (int)cw_div(p0, a.rcp_wo, a.one_wo), oy_last = (int)cw_div(p_last, a.rcp_wo, a.one_wo);
  const int iy0 = oy_first * a.stride - a.pad;
  const int a0 = max(iy0, 0), a1 = min(iy0 + (oy_last - oy_first) * a.stride + 3, a.H);
  const int npx = (a1 - a0) * a.W;                           // at least one row (pad <= 2)
  const unsigned plane = (unsigned)(a.H * a.W) * (unsigned)sizeof(T);
  // task u of a lane: pixels i0 .. i0 + PX - 1 of the run, channels of half th; tasks past the end repeat the last one
  unsigned x_off[NT], x_dst[NT];
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    const int nch = (npx + PX - 1) / PX;
    const int t = min(u * kWave + lane, 2 * nch - 1), th = t >= nch, c = t - th * nch;
    const int i0 = min(c * PX, npx - PX);                    // the last chunk is pulled back to end with the run
    x_off[u] = (unsigned)th * EV * plane + (unsigned)(a0 * a.W + i0) * (unsigned)sizeof(T);
    unsigned dst[2];
#pragma unroll
    for (int e = 0; e < PX; ++e) {
      const int y = (int)cw_div(i0 + e, a.rcp_w, a.one_w), xx = i0 + e - y * a.W;
      dst[e] = (unsigned)((y + a0 - iy0) * a.PW + xx + a.pad + th * a.PS);
    }
    x_dst[u] = PX == 2 ? dst[0] | dst[1] << 16 : dst[0];
  }
  uint32_t xv[NT][EV];
  const glb_u8_t* xp = (const glb_u8_t*)(a.x + (long)b * a.x_image + (long)G * a.x_group) + (long)q * CB * plane;
  auto load_x = [&]() {
    const glb_u8_t* pe = xp;
#pragma unroll
    for (int e = 0; e < EV; ++e) {
      asm volatile("" : "+s"(pe));
#pragma unroll
      for (int u = 0; u < NT; ++u) xv[u][e] = ((glb_any_u32_t*)(pe + here(x_off[u])))->v;
      pe += plane;
    }
    xp += (long)KG * CB * plane;
  };
  if (n > 0) load_x();
  __builtin_amdgcn_sched_barrier(0);
  for (int c = lane; c < 2 * a.PS; c += kWave) *(lds_cw_u32x4_t*)(Ps + c * 16) = cw_u32x4_t{0, 0, 0, 0};
  int b_off[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int p = min(p0 + j * 32 + l32, p_last);            // columns past the end are discarded
    const int oy = (int)cw_div(p, a.rcp_wo, a.one_wo), ox = p - oy * a.Wo;
    b_off[j] = ((oy - oy_first) * a.stride * a.PW + ox * a.stride + half * a.PS) * 16;
  }

  constexpr int CH = conv_wave_chains(F32, KG);
  f32x16_t acc[CH][NB];
#pragma unroll
  for (int h = 0; h < CH; ++h)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[h][j][r] = 0.f;

  // selectors of perm(hi, lo, sel): 16 bits of `lo` (its low or high half) below 16 bits of `hi`
  auto pick = [](int lo_half, int hi_half) -> uint32_t {
    return (lo_half ? 0x0302u : 0x0100u) | ((hi_half ? 0x0706u : 0x0504u) << 16);
  };
  auto to_lds = [&]() {
#pragma unroll
    for (int i = 0; i < 9; ++i) *(lds_cw_u32x4_t*)(Ws + (i * 64 + lane) * 16) = wr[i];
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
      for (int e = 0; e < PX; ++e) {
        cw_u32x4_t o;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if constexpr (F32) o[i] = xv[u][i];
          else o[i] = __builtin_amdgcn_perm(xv[u][2 * i + 1], xv[u][2 * i], pick(e, e));
        }
        *(lds_cw_u32x4_t*)(Ps + (PX == 2 ? (e ? x_dst[u] >> 16 : x_dst[u] & 0xffffu) : x_dst[u]) * 16) = o;
      }
  };
  const int a_off = (18 * l32 + 9 * (half ^ ((l32 >> 3) & 1))) * 16;
  constexpr int kAhead = conv_wave_ahead(F32, NB);
  // One step: its operands move from registers to LDS, the registers are loaded with the next step's (MORE), and the step is
  // multiplied.  A wavefront's LDS accesses take effect in order, so nothing waits between the writes and the reads.
  auto step = [&](auto more) {
    wave_lds_order();                                        // the reads of the step before (or the zero fill)
    to_lds();
    wave_lds_order();
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (decltype(more)::value) {
      load_w();
      __builtin_amdgcn_sched_barrier(0);
      load_x();
      __builtin_amdgcn_sched_barrier(0);
    }
    uint32_t wv[36];
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const cw_u32x4_t v = *(const lds_cw_u32x4_t*)(Ws + a_off + k * 16);
#pragma unroll
      for (int e = 0; e < 4; ++e) wv[4 * k + e] = v[e];
    }
    cw_u32x4_t bv[kAhead + 1][NB];
    bf16x8_t af[2];
    auto read_b = [&](int tap) {
      const lds_u8_t* base = Ps + ((tap / 3) * a.PW + tap % 3) * 16;
#pragma unroll
      for (int j = 0; j < NB; ++j) bv[tap % (kAhead + 1)][j] = *(const lds_cw_u32x4_t*)(base + b_off[j]);
    };
    auto regroup = [&](int tap) {
      cw_u32x4_t o;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int e0 = 9 * (2 * i) + tap, e1 = 9 * (2 * i + 1) + tap;     // elements (channel 2i, tap), (channel 2i+1, tap)
        o[i] = __builtin_amdgcn_perm(wv[e1 / 2], wv[e0 / 2], pick(e0 % 2, e1 % 2));
      }
      af[tap & 1] = __builtin_bit_cast(bf16x8_t, o);
    };
#pragma unroll
    for (int tap = 0; tap < kAhead; ++tap) read_b(tap);
    if constexpr (!F32) regroup(0);
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      if (tap + kAhead < 9) read_b(tap + kAhead);
      if constexpr (!F32) {
        if (tap < 8) regroup(tap + 1);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = 0; c < (F32 ? 4 : 1); ++c)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          const cw_u32x4_t& x = bv[tap % (kAhead + 1)][j];
          if constexpr (F32)
            acc[c % CH][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(x[c]), __uint_as_float(wv[9 * c + tap]), acc[c % CH][j], 0, 0, 0);
          else
            acc[0][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, x), af[tap & 1], acc[0][j], 0, 0, 0);
        }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  for (int s = 0; s + 1 < n; ++s) step(std::true_type{});

  // ---- the four partial sums meet in LDS: [wavefront][row][position].  Everything the epilogue reads from memory is asked for
  // before the last step, so that it does not wait for it: chunks of kEV positions, then the positions behind the last whole chunk.
  constexpr int kPitch = 32 * NB + 4, kPart = 32 * kPitch, kPerRow = 32 * NB / EV, kIter = (32 * kPerRow + KG * kWave - 1) / (KG * kWave);
  const Epilogue& ep = a.ep;
  const long out0 = (long)b * a.y_image + (long)G * a.y_group + (long)row0 * a.HoWo + p0;
  const long rv0 = (long)G * a.cog + row0;
  struct Consts { float bias, scale, shift; };
  auto consts = [&](int row) {
    Consts c{0.f, 1.f, 0.f};
    if (ep.row_bias) c.bias = ep.row_bias[rv0 + row];
    if (ep.row_scale) { c.scale = ep.row_scale[rv0 + row]; c.shift = ep.row_shift[rv0 + row]; }
    return c;
  };
  const int whole = cols_left / EV * EV, tid = threadIdx.x;
  Consts k_it[kIter];
  uint4 r_it[kIter];
  bool live[kIter];
#pragma unroll
  for (int i = 0; i < kIter; ++i) {
    const int t = tid + i * KG * kWave, row = t / kPerRow, c = (t - row * kPerRow) * EV;
    live[i] = row < min(rows_left, 32) && c < whole;
    k_it[i] = consts(min(row, rows_left - 1));
    r_it[i] = make_uint4(0u, 0u, 0u, 0u);
    if (a.R && live[i]) r_it[i] = load_at<uint4>(a.R + out0 + (long)row * a.HoWo + c);
  }
  constexpr int kTail = (32 * EV + KG * kWave - 1) / (KG * kWave);            // fewer than kEV positions of 32 rows
  Consts t_k[kTail];
  float t_res[kTail];
#pragma unroll
  for (int i = 0; i < kTail; ++i) {
    const int t = tid + i * KG * kWave, row = t % 32, c = whole + t / 32;
    t_k[i] = consts(min(row, rows_left - 1));
    t_res[i] = a.R && row < rows_left && c < cols_left ? load_f32<T>(a.R + out0 + (long)row * a.HoWo + c) : 0.f;
  }
  __builtin_amdgcn_sched_barrier(0);
  if (n > 0) step(std::false_type{});

  lds_f32_t* const red = (lds_f32_t*)smem_raw;
  if constexpr (KG > 1) __syncthreads(); else wave_lds_order();
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    if constexpr (CH == 2) acc[0][j] += acc[1][j];
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4)
      *(lds_f32x4_t*)(red + q * kPart + l32 * kPitch + j * 32 + r4 * 8 + half * 4) =
          f32x4v_t{acc[0][j][4 * r4], acc[0][j][4 * r4 + 1], acc[0][j][4 * r4 + 2], acc[0][j][4 * r4 + 3]};
  }
  if constexpr (KG > 1) __syncthreads(); else wave_lds_order();
  static_assert(KG == 1 || KG == 4, "one chain, or four added pairwise");
  auto finish = [&](auto act) {
    constexpr int ACT = decltype(act)::value;
#pragma unroll
    for (int i = 0; i < kIter; ++i) {
      if (!live[i]) continue;
      const int t = tid + i * KG * kWave, row = t / kPerRow, c = (t - row * kPerRow) * EV;
      T res[EV], out[EV];
      __builtin_memcpy(res, &r_it[i], 16);
#pragma unroll
      for (int h = 0; h < EV / 4; ++h) {
        f32x4v_t s[KG];
#pragma unroll
        for (int g = 0; g < KG; ++g) s[g] = *(const lds_f32x4_t*)(red + g * kPart + row * kPitch + c + 4 * h);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float v = s[0][e];
          if constexpr (KG == 4) v = (s[0][e] + s[2][e]) + (s[1][e] + s[3][e]);
          store_f32<T>(&out[4 * h + e], act_const<ACT>(fmaf(v + k_it[i].bias, k_it[i].scale, k_it[i].shift) + load_f32<T>(&res[4 * h + e])));
        }
      }
      uint4 packed;
      __builtin_memcpy(&packed, out, 16);
      store_at(a.y + out0 + (long)row * a.HoWo + c, packed);
    }
#pragma unroll
    for (int i = 0; i < kTail; ++i) {
      const int t = tid + i * KG * kWave, row = t % 32, c = whole + t / 32;
      if (row >= rows_left || c >= cols_left) continue;
      const lds_f32_t* src = red + row * kPitch + c;
      float v = src[0];
      if constexpr (KG == 4) v = (src[0] + src[2 * kPart]) + (src[kPart] + src[3 * kPart]);
      store_f32<T>(a.y + out0 + (long)row * a.HoWo + c, act_const<ACT>(fmaf(v + t_k[i].bias, t_k[i].scale, t_k[i].shift) + t_res[i]));
    }
  };
  if (ep.act == NF_ACT_RELU) finish(std::integral_constant<int, NF_ACT_RELU>{});
  else if (ep.act == NF_ACT_GELU) finish(std::integral_constant<int, NF_ACT_GELU>{});
  else finish(std::integral_constant<int, NF_ACT_NONE>{});
}

}  // namespace nf
