// Decimation ahead of the FFT prefill: contexts of M = 2^m >= 16384 tokens that keep low frequencies only (|k| <= reach, k and M - k
// alike, in every layer) do not need M points.  With a window w of kDecTaps points of a grid of N = 2^LOGN >= 4 reach points, D = M / N tokens apart,
//   y[m] = sum_n w(m - n / D) x[n]   (n modulo M)   gives   U[k] = DFT_N(y)[k] / W(k / N),  |k| <= N / 4,
// up to an aliasing error of 1.4e-9 of a tone at the worst frequency (see interp.h: the same window, the roles of time and frequency
// exchanged; with its eight taps it is 9.7e-8, which a strong tone among the frequencies that are not kept would show).  y is a banded matrix
// product: 16 grid points x (25 D) tokens x 128 channels at a time on the matrix cores, whose left operand is the same everywhere.
// bf16 tokens are exact operands; the window is split into three bf16 parts (24 bits), fp32 tokens as well (six of the nine
// products: what is left out is below 2^-24), sums are fp32.
#include "common.h"

namespace iwdft {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kDecThreads = 256, kDecRun = 8;  // tiles of 16 grid points that a wave walks

__device__ __forceinline__ uint32_t bf16_pair(float lo, float hi) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){lo, hi}, bf16x2));
}

// A wave walks kDecRun tiles of 16 grid points (16 D tokens, D / 2 blocks of 32) of one (slice, tensor), all 128 channels, and reads
// every token once: a block counts for its own tile and, within dec_halo blocks of a tile's end, for the neighbour.  A lane holds 8
// tokens x 8 channels of a block (whole rows over 16 lanes), which are the operand of channel 8 (lane % 16) + j, j = 0 .. 7, after
// a permutation of halves: no LDS trip.  y: [tensor][slice of the launch][N][128].
// What bounds it is HBM: one read of the tokens, 1 / D of twice (bf16) their bytes written; 192 matrix instructions (16 cycles) per 32 KB at D = 8.
// 8 slices of 131072 tokens, K and V, bf16: 135 us, 4.0 TB/s read; 64 of them, 4096 bins, with the transforms: 4200 (sixteen 8192-point transforms
// per channel pair) -> 1665 us.
template <bool BF16, int D, bool WIDE>
__global__ __launch_bounds__(kDecThreads, 2) void decimate_kernel(Params P, const void* __restrict__ K, const void* __restrict__ V,
                                                                 int slice0, int slices) {
  constexpr int BT = D / 2, HB = dec_halo(D), NG = BT + 2 * HB;
  constexpr int kElem = BF16 ? 2 : 4, kRow = kHeadDim * kElem, W = BF16 ? 1 : 2;
  static_assert(HB <= BT, "a block meets three tiles at most");
  __shared__ u32x4 wl[NG * 3 * 64];
  for (int i = threadIdx.x; i < NG * 3 * 64; i += kDecThreads) wl[i] = ((const u32x4*)P.dec_window)[i];
  __syncthreads();
  const uint32_t M = P.M, N = M / D, runs = N / (16 * kDecRun), blocks = M / 32;
  const uint32_t item = __builtin_amdgcn_readfirstlane(blockIdx.x * (kDecThreads / 64) + threadIdx.x / 64);
  if (item >= runs * 2u * (uint32_t)slices) return;  // a whole wave; no barrier follows
  const int lane = threadIdx.x & 63;
  const uint32_t st = item / runs, sl = st >> 1, t0 = (item % runs) * kDecRun;  // st: (slice of the launch, tensor)
  const int64_t tokens = (int64_t)P.S + M + P.R;
  const char* X = (const char*)((st & 1) ? V : K) + ((int64_t)(slice0 + sl) * tokens + P.S) * kRow +
                  (lane >> 4) * 8 * kRow + (lane & 15) * 8 * kElem;
  float* Y = P.dec_scratch + (((int64_t)(st & 1) * slices + sl) * N + (lane >> 4) * 4) * kHeadDim + (lane & 15) * 8;

  u32x4 raw[8 * W], nxt[8 * W];
  auto fetch = [&](u32x4 (&z)[8 * W], int b) {  // block b, modulo the context
    const char* p = X + (int64_t)((uint32_t)b & (blocks - 1)) * (32 * kRow);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
#pragma unroll
      for (int w = 0; w < W; ++w) {
        if constexpr (WIDE) {
          z[i * W + w] = __builtin_nontemporal_load((const u32x4*)(p + i * kRow + w * 16));
        } else {  // tensors that are not 16-byte aligned
#pragma unroll
          for (int c = 0; c < 4; ++c) z[i * W + w][c] = *(const uint32_t*)(p + i * kRow + w * 16 + c * 4);
        }
      }
    }
  };
  f32x4 prev[8], cur[8], next[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) prev[j] = cur[j] = next[j] = (f32x4)(0.f);
  auto window = [&](int g, int s) { return __builtin_bit_cast(bf16x8, wl[(g * 3 + s) * 64 + lane]); };
  // acc[j] += window group g x the tokens of raw
  auto add = [&](f32x4 (&acc)[8], int g) {
    const bf16x8 w0 = window(g, 0), w1 = window(g, 1), w2 = window(g, 2);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if constexpr (BF16) {
        u32x4 f;  // tokens 2 i, 2 i + 1 of channel j
#pragma unroll
        for (int i = 0; i < 4; ++i)
          f[i] = __builtin_amdgcn_perm(raw[2 * i + 1][j / 2], raw[2 * i][j / 2], (j & 1) ? 0x07060302u : 0x05040100u);
        const bf16x8 x = __builtin_bit_cast(bf16x8, f);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2, x, acc[j], 0, 0, 0);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1, x, acc[j], 0, 0, 0);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w0, x, acc[j], 0, 0, 0);
      } else {
        u32x4 f0, f1, f2;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float a = __uint_as_float(raw[4 * i + j / 4][j & 3]), b = __uint_as_float(raw[4 * i + 2 + j / 4][j & 3]);
          const uint32_t h0 = bf16_pair(a, b);
          const float a1 = a - __uint_as_float(h0 << 16), b1 = b - __uint_as_float(h0 & 0xffff0000u);
          const uint32_t h1 = bf16_pair(a1, b1);
          f0[i] = h0;
          f1[i] = h1;
          f2[i] = bf16_pair(a1 - __uint_as_float(h1 << 16), b1 - __uint_as_float(h1 & 0xffff0000u));
        }
        const bf16x8 x0 = __builtin_bit_cast(bf16x8, f0), x1 = __builtin_bit_cast(bf16x8, f1), x2 = __builtin_bit_cast(bf16x8, f2);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2, x0, acc[j], 0, 0, 0);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1, x1, acc[j], 0, 0, 0);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w0, x2, acc[j], 0, 0, 0);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1, x0, acc[j], 0, 0, 0);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w0, x1, acc[j], 0, 0, 0);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w0, x0, acc[j], 0, 0, 0);
      }
    }
  };
  const int first = (int)(t0 * BT) - HB, last = (int)((t0 + kDecRun) * BT) + HB - 1;  // blocks of the run
  fetch(nxt, first);
#pragma unroll 1
  for (int tile = (int)t0 - 1; tile <= (int)t0 + kDecRun; ++tile) {  // the outer two for the blocks they share with the run
#pragma unroll
    for (int bb = 0; bb < BT; ++bb) {
      const int b = tile * BT + bb;
      if (b < first || b > last) continue;  // uniform
#pragma unroll
      for (int i = 0; i < 8 * W; ++i) raw[i] = nxt[i];
      if (b < last) fetch(nxt, b + 1);
      if (bb < HB && tile > (int)t0) add(prev, BT + HB + bb);
      if (tile >= (int)t0 && tile < (int)t0 + kDecRun) add(cur, HB + bb);
      if (bb >= BT - HB && tile + 1 < (int)t0 + kDecRun) add(next, bb - (BT - HB));
      if (bb == HB - 1 && tile > (int)t0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float* y = Y + ((int64_t)(tile - 1) * 16 + r) * kHeadDim;
          *(f32x4*)y = (f32x4){prev[0][r], prev[1][r], prev[2][r], prev[3][r]};
          *(f32x4*)(y + 4) = (f32x4){prev[4][r], prev[5][r], prev[6][r], prev[7][r]};
        }
      }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) prev[j] = cur[j], cur[j] = next[j], next[j] = (f32x4)(0.f);
  }
}

hipError_t launch_decimate(const Params& P, const void* K, const void* V, int slice0, int slices, hipStream_t st) {
  const uint32_t D = P.M >> P.dec_logN;
  const uint64_t waves = (uint64_t)(P.M / D) / (16 * kDecRun) * 2 * slices, blocks = (waves + 3) / 4;
  if (blocks > 0x7fffffffull) return hipErrorInvalidConfiguration;
  const bool wide = (((uintptr_t)K | (uintptr_t)V) & 15u) == 0;
#define IWDFT_DEC_LAUNCH(B16, DV, WIDE) \
  decimate_kernel<B16, DV, WIDE><<<dim3((uint32_t)blocks), dim3(kDecThreads), 0, st>>>(P, K, V, slice0, slices)
#define IWDFT_DEC_CASE(DV)                                \
  case DV:                                                \
    if (P.kv_dtype == 1) {                                \
      if (wide) IWDFT_DEC_LAUNCH(true, DV, true);         \
      else IWDFT_DEC_LAUNCH(true, DV, false);             \
    } else {                                              \
      if (wide) IWDFT_DEC_LAUNCH(false, DV, true);        \
      else IWDFT_DEC_LAUNCH(false, DV, false);            \
    }                                                     \
    break;
  switch (D) {
    IWDFT_DEC_CASE(2)
    IWDFT_DEC_CASE(4)
    IWDFT_DEC_CASE(8)
    IWDFT_DEC_CASE(16)
    default: return hipErrorInvalidValue;
  }
#undef IWDFT_DEC_CASE
#undef IWDFT_DEC_LAUNCH
  return hipGetLastError();
}

}  // namespace iwdft
