// Token rows as channel pairs: several adjacent pairs of a row per load or store, taken in turn by the transform kernels.
#pragma once
#include "common.h"

namespace iwdft {

// One token sample of NP adjacent channel pairs as NW 32-bit words (NW = NP for bf16, 2 NP for fp32), fetched
// with one load of 4 NW bytes.
template <int NW>
struct Raw {
  uint32_t w[NW];
};
template <int NW>
__device__ __forceinline__ Raw<NW> load_raw(const char* p) {
  Raw<NW> r;
  if constexpr (NW == 1) {
    r.w[0] = *(const uint32_t*)p;
  } else if constexpr (NW == 2) {
    const uint2 u = *(const uint2*)p;
    r.w[0] = u.x, r.w[1] = u.y;
  } else {
    static_assert(NW == 4, "1, 2 or 4 words per sample");
    const uint4 u = *(const uint4*)p;
    r.w[0] = u.x, r.w[1] = u.y, r.w[2] = u.z, r.w[3] = u.w;
  }
  return r;
}
// The first channel pair of a sample as a complex number (first channel real, second imaginary), and the
// sample with that pair dropped and the next one moved to the front: the pairs are taken in turn inside a
// run-time loop while the words stay in registers (no run-time index).
template <bool BF16, int NW>
__device__ __forceinline__ float2 raw_front(const Raw<NW>& r) {
  if constexpr (BF16) return make_float2(__uint_as_float(r.w[0] << 16), __uint_as_float(r.w[0] & 0xffff0000u));
  else return make_float2(__uint_as_float(r.w[0]), __uint_as_float(r.w[1]));
}
template <bool BF16, int NW>
__device__ __forceinline__ void raw_pop(Raw<NW>& r) {
  constexpr int W = BF16 ? 1 : 2;
#pragma unroll
  for (int n = 0; n + W < NW; ++n) r.w[n] = r.w[n + W];
}

// Channel pairs per load and store of the kernels that run 8192 / 2^logQ transforms side by side and write samples back
// (ablation, reconstruction), and the workgroups (of four pairs) from which on more than one is faster.  Measured, several
// pairs / one, us: ablation of 64 x 8192 tokens bf16 173 / 294, fp32 253 / 404, 16 x 8192 tokens 55 / 83, 61 / 86; where the
// lanes of one pair already cover 32 bytes of a row (bf16) the longer serial chain costs more: 512 x 1024 tokens 95 / 85;
// fp32 there 512 x 1024 134 / 147, 256 x 1024 61 / 56.
constexpr int side_pairs(int logQ, bool bf16) { return bf16 ? (logQ >= 11 ? 4 : 1) : (logQ >= 10 ? 2 : 1); }
constexpr uint64_t side_pairs_min(int logQ) { return logQ == 10 ? 768 : 256; }

// f32_to_bf16 of both (the hardware conversion rounds to nearest even and keeps NaN, bit for bit the same).
__device__ __forceinline__ uint32_t pack_bf16(float2 v) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){v.x, v.y}, bf16x2));
}
// A pair behind the ones that are still there: after as many pops as pushes the words are a row piece again.
template <bool BF16, int NW>
__device__ __forceinline__ void raw_push(Raw<NW>& r, float2 v) {
  raw_pop<BF16, NW>(r);
  if constexpr (BF16) {
    r.w[NW - 1] = pack_bf16(v);
  } else {
    r.w[NW - 2] = __float_as_uint(v.x);
    r.w[NW - 1] = __float_as_uint(v.y);
  }
}
template <int NW>
__device__ __forceinline__ void store_raw(char* p, const Raw<NW>& r) {
  if constexpr (NW == 1) *(uint32_t*)p = r.w[0];
  else if constexpr (NW == 2) *(uint2*)p = make_uint2(r.w[0], r.w[1]);
  else *(uint4*)p = make_uint4(r.w[0], r.w[1], r.w[2], r.w[3]);
}

}  // namespace iwdft
