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

// Two channels that travel as real and imaginary part of one transform may differ by orders of magnitude, and its rounding
// error goes with the larger one.  The second channel is therefore scaled by a power of two (exact) to the size of the first
// one's largest value, and its spectrum back; a channel that is not finite stays out of the transform (its spectrum is NaN,
// its partner's is not), one that is zero stays exactly zero.  Magnitudes are compared as bits: infinities and NaN come out on
// top.
struct PairScale {
  float up;      // factor of the second channel on the way in
  float h0, h1;  // factors of the sums and differences of mirror entries (1/2 of them each) on the way out
};
__device__ __forceinline__ bool not_finite(uint32_t magnitude) { return magnitude >= 0x7f800000u; }
__device__ __forceinline__ PairScale pair_scale(uint32_t m0, uint32_t m1) {  // largest magnitudes, as float bits
  // 2^(exponent of the first one's maximum - that of the second's); 1 where either is zero, subnormal or not finite
  const int e0 = (int)(m0 >> 23), e1 = (int)(m1 >> 23);
  const int de = (e0 > 0 && e0 < 255 && e1 > 0 && e1 < 255) ? min(max(e0 - e1, -60), 60) : 0;
  PairScale s;
  s.up = __uint_as_float((uint32_t)(127 + de) << 23);
  s.h0 = not_finite(m0) ? NAN : m0 ? 0.5f : 0.f;
  s.h1 = not_finite(m1) ? NAN : m1 ? 0.5f * __uint_as_float((uint32_t)(127 - de) << 23) : 0.f;
  return s;
}
// The same for all pairs of the raw words of a thread's C samples, in a workgroup of WAVES waves with NS transforms interleaved
// over the lanes (this thread's: tid % NS): channels that are not finite are cleared in the words.  red is free again behind the
// next barrier.  One lane reduction and one barrier serve all pairs of a load; the maxima of a bf16 pair are one packed word.
template <bool BF16>
__device__ __forceinline__ uint32_t word_max(uint32_t a, uint32_t b) {  // of magnitudes; per half for bf16
  if constexpr (BF16) {
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
  } else {
    return max(a, b);
  }
}
template <int N>
__device__ __forceinline__ uint32_t row_ror(uint32_t v) {  // the value N lanes further in the row of 16
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x120 + N, 0xf, 0xf, false);
}
template <bool BF16, int NS, int NW, int NP, int C, int WAVES>
__device__ __forceinline__ void scale_pairs(Raw<NW> (&z)[C], int tid, uint32_t (&red)[WAVES][NS][NW], PairScale (&sc)[NP]) {
  static_assert(NW == NP * (BF16 ? 1 : 2) && NS <= 32, "");
  uint32_t m[NW];
#pragma unroll
  for (int n = 0; n < NW; ++n) {
    m[n] = 0u;
#pragma unroll
    for (int i = 0; i < C; ++i) m[n] = word_max<BF16>(m[n], z[i].w[n] & (BF16 ? 0x7fff7fffu : 0x7fffffffu));
    // over the lanes of the same transform: rotations inside the rows of 16 lanes, then the rows
    if constexpr (NS <= 8) m[n] = word_max<BF16>(m[n], row_ror<8>(m[n]));
    if constexpr (NS <= 4) m[n] = word_max<BF16>(m[n], row_ror<4>(m[n]));
    if constexpr (NS <= 2) m[n] = word_max<BF16>(m[n], row_ror<2>(m[n]));
    if constexpr (NS <= 1) m[n] = word_max<BF16>(m[n], row_ror<1>(m[n]));
  }
#pragma unroll
  for (int o = 16; o <= 32; o *= 2) {
#pragma unroll
    for (int n = 0; n < NW; ++n)
      if (o >= NS) m[n] = word_max<BF16>(m[n], (uint32_t)__shfl_xor((int)m[n], o));
  }
  if ((tid & 63) < NS) {
#pragma unroll
    for (int n = 0; n < NW; ++n) red[tid >> 6][tid & (NS - 1)][n] = m[n];
  }
  __syncthreads();
#pragma unroll
  for (int n = 0; n < NW; ++n) {
#pragma unroll
    for (int w = 0; w < WAVES; ++w) m[n] = word_max<BF16>(m[n], red[w][tid & (NS - 1)][n]);
    if constexpr (NS == 1) m[n] = (uint32_t)__builtin_amdgcn_readfirstlane((int)m[n]);
    uint32_t keep;
    if constexpr (BF16) keep = (not_finite(m[n] << 16) ? 0u : 0xffffu) | (not_finite(m[n] & 0xffff0000u) ? 0u : 0xffff0000u);
    else keep = not_finite(m[n]) ? 0u : ~0u;
    if (keep != ~0u) {
#pragma unroll
      for (int i = 0; i < C; ++i) z[i].w[n] &= keep;
    }
  }
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    if constexpr (BF16) sc[p] = pair_scale(m[p] << 16, m[p] & 0xffff0000u);
    else sc[p] = pair_scale(m[2 * p], m[2 * p + 1]);
  }
}

// Channel pairs per load and store of the kernels that run 8192 / 2^logQ transforms side by side and write samples back
// (ablation, reconstruction), and the workgroups (of four pairs) from which on more than one is faster.  Measured, several
// pairs / one, us: ablation of 64 x 8192 tokens bf16 173 / 294, fp32 253 / 404, 16 x 8192 tokens 55 / 83, 61 / 86; where the
// lanes of one pair already cover 32 bytes of a row (bf16) the longer serial chain costs more: 512 x 1024 tokens 95 / 85;
// fp32 there 512 x 1024 134 / 147, 256 x 1024 61 / 56.
constexpr int side_pairs(int logQ, bool bf16) { return bf16 ? (logQ >= 11 ? 4 : 1) : (logQ >= 10 ? 2 : 1); }
constexpr uint64_t side_pairs_min(int logQ) { return logQ == 10 ? 768 : 256; }
// Whether two transforms of 8192 points share a workgroup of 1024 threads (twice as many bytes of a row per line that a load or store
// touches), `blocks` of them per XCD: not where a round of one per CU would stay partly empty -- two of 512 threads are faster where they have a CU
// to themselves.  Us, one / two transforms, by rounds: prefill 1 42 / 36, 1.5 59 / 66, 2 78 / 71, 2.5 122 / 130, 3.5 165 / 171, 8.5 332 / 340, 16
// 724 / 663; fp32 1 31 / 24, 3 77 / 71, 16 532 / 521; reconstruction 1.5 75 / 87, 2 90 / 84, 3 157 / 139, 4 230 / 223; ablation fp32 4 253 / 230
// (bf16, 2: 161 / 157 and 169 / 174, so it stays with one).
constexpr int64_t kTwoRound = 32;  // workgroups that an XCD runs at a time
inline bool two_transforms(int64_t blocks) {
  return blocks >= kTwoRound && (blocks + kTwoRound - 1) / kTwoRound * kTwoRound * 20 <= blocks * 21;
}

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
