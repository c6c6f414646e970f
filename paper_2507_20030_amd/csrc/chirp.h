// Transforms of Q points for any Q <= 8192 through the chirp-z identity  k a = (k^2 + a^2 - (a - k)^2) / 2:
//   sum_k Z[k] e^{+j 2 pi k a / Q} = c[a] * sum_k (Z[k] c[k]) h[a - k],   c[n] = e^{+j pi n^2 / Q},  h = conj c,
// a linear convolution with the chirp h, run as a circular one of length N = 2^LOGN >= 2 Q - 1 in LDS: transform, multiply by
// the transform of h (host-made table, already divided by N, in the order the inverse transform leaves), transform back.  The
// transform of the other sign is the conjugate chain.  Shared by the decode attention and the prefill of lengths that are not
// a power of two.
#pragma once
#include "common.h"
#include "fft_core.h"
#include "interp.h"

namespace iwdft {

// v (entries t + T i of the signal, T = N / 16, zero from Q on) convolved with h (CONJ: with conj h) in place; entries from Q
// on are not meaningful afterwards.  H: [8][T] float4, entry j * T + t = table entries of the positions 16 t + 2 j, 16 t + 2 j + 1.
template <int LOGN, bool CONJ>
__device__ __forceinline__ void chirp_convolve(float2* buf, const TabMem& tab, const float4* __restrict__ H, int t,
                                               float2 (&v)[8]) {
  float2 x[16];
  half_inverse<LOGN>(buf, tab, t, v, x);
  const float4* __restrict__ Ht = H + pin_index(t);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const float4 h = Ht[j * fft_threads(LOGN)];
    x[2 * j] = cmul(x[2 * j], make_float2(h.x, CONJ ? -h.y : h.y));
    x[2 * j + 1] = cmul(x[2 * j + 1], make_float2(h.z, CONJ ? -h.w : h.w));
  }
  half_forward<LOGN>(buf, tab, t, x, v);
}

// e^{+j 2 pi a b / M} to fp32 rounding: M is not a power of two, so the phase is reduced in integers and split in double.
__device__ __forceinline__ float2 cis_exact(uint32_t a, uint32_t b, uint32_t M, double inv_M) {
  const uint64_t p = (uint64_t)a * b;
  int64_t r = (int64_t)(p - (uint64_t)((double)p * inv_M) * M);
  if (r < 0) r += M;
  if (r >= (int64_t)M) r -= M;
  const double x = (double)r * inv_M, q = rint(8.0 * x);
  return cis_octant((float)((x - 0.125 * q) * 6.283185307179586477), (int)q);
}
// e^{+j 2 pi ph} through the hardware sine / cosine (argument in revolutions, ~1e-6 absolute).
__device__ __forceinline__ float2 cis_rev(float ph) {
  return make_float2(__builtin_amdgcn_cosf(ph), __builtin_amdgcn_sinf(ph));
}

}  // namespace iwdft
