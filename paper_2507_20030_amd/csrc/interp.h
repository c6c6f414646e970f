// Transforms of Q points for any Q <= 8192 by interpolation from a power-of-two grid (A. Dutt and V. Rokhlin, "Fast Fourier
// transforms for nonequispaced data", SIAM J. Sci. Comput. 14 (1993); window after Kaiser and Bessel).  With a window w of kTaps
// grid points and its Fourier transform W, and N = 2^LOGN >= 2 Q grid points,
//   sum_n x[n] e^{-j 2 pi r n / Q} = sum_m w(r N / Q - m) Y[m],   Y[m] = sum_n x[n] / W(n / N) e^{-j 2 pi m n / N},  |n| <= Q / 2,
// up to an aliasing error of 1e-7 of a single sample at the worst place, 2e-8 in the 2-norm of noise (eight taps, N >= 2 Q; the sums
// of several blocks take ten, see prefill_any.hip): one N-point transform of a signal that is zero in half of its points, where
// the chirp-z identity takes two.  Tables (tables.hip): 1 / W (one value per sample) and the taps of every r up to Q / 2 -- those of -r are
// the same, mirrored.
#pragma once
#include "common.h"
#include "fft_core.h"

namespace iwdft {

// k mod n for factors below 2^21 (M <= 256 * 8192), without an integer division.
__device__ __forceinline__ uint32_t mod_small(uint32_t k, uint32_t n, float inv_n) {  // k < 2^29, k / n < 2^20
  int32_t r = (int32_t)(k - (uint32_t)((float)k * inv_n) * n);  // the quotient is off by one at most
  if (r < 0) r += (int32_t)n;
  if (r >= (int32_t)n) r -= (int32_t)n;
  return (uint32_t)r;
}
// Samples of thread t: time n0 + i N / 16, i = 0 .. 3 (positions 16 t + 4 i) and i = -4 .. -1 (positions 16 t + 4 (i + 4) + 3), n0 =
// sample_at(16 t); all others are zero.  Index into the signal of sample i = 0 .. 7 (0 .. 3, then -4 .. -1), Q or more: none.
template <int LOGN>
__device__ __forceinline__ uint32_t wing_index(uint32_t n0, int i, uint32_t Q) {
  if (i < 4) {
    const uint32_t a = n0 + ((uint32_t)i << (LOGN - 4));
    return a < ((Q + 1) >> 1) ? a : Q;
  }
  const uint32_t a = n0 + ((uint32_t)(i - 8) << (LOGN - 4)) + Q;  // wraps to a large number where n0 + ... < -Q
  return a >= ((Q + 1) >> 1) ? a : Q;
}
constexpr int wing_position(int i) { return i < 4 ? 4 * i : 4 * (i - 4) + 3; }

// The taps of frequency r as laid out by taps_kernel: NT + 1 weights for the grid points e, e + 1, ..., e + NT with e even (one of the
// outer two is zero) and e itself, -4 <= e: [2][n] float4 | [n] float2 (weight, e as bits) for eight taps, [3][n] float4 for ten, n = Q / 2 + 1.
template <int NT>
struct Taps {
  float w[NT + 1];
  int e;
};
template <int NT = kTaps>
__device__ __forceinline__ Taps<NT> load_taps(const float4* __restrict__ tab, uint32_t r, uint32_t Q) {
  static_assert(NT == 8 || NT == 10, "");
  const uint32_t n = (Q >> 1) + 1;
  const float4 a = tab[r], b = tab[n + r];
  Taps<NT> T;
  T.w[0] = a.x, T.w[1] = a.y, T.w[2] = a.z, T.w[3] = a.w, T.w[4] = b.x, T.w[5] = b.y, T.w[6] = b.z, T.w[7] = b.w;
  if constexpr (NT == 8) {
    const float2 c = ((const float2*)(tab + 2 * n))[r];
    T.w[8] = c.x, T.e = __float_as_int(c.y);
  } else {
    const float4 c = tab[2 * n + r];
    T.w[8] = c.x, T.w[9] = c.y, T.w[10] = c.z, T.e = __float_as_int(c.w);
  }
  return T;
}

// The transform leaves the grid in natural order without padding, kHalo entries of either end repeated beyond the other:
// a window of taps is one address, and lanes with neighbouring bins read neighbouring 16 bytes.
constexpr int kHalo = 16;
constexpr int grid_lds(int logN) { return fft_lds(logN) > (1 << logN) + 2 * kHalo ? fft_lds(logN) : (1 << logN) + 2 * kHalo; }

// Grid of the samples x (wing_position; the others not looked at).  Entry m at buf[kHalo + m].  Entries beyond +-reach need not be formed.
template <int LOGN>
__device__ __forceinline__ void grid_forward(float2* buf, const TabMem& tab, int t, float2 (&x)[16], int reach) {
  constexpr int N = 1 << LOGN, T = fft_threads(LOGN), REM = fft_rem(LOGN), NP = fft_np(LOGN);
  constexpr int SP = T + T / 8;  // distance in LDS of entries T apart
  Tw16 w;
  tab.load<LOGN, 1, false>(w, t);
  dft16_1<false, true>(x);
  write16(buf, t, x);
  __syncthreads();
  constexpr int kLast = REM ? NP - 1 : NP - 2;  // last radix-16 pass that stays in place
  if constexpr (kLast >= 1) fft_pass<LOGN, 1, false, (NP > 2 ? 2 : -1)>(buf, tab, t, w, [] {});
  if constexpr (kLast >= 2) fft_pass<LOGN, 2, false, -1>(buf, tab, t, w, [] {});
  static_assert(NP <= 3, "two passes in place at most");
  const float2* own = buf + fpad(t);  // entries t + T i at i * SP
#pragma unroll
  for (int i = 0; i < 16; ++i) x[i] = own[i * SP];
  const float2* __restrict__ tw = tab.tab + tab_off_rem(LOGN);
  const int k0 = pin_index(t);
  if constexpr (REM == 0) {
    dft16<false>(x, w);
  } else if constexpr (REM == 1) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float2 v = tw[k0 + i * T];
      bfly<false>(x[i], x[i + 8], v.x, v.y);
    }
  } else if constexpr (REM == 2) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float4 v = ((const float4*)tw)[k0 + i * T];
      r4<false>(x[i], x[i + 4], x[i + 8], x[i + 12], v.x, v.y, v.z, v.w);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float4 v = ((const float4*)tw)[k0 + i * T], u = ((const float4*)(tw + N / 4))[k0 + i * T];
      r4<false>(x[i], x[i + 2], x[i + 4], x[i + 6], v.x, v.y, v.z, v.w);
      r4<false>(x[i + 8], x[i + 10], x[i + 12], x[i + 14], v.x, v.y, v.z, v.w);
      bfly<false>(x[i], x[i + 8], u.x, u.y);
      bfly<false>(x[i + 2], x[i + 10], u.z, u.w);
      bfly_j<false>(x[i + 4], x[i + 12], u.x, u.y);
      bfly_j<false>(x[i + 6], x[i + 14], u.z, u.w);
    }
  }
  __syncthreads();
  float2* out = buf + kHalo + t;
#pragma unroll
  for (int i = 0; i < 16; ++i)
    if (i < 8 ? i * T <= reach : (16 - (i + 1)) * T < reach) out[i * T] = x[i];  // uniform
  if (t < kHalo) out[N] = x[0];
  if (t >= T - kHalo) out[15 * T - N] = x[15];
  __syncthreads();
}
// Values of the Q-point transform at r and -r.  ODD: N may be odd, which takes 8-byte reads on the way down.
template <bool ODD = false, int NT = kTaps>
__device__ __forceinline__ void grid_at(const float2* buf, int N, const Taps<NT>& T, float2& zr, float2& zm) {
  const float4* up = (const float4*)(buf + (kHalo + T.e));  // e, e + 1, ...
  const float2* dn = buf + (kHalo + N - T.e - NT);          // -e - NT, -e - NT + 1, ... modulo N
  zr = zm = make_float2(0.f, 0.f);
#pragma unroll
  for (int i = 0; i <= NT / 2; ++i) {
    const float4 p = up[i];  // e + 2 i, e + 2 i + 1
    float4 m;                // -(e + 2 i), -(e + 2 i - 1)
    if constexpr (ODD) {
      const float2 m0 = dn[NT - 2 * i], m1 = dn[NT + 1 - 2 * i];
      m = make_float4(m0.x, m0.y, m1.x, m1.y);
    } else {
      m = ((const float4*)dn)[NT / 2 - i];
    }
    zr = make_float2(fmaf(T.w[2 * i], p.x, zr.x), fmaf(T.w[2 * i], p.y, zr.y));
    zm = make_float2(fmaf(T.w[2 * i], m.x, zm.x), fmaf(T.w[2 * i], m.y, zm.y));
    if (i < NT / 2) zr = make_float2(fmaf(T.w[2 * i + 1], p.z, zr.x), fmaf(T.w[2 * i + 1], p.w, zr.y));
    if (i > 0) zm = make_float2(fmaf(T.w[2 * i - 1], m.z, zm.x), fmaf(T.w[2 * i - 1], m.w, zm.y));
  }
}

}  // namespace iwdft
