// In-LDS complex transforms of 2^LOGQ points (256 .. 16384) by fft_threads(LOGQ) threads t of a workgroup, 16 points per
// thread: radix-16 register passes of multiply-add butterflies.  The narrow end of both directions stays in registers --
// the inverse transform (natural order in) ends with every thread holding 16 consecutive positions of the digit-reversed
// order, the forward one (natural order out) starts from them -- so what a kernel does to the samples costs no LDS trip.
#pragma once
#include "common.h"
#include "fft_tab.h"

namespace iwdft {

constexpr int kFftMaxLogQ = 13;  // longest transform of the power-of-two paths
__host__ __device__ constexpr int fft_threads(int logQ) { return 1 << (logQ - 4); }
// Threads of a workgroup of the decode attention: those of its transform, a whole wave at least -- below 64 the bins are many for the lanes of the
// transform alone (8 slices, 4 heads, a deferred step: M = 512, 384 bins 46 -> 35 us, M = 256, 256 bins 48 -> 33).
__host__ __device__ constexpr int attn_threads(int logQ) { return fft_threads(logQ) < 64 ? 64 : fft_threads(logQ); }

// LDS index of position i: two float2 of padding per 16 keep 16-byte accesses to a thread's 16 positions aligned and spread
// both these and the strided accesses of the wide passes over all banks.
__device__ __forceinline__ int fpad(int i) { return i + ((i >> 4) << 1); }
__host__ __device__ constexpr int fft_lds(int logQ) { return (1 << logQ) + (1 << logQ) / 8; }

// Transforms of 2^logQ points that a workgroup runs side by side, interleaved over the lanes (thread = t NS + g for thread t of
// transform g), its threads, and the distance of the buffers: 8 lanes with 16-byte and 16 lanes with 8-byte accesses fall into
// distinct banks.  512 threads; TWO: two transforms of 8192 points by 1024, see prefill_fft.hip.
__host__ __device__ constexpr int side_ns(int logQ, bool two = false) { return two ? 2 : 1 << (13 - logQ); }
__host__ __device__ constexpr int side_threads(int logQ, bool two = false) { return side_ns(logQ, two) * fft_threads(logQ); }
__host__ __device__ constexpr int side_bs(int logQ, bool two = false) {
  const int ns = side_ns(logQ, two);
  return fft_lds(logQ) + (ns == 1 ? 0 : ns >= 8 ? 2 : 16 / ns);
}
// Time index of position 16 t + m relative to that of position 16 t: the digits of m reversed, times Q / 16.
template <int LOGQ>
__device__ __forceinline__ constexpr int sample_step(int m) { return (((m & 3) << 2) | (m >> 2)) << (LOGQ - 4); }

// Base-4 digit reversal of an even number of bits.
template <int BITS>
__device__ __forceinline__ uint32_t digit_reverse4(uint32_t i) {
  const uint32_t r = __brev(i) >> (32 - BITS);
  return ((r & 0x55555555u) << 1) | ((r >> 1) & 0x55555555u);
}
// Time index of the sample at position p.
template <int LOGQ>
__device__ __forceinline__ uint32_t sample_at(uint32_t p) {
  if constexpr (LOGQ & 1) return (digit_reverse4<LOGQ - 1>(p & ((1u << (LOGQ - 1)) - 1u)) << 1) | (p >> (LOGQ - 1));
  else return digit_reverse4<LOGQ>(p);
}

__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 conjf2(float2 a) { return make_float2(a.x, -a.y); }

// Both transforms are built from butterflies a, b -> a +- w b whose twiddle w = c (1 + j t) comes from a table as
// (c, t) = (cos, tan): with p = b.x - t b.y, q = b.y + t b.x (w b = c (p + j q)) a butterfly is six multiply-adds, where a
// complex product and two additions are eight, and no twiddle is derived at run time.  The forward transform (decimation
// in time, narrow span first) has such butterflies by nature; the inverse one splits the spectrum block by block
// (x^L - z  ->  x^(L/4) - z^(1/4) j^r), so that its twiddles multiply inputs too and depend on the block only.  Where c is
// small t is large, but the rounding of t b.y is scaled by c: nothing is lost.  (It costs range: t reaches 2^30, so sums beyond
// 2^97 overflow.)  The form is E. Linzer and E. Feig's, "Modified FFTs for fused multiply-add architectures", Mathematics of
// Computation 60 (1993).
// INV: w as tabled (sign +), otherwise its conjugate.
template <bool INV>
__device__ __forceinline__ void bfly(float2& a, float2& b, float c, float t) {
  const float s = INV ? t : -t;
  const float p = fmaf(-s, b.y, b.x), q = fmaf(s, b.x, b.y);
  b = make_float2(fmaf(-c, p, a.x), fmaf(-c, q, a.y));
  a = make_float2(fmaf(c, p, a.x), fmaf(c, q, a.y));
}
// The same with j w (INV) or -j conj(w).
template <bool INV>
__device__ __forceinline__ void bfly_j(float2& a, float2& b, float c, float t) {
  const float s = INV ? t : -t, cj = INV ? c : -c;
  const float p = fmaf(-s, b.y, b.x), q = fmaf(s, b.x, b.y);
  b = make_float2(fmaf(cj, q, a.x), fmaf(-cj, p, a.y));
  a = make_float2(fmaf(-cj, q, a.x), fmaf(cj, p, a.y));
}
// ... with w = 1 and with w = +-j.
__device__ __forceinline__ void bfly1(float2& a, float2& b) {
  const float2 u = a;
  a = cadd(u, b);
  b = csub(u, b);
}
template <bool INV>
__device__ __forceinline__ void bfly1_j(float2& a, float2& b) {
  const float2 u = a, v = INV ? make_float2(-b.y, b.x) : make_float2(b.y, -b.x);
  a = cadd(u, v);
  b = csub(u, v);
}
__device__ __forceinline__ void cswap(float2& a, float2& b) {
  const float2 t = a;
  a = b;
  b = t;
}

// Radix-4 butterfly: input m times w^m, then the 4-point transform; (c2, t2): w^2, (c1, t1): w.  W2J: w^2 is j times the
// (c2, t2) given (forward: -j times its conjugate).
template <bool INV, bool W2J = false>
__device__ __forceinline__ void r4(float2& x0, float2& x1, float2& x2, float2& x3, float c2, float t2, float c1, float t1) {
  if constexpr (W2J) {
    bfly_j<INV>(x0, x2, c2, t2);
    bfly_j<INV>(x1, x3, c2, t2);
  } else {
    bfly<INV>(x0, x2, c2, t2);
    bfly<INV>(x1, x3, c2, t2);
  }
  bfly<INV>(x0, x1, c1, t1);
  bfly_j<INV>(x2, x3, c1, t1);
  cswap(x1, x2);
}
template <bool INV>
__device__ __forceinline__ void r4_1(float2& x0, float2& x1, float2& x2, float2& x3) {  // w = 1
  bfly1(x0, x2);
  bfly1(x1, x3);
  bfly1(x0, x1);
  bfly1_j<INV>(x2, x3);
  cswap(x1, x2);
}
constexpr float kCos45 = 0.70710678118654752f;
template <bool INV>
__device__ __forceinline__ void r4_e(float2& x0, float2& x1, float2& x2, float2& x3) {  // w = e^{+-j pi / 4}
  bfly1_j<INV>(x0, x2);
  bfly1_j<INV>(x1, x3);
  bfly<INV>(x0, x1, kCos45, 1.f);
  bfly_j<INV>(x2, x3, kCos45, 1.f);
  cswap(x1, x2);
}

// The eight twiddles of a radix-16 butterfly (see fft_tab.hip).
struct Tw16 {
  float4 s, a, b, c;
};
// Table loads are invariant; without the tie to this place the compiler hoists those of several passes (or out of a loop
// over transforms) and spills.
__device__ __forceinline__ int pin_index(int i) {
  asm volatile("" : "+v"(i) : : "memory");
  return i;
}
// Where a pass finds its twiddles.  TabMem: the tables in constant memory; every pass fetches those of the next one before
// its barrier, so that the latency does not start behind it.
struct TabMem {
  static constexpr bool kEarly = true;
  const float2* __restrict__ tab;  // this length's block
  template <int LOGQ, int K, bool INV>
  __device__ __forceinline__ void load(Tw16& w, int t) const {
    constexpr int N = INV ? tab_n_inv(LOGQ, K) : tab_n_fwd(K);
    constexpr int OFF = INV ? tab_off_inv(LOGQ, K) : tab_off_fwd(LOGQ, K);
    if constexpr (N > 1) {
      const float4* __restrict__ p = (const float4*)(tab + OFF) + pin_index(INV ? t >> (4 * K) : t & (N - 1));
      w.s = p[0];
      w.a = p[N];
      w.b = p[2 * N];
      w.c = p[3 * N];
    }
  }
};
// TabLds: a copy of the forward passes' tables (K = 1, 2, ... behind each other) in LDS, for kernels that keep loads of
// their own in flight: vector memory answers in order, so a table load behind them would wait for them.
struct TabLds {
  static constexpr bool kEarly = false;
  const float2* __restrict__ tab;  // this length's block in memory (the stage at the wide end)
  const float4* lds;
  template <int LOGQ>
  static constexpr int entries() {  // float4
    int n = 0;
    for (int k = 1; k < fft_np(LOGQ); ++k) n += 4 * tab_n_fwd(k);
    return n;
  }
  template <int LOGQ>
  __device__ __forceinline__ void fill(float4* dst, int t) const {  // the tables are adjacent in memory too
    const float4* __restrict__ src = (const float4*)(tab + tab_off_fwd(LOGQ, 1));
    for (int i = t; i < entries<LOGQ>(); i += fft_threads(LOGQ)) dst[i] = src[i];
  }
  template <int LOGQ, int K, bool INV>
  __device__ __forceinline__ void load(Tw16& w, int t) const {
    static_assert(!INV, "forward tables only");
    constexpr int N = tab_n_fwd(K), OFF = (tab_off_fwd(LOGQ, K) - tab_off_fwd(LOGQ, 1)) / 2;
    const float4* p = lds + OFF + (t & (N - 1));
    w.s = p[0];
    w.a = p[N];
    w.b = p[2 * N];
    w.c = p[3 * N];
  }
};

// 16 points at positions p0 + m * span: INV takes the wide radix-4 stage first, the forward transform the narrow one.
template <bool INV>
__device__ __forceinline__ void dft16(float2 (&x)[16], const Tw16& w) {
  constexpr int S = INV ? 4 : 1, G = INV ? 1 : 4;  // element stride inside a group of the first stage, group stride
#pragma unroll
  for (int g = 0; g < 4; ++g)
    r4<INV>(x[g * G], x[g * G + S], x[g * G + 2 * S], x[g * G + 3 * S], w.s.x, w.s.y, w.s.z, w.s.w);
  r4<INV>(x[0], x[G], x[2 * G], x[3 * G], w.a.x, w.a.y, w.b.x, w.b.y);
  r4<INV>(x[S], x[S + G], x[S + 2 * G], x[S + 3 * G], w.a.z, w.a.w, w.b.z, w.b.w);
  r4<INV, true>(x[2 * S], x[2 * S + G], x[2 * S + 2 * G], x[2 * S + 3 * G], w.a.x, w.a.y, w.c.x, w.c.y);
  r4<INV, true>(x[3 * S], x[3 * S + G], x[3 * S + 2 * G], x[3 * S + 3 * G], w.a.z, w.a.w, w.c.z, w.c.w);
}
// WINGS (forward): the samples of the two middle quarters of the time axis, x[4 g + 1] and x[4 g + 2], are zero and not looked at.
template <bool INV, bool WINGS = false>
__device__ __forceinline__ void dft16_1(float2 (&x)[16]) {  // t = 1
  constexpr int S = INV ? 4 : 1, G = INV ? 1 : 4;
  constexpr float kC1 = 0.92387953251128674f, kT1 = 0.41421356237309505f;  // cos, tan 22.5 degrees
  constexpr float kC3 = 0.38268343236508977f, kT3 = 2.41421356237309505f;  // cos, tan 67.5 degrees
  static_assert(!(INV && WINGS), "forward only");
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    if constexpr (WINGS) {
      const float2 a = x[4 * g], b = x[4 * g + 3];
      x[4 * g] = cadd(a, b);
      x[4 * g + 1] = make_float2(a.x - b.y, a.y + b.x);
      x[4 * g + 2] = csub(a, b);
      x[4 * g + 3] = make_float2(a.x + b.y, a.y - b.x);
    } else {
      r4_1<INV>(x[g * G], x[g * G + S], x[g * G + 2 * S], x[g * G + 3 * S]);
    }
  }
  r4_1<INV>(x[0], x[G], x[2 * G], x[3 * G]);
  r4<INV>(x[S], x[S + G], x[S + 2 * G], x[S + 3 * G], kCos45, 1.f, kC1, kT1);
  r4_e<INV>(x[2 * S], x[2 * S + G], x[2 * S + 2 * G], x[2 * S + 3 * G]);
  r4<INV, true>(x[3 * S], x[3 * S + G], x[3 * S + 2 * G], x[3 * S + 3 * G], kCos45, 1.f, kC3, kT3);
}

// The 16 consecutive positions of thread t, 16 bytes at a time.
__device__ __forceinline__ void read16(const float2* buf, int t, float2 (&x)[16]) {
  const float4* b = (const float4*)(buf + 18 * t);
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    const float4 v = b[m];
    x[2 * m] = make_float2(v.x, v.y);
    x[2 * m + 1] = make_float2(v.z, v.w);
  }
}
__device__ __forceinline__ void write16(float2* buf, int t, const float2 (&x)[16]) {
  float4* b = (float4*)(buf + 18 * t);
#pragma unroll
  for (int m = 0; m < 8; ++m) b[m] = make_float4(x[2 * m].x, x[2 * m].y, x[2 * m + 1].x, x[2 * m + 1].y);
}

// One radix-16 pass of span 16^K (K >= 1) in place.  Tab::kEarly: w holds its twiddles on entry and, NEXT >= 0, those of
// the pass of span 16^NEXT on return.  hook(k) runs between the butterflies and the stores.
// HALF: the upper half of the input is zero (only looked at where the radix-2 stage comes with the reads).
// NORM: the input is divided by Q on the way in.
template <int LOGQ, int K, bool INV, int NEXT, bool HALF = false, bool NORM = false, typename Tab, typename Hook>
__device__ __forceinline__ void fft_pass(float2* buf, const Tab& tab, int t, Tw16& w, Hook hook) {
  constexpr int Q = 1 << LOGQ, S = 4 * K, s2 = 1 << S;
  constexpr int SP = s2 + s2 / 8;  // distance in LDS of positions s2 apart
  constexpr bool kOne = (INV ? tab_n_inv(LOGQ, K) : tab_n_fwd(K)) == 1;
  constexpr bool kHalves = INV && fft_rem(LOGQ) == 1 && K == fft_np(LOGQ) - 1;  // the radix-2 stage comes with the reads
  float2 x[16];
  float2* base = buf + fpad(((t >> S) << (S + 4)) + (t & (s2 - 1)));
  if constexpr (!Tab::kEarly) tab.template load<LOGQ, K, INV>(w, t);
  if constexpr (kHalves) {
    const float2* lo = buf + fpad(t & (s2 - 1));
    const float2* hi = lo + Q / 2 + Q / 16;
    const float sg = (t >> S) ? -1.f : 1.f;  // block 0: the even samples, block 1: the odd ones
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      x[m] = lo[m * SP];
      if constexpr (!HALF) {
        const float2 v = hi[m * SP];
        x[m] = make_float2(fmaf(sg, v.x, x[m].x), fmaf(sg, v.y, x[m].y));
      }
    }
    __syncthreads();
  } else {
#pragma unroll
    for (int m = 0; m < 16; ++m) x[m] = base[m * SP];
  }
  if constexpr (NORM) {
#pragma unroll
    for (int m = 0; m < 16; ++m) x[m] = make_float2(x[m].x * (1.f / Q), x[m].y * (1.f / Q));
  }
  if constexpr (kOne) dft16_1<INV>(x);
  else dft16<INV>(x, w);
  if constexpr (NEXT >= 0 && Tab::kEarly) tab.template load<LOGQ, NEXT, INV>(w, t);
  hook();
#pragma unroll
  for (int m = 0; m < 16; ++m) base[m * SP] = x[m];
  __syncthreads();
}

// The stage of radix 2^rem at the wide end as a pass of its own.
template <int LOGQ, bool INV>
__device__ __forceinline__ void fft_wide(float2* buf, const float2* __restrict__ tab, int t) {
  constexpr int Q = 1 << LOGQ, T = fft_threads(LOGQ), REM = fft_rem(LOGQ), R = 1 << REM, NB = Q / R;
  constexpr int SP = NB + NB / 8;
  const float2* __restrict__ tw = tab + tab_off_rem(LOGQ);
#pragma unroll
  for (int it = 0; it < NB / T; ++it) {
    const int k = it * T + t;
    float2* b = buf + fpad(k);
    float2 x[R];
#pragma unroll
    for (int m = 0; m < R; ++m) x[m] = b[m * SP];
    if constexpr (REM == 1) {
      if constexpr (INV) bfly1(x[0], x[1]);
      else {
        const float2 w = tw[pin_index(k)];
        bfly<false>(x[0], x[1], w.x, w.y);
      }
    } else if constexpr (REM == 2) {
      if constexpr (INV) r4_1<true>(x[0], x[1], x[2], x[3]);
      else {
        const float4 w = ((const float4*)tw)[pin_index(k)];
        r4<false>(x[0], x[1], x[2], x[3], w.x, w.y, w.z, w.w);
      }
    } else {
      static_assert(REM == 3, "radix 2, 4 or 8");
      if constexpr (INV) {
#pragma unroll
        for (int m = 0; m < 4; ++m) bfly1(x[m], x[m + 4]);
        r4_1<true>(x[0], x[1], x[2], x[3]);
        r4_e<true>(x[4], x[5], x[6], x[7]);
      } else {
        const int i = pin_index(k);
        const float4 w = ((const float4*)tw)[i], v = ((const float4*)(tw + Q / 4))[i];
        r4<false>(x[0], x[1], x[2], x[3], w.x, w.y, w.z, w.w);
        r4<false>(x[4], x[5], x[6], x[7], w.x, w.y, w.z, w.w);
        bfly<false>(x[0], x[4], v.x, v.y);
        bfly<false>(x[1], x[5], v.z, v.w);
        bfly_j<false>(x[2], x[6], v.x, v.y);
        bfly_j<false>(x[3], x[7], v.z, v.w);
      }
    }
#pragma unroll
    for (int m = 0; m < R; ++m) b[m * SP] = x[m];
  }
  __syncthreads();
}

// Inverse transform of the natural-order spectrum in buf (complete: behind a barrier); on return x holds the samples at
// positions 16 t + m.  buf may be overwritten position by position by the same thread without a
// barrier, otherwise only behind one.  tab: this length's block of the tables.  NORM: with the factor 1 / Q, applied
// ahead of the first stage whose twiddles are not constant, so that no sum exceeds the range of the samples and their spectrum.
template <int LOGQ, int K = fft_np(LOGQ) - 1, bool NORM = false>
__device__ __forceinline__ void fft_inv_passes(float2* buf, const TabMem& tab, int t, Tw16& w) {
  if constexpr (K >= 1) {
    fft_pass<LOGQ, K, true, K - 1, false, NORM>(buf, tab, t, w, [] {});
    fft_inv_passes<LOGQ, K - 1>(buf, tab, t, w);
  }
}
template <int LOGQ, bool NORM = false>
__device__ __forceinline__ void fft_inverse(float2* buf, const float2* __restrict__ tab, int t, float2 (&x)[16]) {
  static_assert(fft_np(LOGQ) >= 2, "256 points at least");
  Tw16 w;
  if constexpr (fft_rem(LOGQ) >= 2) fft_wide<LOGQ, true>(buf, tab, t);
  const TabMem tm{tab};
  tm.load<LOGQ, fft_np(LOGQ) - 1, true>(w, t);
  fft_inv_passes<LOGQ, fft_np(LOGQ) - 1, NORM>(buf, tm, t, w);
  read16(buf, t, x);
  dft16<true>(x, w);
}

// Forward transform of the samples x at positions 16 t + m; buf is free (behind a barrier, or last read by
// fft_inverse).  On return buf holds the natural-order spectrum, complete for even LOGQ and for WIDE; otherwise the last
// radix-2 stage is left to spectrum_pair, which forms it for the entries that are wanted.
template <int LOGQ, int K, typename Tab, typename Hook>
__device__ __forceinline__ void fft_fwd_passes(float2* buf, const Tab& tab, int t, Tw16& w, Hook hook) {
  auto h = [&] { hook(K); };
  if constexpr (K + 1 < fft_np(LOGQ)) {
    fft_pass<LOGQ, K, false, K + 1>(buf, tab, t, w, h);
    fft_fwd_passes<LOGQ, K + 1>(buf, tab, t, w, hook);
  } else {
    fft_pass<LOGQ, K, false, -1>(buf, tab, t, w, h);
  }
}
// hook(k) runs between the butterflies of radix-16 pass k = 0 .. fft_np(LOGQ) - 1 and its stores.
template <int LOGQ, bool WIDE = false, typename Tab, typename Hook>
__device__ __forceinline__ void fft_forward(float2* buf, const Tab& tab, int t, float2 (&x)[16], Hook hook) {
  Tw16 w;
  if constexpr (Tab::kEarly) tab.template load<LOGQ, 1, false>(w, t);
  dft16_1<false>(x);
  hook(0);
  write16(buf, t, x);
  __syncthreads();
  fft_fwd_passes<LOGQ, 1>(buf, tab, t, w, hook);
  if constexpr (fft_rem(LOGQ) >= 2 || (WIDE && fft_rem(LOGQ) == 1)) fft_wide<LOGQ, false>(buf, tab.tab, t);
}

// Workgroup barriers inside the two, for waves beside them that have no transform.
constexpr int fft_inverse_barriers(int logQ) { return (fft_rem(logQ) >= 2) + (fft_np(logQ) - 1) + (fft_rem(logQ) == 1); }
constexpr int fft_forward_barriers(int logQ) { return 1 + (fft_np(logQ) - 1) + (fft_rem(logQ) >= 2); }

// The two transforms between signals of at most N / 2 points, for convolutions of length N = 2^LOGN (chirp.h): thread t holds
// entries t + T i, i < 8, T = N / 16, in registers; the upper half of the inverse transform's input is zero, that of the
// forward transform's output is not formed.  Neither needs a barrier in front as long as buf was last touched at these and
// the thread's other entries t + T i, i < 16, only.
template <int LOGN>
__device__ __forceinline__ void half_inverse(float2* buf, const TabMem& tab, int t, const float2 (&v)[8], float2 (&x)[16]) {
  constexpr int N = 1 << LOGN, T = fft_threads(LOGN), REM = fft_rem(LOGN), NP = fft_np(LOGN);
  constexpr int SP = T + T / 8;  // distance in LDS of entries T apart
  static_assert(NP >= 2 && T >= 16, "256 points at least");
  Tw16 w;
  float2* b = buf + fpad(t);
  if constexpr (REM == 0) {  // the wide pass starts from the registers
#pragma unroll
    for (int m = 0; m < 8; ++m) x[m] = v[m], x[m + 8] = make_float2(0.f, 0.f);
    dft16_1<true>(x);
    tab.load<LOGN, NP - 2, true>(w, t);
#pragma unroll
    for (int m = 0; m < 16; ++m) b[m * SP] = x[m];
    __syncthreads();
    fft_inv_passes<LOGN, NP - 2>(buf, tab, t, w);
  } else {
    tab.load<LOGN, NP - 1, true>(w, t);
    if constexpr (REM == 1) {
#pragma unroll
      for (int i = 0; i < 8; ++i) b[i * SP] = v[i];
      __syncthreads();
      fft_pass<LOGN, NP - 1, true, NP - 2, true>(buf, tab, t, w, [] {});
      fft_inv_passes<LOGN, NP - 2>(buf, tab, t, w);
    } else {
      if constexpr (REM == 2) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float2 u = v[i], z = v[i + 4];
          b[i * SP] = cadd(u, z);
          b[(i + 4) * SP] = make_float2(u.x - z.y, u.y + z.x);
          b[(i + 8) * SP] = csub(u, z);
          b[(i + 12) * SP] = make_float2(u.x + z.y, u.y - z.x);
        }
      } else {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          float2 y[8];
#pragma unroll
          for (int m = 0; m < 4; ++m) y[m] = y[m + 4] = v[i + 2 * m];
          r4_1<true>(y[0], y[1], y[2], y[3]);
          r4_e<true>(y[4], y[5], y[6], y[7]);
#pragma unroll
          for (int m = 0; m < 8; ++m) b[(i + 2 * m) * SP] = y[m];
        }
      }
      __syncthreads();
      fft_inv_passes<LOGN, NP - 1>(buf, tab, t, w);
    }
  }
  static_assert(N == 16 * T, "");
  read16(buf, t, x);
  dft16<true>(x, w);
}
// buf: last read by half_inverse.
template <int LOGN>
__device__ __forceinline__ void half_forward(float2* buf, const TabMem& tab, int t, float2 (&x)[16], float2 (&v)[8]) {
  constexpr int N = 1 << LOGN, T = fft_threads(LOGN), REM = fft_rem(LOGN), NP = fft_np(LOGN);
  constexpr int SP = T + T / 8;
  const float2* b = buf + fpad(t);
  const float2* __restrict__ tw = tab.tab + tab_off_rem(LOGN);
  Tw16 w;
  tab.load<LOGN, 1, false>(w, t);
  dft16_1<false>(x);
  write16(buf, t, x);
  __syncthreads();
  if constexpr (REM == 0) {
    if constexpr (NP == 3) fft_pass<LOGN, 1, false, 2>(buf, tab, t, w, [] {});
    static_assert(NP <= 3, "one pass between the two ends at most");
#pragma unroll
    for (int m = 0; m < 16; ++m) x[m] = b[m * SP];
    dft16<false>(x, w);
#pragma unroll
    for (int m = 0; m < 8; ++m) v[m] = x[m];
  } else if constexpr (REM == 1) {
    float2 wt[8];  // fetched before the last barrier
    fft_fwd_passes<LOGN, 1>(buf, tab, t, w, [&](int k) {
      if (k != NP - 1) return;
      const int i0 = pin_index(t);
#pragma unroll
      for (int i = 0; i < 8; ++i) wt[i] = tw[i0 + i * T];
    });
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      float2 o = b[(i + 8) * SP];
      v[i] = b[i * SP];
      bfly<false>(v[i], o, wt[i].x, wt[i].y);
    }
  } else if constexpr (REM == 2) {
    float4 wt[4];
    fft_fwd_passes<LOGN, 1>(buf, tab, t, w, [&](int k) {
      if (k != NP - 1) return;
      const int i0 = pin_index(t);
#pragma unroll
      for (int i = 0; i < 4; ++i) wt[i] = ((const float4*)tw)[i0 + i * T];
    });
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float2 y0 = b[i * SP], y1 = b[(i + 4) * SP], y2 = b[(i + 8) * SP], y3 = b[(i + 12) * SP];
      r4<false>(y0, y1, y2, y3, wt[i].x, wt[i].y, wt[i].z, wt[i].w);
      v[i] = y0;
      v[i + 4] = y1;
    }
  } else {
    float4 wt[2], wu[2];
    fft_fwd_passes<LOGN, 1>(buf, tab, t, w, [&](int k) {
      if (k != NP - 1) return;
      const int i0 = pin_index(t);
#pragma unroll
      for (int i = 0; i < 2; ++i) wt[i] = ((const float4*)tw)[i0 + i * T], wu[i] = ((const float4*)(tw + N / 4))[i0 + i * T];
    });
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      float2 y[8];
#pragma unroll
      for (int m = 0; m < 8; ++m) y[m] = b[(i + 2 * m) * SP];
      r4<false>(y[0], y[1], y[2], y[3], wt[i].x, wt[i].y, wt[i].z, wt[i].w);
      r4<false>(y[4], y[5], y[6], y[7], wt[i].x, wt[i].y, wt[i].z, wt[i].w);
      bfly<false>(y[0], y[4], wu[i].x, wu[i].y);
      bfly<false>(y[1], y[5], wu[i].z, wu[i].w);
      bfly_j<false>(y[2], y[6], wu[i].x, wu[i].y);
      bfly_j<false>(y[3], y[7], wu[i].z, wu[i].w);
#pragma unroll
      for (int m = 0; m < 4; ++m) v[i + 2 * m] = y[m];
    }
  }
}

// Table entry that spectrum_pair needs for entry r (nothing when the spectrum is complete).
template <int LOGQ>
__device__ __forceinline__ float2 pair_twiddle(const float2* __restrict__ tab, uint32_t r) {
  if constexpr (fft_rem(LOGQ) == 1) return tab[tab_off_rem(LOGQ) + (r & ((1u << (LOGQ - 1)) - 1u))];
  else return make_float2(1.f, 0.f);
}
// Entries r and -r (mod Q) of the spectrum that fft_forward left in buf; w = pair_twiddle(r).
template <int LOGQ>
__device__ __forceinline__ void spectrum_pair(const float2* buf, uint32_t r, float2 w, float2& zr, float2& zm) {
  constexpr uint32_t Q = 1u << LOGQ, H = Q / 2;
  if constexpr (fft_rem(LOGQ) == 1) {
    // Z[k + H s] = E[k] + (-1)^s W^k O[k]; the mirror entry is H - k with W^(H - k) = -conj(W^k)
    const uint32_t k = r & (H - 1), km = (H - k) & (H - 1);
    const float c = (r & H) ? -w.x : w.x;
    const float2 e = buf[fpad(k)], o = buf[fpad(k) + (int)(H + H / 8)], em = buf[fpad(km)], om = buf[fpad(km) + (int)(H + H / 8)];
    zr = make_float2(fmaf(c, fmaf(w.y, o.y, o.x), e.x), fmaf(c, fmaf(-w.y, o.x, o.y), e.y));
    zm = make_float2(fmaf(c, fmaf(-w.y, om.y, om.x), em.x), fmaf(c, fmaf(w.y, om.x, om.y), em.y));
  } else {
    zr = buf[fpad((int)r)];
    zm = buf[fpad((int)((Q - r) & (Q - 1)))];
  }
}

}  // namespace iwdft
