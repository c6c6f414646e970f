// Prefill of contexts of M = 2^m >= 16384 tokens that keep low frequencies only (|k| <= reach, k and M - k alike, in every layer):
// they do not need M points.  With a window w of kDecTaps points of a grid of N = 2^LOGN >= 4 reach points, D = M / N tokens apart,
//   y[m] = sum_n w(m - n / D) x[n]   (n modulo M)   gives   U[k] = DFT_N(y)[k] / W(k / N),  |k| <= N / 4,
// up to an aliasing error of 1.4e-9 of a tone at the worst frequency (see interp.h: the same window, the roles of time and frequency
// exchanged; with its eight taps it is 9.7e-8, which a strong tone among the frequencies that are not kept would show).
//
// All of it is in 64 bits, which gfx950 issues at the rate of unpacked fp32.  The grid concentrates what the kept bins hold: a rounding of the
// size of an offset or a strong tone is white over N points instead of M and 1 / W multiplies it, so that 32-bit sums
// and transforms of the grid showed up to 10 times the error of 32-bit transforms of the tokens (bf16 tokens with an offset, whose sums
// cancel exactly there, up to 300 times).  In 64 bits nothing is left but the rounding of the result.
#include "common.h"

namespace iwdft {

namespace {

constexpr int kDecThreads = 256, kDecRun = 64;  // grid points of a wave
constexpr int kDecTile = 16, kDecPitch = kDecTile + 1;  // grid points of a channel that leave together, a whole line; padding: distinct banks
typedef const __attribute__((address_space(4))) double* ScalarDoubles;

// A wave forms kDecRun grid points of 64 channels of one (slice, tensor), one channel a lane; token q D + d counts for the grid points
// q - 4 .. q + 5, whose sums are a window of ten registers that a loop unrolled ten times shifts by renaming.  The weights are wave-uniform
// and come through scalar loads, which the products of a token and the other waves cover.  y: [slice of the launch, tensor][channel][N].
// What bounds it is the vector ALU (82 % of the wave cycles of four waves per SIMD; ten products a token and channel, 14 % of them for the runs'
// ends) beside HBM: 4 slices of 131072 tokens, K and V, bf16: 87 us, 0.31 GB read and 0.13 written.  64 slices with the transforms: two
// channels a lane 2440 us against 2370, plain loads 2370 against 2310 with non-temporal ones, 64 bytes of a channel at a time and two steps in
// flight 2300 against 2210, twice the slices per launch, whose grids no longer fit the memory-side cache, 2580 against 2370.
template <bool BF16, int D>
__global__ __launch_bounds__(kDecThreads, 4) void decimate_kernel(Params P, const void* __restrict__ K, const void* __restrict__ V,
                                                                 int slice0, int slices) {
  constexpr int kElem = BF16 ? 2 : 4, kRow = kHeadDim * kElem;
  constexpr int kAhead = D >= 16 ? 2 : 5;  // steps of D tokens in flight; a divisor of 10
  static_assert(kDecTaps == 10 && kDecRun % kDecTile == 0, "");
  __shared__ double tiles[kDecThreads / 64][64 * kDecPitch];
  const uint32_t M = P.M, N = M / D, runs = N / kDecRun;
  const uint32_t item = __builtin_amdgcn_readfirstlane(blockIdx.x * (kDecThreads / 64) + threadIdx.x / 64);
  if (item >= runs * 4u * (uint32_t)slices) return;  // a whole wave; no barrier follows
  const int lane = threadIdx.x & 63;
  double* tile = tiles[threadIdx.x >> 6];
  const uint32_t half = item & 1u, run = (item >> 1) % runs, st = (item >> 1) / runs;  // st: (slice of the launch, tensor)
  const uint32_t m0 = run * kDecRun;
  const char* X = (const char*)((st & 1) ? V : K) + ((int64_t)(slice0 + (int)(st >> 1)) * ((int64_t)P.S + M + P.R) + P.S) * kRow +
                  (int)(half * 64u + (uint32_t)lane) * kElem;
  double* Y = P.dec_scratch + ((int64_t)st * kHeadDim + half * 64u) * N + m0;

  uint32_t raw[kAhead][D];
  auto fetch = [&](uint32_t (&z)[D], uint32_t q) {  // tokens q D .. q D + D - 1, modulo the context
    const char* p = X + (int64_t)((q & (N - 1u)) * (uint32_t)D) * kRow;
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if constexpr (BF16) z[d] = __builtin_nontemporal_load((const uint16_t*)(p + d * kRow));
      else z[d] = __builtin_nontemporal_load((const uint32_t*)(p + d * kRow));
    }
  };
  double acc[kDecTaps];
#pragma unroll
  for (int i = 0; i < kDecTaps; ++i) acc[i] = 0.0;
  const uint32_t q0 = m0 - 5u;  // first step that reaches grid point m0
#pragma unroll
  for (int a = 0; a < kAhead; ++a) fetch(raw[a], q0 + (uint32_t)a);
  // The next token's weights, behind the products of the token before: the scalar registers hold two tokens'.
  auto load_weights = [&](double (&w)[kDecTaps], int d) {
    uint64_t p = (uint64_t)(uintptr_t)(P.dec_weights + d * kDecTaps);
    asm volatile(""
                 : "+s"(p), "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]), "+v"(acc[4]), "+v"(acc[5]), "+v"(acc[6]), "+v"(acc[7]),
                   "+v"(acc[8]), "+v"(acc[9]));
#pragma unroll
    for (int i = 0; i < kDecTaps; ++i) w[i] = ((ScalarDoubles)p)[i];
  };
  double w[kDecTaps];
  load_weights(w, 0);
  constexpr int kSteps = kDecRun + kDecTaps - 1;
#pragma unroll 1
  for (int s0 = 0; s0 < kSteps; s0 += 10) {
#pragma unroll
    for (int u = 0; u < 10; ++u) {
      const int s = s0 + u;
      if (s >= kSteps) break;  // uniform
      uint32_t (&z)[D] = raw[u % kAhead];
#pragma unroll
      for (int d = 0; d < D; ++d) {
        double wn[kDecTaps];
        load_weights(wn, (d + 1) % D);
        const double x = (double)__uint_as_float(BF16 ? z[d] << 16 : z[d]);
#pragma unroll
        for (int i = 0; i < kDecTaps; ++i) acc[(u + i) % 10] = fma(w[i], x, acc[(u + i) % 10]);
#pragma unroll
        for (int i = 0; i < kDecTaps; ++i) w[i] = wn[i];
      }
      if (s + kAhead < kSteps) fetch(z, q0 + (uint32_t)(s + kAhead));
      // grid point q - 4 = m0 + s - 9 is complete
      const int o = s - (kDecTaps - 1);
      if (o >= 0) tile[lane * kDecPitch + (o & (kDecTile - 1))] = acc[u];
      acc[u] = 0.0;
      if (o >= 0 && (o & (kDecTile - 1)) == kDecTile - 1) {
        constexpr int kLanes = kDecTile / 2;
        const int c0 = lane / kLanes, m = (lane & (kLanes - 1)) * 2;
        double* y = Y + (int64_t)c0 * N + (o - (kDecTile - 1)) + m;
#pragma unroll
        for (int c = 0; c < 64; c += 64 / kLanes) {
          const double* t = tile + (c0 + c) * kDecPitch + m;
          *(double2*)(y + (int64_t)c * N) = make_double2(t[0], t[1]);
        }
      }
    }
  }
}

// ------------------------------------------------------------------------------------------ transforms
__device__ __forceinline__ double2 add(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 sub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 mul(double2 a, double2 b) { return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }
__device__ __forceinline__ double2 mul_mj(double2 a) { return make_double2(a.y, -a.x); }  // -j a

__device__ __forceinline__ void dft4(double2& a, double2& b, double2& c, double2& d) {
  const double2 s = add(a, c), t = sub(a, c), u = add(b, d), v = mul_mj(sub(b, d));
  a = add(s, u), b = add(t, v), c = sub(s, u), d = sub(t, v);
}
// In place, entry k of the transform at x[4 (k % 4) + k / 4] (swap16).
__device__ __forceinline__ void dft16(double2 (&x)[16]) {
  constexpr double c1 = 0.92387953251128675613, s1 = 0.38268343236508977173, h = 0.70710678118654752440;
#pragma unroll
  for (int n = 0; n < 4; ++n) dft4(x[n], x[n + 4], x[n + 8], x[n + 12]);  // x[n + 4 k]: entry k of the samples n, n + 4, ...
  x[5] = mul(x[5], make_double2(c1, -s1));
  x[6] = make_double2((x[6].x + x[6].y) * h, (x[6].y - x[6].x) * h);
  x[7] = mul(x[7], make_double2(s1, -c1));
  x[9] = make_double2((x[9].x + x[9].y) * h, (x[9].y - x[9].x) * h);
  x[10] = mul_mj(x[10]);
  x[11] = make_double2((x[11].y - x[11].x) * h, -(x[11].x + x[11].y) * h);
  x[13] = mul(x[13], make_double2(s1, -c1));
  x[14] = make_double2((x[14].y - x[14].x) * h, -(x[14].x + x[14].y) * h);
  x[15] = mul(x[15], make_double2(-c1, s1));
#pragma unroll
  for (int k = 0; k < 4; ++k) dft4(x[4 * k], x[4 * k + 1], x[4 * k + 2], x[4 * k + 3]);
}
__device__ constexpr int swap16(int k) { return 4 * (k & 3) + (k >> 2); }
// The even and the odd entries of an eight-point transform of x[0], x[S], ..., x[7 S] in place, entry k at x[S swap8(k)].
template <int S>
__device__ __forceinline__ void dft8(double2* x) {
  constexpr double h = 0.70710678118654752440;
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    const double2 a = x[n * S], b = x[(n + 4) * S];
    x[n * S] = add(a, b), x[(n + 4) * S] = sub(a, b);
  }
  double2 &p = x[5 * S], &q = x[6 * S], &r = x[7 * S];
  p = make_double2((p.x + p.y) * h, (p.y - p.x) * h);
  q = mul_mj(q);
  r = make_double2((r.y - r.x) * h, -(r.x + r.y) * h);
  dft4(x[0], x[S], x[2 * S], x[3 * S]);
  dft4(x[4 * S], x[5 * S], x[6 * S], x[7 * S]);
}
__device__ constexpr int swap8(int k) { return (k >> 1) + 4 * (k & 1); }

__device__ __forceinline__ int lpad(int i) { return i + (i >> 4); }  // 16-byte entries; consecutive threads' stores fall into distinct banks

// One channel's grid: its N real points are C = N / 2 complex ones z[n] = y[2 n] + j y[2 n + 1], transformed in LDS (Stockham, radix 16; a
// pass of radix 8 ahead for C = 2048, the last radix-2 stage of C = 8192 at the kept bins only) and taken apart at the kept bins,
//   2 Y[k] = Z[k] + conj Z[-k] - j e^{-j 2 pi k / N} (Z[k] - conj Z[-k]).
// A persistent workgroup of C / 16 threads walks the (slice, tensor, channel) rows; the next row is fetched under the current one.
// Twiddles are the powers of one table entry a pass.  What bounds it: waits (three quarters of the wave cycles) of the one workgroup that the LDS of
// a CU holds; vector ALU 18 us, LDS 12 and memory 28 of 51 us for 1024 rows of 16384 points.
// 8 x 8 slices of 131072 tokens, 4096 bins, bf16, with the decimation: 4170 us (sixteen 8192-point transforms per channel pair) -> 2210.
constexpr int low_threads(int logN) { return 1 << (logN - 5); }
constexpr int low_lds(int logN) { return ((1 << (logN - 1)) + (1 << (logN - 5))) * (int)sizeof(double2); }
template <int LOGN>
__global__ __launch_bounds__(low_threads(LOGN), 2) void prefill_low_kernel(Params P, int slice0, int rows) {
  constexpr int N = 1 << LOGN, C = N / 2, T = low_threads(LOGN), LOGC = LOGN - 1;
  constexpr int R0 = LOGC % 4 == 3 ? 8 : 16;  // radix of the first pass
  constexpr bool kLast2 = LOGC % 4 == 1;      // a last radix-2 stage, formed at the kept bins
  static_assert(LOGN >= 12 && LOGN <= 14, "");
  extern __shared__ __attribute__((aligned(16))) double2 lds[];
  const int t = threadIdx.x;
  const double2* __restrict__ tw = P.dec_tw;  // e^{-j 2 pi m / N}, m <= N / 4
  const int spl = P.batch * P.n_kv;
  double2 x[16], nx[16];
  auto fetch = [&](int row) {
    const double2* z = (const double2*)(P.dec_scratch + (int64_t)row * N) + t;
#pragma unroll
    for (int i = 0; i < 16; ++i) nx[i] = z[i * T];
  };
  int row = blockIdx.x;
  if (row >= rows) return;  // the whole workgroup
  fetch(row);
#pragma unroll 1
  for (;;) {
#pragma unroll
    for (int i = 0; i < 16; ++i) x[i] = nx[i];
    const int next = row + (int)gridDim.x;
    if (next < rows) fetch(next);
    __syncthreads();  // the bins of the row before have been read
    if constexpr (R0 == 16) {
      dft16(x);
#pragma unroll
      for (int k = 0; k < 16; ++k) lds[lpad(16 * t + k)] = x[swap16(k)];
    } else {  // two transforms of eight points a thread: samples t + T (i + 2 r)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        dft8<2>(x + i);
#pragma unroll
        for (int k = 0; k < 8; ++k) lds[lpad(8 * (t + T * i) + k)] = x[i + 2 * swap8(k)];
      }
    }
#pragma unroll
    for (int ns = R0; ns * 16 <= C; ns *= 16) {
      const int j = t & (ns - 1);
      const double2 w1 = tw[j * (N / (16 * ns))];
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 16; ++i) x[i] = lds[lpad(t + i * T)];
      double2 w[16];
      w[1] = w1;
#pragma unroll
      for (int i = 2; i < 16; ++i) w[i] = mul(w[i / 2], w[i - i / 2]);
#pragma unroll
      for (int i = 1; i < 16; ++i) x[i] = mul(x[i], w[i]);
      dft16(x);
      __syncthreads();
      const int base = (t - j) * 16 + j;
#pragma unroll
      for (int k = 0; k < 16; ++k) lds[lpad(base + k * ns)] = x[swap16(k)];
    }
    __syncthreads();
    const int channel = row & (kHeadDim - 1), st = row >> 7, slice = slice0 + (st >> 1), layer = slice / spl;
    const LayerInfo L = layer_info(P, layer);
    const int32_t* __restrict__ bins = P.bins + L.bin_off;
    float2* F = ((st & 1) ? P.FV : P.FK) + L.coef_off + ((int64_t)(slice - layer * spl) * kHeadDim + channel) * L.Bp;
    constexpr int U = 4;
    for (int i0 = t; i0 < L.nb; i0 += U * T) {
      uint32_t k[U];
      double2 wk[U];
      double g[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + u * T;
        k[u] = (uint32_t)bins[i < L.nb ? i : L.nb - 1];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t f = 2u * k[u] <= P.M ? k[u] : P.M - k[u];  // <= N / 4
        wk[u] = tw[f];
        g[u] = P.dec_gain[f];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + u * T;
        if (i >= L.nb) continue;
        const bool up = 2u * k[u] > P.M;  // the conjugate of its mirror
        const int f = (int)(up ? P.M - k[u] : k[u]);
        double2 a, b;  // Z[f], Z[-f]
        if constexpr (kLast2) {
          constexpr int H = C / 2;
          const int r = f & (H - 1), rm = (H - r) & (H - 1);
          const double2 w2 = mul(wk[u], wk[u]);  // e^{-j 2 pi f / C}
          a = add(lds[lpad(r)], mul(w2, lds[lpad(r + H)]));
          b = add(lds[lpad(rm)], mul(make_double2(w2.x, -w2.y), lds[lpad(rm + H)]));
        } else {
          a = lds[lpad(f)];
          b = lds[lpad((C - f) & (C - 1))];
        }
        const double2 e = make_double2(a.x + b.x, a.y - b.y), o = mul(wk[u], make_double2(a.y + b.y, b.x - a.x));
        const double h = 0.5 * g[u];
        const float re = (float)(h * (e.x + o.x)), im = (float)(h * (e.y + o.y));
        F[i] = make_float2(re, up ? -im : im);
      }
    }
    if (next >= rows) break;
    row = next;
  }
}

template <int LOGN>
hipError_t launch_transforms(const Params& P, int slice0, int slices, hipStream_t st) {
  constexpr int bytes = low_lds(LOGN), kSlots = 256 << (14 - LOGN);  // workgroups that the device holds at once
  const int rows = slices * 2 * kHeadDim;
  static LdsLimit lim;
  const hipError_t e = lim.ensure((const void*)prefill_low_kernel<LOGN>, bytes);
  if (e != hipSuccess) return e;
  prefill_low_kernel<LOGN><<<dim3((uint32_t)(rows < kSlots ? rows : kSlots)), dim3(low_threads(LOGN)), bytes, st>>>(P, slice0, rows);
  return hipGetLastError();
}

template <bool BF16>
hipError_t launch_decimate(const Params& P, const void* K, const void* V, int slice0, int slices, hipStream_t st) {
  const uint32_t N = 1u << P.dec_logN, waves = N / kDecRun * 4 * (uint32_t)slices;
  const dim3 grid((waves + kDecThreads / 64 - 1) / (kDecThreads / 64)), block(kDecThreads);
  switch (P.M >> P.dec_logN) {
    case 4: decimate_kernel<BF16, 4><<<grid, block, 0, st>>>(P, K, V, slice0, slices); break;
    case 8: decimate_kernel<BF16, 8><<<grid, block, 0, st>>>(P, K, V, slice0, slices); break;
    case 16: decimate_kernel<BF16, 16><<<grid, block, 0, st>>>(P, K, V, slice0, slices); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_prefill_low(const Params& P, const void* K, const void* V, hipStream_t st) {
  for (int s0 = 0; s0 < P.n_slices; s0 += P.dec_slices) {
    const int n = P.n_slices - s0 < P.dec_slices ? P.n_slices - s0 : P.dec_slices;
    hipError_t e = P.kv_dtype == 1 ? launch_decimate<true>(P, K, V, s0, n, st) : launch_decimate<false>(P, K, V, s0, n, st);
    if (e != hipSuccess) return e;
    switch (P.dec_logN) {
      case 12: e = launch_transforms<12>(P, s0, n, st); break;
      case 13: e = launch_transforms<13>(P, s0, n, st); break;
      case 14: e = launch_transforms<14>(P, s0, n, st); break;
      default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace iwdft
