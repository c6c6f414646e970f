// Tables that a context holds in device memory, made there when it is created: they depend on its lengths alone, and a thousand threads take
// microseconds where one on the host takes longer than a prefill gains by them (iwdft_create at M = 8132, 2033 bins, one layer 1380 -> 97 us, with 32 layers
// 1780 -> 530).  In 64 bits, rounded at the end.  Launched on the null stream; the caller waits.
#include "tables.h"

namespace iwdft {

namespace {

constexpr double kPi = 3.14159265358979323846;
constexpr int kThreads = 256;

// Transform of the window I0(beta sqrt(1 - (2 x / taps)^2)), |x| < taps / 2, at k / N, up to a factor; W0: its value at 0.
__device__ double window_transform(const Window& w, double k) {
  const double y = kPi * w.taps * k / (double)w.N, r2 = w.beta * w.beta - y * y, r = sqrt(fabs(r2));
  return r2 > 0.0 ? sinh(r) / r : r > 0.0 ? sin(r) / r : 1.0;
}
// The window at x grid points.  I0(2 sqrt(q)) by its series: for q <= 250 (ten taps, lowest frequencies only) term 50 is below 1e-18 of the sum.
__device__ double window_at(const Window& w, double x) {
  if (fabs(x) >= 0.5 * w.taps) return 0.0;
  const double z = 1.0 - x * x * 4.0 / (double)(w.taps * w.taps), q = z > 0.0 ? 0.25 * w.beta * w.beta * z : 0.0;
  double s = 1.0;
#pragma unroll
  for (int k = 49; k >= 1; --k) s = fma(s * q, 1.0 / ((double)k * k), 1.0);
  return s / (w.taps * w.W0);
}

__global__ void chirp_kernel(float2* c, int64_t Q) {
  const int64_t n = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (n >= Q) return;
  double s, co;
  sincospi((double)((n * n) % (2 * Q)) / (double)Q, &s, &co);  // exact phase reduction
  c[n] = make_float2((float)co, (float)s);
}

// 1 / W at the samples of every thread of the transform (interp.h), [8][N / 16].
__global__ void samples_kernel(float* dec, int64_t Q, int logN, Window w) {
  const int64_t T = w.N / 16, g = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (g >= 8 * T) return;
  const int i = (int)(g / T);
  const int64_t p = 16 * (g % T);  // time index of position p (fft_core.h, sample_at)
  const int odd = logN & 1, even = logN - odd;
  int64_t n0 = 0;
  for (int b = 0; b < even; b += 2) n0 |= ((p >> b) & 3) << (even - 2 - b);
  if (odd) n0 = (n0 << 1) | (p >> (logN - 1));
  const int64_t m = n0 + (i < 4 ? i : i - 8) * (w.N / 16);
  dec[g] = (m >= 0 ? m < (Q + 1) / 2 : -m <= Q / 2) ? (float)(w.W0 / window_transform(w, (double)m)) : 0.f;
}

// Taps of points r = 0 .. P / 2 of one period P on a grid of G, [2][n][4] | [n][2] (eight taps) or [3][n][4] (ten; interp.h), n = P / 2 + 1;
// unit: a step of G in points of the window's grid.  A thread per weight; the extra one of the two outer ones is 0.
__global__ void taps_kernel(float* taps, int64_t P, int64_t G, double unit, Window w) {
  const int64_t n = P / 2 + 1, g = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int NT = w.taps;
  if (g >= n * (NT + 1)) return;
  const int64_t r = g / (NT + 1);
  const int e = (int)(g % (NT + 1));
  const int64_t first = r * G / P - (NT / 2 - 1);
  const int odd = (int)(first & 1), j = e - odd;
  const auto at = [&](int f) { return f < 8 || NT > 8 ? (f / 4 * n + r) * 4 + f % 4 : 8 * n + 2 * r + (f - 8); };
  taps[at(e)] = j >= 0 && j < NT ? (float)window_at(w, (double)(r * G - (first + j) * P) / (double)P * unit) : 0.f;
  if (e == 0) taps[at(NT > 8 ? 11 : 9)] = __int_as_float((int)(first - odd));
}

// Taps of the tokens d = 0 .. D - 1 behind a grid point, [d][i]: grid point i - (taps / 2 - 1).
template <typename F>
__global__ void token_taps_kernel(F* taps, int64_t D, Window w) {
  const int64_t g = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (g >= D * w.taps) return;
  taps[g] = (F)window_at(w, (double)(g % w.taps - (w.taps / 2 - 1)) - (double)(g / w.taps) / (double)D);
}

__global__ void gain_kernel(float* gain, Window w) {
  const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (k > w.N / 4) return;
  gain[k] = (double)k <= w.reach ? (float)(w.W0 / window_transform(w, (double)k)) : 0.f;
}

// e^{-j 2 pi k / N} and 1 / W(k / N), k = 0 .. N / 4 (0 beyond the reach), in 64 bits.
__global__ void low_kernel(double2* tw, double* gain, Window w) {
  const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (k > w.N / 4) return;
  double s, c;
  sincospi(2.0 * (double)k / (double)w.N, &s, &c);
  tw[k] = make_double2(c, -s);
  gain[k] = (double)k <= w.reach ? w.W0 / window_transform(w, (double)k) : 0.0;
}

dim3 blocks(int64_t n) { return dim3((uint32_t)((n + kThreads - 1) / kThreads)); }

}  // namespace

hipError_t make_chirp(float2* c, int64_t Q) {
  chirp_kernel<<<blocks(Q), dim3(kThreads), 0, nullptr>>>(c, Q);
  return hipGetLastError();
}
hipError_t make_samples(float* dec, int64_t Q, int logN, const Window& w) {
  samples_kernel<<<blocks(w.N / 2), dim3(kThreads), 0, nullptr>>>(dec, Q, logN, w);
  return hipGetLastError();
}
hipError_t make_taps(float* taps, int64_t P, int64_t G, double unit, const Window& w) {
  taps_kernel<<<blocks((P / 2 + 1) * (w.taps + 1)), dim3(kThreads), 0, nullptr>>>(taps, P, G, unit, w);
  return hipGetLastError();
}
hipError_t make_token_taps(float* taps, int64_t D, const Window& w) {
  token_taps_kernel<<<blocks(D * w.taps), dim3(kThreads), 0, nullptr>>>(taps, D, w);
  return hipGetLastError();
}
hipError_t make_token_taps(double* taps, int64_t D, const Window& w) {
  token_taps_kernel<<<blocks(D * w.taps), dim3(kThreads), 0, nullptr>>>(taps, D, w);
  return hipGetLastError();
}
hipError_t make_gain(float* gain, const Window& w) {
  gain_kernel<<<blocks(w.N / 4 + 1), dim3(kThreads), 0, nullptr>>>(gain, w);
  return hipGetLastError();
}
hipError_t make_low(double2* tw, double* gain, const Window& w) {
  low_kernel<<<blocks(w.N / 4 + 1), dim3(kThreads), 0, nullptr>>>(tw, gain, w);
  return hipGetLastError();
}

}  // namespace iwdft
