// The twiddle tables of the in-LDS transforms, evaluated by the compiler in double precision and placed in the code
// object: constant data of the library, nothing to fill at run time and nothing a stream would have to wait for.
#include "fft_tab.h"

#include <mutex>

namespace iwdft {

namespace {

struct Entry {
  float c, t;
};

// (cos, tan) of 2 pi num / den.  A vanishing cosine is replaced by 2^-30: cos (b.x - tan b.y) then misses b.x by 2^-30 of
// its size, far below fp32 rounding.
constexpr Entry entry(long num, long den) {
  num %= den;
  const long oct = (8 * num + den / 2) / den;                  // nearest multiple of 45 degrees
  const double th = 6.28318530717958647692 * ((double)(8 * num - oct * den) / (8.0 * (double)den));  // |th| <= pi / 8
  const double t2 = th * th;
  double s = 1.0, c = 1.0;
  for (int k = 15; k >= 3; k -= 2) s = 1.0 - s * t2 / (double)(k * (k - 1));
  for (int k = 16; k >= 2; k -= 2) c = 1.0 - c * t2 / (double)(k * (k - 1));
  s *= th;
  if (oct & 1) {
    const double r = 0.70710678118654752440, c1 = (c - s) * r, s1 = (c + s) * r;
    c = c1, s = s1;
  }
  if (oct & 2) {
    const double c1 = -s;
    s = c, c = c1;
  }
  if (oct & 4) c = -c, s = -s;
  if (c < 1e-9 && c > -1e-9) c = 1.0 / (double)(1 << 30);
  return Entry{(float)c, (float)(s / c)};
}

// Residue a mod 2^bits of the samples that block i of 2^bits blocks holds: the stage at the wide end splits by the low
// bit (rem odd), everything else by base-4 digits, least significant first.
constexpr long block_residue(long i, int bits) {
  long a = 0;
  int taken = 0;
  if (bits & 1) a = (i >> (bits - 1)) & 1, taken = 1;
  for (; taken < bits; taken += 2) a |= ((i >> (bits - taken - 2)) & 3) << taken;
  return a;
}

struct alignas(16) Table {
  Entry e[tab_base(kTabMaxLogQ + 1)];
};

// The eight twiddles of a radix-16 butterfly with t = e^{2 pi j num / (16 n)}, e = e^{j pi / 4}, c = e^{j pi / 8}:
// (t^8, t^4), (t^2, t^2 e), (t, t c), (t c^2, t c^3) -- four 16-byte loads, set index fastest.
constexpr void put16(Table& T, int off, long n, long i, long num) {
  const long a[8] = {8 * num, 4 * num, 2 * num, 2 * num + 2 * n, num, num + n, num + 2 * n, num + 3 * n};
  for (int v = 0; v < 8; ++v) T.e[off + ((v >> 1) * n + i) * 2 + (v & 1)] = entry(a[v], 16 * n);
}

constexpr Table make_table() {
  Table T{};
  for (int l = kTabMinLogQ; l <= kTabMaxLogQ; ++l) {
    const int base = tab_base(l), off = base + tab_off_rem(l);
    const long Q = 1l << l;
    for (int q = 0; q < fft_np(l); ++q) {
      const long ni = tab_n_inv(l, q), nf = tab_n_fwd(q);
      for (long i = 0; ni > 1 && i < ni; ++i) put16(T, base + tab_off_inv(l, q), ni, i, block_residue(i, l - 4 * (q + 1)));
      for (long i = 0; nf > 1 && i < nf; ++i) put16(T, base + tab_off_fwd(l, q), nf, i, i);
    }
    // w = e^{2 pi j k / Q}: radix 2: w; radix 4: (w^2, w); radix 8: (w^4, w^2) and, behind all of these, (w, w e)
    if (fft_rem(l) == 1)
      for (long k = 0; k < Q / 2; ++k) T.e[off + k] = entry(k, Q);
    if (fft_rem(l) == 2)
      for (long k = 0; k < Q / 4; ++k) T.e[off + 2 * k] = entry(2 * k, Q), T.e[off + 2 * k + 1] = entry(k, Q);
    if (fft_rem(l) == 3)
      for (long k = 0; k < Q / 8; ++k) {
        T.e[off + 2 * k] = entry(4 * k, Q), T.e[off + 2 * k + 1] = entry(2 * k, Q);
        T.e[off + Q / 4 + 2 * k] = entry(k, Q), T.e[off + Q / 4 + 2 * k + 1] = entry(k + Q / 8, Q);
      }
  }
  return T;
}

constexpr Table kTable = make_table();
static __device__ Table kTwiddles = kTable;  // not const: a constant that only host code names is left out of the device code

constexpr int kMaxDevices = 64;
std::mutex g_mu;
const float2* g_ptr[kMaxDevices] = {};

}  // namespace

hipError_t fft_table(const float2** tab) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_mu);
  if (!g_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(kTwiddles));
    if (e != hipSuccess) return e;
    g_ptr[dev] = (const float2*)p;
  }
  *tab = g_ptr[dev];
  return hipSuccess;
}

}  // namespace iwdft
