// Layout of the twiddle tables of the in-LDS transforms (fft_core.h): one block per length 2^LOGQ, each entry a twiddle
// w = e^{+j phi} as the pair (cos phi, tan phi) that a multiply-add butterfly consumes.  The array itself lives in
// fft_tab.hip; kernels get its address as an argument.
#pragma once
#include <hip/hip_runtime.h>

namespace iwdft {

constexpr int kTabMinLogQ = 8, kTabMaxLogQ = 14;

// Stage plan of 2^LOGQ points: one stage of radix 2^rem at the wide end (rem = LOGQ mod 4; none for 0), then np radix-16
// passes of span 16^(np - 1), ..., 16, 1 (the inverse transform runs them in this order, the forward one backwards).
constexpr int fft_np(int logQ) { return logQ / 4; }
constexpr int fft_rem(int logQ) { return logQ % 4; }

// Distinct twiddle sets of a radix-16 pass of span 16^q: the inverse transform's depend on the block a butterfly belongs
// to, the forward one's on the position inside a block.  A single set is constant and has no table.
constexpr int tab_n_inv(int logQ, int q) { return 1 << (logQ - 4 * (q + 1)); }
constexpr int tab_n_fwd(int q) { return 1 << (4 * q); }
constexpr int tab_sz16(int n) { return n > 1 ? 8 * n : 0; }

// Offsets in float2 from the start of a length's block: inverse passes (narrow span first) | forward passes | forward
// stage of radix 2^rem (the inverse one has constant twiddles), all entries in natural order.
constexpr int tab_off_inv(int logQ, int q) {
  int o = 0;
  for (int i = 0; i < q; ++i) o += tab_sz16(tab_n_inv(logQ, i));
  return o;
}
constexpr int tab_off_fwd(int logQ, int q) {
  int o = tab_off_inv(logQ, fft_np(logQ));
  for (int i = 0; i < q; ++i) o += tab_sz16(tab_n_fwd(i));
  return o;
}
constexpr int tab_off_rem(int logQ) { return tab_off_fwd(logQ, fft_np(logQ)); }
constexpr int tab_size(int logQ) { return tab_off_rem(logQ) + (fft_rem(logQ) ? 1 << (logQ - 1) : 0); }
constexpr int tab_base(int logQ) {
  int o = 0;
  for (int l = kTabMinLogQ; l < logQ; ++l) o += tab_size(l);
  return o;
}

// Device address of the tables on the current device (looked up once per device); the block of length 2^LOGQ starts at
// tab_base(LOGQ).
hipError_t fft_table(const float2** tab);

}  // namespace iwdft
