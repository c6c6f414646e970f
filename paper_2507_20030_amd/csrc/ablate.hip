// The frequency-ablation tools of Sec. 3.2: the greedy per-layer mask (host integer work) and the
// device routine that removes one frequency chunk from a K or V tensor (Eq. freq-zero followed by the
// inverse DFT), which the offline study runs once per (layer, chunk).
#include <algorithm>
#include <cmath>
#include <vector>

#include "common.h"
#include "fft_core.h"
#include "fft_lds.h"
#include "pair_io.h"

namespace iwdft {

namespace {
constexpr int kAbPairs = kHeadDim / 2;
constexpr int kCusPerXcd = 32;
}  // namespace

// Two adjacent channels of a slice travel as one complex signal: forward transform, weights
// h[k] = 1 - ([k in chunk] + [M-k in chunk]) / 2 (the real part of the inverse transform of a real signal's spectrum with the
// chunk zeroed; symmetric, so both packed channels stay real), 1/M (on the spectrum: M times the samples may be out of range), inverse transform.  Block
// ids are dealt so that the workgroups of a slice share one XCD's L2.
// As in the FFT prefill a workgroup runs NS = 8192 / Q transforms side by side, interleaved over the lanes, on NP channel
// pairs one after the other: what bounded this kernel was one pair per workgroup, 4 bytes of every 128-byte line per load and
// per store.  A thread's 16 samples are 16 consecutive positions of the digit-reversed order, where the forward transform
// starts and the inverse one ends in registers, so samples cross LDS only inside the transforms; results take the place of
// the inputs in the loaded words.  Only the chunk's entries and their mirrors are weighed.  64 slices of 8192 tokens, bf16:
// 310 -> 167 us (0.27 GB read and written: 1.6 TB/s); what is left is the vector arithmetic of the two transforms.
// TWO (8192 points, fp32): two transforms by 1024 threads, see prefill_fft.hip.
template <int LOGQ, bool BF16, int NP, bool TWO = false>
__global__ __launch_bounds__(side_threads(LOGQ, TWO), 4) void ablate_kernel(const char* __restrict__ x, char* __restrict__ out,
                                                       const float2* __restrict__ tabs, int n_slices, int per_xcd, int lo,
                                                       int hi) {
  extern __shared__ __attribute__((aligned(16))) float2 smem[];
  constexpr int Q = 1 << LOGQ, T = fft_threads(LOGQ), NS = side_ns(LOGQ, TWO), BS = side_bs(LOGQ, TWO);
  static_assert(T * NS == (TWO ? 1024 : 512) && NS * NP <= kAbPairs, "");
  constexpr int kElem = BF16 ? 2 : 4;
  constexpr int kRow = kHeadDim * kElem;
  constexpr int NW = NP * (BF16 ? 1 : 2);
  constexpr int kGroups = kAbPairs / (NP * NS);  // workgroups per slice
  const TabMem tab{tabs + tab_base(LOGQ)};
  const int t = threadIdx.x / NS, g = threadIdx.x % NS;
  const uint32_t idx = blockIdx.x >> 3;
  const uint32_t slice = (blockIdx.x & 7u) * (uint32_t)per_xcd + idx / kGroups;
  if (slice >= (uint32_t)n_slices) return;  // the whole workgroup
  const int64_t base = ((int64_t)slice * Q + sample_at<LOGQ>(16 * t)) * kRow + ((idx % kGroups) * NS + g) * (NP * 2 * kElem);
  float2* buf = smem + g * BS;

  Raw<NW> z[16];
#pragma unroll
  for (int m = 0; m < 16; ++m) z[m] = load_raw<NW>(x + base + sample_step<LOGQ>(m) * kRow);
#pragma unroll 1
  for (int p = 0; p < NP; ++p) {
    float2 v[16];
#pragma unroll
    for (int m = 0; m < 16; ++m) v[m] = raw_front<BF16, NW>(z[m]);
    fft_forward<LOGQ, true>(buf, tab, t, v, [](int) {});
    for (int k = lo + t; k < hi; k += T) {  // every entry has one writer: a mirror inside the chunk is its own k
      const int km = (Q - k) & (Q - 1);
      const bool both = km >= lo && km < hi;
      float2& a = buf[fpad(k)];
      a = both ? make_float2(0.f * a.x, 0.f * a.y) : make_float2(0.5f * a.x, 0.5f * a.y);
      if (!both) {
        float2& b = buf[fpad(km)];
        b = make_float2(0.5f * b.x, 0.5f * b.y);
      }
    }
    __syncthreads();
    fft_inverse<LOGQ, true>(buf, tab.tab, t, v);
#pragma unroll
    for (int m = 0; m < 16; ++m) raw_push<BF16, NW>(z[m], v[m]);
  }
#pragma unroll
  for (int m = 0; m < 16; ++m) store_raw<NW>(out + base + sample_step<LOGQ>(m) * kRow, z[m]);
}

// M > 8192 (a power of two): the subtractive form.  Zeroing the chunk and taking the real part equals
//   x[n] - (1/M) Re sum_{k in chunk} X[k] e^{+j 2 pi k n / M},
// so only the chunk's coefficients are needed: they are formed like the FFT prefill does it (M / 8192
// decimated 8192-point transforms per channel pair, accumulated per bin in registers, at most 4096 bins at
// a time) and turned back like the FFT reconstruction does it (Hermitian halves folded modulo 8192, one
// inverse transform per residue of the token index), subtracting from the input row (first piece of the
// chunk) or from what the previous piece left in the output.
template <bool BF16>
__global__ __launch_bounds__(kFftThreads, 2) void ablate_long_kernel(const char* __restrict__ x, char* __restrict__ out,
                                                                    int n_slices, int per_xcd, uint32_t M, int lo,
                                                                    int hi) {
  extern __shared__ __attribute__((aligned(16))) float2 smem[];
  constexpr int LOGQ = kFftMaxLogQ, Q = 1 << LOGQ, H = Q / 2, IT = H / kFftThreads;
  static_assert(LOGQ & 1, "written for the odd transform length 2^13");
  constexpr int kElem = BF16 ? 2 : 4;
  constexpr int kRow = kHeadDim * kElem;
  constexpr int kPiece = kFftNBT * kFftThreads;  // bins handled at a time
  float2* buf = smem;
  float2* tab = smem + Q + (Q >> 5);
  const int tid = threadIdx.x;
  const uint32_t idx = blockIdx.x >> 3;
  const uint32_t slice = (blockIdx.x & 7u) * (uint32_t)per_xcd + idx / kAbPairs;
  if (slice >= (uint32_t)n_slices) return;
  const int64_t base = (int64_t)slice * M * kRow + (idx % kAbPairs) * 2 * kElem;
  const char* X = x + base;
  char* Y = out + base;
  const uint32_t Pb = M >> LOGQ;
  const int64_t step = (int64_t)Pb * kRow;  // bytes between consecutive samples of one residue
  const float gain = 0.5f / (float)M;

  for (int m = tid; m <= (Q >> 3); m += kFftThreads) tab[m] = cis((uint32_t)m, (uint32_t)Q);

  for (int lo_p = lo; lo_p < hi; lo_p += kPiece) {
    const int hi_p = hi < lo_p + kPiece ? hi : lo_p + kPiece;
    float2 acc0[kFftNBT], acc1[kFftNBT];
#pragma unroll
    for (int j = 0; j < kFftNBT; ++j) acc0[j] = acc1[j] = make_float2(0.f, 0.f);

    // forward: X[k] of both channels for the bins of this piece
    for (uint32_t b = 0; b < Pb; ++b) {
      int lt = tid;
      asm volatile("" : "+v"(lt));  // keeps the passes' address arithmetic out of long-lived registers
      const char* Xb = X + (int64_t)b * kRow;
#pragma unroll
      for (int g0 = 0; g0 < IT; g0 += 4) {
        float2 za[4], zc[4];
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const int a = (g0 + it) * kFftThreads + lt;
          za[it] = load_pair<BF16>(Xb + (int64_t)a * step);
          zc[it] = load_pair<BF16>(Xb + (int64_t)(a + H) * step);
        }
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const int p = digit_pos<LOGQ>((g0 + it) * kFftThreads + lt);
          buf[pad(p)] = cadd(za[it], zc[it]);
          buf[pad(p + 1)] = csub(za[it], zc[it]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      __syncthreads();
      fft_dit<LOGQ>(buf, tab, lt);
#pragma unroll
      for (int j = 0; j < kFftNBT; ++j) {
        const uint32_t k = (uint32_t)(lo_p + j * kFftThreads + tid);
        if ((int)k < hi_p) {
          const int r = k & (Q - 1), rm = (Q - r) & (Q - 1);
          const float2 w1 = buf[pad(r)], w2 = buf[pad(rm)];
          const float2 d0 = make_float2(0.5f * (w1.x + w2.x), 0.5f * (w1.y - w2.y));
          const float2 d1 = make_float2(0.5f * (w1.y + w2.y), 0.5f * (w2.x - w1.x));
          const float2 tw = conjf2(cis_poly2((k * b) & (M - 1u), M));
          acc0[j] = cadd(acc0[j], cmul(tw, d0));
          acc1[j] = cadd(acc1[j], cmul(tw, d1));
        }
      }
      __syncthreads();
    }

    // inverse: y[n] = (1/M) Re sum_k X[k] e^{+j 2 pi k n / M}, residue by residue, subtracted in place
    for (uint32_t b = 0; b < Pb; ++b) {
      int lt = tid;
      asm volatile("" : "+v"(lt));
      for (int e = tid; e < Q + (Q >> 5); e += kFftThreads) buf[e] = make_float2(0.f, 0.f);
      __syncthreads();
      // the bins of a piece are consecutive and at most Q many: distinct slots k mod Q, and distinct mirror
      // slots; a mirror slot may coincide with a direct one, so the mirrors are added in a second round
#pragma unroll
      for (int round = 0; round < 2; ++round) {
#pragma unroll
        for (int j = 0; j < kFftNBT; ++j) {
          const uint32_t k = (uint32_t)(lo_p + j * kFftThreads + tid);
          if ((int)k < hi_p) {
            const float2 tw = cis_poly2((k * b) & (M - 1u), M);
            const float2 z0 = cmul(make_float2(acc0[j].x * gain, acc0[j].y * gain), tw);
            const float2 z1 = cmul(make_float2(acc1[j].x * gain, acc1[j].y * gain), tw);
            const int r = k & (Q - 1), rm = (Q - r) & (Q - 1);
            if (round == 0) buf[pad(r)] = make_float2(z0.x - z1.y, z0.y + z1.x);                 //      z0 + j z1
            else buf[pad(rm)] = cadd(buf[pad(rm)], make_float2(z0.x + z1.y, z1.x - z0.y));       // conj z0 + j conj z1
          }
        }
        __syncthreads();
      }
      ifft_dif<LOGQ>(buf, tab, lt);
      const char* src = (lo_p == lo) ? X : (const char*)Y;  // later pieces continue from their own output
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int a = it * kFftThreads + tid;
        const int p = digit_pos<LOGQ>(a);
        const float2 u = buf[pad(p)], w = buf[pad(p + 1)];
        const int64_t o0 = ((int64_t)a * Pb + b) * kRow, o1 = ((int64_t)(a + H) * Pb + b) * kRow;
        const float2 x0 = load_pair<BF16>(src + o0), x1 = load_pair<BF16>(src + o1);
        store_pair<BF16>(Y + o0, csub(x0, cadd(u, w)));
        store_pair<BF16>(Y + o1, csub(x1, csub(u, w)));
      }
      __syncthreads();
    }
  }
}

template <bool BF16>
static hipError_t launch_ablate_t(const void* x, void* out, int n_slices, int logQ, int lo, int hi, hipStream_t st) {
  const int per_xcd = (n_slices + 7) / 8;
  // several pairs per load need 16-byte aligned tensors; not where the device would not be full (pair_io.h): the pairs spread over
  // more workgroups then, two per load at 4096 and 8192 points as long as every CU has one (8 x 8192 tokens, one / two, us: bf16
  // 44.5 / 34.2, fp32 48.3 / 38.6; 12 x 4096: 26.5 / 22.2, 26.2 / 23.8; but 48 x 2048 in fp32 27.2 / 29.5)
  const bool aligned = (((uintptr_t)x | (uintptr_t)out) & 15u) == 0;
  const bool wide = aligned && (uint64_t)n_slices * (kAbPairs / 4) >= side_pairs_min(logQ) * (uint64_t)side_ns(logQ);
  const bool two = aligned && (int64_t)per_xcd * (kAbPairs / 2) >= kCusPerXcd * side_ns(logQ);
  const bool side = logQ == 13 && !BF16 && two_transforms((int64_t)per_xcd * (kAbPairs / 4));
  const float2* tab = nullptr;
  hipError_t e = fft_table(&tab);
  if (e != hipSuccess) return e;
#define IWDFT_AB_LAUNCH(LQ, NP, TWO)                                                                            \
  {                                                                                                             \
    const size_t lds = sizeof(float2) * (size_t)(side_ns(LQ, TWO) * side_bs(LQ, TWO));                          \
    const uint64_t blocks = (uint64_t)per_xcd * (kAbPairs / ((NP) * side_ns(LQ, TWO))) * 8;                     \
    if (blocks > 0x7fffffffull) return hipErrorInvalidConfiguration;                                            \
    static LdsLimit lim;                                                                                        \
    e = lim.ensure((const void*)ablate_kernel<LQ, BF16, NP, TWO>, (int)lds);                                    \
    if (e != hipSuccess) return e;                                                                              \
    ablate_kernel<LQ, BF16, NP, TWO><<<dim3((uint32_t)blocks), dim3(side_threads(LQ, TWO)), lds, st>>>(         \
        (const char*)x, (char*)out, tab, n_slices, per_xcd, lo, hi);                                            \
  }
#define IWDFT_AB_CASE(LQ)                                                             \
  {                                                                                   \
    constexpr int kNp = side_pairs(LQ, BF16), kTwo = LQ < 12 ? 1 : 2;                 \
    if (wide && side) IWDFT_AB_LAUNCH(LQ, kNp, LQ == 13 && !BF16)                     \
    else if (wide) IWDFT_AB_LAUNCH(LQ, kNp, false)                                    \
    else if (two) IWDFT_AB_LAUNCH(LQ, kTwo, false)                                    \
    else IWDFT_AB_LAUNCH(LQ, 1, false)                                                \
  }
  switch (logQ) {
    case 8: IWDFT_AB_CASE(8) break;
    case 9: IWDFT_AB_CASE(9) break;
    case 10: IWDFT_AB_CASE(10) break;
    case 11: IWDFT_AB_CASE(11) break;
    case 12: IWDFT_AB_CASE(12) break;
    case 13: IWDFT_AB_CASE(13) break;
    default: return hipErrorInvalidValue;
  }
#undef IWDFT_AB_CASE
#undef IWDFT_AB_LAUNCH
  return hipGetLastError();
}

hipError_t launch_ablate(const void* x, void* out, int n_slices, uint32_t M, int kv_dtype, int lo, int hi,
                         hipStream_t st) {
  int logM = 0;
  while ((1u << logM) < M) ++logM;
  if (logM <= kFftMaxLogQ)
    return kv_dtype == 1 ? launch_ablate_t<true>(x, out, n_slices, logM, lo, hi, st)
                         : launch_ablate_t<false>(x, out, n_slices, logM, lo, hi, st);
  const int per_xcd = (n_slices + 7) / 8;
  const uint64_t blocks = (uint64_t)per_xcd * kAbPairs * 8;
  if (blocks > 0x7fffffffull) return hipErrorInvalidConfiguration;
  const size_t lds = sizeof(float2) * (size_t)fft_lds_float2(kFftMaxLogQ);
  static LdsLimit lim16, lim32;
  hipError_t e = kv_dtype == 1 ? lim16.ensure((const void*)ablate_long_kernel<true>, (int)lds)
                               : lim32.ensure((const void*)ablate_long_kernel<false>, (int)lds);
  if (e != hipSuccess) return e;
  if (kv_dtype == 1)
    ablate_long_kernel<true><<<dim3((uint32_t)blocks), dim3(kFftThreads), lds, st>>>((const char*)x, (char*)out, n_slices,
                                                                                   per_xcd, M, lo, hi);
  else
    ablate_long_kernel<false><<<dim3((uint32_t)blocks), dim3(kFftThreads), lds, st>>>((const char*)x, (char*)out, n_slices,
                                                                                    per_xcd, M, lo, hi);
  return hipGetLastError();
}

// chunk c of C = bins [floor(c M / C), floor((c + 1) M / C))
int64_t chunk_edge(int64_t c, int64_t M, int64_t C) { return (c * M) / C; }

int select_chunks(const float* delta, int n_chunks, double r, std::vector<int>* keep) {
  for (int c = 0; c < n_chunks; ++c)
    if (std::isnan(delta[c])) return -1;
  volatile double scaled = r * (double)n_chunks;  // volatile: the product is rounded before the add
  double n = std::floor(scaled + 0.5);
  if (n < 1.0) n = 1.0;
  if (n > (double)n_chunks) n = (double)n_chunks;
  std::vector<int> order(n_chunks);
  for (int c = 0; c < n_chunks; ++c) order[c] = c;
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return delta[a] > delta[b]; });
  keep->assign(order.begin(), order.begin() + (int)n);
  std::sort(keep->begin(), keep->end());
  return 0;
}

}  // namespace iwdft
