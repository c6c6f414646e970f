// Prefill transform (Sec. 3.1.2 Eq. dft-full at the kept bins, Sec. 4.2.1 Eq. prefill-dft) for DFT lengths that are not a
// power of two, e.g. M = context - sink - recent: U_M[k] = sum_n x[n] e^{-j 2 pi k n / M} interpolated from the transform of a
// power-of-two grid (interp.h), O(M log M) per channel where the dense contraction costs O(M |B|).
//
// Two channels of a slice travel as real and imaginary part of one signal and are separated at the kept bins, as in the
// power-of-two prefill; the second one is scaled to the first one's size on the way (scale_pairs).
// M > 8192 runs in Pb decimated blocks of up to A = ceil(M / Pb) samples, n = Pb a + b, centred at c = floor(A / 2):
//   U[k] = sum_b e^{-j 2 pi k (Pb c + b) / M} sum_a x[Pb a + b] e^{-j 2 pi (k Pb / M) (a - c)},
// where Pb need not divide M: the inner sum is wanted at the frequencies k Pb / M, wherever they lie on the grid.  Where Pb divides M, a is
// taken modulo A about 0 (c = 0).
// The running sums live in the output rows (every bin belongs to one thread, which reads back its own earlier store).  There the taps are
// ten: what an offset or a low tone leaves on its neighbours (1.6e-7 of it with eight taps, N / Q = 2) is the same in every block
// and adds up, where roundings of different samples do not (noise beside an offset of 30, error of the bins 1 .. 63 in units of it and of
// the noise: 3 blocks of 8191 1.6e-6 -> 5.4e-7, 64 blocks 7.1e-6 -> 2.2e-6).
#include "interp.h"
#include "pair_io.h"

namespace iwdft {

// A workgroup of N / 16 threads walks the (slice, tensor, NP channel pairs) items of its XCD; token rows are fetched 4 NP
// (bf16) or 8 NP (fp32) bytes at a time, the next item's while the last pair of the current one is transformed.
// What bounds it: vector ALU and LDS, each busy 52 % of the time with one workgroup of 16384 points per CU (936 vector and 110
// LDS instructions per wave and pair).  The pairs are unrolled (a rolled loop moves their words: 1.62 ms against 1.56), the
// maxima of all pairs are reduced at once (one by one: 1.66), the next pair's 1 / W is fetched while the bins are read.
// 32 x 8 slices, M = 8132, 2033 bins, bf16: 2.30 ms (two chirp-z transforms of the same length) -> 1.56 ms, dense contraction
// 7.43; relative error 2.3e-7 -> 1.5e-7, dense 8.5e-7.
// ODD: blocks that do not divide M.
template <int LOGN, bool BF16, int NP, int NT, bool ODD>
__global__ __launch_bounds__(fft_threads(LOGN), 4) void prefill_any_kernel(Params P, const void* __restrict__ K,
                                                                       const void* __restrict__ V, int per_xcd,
                                                                       int n_st, int slots) {
  constexpr int T = fft_threads(LOGN), NWV = T < 64 ? 1 : T / 64;
  constexpr int kElem = BF16 ? 2 : 4;
  constexpr int kRow = kHeadDim * kElem;  // bytes per token row
  constexpr int NW = NP * (BF16 ? 1 : 2);
  constexpr int kGroups = kHeadDim / 2 / NP;
  extern __shared__ __attribute__((aligned(16))) float2 buf[];
  __shared__ uint32_t maxima[NWV][1][NW];
  const TabMem tab{P.tab + tab_base(LOGN)};
  const int t = threadIdx.x;
  const uint32_t xcd = blockIdx.x & 7u;
  const int st_first = (int)xcd * per_xcd, st_count = min(per_xcd, n_st - st_first);
  const int n_items = st_count * kGroups;
  int n = (int)(blockIdx.x >> 3);
  if (n >= n_items) return;  // the whole workgroup
  const uint32_t M = P.M, Q = P.pf_period, A = ODD ? P.pf_A : Q, Pb = ODD ? P.pf_Pb : M / Q;
  const float inv_Mf = 1.0f / (float)M, inv_Q = 1.0f / (float)Q;
  const int spl = P.batch * P.n_kv;
  const int64_t N = (int64_t)P.S + M + P.R;  // tokens per slice in the caller's tensor
  const int64_t step = (int64_t)Pb * kRow;   // bytes between consecutive samples of one block

  Raw<NW> z[8];
  auto fetch = [&](int item, uint32_t b) {
    const int st = st_first + item / kGroups;
    const char* X = (const char*)((st & 1) ? V : K) + ((int64_t)(st >> 1) * N + P.S + b) * kRow +
                    (item % kGroups) * (NP * 2 * kElem);
    const uint32_t n0 = sample_at<LOGN>(16u * (uint32_t)pin_index(t));
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      uint32_t a = wing_index<LOGN>(n0, i, A);
      if constexpr (ODD) {  // that index is modulo A
        if (a < A) a = a < ((A + 1) >> 1) ? a + (A >> 1) : a - ((A + 1) >> 1);
        if (a < A && a * Pb + b >= M) a = A;
      }
      if (a < A) z[i] = load_raw<NW>(X + (int64_t)a * step);
      else z[i] = Raw<NW>{};
    }
  };
  // 1 / W at the thread's samples, 0 where there is none
  float dec[8];
  auto fetch_dec = [&] {
    const float* __restrict__ d = P.any_dec + pin_index(t);
#pragma unroll
    for (int i = 0; i < 8; ++i) dec[i] = d[i * T];
  };
  fetch(n, 0);
  fetch_dec();
  uint32_t b = 0;
#pragma unroll 1
  for (;;) {
    const int st = st_first + n / kGroups, slice = st >> 1;
    const int layer = slice / spl, s = slice - layer * spl;
    const LayerInfo L = layer_info(P, layer);
    const int32_t* bins = P.bins + L.bin_off;
    float2* F = ((st & 1) ? P.FV : P.FK) + L.coef_off + ((int64_t)s * kHeadDim + (n % kGroups) * (NP * 2)) * L.Bp;
    const bool last_b = b + 1 == Pb;
    const int n1 = last_b ? n + slots : n;
    const uint32_t b1 = last_b ? 0u : b + 1;
    const bool more = n1 < n_items;
    const uint32_t k_max = (uint32_t)bins[L.nb - 1];  // ascending
    const int reach = !ODD && Pb == 1 && 2 * k_max < Q ? (int)((k_max << LOGN) / Q) + kTaps + 1 : 1 << LOGN;
    PairScale sc[NP];
    scale_pairs<BF16>(z, t, maxima, sc);
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      float2 x[16];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float2 v = raw_front<BF16, NW>(z[i]);
        raw_pop<BF16, NW>(z[i]);
        x[wing_position(i)] = make_float2(v.x * dec[i], v.y * (dec[i] * sc[p].up));
      }
      if (p == NP - 1 && more) fetch(n1, b1);
      const float h0 = sc[p].h0, h1 = sc[p].h1;
      // kept bins of this thread, two at a time; the first two are fetched while the transform runs
      constexpr int U = 2;
      uint32_t k[U];
      auto fetch_bins = [&](int i0) {
#pragma unroll
        for (int j = 0; j < U; ++j) {
          const int i = i0 + j * T;
          k[j] = (uint32_t)bins[i < L.nb ? i : L.nb - 1];
        }
      };
      fetch_bins(pin_index(t));
      grid_forward<LOGN>(buf, tab, t, x, reach);
      fetch_dec();
      float2* F0 = F + (int64_t)(2 * p) * L.Bp;
      for (int i0 = t; i0 < L.nb; i0 += U * T) {
        if (i0 >= U * T) fetch_bins(i0);
        Taps<NT> taps[U];
        bool up[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
          const uint32_t r = ODD ? mod_small(k[j] * P.pf_step, Q, inv_Q) : Pb == 1 ? k[j] : mod_small(k[j], Q, inv_Q);
          up[j] = 2u * r > Q;  // upper half: the taps of the mirror
          taps[j] = load_taps<NT>(P.any_taps, up[j] ? Q - r : r, Q);
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
          const int i = i0 + j * T;
          if (i >= L.nb) continue;
          float2 wl, wh;
          grid_at<false, NT>(buf, 1 << LOGN, taps[j], wl, wh);
          const float2 w1 = up[j] ? wh : wl, w2 = up[j] ? wl : wh;
          float2 d0 = make_float2(h0 * (w1.x + w2.x), h0 * (w1.y - w2.y));
          float2 d1 = make_float2(h1 * (w1.y + w2.y), h1 * (w2.x - w1.x));
          if (ODD || Pb > 1) {
            uint32_t ph;  // k (Pb c + b) mod M
            if constexpr (!ODD) {
              ph = mod_small(k[j] * b, M, inv_Mf);
            } else {  // M <= kAnyMaxPeriod * Pb: the product needs 64 bits, the quotient is off by one at most
              const uint64_t u = (uint64_t)k[j] * (Pb * (A >> 1) + b);
              int32_t q = (int32_t)(uint32_t)(u - (uint64_t)((double)u * (1.0 / (double)M)) * M);
              if (q < 0) q += (int32_t)M;
              if (q >= (int32_t)M) q -= (int32_t)M;
              ph = (uint32_t)q;
            }
            const float2 tw = conjf2(cis_poly_x((float)ph / (float)M));
            d0 = cmul(tw, d0);
            d1 = cmul(tw, d1);
            if (b) {
              d0 = cadd(F0[i], d0);
              d1 = cadd(F0[L.Bp + i], d1);
            }
          }
          F0[i] = d0;
          F0[L.Bp + i] = d1;
        }
      }
      __syncthreads();  // the next transform overwrites buf
    }
    if (!more) break;
    n = n1;
    b = b1;
  }
}

constexpr int kCusPerXcd = 32;

template <bool BF16, int NT, bool ODD>
static hipError_t launch_prefill_any_t(const Params& P, const void* K, const void* V, hipStream_t st) {
  const int n_st = P.n_slices * 2;
  const int per_xcd = (n_st + 7) / 8;
  constexpr int kNp = BF16 ? 4 : 2;
  const int logN = P.pf_logN;
  const int max_slots = kCusPerXcd << (kTabMaxLogQ - logN);  // workgroups that an XCD holds at once
  // one pair per item where the device would not be full with several, and on grids of 1024 points
  const bool few = logN == 10 || (int64_t)per_xcd * (kHeadDim / 2 / kNp) < max_slots;
#define IWDFT_PA_LAUNCH(LN, NP)                                                                                  \
  {                                                                                                              \
    constexpr int bytes = (int)sizeof(float2) * grid_lds(LN);                                                     \
    const int64_t items = (int64_t)per_xcd * (kHeadDim / 2 / (NP));                                              \
    const int slots = items < max_slots ? (int)items : max_slots;                                                \
    static LdsLimit lim;                                                                                         \
    const hipError_t e = lim.ensure((const void*)prefill_any_kernel<LN, BF16, NP, NT, ODD>, bytes);                 \
    if (e != hipSuccess) return e;                                                                               \
    prefill_any_kernel<LN, BF16, NP, NT, ODD><<<dim3((uint32_t)slots * 8), dim3(fft_threads(LN)), bytes, st>>>(     \
        P, K, V, per_xcd, n_st, slots);                                                                          \
  }
#define IWDFT_PA_CASE(LN)                             \
  case LN:                                            \
    if (few) IWDFT_PA_LAUNCH(LN, 1)                   \
    else IWDFT_PA_LAUNCH(LN, kNp)                     \
    break;
  switch (logN) {
    case 10: IWDFT_PA_LAUNCH(10, 1) break;
    IWDFT_PA_CASE(11)
    IWDFT_PA_CASE(12)
    IWDFT_PA_CASE(13)
    IWDFT_PA_CASE(14)
    default: return hipErrorInvalidValue;
  }
#undef IWDFT_PA_CASE
#undef IWDFT_PA_LAUNCH
  return hipGetLastError();
}

hipError_t launch_prefill_any(const Params& P, const void* K, const void* V, hipStream_t st) {
  if (!P.any_dec) return hipErrorInvalidValue;
  const hipError_t e = launch_prefill_edges(P, K, V, st);
  if (e != hipSuccess) return e;
  const bool b16 = P.kv_dtype == 1;
  if (P.pf_Pb == 1) return b16 ? launch_prefill_any_t<true, kTaps, false>(P, K, V, st) : launch_prefill_any_t<false, kTaps, false>(P, K, V, st);
  if (P.M % P.pf_Pb == 0)
    return b16 ? launch_prefill_any_t<true, kSumTaps, false>(P, K, V, st) : launch_prefill_any_t<false, kSumTaps, false>(P, K, V, st);
  return b16 ? launch_prefill_any_t<true, kSumTaps, true>(P, K, V, st) : launch_prefill_any_t<false, kSumTaps, true>(P, K, V, st);
}

}  // namespace iwdft
