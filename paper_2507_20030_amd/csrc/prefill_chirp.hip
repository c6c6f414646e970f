// Prefill transform (Sec. 3.1.2 Eq. dft-full at the kept bins, Sec. 4.2.1 Eq. prefill-dft) for DFT lengths that are not a
// power of two, e.g. M = context - sink - recent: U_M[k] = sum_n x[n] e^{-j 2 pi k n / M} through chirp-z transforms
// (chirp.h), O(M log M) per channel where the dense contraction costs O(M |B|).
//
// Two channels of a slice travel as real and imaginary part of one signal and are separated at the kept bins, as in the
// power-of-two prefill; the second one is scaled to the first one's size on the way (pair_scale).
// M > 8192 runs in Pb = M / Q decimated blocks (chirp.h's Q): U[k] = sum_b e^{-j 2 pi k b / M} DFT_Q(x[Pb a + b])[k mod Q],
// the running sums live in the output rows (every bin belongs to one thread, which reads back its own earlier store).
#include "chirp.h"
#include "pair_io.h"

namespace iwdft {

// A workgroup of N / 16 threads walks the (slice, tensor, NP channel pairs) items of its XCD; token rows are fetched 4 NP
// (bf16) or 8 NP (fp32) bytes at a time, the next item's while the last pair of the current one is transformed.
// What bounds it is the vector arithmetic and the barriers of two N-point transforms per pair (240 points of convolution per
// ns over the chip, whatever N).  32 x 8 slices, M = 8132, 2033 bins, bf16: 7.43 ms (dense contraction) -> 2.30 ms, relative
// error 8.5e-7 -> 2.3e-7.
template <int LOGN, bool BF16, int NP>
__global__ __launch_bounds__(fft_threads(LOGN), 4) void prefill_chirp_kernel(Params P, const void* __restrict__ K,
                                                                         const void* __restrict__ V, int per_xcd,
                                                                         int n_st, int slots) {
  constexpr int T = fft_threads(LOGN), NWV = T < 64 ? 1 : T / 64;
  constexpr int SP = T + T / 8;  // distance in LDS of entries T apart
  constexpr int kElem = BF16 ? 2 : 4;
  constexpr int kRow = kHeadDim * kElem;  // bytes per token row
  constexpr int NW = NP * (BF16 ? 1 : 2);
  constexpr int kGroups = kHeadDim / 2 / NP;
  extern __shared__ __attribute__((aligned(16))) float2 buf[];
  __shared__ uint2 smax[NWV];
  const TabMem tab{P.tab + tab_base(LOGN)};
  const float4* __restrict__ H = P.chirpW;
  const int t = threadIdx.x;
  const uint32_t xcd = blockIdx.x & 7u;
  const int st_first = (int)xcd * per_xcd, st_count = min(per_xcd, n_st - st_first);
  const int n_items = st_count * kGroups;
  int n = (int)(blockIdx.x >> 3);
  if (n >= n_items) return;  // the whole workgroup
  const uint32_t M = P.M, Q = P.chirp_Q, Pb = M / Q;
  const float inv_Mf = 1.0f / (float)M, inv_Q = 1.0f / (float)Q;
  const int spl = P.batch * P.n_kv;
  const int64_t N = (int64_t)P.S + M + P.R;  // tokens per slice in the caller's tensor
  const int64_t step = (int64_t)Pb * kRow;   // bytes between consecutive samples of one block
  float2* own = buf + fpad(t);               // this thread's entries t + T i at i * SP

  Raw<NW> z[8];
  auto fetch = [&](int item, uint32_t b) {
    const int st = st_first + item / kGroups;
    const char* X = (const char*)((st & 1) ? V : K) + ((int64_t)(st >> 1) * N + P.S + b) * kRow +
                    (item % kGroups) * (NP * 2 * kElem);
    const int o = pin_index(t);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t a = (uint32_t)(o + T * i);
      if (a < Q) z[i] = load_raw<NW>(X + (int64_t)a * step);
      else z[i] = Raw<NW>{};
    }
  };
  auto max2 = [](uint2 a, uint2 b) { return make_uint2(max(a.x, b.x), max(a.y, b.y)); };

  fetch(n, 0);
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
#pragma unroll 1
    for (int p = 0; p < NP; ++p) {
      float2 v[8];
      uint2 m = make_uint2(0u, 0u);  // largest magnitude of either channel, as bits: infinities and NaN come out on top
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        v[i] = raw_front<BF16, NW>(z[i]);
        raw_pop<BF16, NW>(z[i]);
        m = max2(m, make_uint2(__float_as_uint(v[i].x) & 0x7fffffffu, __float_as_uint(v[i].y) & 0x7fffffffu));
      }
      if (p == NP - 1 && more) fetch(n1, b1);
#pragma unroll
      for (int o = (T < 64 ? T : 64) / 2; o >= 1; o >>= 1) m = max2(m, make_uint2(__shfl_xor(m.x, o), __shfl_xor(m.y, o)));
      if (NWV > 1) {
        if ((t & 63) == 0) smax[t >> 6] = m;
        __syncthreads();
        m = smax[0];
#pragma unroll
        for (int w = 1; w < NWV; ++w) m = max2(m, smax[w]);
      }
      const PairScale sc = pair_scale(m.x, m.y);
      const bool bad0 = not_finite(m.x), bad1 = not_finite(m.y);
      const float h0 = sc.h0, h1 = sc.h1;
      const int o = pin_index(t);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uint32_t a = (uint32_t)(o + T * i);
        const float2 c = a < Q ? P.chirp[a] : make_float2(0.f, 0.f);
        v[i] = cmul(make_float2(bad0 ? 0.f : v[i].x, bad1 ? 0.f : v[i].y * sc.up), conjf2(c));
      }
      chirp_convolve<LOGN, true>(buf, tab, H, t, v);
      const int o2 = pin_index(t);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uint32_t a = (uint32_t)(o2 + T * i);
        const float2 c = a < Q ? P.chirp[a] : make_float2(0.f, 0.f);
        own[i * SP] = cmul(v[i], conjf2(c));
      }
      __syncthreads();
      float2* F0 = F + (int64_t)(2 * p) * L.Bp;
      constexpr int U = 4;
      for (int i0 = t; i0 < L.nb; i0 += U * T) {
        uint32_t k[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
          const int i = i0 + j * T;
          k[j] = (uint32_t)bins[i < L.nb ? i : L.nb - 1];
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
          const int i = i0 + j * T;
          if (i >= L.nb) continue;
          const uint32_t r = Pb == 1 ? k[j] : mod_small(k[j], Q, inv_Q), rm = r ? Q - r : 0u;
          const float2 w1 = buf[fpad((int)r)], w2 = buf[fpad((int)rm)];
          float2 d0 = make_float2(h0 * (w1.x + w2.x), h0 * (w1.y - w2.y));
          float2 d1 = make_float2(h1 * (w1.y + w2.y), h1 * (w2.x - w1.x));
          if (Pb > 1) {
            const float2 tw = conjf2(cis_poly_x((float)mod_small(k[j] * b, M, inv_Mf) / (float)M));  // e^{-j 2 pi k b / M}
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

template <bool BF16>
static hipError_t launch_prefill_chirp_t(const Params& P, const void* K, const void* V, hipStream_t st) {
  const int n_st = P.n_slices * 2;
  const int per_xcd = (n_st + 7) / 8;
  constexpr int kNp = BF16 ? 4 : 2;
  const int logN = P.chirp_logN;
  const int max_slots = kCusPerXcd << (kTabMaxLogQ - logN);  // workgroups that an XCD holds at once
  // one pair per item where the device would not be full with several; 1024 points only come with few slices (see the plan)
  const bool few = logN == 10 || (int64_t)per_xcd * (kHeadDim / 2 / kNp) < max_slots;
#define IWDFT_PC_LAUNCH(LN, NP)                                                                                  \
  {                                                                                                              \
    constexpr int bytes = (int)sizeof(float2) * fft_lds(LN);                                                     \
    const int64_t items = (int64_t)per_xcd * (kHeadDim / 2 / (NP));                                              \
    const int slots = items < max_slots ? (int)items : max_slots;                                                \
    static LdsLimit lim;                                                                                         \
    const hipError_t e = lim.ensure((const void*)prefill_chirp_kernel<LN, BF16, NP>, bytes);                     \
    if (e != hipSuccess) return e;                                                                               \
    prefill_chirp_kernel<LN, BF16, NP><<<dim3((uint32_t)slots * 8), dim3(fft_threads(LN)), bytes, st>>>(         \
        P, K, V, per_xcd, n_st, slots);                                                                          \
  }
#define IWDFT_PC_CASE(LN)                             \
  case LN:                                            \
    if (few) IWDFT_PC_LAUNCH(LN, 1)                   \
    else IWDFT_PC_LAUNCH(LN, kNp)                     \
    break;
  switch (logN) {
    case 10: IWDFT_PC_LAUNCH(10, 1) break;
    IWDFT_PC_CASE(11)
    IWDFT_PC_CASE(12)
    IWDFT_PC_CASE(13)
    IWDFT_PC_CASE(14)
    default: return hipErrorInvalidValue;
  }
#undef IWDFT_PC_CASE
#undef IWDFT_PC_LAUNCH
  return hipGetLastError();
}

hipError_t launch_prefill_chirp(const Params& P, const void* K, const void* V, hipStream_t st) {
  if (!P.chirp) return hipErrorInvalidValue;
  const hipError_t e = launch_prefill_edges(P, K, V, st);
  if (e != hipSuccess) return e;
  return P.kv_dtype == 1 ? launch_prefill_chirp_t<true>(P, K, V, st) : launch_prefill_chirp_t<false>(P, K, V, st);
}

}  // namespace iwdft
