// Materialising reconstruction (Sec. 3.1.2 Eq. inverse-swdft over the kept bins; Sec. 4.2.2
// Eq. reconstruct-idft): x~[a] = (1/M) Re sum_k w_k U_T[k] exp(+j 2 pi k a / M).
// With the fixed-frame storage U_T[k] = exp(-j 2 pi k t/M) F_T[k], t = (T-M) mod M, so the
// sum runs over F_T with the slot index shifted by t.  This is the sparse inverse DFT written
// as a tiled contraction [slots x bins] * [bins x channels]; decode attention never calls it
// (it consumes the coefficients directly), it exists to inspect / verify the state.
//
// Two kernels: the tiled direct contraction (any M, any slot range) and, for power-of-two M and long
// ranges, in-LDS inverse FFTs (reconstruct_fft_kernel below).
#include "common.h"
#include "fft_core.h"
#include "pair_io.h"

namespace iwdft {

constexpr int kRecSlots = 64;  // slots per block
constexpr int kRecBins = 32;   // bins per LDS tile
constexpr int kRecPairs = kHeadDim / 2;

// grid: ((s * atiles) + atile) * 2 + tensor ; 256 threads, each 4 channels x 8 slots.
template <bool BF16>
__global__ __launch_bounds__(256) void reconstruct_kernel(Params P, int layer, uint32_t a0, uint32_t stride,
                                                         uint32_t n_slots, void* __restrict__ Kt,
                                                         void* __restrict__ Vt, uint32_t tsh, int atiles) {
  __shared__ float2 Fs[kRecBins][kHeadDim + 1];
  __shared__ float2 Tw[kRecBins][kRecSlots];
  uint32_t bid = blockIdx.x;
  const int tensor = bid & 1;
  bid >>= 1;
  const int at = bid % atiles;
  const int s = bid / atiles;
  void* out = tensor ? Vt : Kt;
  if (!out) return;
  const LayerInfo L = P.layers[layer];
  const float2* F = (tensor ? P.FV : P.FK) + L.coef_off + (int64_t)s * kHeadDim * L.Bp;
  const float inv_M = P.gain / (float)P.M;
  const int tid = threadIdx.x;
  const int td = tid & 31, ta = tid >> 5;

  float acc[8][4];
#pragma unroll
  for (int a = 0; a < 8; ++a)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[a][c] = 0.f;

  for (int i0 = 0; i0 < L.nb; i0 += kRecBins) {
    __syncthreads();
    {  // coefficient tile, pre-multiplied by w_k / M
      const int i = i0 + (tid & 31);
      const float w = (i < L.nb) ? P.weights[L.bin_off + i] * inv_M : 0.f;
      for (int d = tid >> 5; d < kHeadDim; d += 8) {
        float2 f = (i < L.nb) ? F[(int64_t)d * L.Bp + i] : make_float2(0.f, 0.f);
        Fs[tid & 31][d] = make_float2(f.x * w, f.y * w);
      }
    }
    for (int e = tid; e < kRecBins * kRecSlots; e += 256) {  // twiddle tile
      const int i = i0 + e / kRecSlots, a = e % kRecSlots;
      float2 w = make_float2(0.f, 0.f);
      const uint32_t rel = at * kRecSlots + a;            // output row; its slot is a0 + stride * rel < M
      const uint32_t slot = a0 + stride * rel;
      if (i < L.nb && rel < n_slots) {
        const uint32_t k = (uint32_t)P.bins[L.bin_off + i];
        const uint32_t sh = (slot % P.M + P.M - tsh) % P.M;  // (slot - t) mod M
        w = cis(mulmod(k, sh, P.M, P.Mmask), P.M);
      }
      Tw[e / kRecSlots][a] = w;
    }
    __syncthreads();
#pragma unroll 4
    for (int i = 0; i < kRecBins; ++i) {
      float2 f[4], w[8];
#pragma unroll
      for (int c = 0; c < 4; ++c) f[c] = Fs[i][td * 4 + c];
#pragma unroll
      for (int a = 0; a < 8; ++a) w[a] = Tw[i][ta * 8 + a];
#pragma unroll
      for (int a = 0; a < 8; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[a][c] += f[c].x * w[a].x - f[c].y * w[a].y;
    }
  }
#pragma unroll
  for (int a = 0; a < 8; ++a) {
    const uint32_t rel = at * kRecSlots + ta * 8 + a;
    if (rel < n_slots) {
      const int64_t o = ((int64_t)s * n_slots + rel) * kHeadDim + td * 4;
#pragma unroll
      for (int c = 0; c < 4; ++c) store_kv<BF16>(out, o + c, acc[a][c]);
    }
  }
}

// All M slots of two adjacent channels of one slice at a time: the kept coefficients (times w_k / (2M))
// go to bin k and, conjugated, to bin M - k of an LDS spectrum -- channel c0 as it is, channel c1 times j,
// so that after the inverse transform the real part is channel c0 and the imaginary part channel c1 --
// folded modulo Q = min(M, 8192) with the collision rounds the attention kernel uses (Params::fold).
// M > Q: block b of the token axis, slots Pb a + b, comes from the spectrum with bin k turned by
// e^{j 2 pi k b / M}.  Rows go out rotated by the slot shift (T - M) mod M; slots outside [a0, a0 + n_slots)
// are skipped.  Block ids are dealt so that the workgroups of a (slice, tensor) share one XCD's L2.
// A workgroup runs NS = 8192 / Q transforms side by side, interleaved over the lanes, on NP channel pairs one after the other
// (as the FFT prefill does), so that a lane stores 16 bytes and NS lanes 16 NS adjacent bytes of an output row at a time: with
// one pair per workgroup every 128-byte line was written in 32 pieces.  K and V of 64 slices, 8192 slots, 2048 bins, bf16:
// 408 -> 232 us (0.54 GB, 2.3 TB/s); what is left is vector arithmetic, the coefficients are read once per pair.
// TWO (8192 points): two transforms by 1024 threads, see prefill_fft.hip.
template <int LOGQ, bool BF16, bool MULTI, int NP, bool TWO = false>
__global__ __launch_bounds__(side_threads(LOGQ, TWO), 4) void reconstruct_fft_kernel(Params P, int layer, uint32_t a0, uint32_t n_slots,
                                                                void* __restrict__ Kt, void* __restrict__ Vt,
                                                                uint32_t tsh, int per_xcd, int n_st) {
  extern __shared__ __attribute__((aligned(16))) float2 smem[];
  constexpr int Q = 1 << LOGQ, T = fft_threads(LOGQ), NS = side_ns(LOGQ, TWO), BS = side_bs(LOGQ, TWO);
  static_assert(T * NS == (TWO ? 1024 : 512) && NS * NP <= kRecPairs, "");
  constexpr int kElem = BF16 ? 2 : 4;
  constexpr int kRow = kHeadDim * kElem;
  constexpr int NW = NP * (BF16 ? 1 : 2);
  constexpr int kGroups = kRecPairs / (NP * NS);  // workgroups per (slice, tensor)
  const float2* tab = P.tab + tab_base(LOGQ);
  const int tid = threadIdx.x;
  const uint32_t idx = blockIdx.x >> 3;
  const uint32_t stn = (blockIdx.x & 7u) * (uint32_t)per_xcd + idx / kGroups;
  if (stn >= (uint32_t)n_st) return;
  const int pair0 = (idx % kGroups) * (NS * NP);
  const int tensor = stn & 1;
  const int s = stn >> 1;  // slice within the layer
  char* out = (char*)(tensor ? Vt : Kt);
  if (!out) return;
  const LayerInfo L = layer_info(P, layer);
  const int32_t* bins = P.bins + L.bin_off;
  const float* wts = P.weights + L.bin_off;
  const uint16_t* fold = P.fold + L.bin_off;
  const uint32_t Pb = MULTI ? (P.M >> LOGQ) : 1u;
  const float gain = 0.5f * P.gain / (float)P.M;
  const int t = tid / NS;  // thread of transform tid % NS
  float2* buf = smem + (tid % NS) * BS;
  char* orow = out + (int64_t)s * n_slots * kRow + (pair0 + (tid % NS) * NP) * 2 * kElem;
  // the coefficients go through the transforms one after the other: consecutive threads, consecutive bins
  const int tp = tid % T;
  float2* spec = smem + (tid / T) * BS;
  const float2* F = (tensor ? P.FV : P.FK) + L.coef_off + ((int64_t)s * kHeadDim + (pair0 + (tid / T) * NP) * 2) * L.Bp;

#pragma unroll 1
  for (uint32_t b = 0; b < Pb; ++b) {
    Raw<NW> z[16] = {};
#pragma unroll 1
    for (int p = 0; p < NP; ++p) {
      float2 x[16] = {};
      write16(buf, t, x);  // this thread read these positions last
      __syncthreads();
      const float2 *F0 = F + (int64_t)(2 * p) * L.Bp, *F1 = F0 + L.Bp;
      for (int round = 0; round < L.fold_rounds; ++round) {
        constexpr int U = 4;  // bins whose loads are in flight together
        for (int i0 = tp; i0 < L.nb; i0 += U * T) {
          uint32_t k[U], fr[U];
          float w[U];
          float2 f0[U], f1[U];
#pragma unroll
          for (int j = 0; j < U; ++j) {
            const int i = i0 + j * T < L.nb ? i0 + j * T : L.nb - 1;
            k[j] = (uint32_t)bins[i], fr[j] = fold[i], w[j] = wts[i], f0[j] = F0[i], f1[j] = F1[i];
          }
#pragma unroll
          for (int j = 0; j < U; ++j) {
            if (i0 + j * T >= L.nb) continue;
            const float wg = w[j] * gain;
            float2 z0 = make_float2(f0[j].x * wg, f0[j].y * wg), z1 = make_float2(f1[j].x * wg, f1[j].y * wg);
            if constexpr (MULTI) {
              const float2 tw = cis_poly2((k[j] * b) & (P.M - 1u), P.M);
              z0 = cmul(z0, tw);
              z1 = cmul(z1, tw);
            }
            const int r = k[j] & (Q - 1), rm = (Q - r) & (Q - 1);
            if ((fr[j] & 0xffu) == (uint32_t)round) {  //      z0  + j z1
              float2 v = make_float2(z0.x - z1.y, z0.y + z1.x);
              if (r == rm) v = make_float2(2.f * z0.x, 2.f * z1.x);  // ... plus the mirror term, same slot
              if (round) v = cadd(v, spec[fpad(r)]);
              spec[fpad(r)] = v;
            }
            if ((fr[j] >> 8) == (uint32_t)round) {     // conj z0  + j conj z1
              float2 v = make_float2(z0.x + z1.y, z1.x - z0.y);
              if (round) v = cadd(v, spec[fpad(rm)]);
              spec[fpad(rm)] = v;
            }
          }
        }
        __syncthreads();
      }
      fft_inverse<LOGQ>(buf, tab, t, x);
#pragma unroll
      for (int m = 0; m < 16; ++m) raw_push<BF16, NW>(z[m], x[m]);
    }
    const uint32_t first = sample_at<LOGQ>(16 * t);
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      const uint32_t ap = (first + sample_step<LOGQ>(m)) * Pb + b;  // index of the un-shifted transform
      const uint32_t slot = (ap + tsh) & (P.M - 1u);                // where it sits after T - M appends
      const uint32_t rel = slot - a0;                                // wraps for slot < a0
      if (rel < n_slots) store_raw<NW>(orow + (int64_t)rel * kRow, z[m]);
    }
  }
}

constexpr int kRecMaxBins = 4096;  // layers with more have always taken the contraction (the transforms walk any list; not measured)
bool reconstruct_fft_ok(const Params& P) { return P.Mmask != 0 && P.M >= 256 && P.max_nb <= kRecMaxBins; }

template <bool BF16>
static hipError_t launch_reconstruct_fft_t(const Params& P, int layer, uint32_t a0, uint32_t n_slots, void* Kt,
                                           void* Vt, uint32_t tsh, hipStream_t st) {
  int logM = 0;
  while ((1u << logM) < P.M) ++logM;
  const int logQ = logM < kFftMaxLogQ ? logM : kFftMaxLogQ;
  const int n_st = P.batch * P.n_kv * 2;
  const int per_xcd = (n_st + 7) / 8;
  // several pairs per store need 16-byte aligned outputs (a null one is skipped); not where the device would not be full (pair_io.h):
  // the pairs spread over more workgroups then
  const bool wide = (((uintptr_t)Kt | (uintptr_t)Vt) & 15u) == 0 &&
                    (uint64_t)n_st * (kRecPairs / 4) >= side_pairs_min(logQ) * (uint64_t)side_ns(logQ);
  // One / two transforms a workgroup.  Longer contexts than 16384 gather more bins per transform (16 slices, M = 32768, 4096 bins 295 / 310 us).  One round of
  // workgroups only (bf16: 16 slices) has nothing to hide the gather behind: M = 8192, 1500 bins 1.12 times as fast, 1900 1.01 (behind other data
  // in the caches 0.91), 2000 0.95, 2048 53 / 60; M = 16384, 1024 bins 1.01, 1.05, 1500 121 / 130, 2402 135 / 146, 4096 151 / 159, low and mixed
  // masks alike (the first outputs of a context 138 / 135, 160 / 154, 187 / 175; three outputs in turn 1.0 to 1.2 times as fast).
  // Two rounds and more have: M = 16384, 32 slices, 1024 bins 248 / 234, 2402 282 / 275, 4096 323 / 298; at 8192 long rows only, 32 slices, 400 bins 0.99
  // times as fast, 800 103 / 107, 1200 0.98, 1600 0.99, 1800 1.01, 2048 123 / 121, 48 slices, 800 159 / 165, 64, 2048 232 / 225.  fp32, 16384 slots, 8
  // slices, 1024 bins 77 / 72, 1800 88 / 86, 2402 to 4096 0.99 to 1.00, 16 slices, 2481 bins 209 / 195.
  const int64_t blocks = (int64_t)per_xcd * (kRecPairs / (BF16 ? 8 : 4));
  const bool once = blocks <= kTwoRound;
  const bool pays = !BF16 || (P.M == 8192 ? once == (P.max_nb <= 1792) : !once || P.max_nb <= 1024);
  const bool two = logQ == 13 && P.M <= 16384 && two_transforms(blocks) && pays;
  hipError_t e = hipSuccess;
#define IWDFT_RC_LAUNCH(LQ, MULTI, NP, TWO)                                                             \
  {                                                                                                     \
    const size_t lds = sizeof(float2) * (size_t)(side_ns(LQ, TWO) * side_bs(LQ, TWO));                  \
    const uint64_t blocks = (uint64_t)per_xcd * (kRecPairs / ((NP) * side_ns(LQ, TWO))) * 8;            \
    if (blocks > 0x7fffffffull) return hipErrorInvalidConfiguration;                                    \
    static LdsLimit lim;                                                                                \
    e = lim.ensure((const void*)reconstruct_fft_kernel<LQ, BF16, MULTI, NP, TWO>, (int)lds);            \
    if (e != hipSuccess) return e;                                                                      \
    reconstruct_fft_kernel<LQ, BF16, MULTI, NP, TWO>                                                    \
        <<<dim3((uint32_t)blocks), dim3(side_threads(LQ, TWO)), lds, st>>>(                             \
            P, layer, a0, n_slots, Kt, Vt, tsh, per_xcd, n_st);                                         \
  }
#define IWDFT_RC_CASE(LQ, MULTI)                                                      \
  {                                                                                   \
    constexpr int kNp = side_pairs(LQ, BF16);                                   \
    if (wide && two) IWDFT_RC_LAUNCH(LQ, MULTI, kNp, LQ == 13)                        \
    else if (wide) IWDFT_RC_LAUNCH(LQ, MULTI, kNp, false)                             \
    else IWDFT_RC_LAUNCH(LQ, MULTI, 1, false)                                         \
  }
  if (logM > logQ) IWDFT_RC_CASE(kFftMaxLogQ, true)
  else switch (logQ) {
    case 8: IWDFT_RC_CASE(8, false) break;
    case 9: IWDFT_RC_CASE(9, false) break;
    case 10: IWDFT_RC_CASE(10, false) break;
    case 11: IWDFT_RC_CASE(11, false) break;
    case 12: IWDFT_RC_CASE(12, false) break;
    default: IWDFT_RC_CASE(13, false) break;
  }
#undef IWDFT_RC_CASE
#undef IWDFT_RC_LAUNCH
  return hipGetLastError();
}

// use_fft: the caller knows the layer's fold schedule is valid (the attention path uses FFTs too).
hipError_t launch_reconstruct(const Params& P, int layer, uint32_t a0, uint32_t stride, uint32_t n_slots, void* Kt,
                              void* Vt, uint32_t tsh, bool use_fft, hipStream_t st) {
  // The transform produces all M slots; the direct contraction costs O(|B|) per requested slot.
  if (stride == 1 && use_fft && reconstruct_fft_ok(P) && (uint64_t)n_slots * 8 >= P.M)
    return P.kv_dtype == 1 ? launch_reconstruct_fft_t<true>(P, layer, a0, n_slots, Kt, Vt, tsh, st)
                           : launch_reconstruct_fft_t<false>(P, layer, a0, n_slots, Kt, Vt, tsh, st);
  const int atiles = (int)((n_slots + kRecSlots - 1) / kRecSlots);
  const uint64_t blocks = (uint64_t)P.batch * P.n_kv * atiles * 2;
  if (blocks > 0x7fffffffull) return hipErrorInvalidConfiguration;
  if (P.kv_dtype == 1)
    reconstruct_kernel<true><<<dim3((uint32_t)blocks), dim3(256), 0, st>>>(P, layer, a0, stride, n_slots, Kt, Vt, tsh, atiles);
  else
    reconstruct_kernel<false><<<dim3((uint32_t)blocks), dim3(256), 0, st>>>(P, layer, a0, stride, n_slots, Kt, Vt, tsh, atiles);
  return hipGetLastError();
}

}  // namespace iwdft
