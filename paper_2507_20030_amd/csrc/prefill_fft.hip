// Prefill transform through FFTs (Sec. 3.1.2 Eq. dft-full computed the way Sec. 3.1.2 / Sec. 4.2.1
// suggest, O(M log M) per channel, followed by the pruning of Eq. freq-zero): for every slice, channel
// and kept bin k the same U_M[k] = sum_n x[n] e^{-j 2 pi k n / M} as the dense contraction, for DFT
// lengths that are a power of two.
//
// One workgroup transforms two channels of one slice at a time, packed as the real and imaginary part
// of one complex signal z = x_c0 + j x_c1; the two spectra are separated afterwards with
// X_c0[k] = (Z[k] + conj Z[-k]) / 2, X_c1[k] = (Z[k] - conj Z[-k]) / (2j).  M > 8192: the token axis is
// decimated by Pb = M / 8192, n = Pb a + b, so that
//   U[k] = sum_b e^{-j 2 pi k b / M} * DFT_8192( x[Pb a + b] )[k mod 8192],
// one in-LDS transform per residue b (only the kept bins are ever formed).  Each lane reads 4 to 16 bytes
// of a token row (256 or 512), so the workgroups of one (slice, tensor) are placed on one XCD next to each
// other in time and share the rows in that XCD's L2: HBM delivers every row once.
//
// Three kernels: prefill_fft_kernel (M <= 8192), prefill_stream_kernel (longer M, running sums in
// registers, 4096 bins a launch) and prefill_rows_kernel (longer M and more bins, sums in the output rows).
#include "common.h"
#include "fft_core.h"
#include "fft_lds.h"
#include "pair_io.h"

namespace iwdft {

constexpr int kPairs = kHeadDim / 2;  // channel pairs per (slice, tensor)

// hardware block id -> (xcd = id & 7, idx = id >> 3); XCD x owns the (slice, tensor) pairs
// x * per_xcd .. (x + 1) * per_xcd - 1, 64 / (NS NP) consecutive idx each.
// A workgroup of 512 threads runs NS = 8192 / Q transforms side by side, each on NP channel pairs one after the other.  The
// transforms are interleaved over the lanes (thread = t NS + g), so that NS lanes fetch 4 NP NS adjacent bytes of a token
// row (bf16) with one load each: a token row is two 128-byte lines, and what bounds the loads is the number of lines that
// are asked for, not their bytes (measured on 1.07 GB: 16 bytes of every line per load 0.37 ms, 32 0.28, 64 0.19, 128 0.18).
// A thread's 16 samples are the 16 consecutive positions that the first radix-16 pass combines: that pass runs on the
// loaded words and the samples go to LDS once, behind it; the last radix-2 stage (M >= 8192, M = 512) is formed at the kept
// bins only (spectrum_pair).  32 x 8 slices of 8192 tokens, 2048 bins: 0.80 -> 0.72 ms; 0.33 ms of it are the transforms.
// EQ: the two channels of a pair are scaled to one size on the way (pair_scale), each as exact as alone; see the launcher.
// TWO (M = 8192): 1024 threads run two transforms, so that 32 adjacent bytes of a row are fetched at a time.  There the loads weigh most, 380 us
// of the 727 that 32 x 8 slices take with one (the transforms alone 260, loads and stores without transforms 576); with two 668 us (469).
// At 4096 points and below, where several transforms share a workgroup anyway, twice as many are slower (4096 points 0.93 .. 0.97, 1024 0.7).
template <int LOGQ, bool BF16, int NP, bool EQ, bool TWO = false>
__global__ __launch_bounds__(side_threads(LOGQ, TWO), 4) void prefill_fft_kernel(Params P, const void* __restrict__ K,
                                                            const void* __restrict__ V, int per_xcd, int n_st) {
  extern __shared__ __attribute__((aligned(16))) float2 smem[];
  constexpr int Q = 1 << LOGQ, T = fft_threads(LOGQ), NS = side_ns(LOGQ, TWO), BS = side_bs(LOGQ, TWO);
  static_assert(T * NS == (TWO ? 1024 : 512) && NS * NP <= kPairs, "");
  constexpr int kElem = BF16 ? 2 : 4;
  constexpr int kRow = kHeadDim * kElem;  // bytes per token row
  constexpr int NW = NP * (BF16 ? 1 : 2);
  __shared__ uint32_t maxima[EQ ? T * NS / 64 : 1][EQ ? NS : 1][EQ ? NW : 1];
  __shared__ float2 halves[EQ ? NS : 1][EQ ? NP : 1];  // (h0, h1): transforms are pruned by other threads than those that fetch
  constexpr int kGroups = kPairs / (NP * NS);  // workgroups per (slice, tensor)
  const TabMem tab{P.tab + tab_base(LOGQ)};
  const int tid = threadIdx.x;
  const uint32_t idx = blockIdx.x >> 3;
  const uint32_t st = (blockIdx.x & 7u) * (uint32_t)per_xcd + idx / kGroups;
  if (st >= (uint32_t)n_st) return;
  const int pair0 = (idx % kGroups) * (NS * NP);
  const int tensor = st & 1;
  const int slice = st >> 1;
  const int spl = P.batch * P.n_kv;
  const int layer = slice / spl;
  const int s = slice - layer * spl;
  const LayerInfo L = layer_info(P, layer);
  const int32_t* bins = P.bins + L.bin_off;
  const int64_t N = (int64_t)P.S + P.M + P.R;  // tokens per slice in the caller's tensor
  const int t = tid / NS;                      // thread of transform tid % NS
  float2* buf = smem + (tid % NS) * BS;
  const char* X = (const char*)(tensor ? V : K) + ((int64_t)slice * N + P.S) * kRow + (pair0 + (tid % NS) * NP) * 2 * kElem;
  // the pruning goes through the transforms one after the other: consecutive threads, consecutive bins
  const int tp = tid % T;
  const float2* spec = smem + (tid / T) * BS;
  float2* F = (tensor ? P.FV : P.FK) + L.coef_off + ((int64_t)s * kHeadDim + (pair0 + (tid / T) * NP) * 2) * L.Bp;

  Raw<NW> z[16];
  const char* X0 = X + (int64_t)sample_at<LOGQ>(16 * t) * kRow;
#pragma unroll
  for (int m = 0; m < 16; ++m) z[m] = load_raw<NW>(X0 + sample_step<LOGQ>(m) * kRow);
  PairScale sc[NP];
  if constexpr (EQ) {
    scale_pairs<BF16>(z, tid, maxima, sc);
    if (NS > 1 && tid < NS) {
#pragma unroll
      for (int p = 0; p < NP; ++p) halves[tid][p] = make_float2(sc[p].h0, sc[p].h1);
    }
  }
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    float2 x[16];
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      x[m] = raw_front<BF16, NW>(z[m]);
      if constexpr (EQ) x[m].y *= sc[p].up;
      raw_pop<BF16, NW>(z[m]);
    }
    float2* F0 = F + (int64_t)(2 * p) * L.Bp;
    // kept bins of this thread, four at a time; the first four are fetched while the transform runs
    constexpr int U = 4;
    uint32_t kj[U];
    float2 wj[U];
    auto fetch_bins = [&](int i0) {
#pragma unroll
      for (int j = 0; j < U; ++j) {
        const int i = i0 + j * T;
        kj[j] = (uint32_t)bins[i < L.nb ? i : L.nb - 1];
      }
    };
    auto fetch_tw = [&](int k) {
      if (k != fft_np(LOGQ) - 1) return;
#pragma unroll
      for (int j = 0; j < U; ++j) wj[j] = pair_twiddle<LOGQ>(tab.tab, kj[j] & (Q - 1));
    };
    fetch_bins(pin_index(tp));
    fft_forward<LOGQ>(buf, tab, t, x, fetch_tw);
    float2 h = make_float2(0.5f, 0.5f);
    if constexpr (EQ) h = NS > 1 ? halves[tid / T][p] : make_float2(sc[p].h0, sc[p].h1);
    for (int i0 = tp; i0 < L.nb; i0 += U * T) {
      if (i0 >= U * T) {
        fetch_bins(i0);
        fetch_tw(fft_np(LOGQ) - 1);
      }
#pragma unroll
      for (int j = 0; j < U; ++j) {
        const int i = i0 + j * T;
        if (i < L.nb) {
          float2 w1, w2;
          spectrum_pair<LOGQ>(spec, kj[j] & (Q - 1), wj[j], w1, w2);
          F0[i] = make_float2(h.x * (w1.x + w2.x), h.x * (w1.y - w2.y));
          F0[L.Bp + i] = make_float2(h.y * (w1.y + w2.y), h.y * (w2.x - w1.x));
        }
      }
    }
    __syncthreads();  // the next transform overwrites buf
  }
}

// M > 8192 and more kept bins than registers hold (prefill_stream_kernel): the running sums over the residues live in the output
// rows, every bin belongs to one thread, which reads back its own earlier store.  On the transforms of fft_lds.h, whose twiddles
// sit in LDS: vector memory answers in order, and table loads between the stores of the sums and the next transform waited for
// these (on fft_core.h, 256 slices of 16384 tokens, 4200 bins: bf16 3.03 ms, fp32 4.18; here 2.65 and 3.51).
template <bool BF16, int NP>
__global__ __launch_bounds__(kFftThreads, 4) void prefill_rows_kernel(Params P, const void* __restrict__ K,
                                                                     const void* __restrict__ V, int per_xcd, int n_st) {
  extern __shared__ __attribute__((aligned(16))) float2 buf[];
  constexpr int LOGQ = kFftMaxLogQ, Q = 1 << LOGQ, H = Q / 2, IT = H / kFftThreads;
  static_assert(LOGQ & 1, "written for the odd transform length 2^13");
  constexpr int kElem = BF16 ? 2 : 4;
  constexpr int kRow = kHeadDim * kElem;  // bytes per token row
  constexpr int NW = NP * (BF16 ? 1 : 2);
  constexpr int kGroups = kPairs / NP;    // workgroups per (slice, tensor)
  float2* tab = buf + Q + (Q >> 5);
  const int tid = threadIdx.x;
  const uint32_t idx = blockIdx.x >> 3;
  const uint32_t st = (blockIdx.x & 7u) * (uint32_t)per_xcd + idx / kGroups;
  if (st >= (uint32_t)n_st) return;
  const int pair0 = (idx % kGroups) * NP;
  const int slice = st >> 1;
  const int spl = P.batch * P.n_kv;
  const int layer = slice / spl;
  const LayerInfo L = layer_info(P, layer);
  const int32_t* bins = P.bins + L.bin_off;
  const int64_t N = (int64_t)P.S + P.M + P.R;  // tokens per slice in the caller's tensor
  const char* X = (const char*)((st & 1) ? V : K) + ((int64_t)slice * N + P.S) * kRow + pair0 * 2 * kElem;
  const uint32_t Pb = P.M >> LOGQ;
  const int64_t step = (int64_t)Pb * kRow;  // bytes between consecutive samples of one residue
  float2* F = ((st & 1) ? P.FV : P.FK) + L.coef_off + ((int64_t)(slice - layer * spl) * kHeadDim + pair0 * 2) * L.Bp;

  for (int m = tid; m <= (Q >> 3); m += kFftThreads) tab[m] = P.tw8[m];  // e^{j 2 pi m / Q}, host-made

  for (uint32_t b = 0; b < Pb; ++b) {
    int lt = tid;
    asm volatile("" : "+v"(lt));  // keeps the passes' address arithmetic out of long-lived registers
    const char* Xb = X + (int64_t)b * kRow;
    // Consecutive threads own consecutive LDS positions (their stores fall into distinct banks) and fetch the samples that
    // belong there, a and a + Q / 2 for the first radix-2 stage.
    Raw<NW> za[IT], zc[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int a = digit_pos<LOGQ - 1>(it * kFftThreads + lt);  // digit reversal is its own inverse
      za[it] = load_raw<NW>(Xb + (int64_t)a * step);
      zc[it] = load_raw<NW>(Xb + (int64_t)(a + H) * step);
    }
#pragma unroll
    for (int p = 0; p < NP; ++p) {
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int pos = 2 * (it * kFftThreads + lt);
        const float2 u = raw_front<BF16, NW>(za[it]), v = raw_front<BF16, NW>(zc[it]);
        raw_pop<BF16, NW>(za[it]);
        raw_pop<BF16, NW>(zc[it]);
        buf[pad(pos)] = cadd(u, v);
        buf[pad(pos + 1)] = csub(u, v);
      }
      __syncthreads();  // (the first time also publishes tab)
      fft_dit<LOGQ>(buf, tab, lt);
      float2* F0 = F + (int64_t)(2 * p) * L.Bp;
      for (int i = tid; i < L.nb; i += kFftThreads) {
        const uint32_t kj = (uint32_t)bins[i];
        const int r = kj & (Q - 1), rm = (Q - r) & (Q - 1);
        const float2 w1 = buf[pad(r)], w2 = buf[pad(rm)];
        const float2 tw = conjf2(cis_poly2((kj * b) & (P.M - 1u), P.M));  // e^{-j 2 pi k b / M}
        float2 d0 = cmul(tw, make_float2(0.5f * (w1.x + w2.x), 0.5f * (w1.y - w2.y)));
        float2 d1 = cmul(tw, make_float2(0.5f * (w1.y + w2.y), 0.5f * (w2.x - w1.x)));
        if (b) {
          d0 = cadd(F0[i], d0);
          d1 = cadd(F0[L.Bp + i], d1);
        }
        F0[i] = d0;
        F0[L.Bp + i] = d1;
      }
      __syncthreads();  // the next pair overwrites buf
    }
  }
}

// M > 8192, NBT * 512 kept bins per layer and launch: one persistent workgroup per CU walks the (slice, tensor, NP channel
// pairs) items of its XCD and their residues with the running sums of all kept bins in registers (which is why there is
// one), and fetches the samples of the next step while it transforms the pairs of the current one, a row or so per phase: a
// wave that issues more than the address queue takes stalls, and the barriers make the others wait.  Vector memory answers
// in order, so nothing else in the loop may be a load that is waited for at once: the passes' twiddles and the bin
// twiddles sit in LDS.  8 x 8 slices of 131072 tokens, 4096 bins: 4.77 -> 4.27 ms; with the token loads taken out 2.2.
// The last radix-2 stage of the transform and the residue sum are one thing: sample n = Pb (2 a + h) + b, so every bin takes
// two products, with e^{-j 2 pi k b / M} for the even half spectrum E and e^{-j 2 pi k (b + Pb) / M} for the odd one O; with
// r = k mod 4096 and the mirror entry r' = -r mod 4096, the first channel's part is (E[r] + conj E[r']) / 2 and so on.
template <bool BF16, int NBT, int NP, bool EQ>
__global__ __launch_bounds__(512, 2) void prefill_stream_kernel(Params P, const void* __restrict__ K,
                                                               const void* __restrict__ V, int per_xcd, int n_st,
                                                               int slots, int bin0) {
  constexpr int LOGQ = 13, Q = 1 << LOGQ, H = Q / 2, T = 512;
  static_assert(fft_threads(LOGQ) == T && kFftMaxLogQ == LOGQ, "");
  constexpr int kElem = BF16 ? 2 : 4;
  constexpr int kRow = kHeadDim * kElem;
  constexpr int NW = NP * (BF16 ? 1 : 2);  // words per sample: 16 bytes, one pair's for tensors that are not 16-byte aligned
  constexpr int kGroups = kPairs / NP;
  extern __shared__ __attribute__((aligned(16))) float2 buf[];
  __shared__ uint32_t maxima[EQ ? 8 : 1][1][EQ ? NW : 1];
  float4* ltab = (float4*)(buf + fft_lds(LOGQ));
  float4* btw = ltab + TabLds::entries<LOGQ>();  // [NBT * T] bin twiddles (even, odd), halves of them without EQ; a thread's own entries only
  const TabLds tab{P.tab + tab_base(LOGQ), ltab};
  const int tid = threadIdx.x;
  const uint32_t xcd = blockIdx.x & 7u;
  const int st_first = (int)xcd * per_xcd, st_count = min(per_xcd, n_st - st_first);
  const int n_items = st_count * kGroups;
  const int spl = P.batch * P.n_kv;
  auto layer_of = [&](int item) {  // this launch's bins of the item's layer: NBT * T from bin0 on
    LayerInfo L = layer_info(P, ((st_first + item / kGroups) >> 1) / spl);
    L.bin_off += bin0;
    L.coef_off += bin0;
    L.nb = min(L.nb - bin0, NBT * T);
    return L;
  };
  auto with_bins = [&](int item) {  // the first of items item, item + slots, ... whose layer has any
    while (item < n_items && layer_of(item).nb <= 0) item += slots;
    return item;
  };
  int n = with_bins((int)(blockIdx.x >> 3));
  if (n >= n_items) return;  // the whole workgroup
  tab.fill<LOGQ>(ltab, tid);

  const uint32_t M = P.M, Pb = M >> LOGQ;
  const int64_t N = (int64_t)P.S + M + P.R;      // tokens per slice in the caller's tensor
  const uint32_t step = Pb * (uint32_t)kRow;     // bytes between consecutive samples of one residue
  const uint32_t voff = sample_at<LOGQ>(16 * tid) * step;  // < 2^32: the launcher checks M
  auto rows = [&](int item, uint32_t b) {        // first sample of residue b of an item
    const int st = st_first + item / kGroups;
    return (const char*)((st & 1) ? V : K) + ((int64_t)(st >> 1) * N + P.S + b) * kRow + (item % kGroups) * (NP * 2 * kElem);
  };
  auto fetch = [&](Raw<NW>& z, const char* base, uint32_t off, int m) {
    z = load_raw<NW>(base + (int64_t)((((m & 3) << 2) | (m >> 2)) * (Q / 16)) * step + off);
  };

  uint32_t kk[NBT];
  auto fetch_bins = [&](uint32_t (&k)[NBT], int bin_off, int nb) {
    const int o = pin_index(tid);
#pragma unroll
    for (int j = 0; j < NBT; ++j) {
      const int i = j * T + o;
      k[j] = (uint32_t)P.bins[bin_off + (i < nb ? i : nb - 1)];
    }
  };
  Raw<NW> z[16];
  LayerInfo L = layer_of(n);
  fetch_bins(kk, L.bin_off, L.nb);
#pragma unroll
  for (int m = 0; m < 16; ++m) fetch(z[m], rows(n, 0), voff, m);
  float2 acc[NP][2][NBT];  // running sums over the residues
#pragma unroll
  for (int p = 0; p < NP; ++p)
#pragma unroll
    for (int j = 0; j < NBT; ++j) acc[p][0][j] = acc[p][1][j] = make_float2(0.f, 0.f);
  __syncthreads();

  uint32_t b = 0;
#pragma unroll 1
  for (;;) {
    const int st = st_first + n / kGroups;
    const int s = (st >> 1) - ((st >> 1) / spl) * spl;
    float2* F = ((st & 1) ? P.FV : P.FK) + L.coef_off + ((int64_t)s * kHeadDim + (n % kGroups) * (NP * 2)) * L.Bp;
    const bool last_b = b + 1 == Pb;
    const int n1 = last_b ? with_bins(n + slots) : n;
    const bool more = n1 < n_items;
    const uint32_t b1 = last_b ? 0u : b + 1;
    // at the very end the current rows are fetched once more instead of a branch
    const char* nx = more ? rows(n1, b1) : rows(n, b);
    const LayerInfo Ln = layer_of(more ? n1 : n);
    Raw<NW> zn[16];

#pragma unroll
    for (int j = 0; j < NBT; ++j) {
      const float2 t0 = cis_poly2((kk[j] * b) & (M - 1u), M), t1 = cis_poly2((kk[j] * (b + Pb)) & (M - 1u), M);
      constexpr float kHalf = EQ ? 1.f : 0.5f;
      btw[j * T + tid] = make_float4(kHalf * t0.x, -kHalf * t0.y, kHalf * t1.x, -kHalf * t1.y);
    }
    PairScale sc[NP];
    if constexpr (EQ) scale_pairs<BF16>(z, tid, maxima, sc);
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      float2 x[16];
#pragma unroll
      for (int m = 0; m < 16; ++m) {
        x[m] = raw_front<BF16, NW>(z[m]);
        if constexpr (EQ) x[m].y *= sc[p].up;
        raw_pop<BF16, NW>(z[m]);
      }
      // The next step's samples, one row or so per phase (three passes and the pruning): a wave that issues more than the
      // address queue takes stalls.  In this order every word lands in a register that the current samples have left.
      auto fetch_next = [&](int phase) {
        constexpr int kPhases = 4 * NP;
        const int at = 4 * p + phase;
        const uint32_t off = (uint32_t)pin_index((int)voff);
#pragma unroll
        for (int m = at * 16 / kPhases; m < (at + 1) * 16 / kPhases; ++m) fetch(zn[m], nx, off, m);
      };
      fft_forward<LOGQ>(buf, tab, tid, x, fetch_next);
      fetch_next(3);
      float2 h = make_float2(1.f, 1.f);  // without EQ the bin twiddles hold the halves
      if constexpr (EQ) h = make_float2(sc[p].h0, sc[p].h1);
#pragma unroll
      for (int j = 0; j < NBT; ++j) {
        const uint32_t r = kk[j] & (H - 1), rm = (H - r) & (H - 1);
        const float2 *u = buf + fpad((int)r), *v = buf + fpad((int)rm);
        const float2 e = u[0], o = u[H + H / 8], em = v[0], om = v[H + H / 8];
        const float4 w = btw[j * T + tid];
        const float2 se = make_float2(h.x * (e.x + em.x), h.x * (e.y - em.y));
        const float2 de = make_float2(h.y * (e.y + em.y), h.y * (em.x - e.x));  // -j (E - conj E')
        const float2 so = make_float2(h.x * (o.x + om.x), h.x * (o.y - om.y));
        const float2 dd = make_float2(h.y * (o.y + om.y), h.y * (om.x - o.x));
        float2 &a0 = acc[p][0][j], &a1 = acc[p][1][j];
        a0 = make_float2(fmaf(w.x, se.x, fmaf(-w.y, se.y, a0.x)), fmaf(w.x, se.y, fmaf(w.y, se.x, a0.y)));
        a1 = make_float2(fmaf(w.x, de.x, fmaf(-w.y, de.y, a1.x)), fmaf(w.x, de.y, fmaf(w.y, de.x, a1.y)));
        a0 = make_float2(fmaf(w.z, so.x, fmaf(-w.w, so.y, a0.x)), fmaf(w.z, so.y, fmaf(w.w, so.x, a0.y)));
        a1 = make_float2(fmaf(w.z, dd.x, fmaf(-w.w, dd.y, a1.x)), fmaf(w.z, dd.y, fmaf(w.w, dd.x, a1.y)));
      }
      __syncthreads();  // the next transform overwrites buf
    }
    if (last_b) {
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        float2* F0 = F + (int64_t)(2 * p) * L.Bp;
#pragma unroll
        for (int j = 0; j < NBT; ++j) {
          const int i = j * T + tid;
          if (i < L.nb) {
            F0[i] = acc[p][0][j];
            F0[L.Bp + i] = acc[p][1][j];
          }
          acc[p][0][j] = acc[p][1][j] = make_float2(0.f, 0.f);
        }
      }
    }
    if (!more) break;
    if (last_b) fetch_bins(kk, Ln.bin_off, Ln.nb);
    n = n1;
    b = b1;
    L = Ln;
#pragma unroll
    for (int m = 0; m < 16; ++m) z[m] = zn[m];
  }
}

constexpr int kCusPerXcd = 32;
constexpr uint64_t kFewWorkgroups = 256;
bool prefill_fft_ok(const Params& P) { return P.Mmask != 0 && P.M >= 256; }

template <bool BF16>
static hipError_t launch_prefill_fft_t(const Params& P, const void* K, const void* V, hipStream_t st) {
  int logM = 0;
  while ((1u << logM) < P.M) ++logM;
  const int n_st = P.n_slices * 2;
  const int per_xcd = (n_st + 7) / 8;
  // several pairs per load need 16-byte aligned tensors (and rows, which are 256 or 512 bytes)
  const bool wide = (((uintptr_t)K | (uintptr_t)V) & 15u) == 0;
  // Contexts of few bins take the FFT for its speed only, and the contraction it replaces keeps every channel alone (8192 points,
  // a channel 2^11 below its partner: 1.8e-4 relative error in an unscaled transform): there the channels of a pair are scaled to
  // one size.  It costs 31 packed maxima and 16 products per pair and a barrier: 256 slices of 8192 tokens, 128 bins, bf16 622 us
  // against 547 without, fp32 876 / 861.
  const bool eq = P.scale_pairs != 0;
  hipError_t e = hipSuccess;
  // More than 4096 bins: twice through the tokens where that takes less time than the sums in the output rows (launches / rows,
  // ms; 64 slices, M = 32768, 8192 bins: bf16 2.37 / 2.40, fp32 2.16 / 2.57; 8 slices: 0.277 / 0.240, 0.287 / 0.345; M = 262144,
  // 8192 bins, 8 slices: 2.14 / 2.26, 2.03 / 3.63, one slice: 1.37 / 1.01, 0.75 / 1.25).  More launches do not pay (M = 65536,
  // 16384 bins, 8 slices: 1.06 / 1.06, 1.12 / 1.13, one slice 0.44 / 0.39, 0.38 / 0.35; M = 262144, 65536 bins, one slice: 11.0 /
  // 5.7, 6.3 / 4.5).
  const bool twice = P.max_nb <= 8192 && (BF16 ? P.M >= 131072u && P.n_slices >= 8 : P.M >= 32768u);
  const bool stream = P.M <= kStreamMaxM && (P.max_nb <= 4096 || twice);
  if (logM > kFftMaxLogQ && stream) {
#define IWDFT_PF_STREAM(NBT, NP, EQ)                                                                          \
  {                                                                                                           \
    const size_t bytes = sizeof(float2) * fft_lds(kFftMaxLogQ) +                                              \
                         sizeof(float4) * (TabLds::entries<kFftMaxLogQ>() + (NBT) * 512);                     \
    const int items = per_xcd * (kPairs / (NP)), slots = items < kCusPerXcd ? items : kCusPerXcd;             \
    static LdsLimit lim;                                                                                      \
    e = lim.ensure((const void*)prefill_stream_kernel<BF16, NBT, NP, EQ>, (int)bytes);                        \
    if (e != hipSuccess) return e;                                                                            \
    prefill_stream_kernel<BF16, NBT, NP, EQ><<<dim3((uint32_t)slots * 8), dim3(512), bytes, st>>>(            \
        P, K, V, per_xcd, n_st, slots, bin0);                                                                 \
  }
    constexpr int kNp = BF16 ? 4 : 2;
    for (int bin0 = 0; bin0 < P.max_nb; bin0 += 4096) {
      if (P.max_nb - bin0 > 2048) {
        if (wide) IWDFT_PF_STREAM(8, kNp, false) else IWDFT_PF_STREAM(8, 1, false)
      } else if (!eq) {
        if (wide) IWDFT_PF_STREAM(4, kNp, false) else IWDFT_PF_STREAM(4, 1, false)
      } else {
        if (wide) IWDFT_PF_STREAM(4, kNp, true) else IWDFT_PF_STREAM(4, 1, true)
      }
      e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
#undef IWDFT_PF_STREAM
    return hipSuccess;
  }
  if (logM > kFftMaxLogQ) {
    const size_t bytes = sizeof(float2) * (size_t)fft_lds_float2(kFftMaxLogQ);
#define IWDFT_PF_ROWS(NP)                                                                                          \
  {                                                                                                                \
    const uint64_t blocks = (uint64_t)per_xcd * (kPairs / (NP)) * 8;                                               \
    if (blocks > 0x7fffffffull) return hipErrorInvalidConfiguration;                                               \
    static LdsLimit lim;                                                                                           \
    e = lim.ensure((const void*)prefill_rows_kernel<BF16, NP>, (int)bytes);                                        \
    if (e != hipSuccess) return e;                                                                                 \
    prefill_rows_kernel<BF16, NP><<<dim3((uint32_t)blocks), dim3(kFftThreads), bytes, st>>>(P, K, V, per_xcd, n_st); \
  }
    constexpr int kNp = BF16 ? 2 : 1;  // what the register budget holds
    if (wide) IWDFT_PF_ROWS(kNp) else IWDFT_PF_ROWS(1)
#undef IWDFT_PF_ROWS
    return hipGetLastError();
  }
  const int logQ = logM;
  // Pairs per thread: as many as the register budget (128) holds next to the transform (the staged samples take 16
  // registers per further bf16 pair), unless the device would not be full: then the pairs spread over more workgroups.  At 256
  // points the 32 transforms side by side cover 128 bytes of a row with one pair each (512 slices, 64 bins, two pairs / one:
  // 30 / 25 us, fp32 40 / 33).
  const bool few = (uint64_t)n_st * (kPairs / 4) < kFewWorkgroups * (uint64_t)side_ns(logQ);
  const bool two = logQ == 13 && two_transforms((int64_t)per_xcd * (kPairs / (BF16 ? 8 : 4)));
#define IWDFT_PF_CASE(LQ, NP, EQ, TWO)                                                                      \
  {                                                                                                         \
    const size_t lds = sizeof(float2) * (size_t)(side_ns(LQ, TWO) * side_bs(LQ, TWO));                      \
    const uint64_t blocks = (uint64_t)per_xcd * (kPairs / ((NP) * side_ns(LQ, TWO))) * 8;                   \
    if (blocks > 0x7fffffffull) return hipErrorInvalidConfiguration;                                        \
    static LdsLimit lim;                                                                                    \
    e = lim.ensure((const void*)prefill_fft_kernel<LQ, BF16, NP, EQ, TWO>, (int)lds);                       \
    if (e != hipSuccess) return e;                                                                          \
    prefill_fft_kernel<LQ, BF16, NP, EQ, TWO>                                                               \
        <<<dim3((uint32_t)blocks), dim3(side_threads(LQ, TWO)), lds, st>>>(P, K, V, per_xcd, n_st);         \
  }
#define IWDFT_PF_SINGLE(LQ)                                                        \
  {                                                                                \
    constexpr int kNp = LQ == 8 ? 1 : BF16 ? 4 : 2;                                \
    constexpr bool kTwo = LQ == 13;                                                \
    if (!eq) {                                                                     \
      if (wide && two) IWDFT_PF_CASE(LQ, kNp, false, kTwo)                         \
      else if (wide && !few) IWDFT_PF_CASE(LQ, kNp, false, false)                  \
      else IWDFT_PF_CASE(LQ, 1, false, false)                                      \
    } else if (wide && two) {                                                      \
      IWDFT_PF_CASE(LQ, kNp, true, kTwo)                                           \
    } else if (wide && !few) {                                                     \
      IWDFT_PF_CASE(LQ, kNp, true, false)                                          \
    } else {                                                                       \
      IWDFT_PF_CASE(LQ, 1, true, false)                                            \
    }                                                                              \
  }
  switch (logQ) {
    case 8: IWDFT_PF_SINGLE(8) break;
    case 9: IWDFT_PF_SINGLE(9) break;
    case 10: IWDFT_PF_SINGLE(10) break;
    case 11: IWDFT_PF_SINGLE(11) break;
    case 12: IWDFT_PF_SINGLE(12) break;
    default: IWDFT_PF_SINGLE(13) break;
  }
#undef IWDFT_PF_SINGLE
#undef IWDFT_PF_CASE
  return hipGetLastError();
}

hipError_t launch_prefill_fft(const Params& P, const void* K, const void* V, hipStream_t st) {
  if (!prefill_fft_ok(P)) return hipErrorInvalidValue;
  hipError_t e = launch_prefill_edges(P, K, V, st);
  if (e != hipSuccess) return e;
  if (P.dec_logN) return launch_prefill_low(P, K, V, st);
  return P.kv_dtype == 1 ? launch_prefill_fft_t<true>(P, K, V, st) : launch_prefill_fft_t<false>(P, K, V, st);
}

}  // namespace iwdft
