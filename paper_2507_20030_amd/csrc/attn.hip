// Decode attention over the reconstructed segment (Sec. 3.1.1 Eq. kv-attn over the middle part
// of Sec. 4.2.2 Eq. kv-concat) without ever writing K~ or V~ (Eq. reconstruct-idft) to memory.
//
// For one slice and one query head, with F the stored coefficients and gain folded in:
//   scores  s[a] = scale * q . K~[a]        = Re sum_k Y[k] e^{+j 2 pi k a / M},
//                                             Y[k] = (w_k scale / M) * sum_c q[c] F_K[c][k]
//   weights p[a] = exp(s[a] - max) ,  Z = sum_a p[a]
//   output  o[c] = sum_a p[a] V~[a][c] / Z  = Re sum_k F_V[c][k] * Pn[k],
//                                             Pn[k] = (w_k / (M Z)) * conj( sum_a p[a] e^{-j 2 pi k a / M} )
// The common slot shift (T-M) of the fixed-frame storage moves K~ and V~ together and drops out
// of softmax attention.  The S sink and R recent tokens that Eq. kv-concat keeps exact join the same
// softmax: kernel A also writes their raw scores q.k_e, kernel B folds them into max / Z and turns
// them into weights p_e / Z, kernel C adds sum_e (p_e / Z) v_e.  Three kernels:
//   A  attn_qc_kernel   streams F_K once, produces qc[k] = sum_c q[c] F_K[c][k]    (HBM-bound)
//   B  attn_fft_kernel  per (slice, pair of query heads): sparse spectrum -> M scores by
//                       inverse FFT in LDS, softmax, forward FFT, gather the kept bins -> Pn
//      attn_chirp_kernel   the same for M that is not a power of two (attn_chirp.hip)
//      attn_direct_kernel  same result by direct O(M |B|) sums (any M; reference path)
//   C  attn_out_kernel  streams F_V once, o[c] = Re sum_k F_V[c][k] Pn[k]           (HBM-bound)
// The fused decode step (launch_step) runs the same three kernels with the streaming update of
// Eq. infi-dft folded in: A and C either add the step's token(s) to every coefficient on its way through
// and write it back, or -- deferred write-back -- leave the coefficients alone and add the exact
// contribution of the tokens they do not hold yet (see StepUpdate).
#include "attn_step.h"
#include "fft_core.h"

namespace iwdft {

// ------------------------------------------------------------------------------------------ A
// Block size of kernel A: the read-only form streams best with 256 threads; the read-modify-write
// form of the fused step measured ~10 % faster with 512 (206 -> 186 us on 32 x 8 x 2048 bins).
constexpr int qc_threads(bool upd) { return upd ? 512 : 256; }
constexpr int qc_bins(bool upd) { return qc_threads(upd) * 2; }

// grid: (slice * chunks + chunk) * passes + pass.  Lane = two adjacent bins, loop over channels.
// Update modes (fused decode step): every K coefficient first absorbs the pending token(s) (the
// streaming update, Eq. infi-dft in the fixed frame: F += x e^{+j 2 pi k (T-M)/M}), is written back, and
// the updated value feeds qc, so that K coefficients are read once per step instead of twice (needs
// passes == 1).  kPlain with pending tokens: qc[k] += sum_j (q . k_j) e^{j theta_jk} instead.
// Shared memory of one block, in floats: q rows, pending K rows, the dots q . k_j.
constexpr int qc_smem_floats(int GT, int MODE) {
  return GT * kHeadDim + (MODE == kUpdate1 ? 1 : kMaxPend) * kHeadDim + (MODE == kPlain ? kMaxPend : 1) * GT;
}
// The work of logical block `bid` (wave-uniform) with THREADS threads; `sm` holds qc_smem_floats floats.  RL lanes (whole waves) run
// along the bins, THREADS / RL groups of them share the channels; their sums meet in `part` ([THREADS][GT], with several groups).
template <bool BF16, int GT, int MODE, int THREADS, int RL = THREADS>
__device__ __forceinline__ void qc_body(const Params& P, const void* __restrict__ q, float2* __restrict__ qc,
                                        float* __restrict__ pe, int chunks, int passes, const StepUpdate& up,
                                        uint32_t bid, float* sm, v4f* part = nullptr) {
  constexpr bool UPD = MODE != kPlain;
  constexpr int kQcThreads = THREADS, kQcBins = RL * 2, kGroups = THREADS / RL, kChannels = kHeadDim / kGroups;
  constexpr int U = kGroups > 1 ? 16 : 8;  // rows in flight
  static_assert(RL % 64 == 0 && kChannels % U == 0, "");
  float (*qs)[kHeadDim] = (float (*)[kHeadDim])sm;                            // [GT][128]
  float (*xs)[kHeadDim] = qs + GT;                                             // pending K rows
  float (*dq)[GT] = (float (*)[GT])(xs + (MODE == kUpdate1 ? 1 : kMaxPend));   // q . k_j of the pending tokens
  const int pass = bid % passes;
  bid /= passes;
  const int chunk = bid % chunks;
  const int slice = bid / chunks;
  const int spl = P.batch * P.n_kv;
  const int layer = slice / spl;
  const int s = slice - layer * spl;
  const LayerInfo L = P.layers[layer];
  const int g0 = pass * GT;
  const int i0 = chunk * kQcBins + (threadIdx.x % RL) * 2;
  const int d0 = kGroups > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / RL) * kChannels : 0;
  v4f* row = (v4f*)(P.FK + L.coef_off + (int64_t)s * kHeadDim * L.Bp + i0);
  const int64_t stride = L.Bp / 2;
  v4f f[U];
  if constexpr (kGroups > 1) {  // few blocks: the first rows are on their way while the queries are
    if (i0 < L.Bp) {
#pragma unroll
      for (int u = 0; u < U; ++u) f[u] = __builtin_nontemporal_load(row + (d0 + u) * stride);
    }
  }
  for (int e = threadIdx.x; e < GT * kHeadDim; e += kQcThreads) {
    const int g = g0 + e / kHeadDim;
    qs[e / kHeadDim][e % kHeadDim] =
        (g < P.G) ? load_kv<BF16>(q, ((int64_t)slice * P.G + g) * kHeadDim + (e % kHeadDim)) : 0.f;
  }
  __syncthreads();
  if constexpr (MODE == kUpdateN) {
    for (int e = threadIdx.x; e < up.np * kHeadDim; e += kQcThreads)
      xs[e / kHeadDim][e % kHeadDim] = pend_elem<BF16>(P, up, false, slice, e / kHeadDim, e % kHeadDim);
    __syncthreads();
  }
  if constexpr (MODE == kPlain) {
    if (up.np > 0) {  // block-uniform
      // the pending rows go through LDS (coalesced loads, one per element), then one (token, head) dot per thread
      for (int e = threadIdx.x; e < up.np * kHeadDim; e += kQcThreads)
        xs[e / kHeadDim][e % kHeadDim] = pend_elem<BF16>(P, up, false, slice, e / kHeadDim, e % kHeadDim);
      __syncthreads();
      for (int idx = threadIdx.x; idx < up.np * GT; idx += kQcThreads) {
        const int j = idx / GT, g = idx % GT;
        float dot = 0.f;
#pragma unroll 8
        for (int c = 0; c < kHeadDim; ++c) dot += qs[g][c] * xs[j][c];
        dq[j][g] = dot;
      }
      if (chunk == 0 && pass == 0 && up.nk && (int)threadIdx.x < kHeadDim)  // keep the newest pending K row
        store_kv<BF16>(const_cast<void*>(up.xk),
                       (int64_t)slice * up.stride + (int64_t)(up.np - 1) * kHeadDim + threadIdx.x, xs[up.np - 1][threadIdx.x]);
      __syncthreads();
    }
  }
  const int E = P.S + P.R;
  if (chunk == 0 && E > 0) {  // raw scores q . k_e of the exact tokens, one (token, head) per thread
    for (int idx = threadIdx.x; idx < E * GT; idx += kQcThreads) {
      const int e = idx / GT, g = idx % GT;
      if (g0 + g >= P.G) continue;
      const void* kr = exact_row_step<BF16>(P, up, false, slice, e);
      float dot = 0.f;
      for (int c = 0; c < kHeadDim; c += 8) {
        if constexpr (BF16) {
          const uint4 w = *(const uint4*)((const uint16_t*)kr + c);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const uint32_t u = (&w.x)[j];
            dot += qs[g][c + 2 * j] * __uint_as_float(u << 16) + qs[g][c + 2 * j + 1] * __uint_as_float(u & 0xffff0000u);
          }
        } else {
          const float4 w0 = *(const float4*)((const float*)kr + c), w1 = *(const float4*)((const float*)kr + c + 4);
          dot += qs[g][c] * w0.x + qs[g][c + 1] * w0.y + qs[g][c + 2] * w0.z + qs[g][c + 3] * w0.w +
                 qs[g][c + 4] * w1.x + qs[g][c + 5] * w1.y + qs[g][c + 6] * w1.z + qs[g][c + 7] * w1.w;
        }
      }
      pe[((int64_t)slice * P.G + g0 + g) * E + e] = dot;
    }
  }
  if (kGroups == 1 && i0 >= L.Bp) return;
  v4f acc[GT];
#pragma unroll
  for (int g = 0; g < GT; ++g) acc[g] = (v4f)(0.f);
  if (kGroups == 1 || i0 < L.Bp) {
  // twiddles of this lane's two bins; padding entries keep 0 and are not written
  const bool live = i0 < L.nb;
  v4f tw = (v4f)(0.f);
  if (UPD || up.np > 0) tw = lane_twiddles(P, L, i0, up.tsh);
  // kUpdateN: twiddles of the first kTwGroup pending tokens; the later groups are these times w^(8 g)
  constexpr int kTwGroup = 8;
  static_assert(kMaxPend % kTwGroup == 0, "pending tokens are handled in groups");
  v4f twn[MODE == kUpdateN ? kTwGroup : 1];
  v4f w8 = (v4f)(0.f);
  if constexpr (MODE == kUpdateN) {
    const v4f w = lane_twiddles(P, L, i0, 1u);  // one slot further per token
    twn[0] = tw;
#pragma unroll
    for (int j = 1; j < kTwGroup; ++j) twn[j] = cmul2(twn[j - 1], w);
    const v4f w2 = cmul2(w, w), w4 = cmul2(w2, w2);
    w8 = cmul2(w4, w4);
  }
  if constexpr (MODE == kPlain) {
    if (up.np > 0 && d0 == 0) {  // the pending tokens' share of qc
      const v4f w = lane_twiddles(P, L, i0, 1u);
      v4f t = tw;
      for (int j = 0; j < up.np; ++j) {
#pragma unroll
        for (int g = 0; g < GT; ++g) acc[g] += dq[j][g] * t;
        t = cmul2(t, w);
      }
    }
  }
#pragma unroll 1
  for (int d = d0; d < d0 + kChannels; d += U) {
    if (kGroups == 1 || d > d0) {
#pragma unroll
      for (int u = 0; u < U; ++u) f[u] = __builtin_nontemporal_load(row + (d + u) * stride);
    }
    if constexpr (MODE == kUpdate1) {
      float x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = pend_elem<BF16>(P, up, false, slice, 0, d + u);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        f[u] += x[u] * tw;
        if (live) __builtin_nontemporal_store(f[u], row + (d + u) * stride);
      }
    }
    if constexpr (MODE == kUpdateN) {
      v4f shift = (v4f)(0.f);  // w^(8 g) of the current group of 8 tokens
      shift.x = shift.z = 1.f;
#pragma unroll
      for (int g8 = 0; g8 < kMaxPend; g8 += kTwGroup) {
        if (g8 < up.np) {
#pragma unroll
          for (int j = 0; j < kTwGroup; ++j) {
            if (g8 + j < up.np) {
              const v4f t = g8 ? cmul2(twn[j], shift) : twn[j];
#pragma unroll
              for (int u = 0; u < U; ++u) f[u] += xs[g8 + j][d + u] * t;
            }
          }
          shift = cmul2(shift, w8);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (live) __builtin_nontemporal_store(f[u], row + (d + u) * stride);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int g = 0; g < GT; ++g) acc[g] += qs[g][d + u] * f[u];
  }
  }
  if constexpr (kGroups > 1) {
#pragma unroll
    for (int g = 0; g < GT; ++g) part[g * THREADS + threadIdx.x] = acc[g];
    __syncthreads();
    for (int e = threadIdx.x; e < GT * RL; e += kQcThreads) {
      const int g = e / RL, l = e % RL, i = chunk * kQcBins + l * 2;
      if (g0 + g >= P.G || i >= L.Bp) continue;
      v4f sum = part[g * THREADS + l];
#pragma unroll
      for (int k = 1; k < kGroups; ++k) sum += part[g * THREADS + k * RL + l];
      *(v4f*)(qc + L.ws_off + ((int64_t)s * P.G + g0 + g) * L.Bp + i) = sum;
    }
    return;
  }
#pragma unroll
  for (int g = 0; g < GT; ++g)
    if (g0 + g < P.G)
      *(v4f*)(qc + L.ws_off + ((int64_t)s * P.G + g0 + g) * L.Bp + i0) = acc[g];
}

template <bool BF16, int GT, int MODE>
__global__ __launch_bounds__(qc_threads(MODE != kPlain)) void attn_qc_kernel(Params P, const void* __restrict__ q,
                                                            float2* __restrict__ qc, float* __restrict__ pe,
                                                            int chunks, int passes, StepUpdate up) {
  __shared__ float sm[qc_smem_floats(GT, MODE)];
  qc_body<BF16, GT, MODE, qc_threads(MODE != kPlain)>(P, q, qc, pe, chunks, passes, up, blockIdx.x, sm);
}
// The same for few blocks: 128 bins a block and its channels over the waves.  What bounds a call of few slices is the serial chain
// of a thread, 16 rounds of 8 rows and a trip to memory each; here it has two rounds of 16 rows (read-only) or one (update
// modes), the first of them on its way before the queries are.  One slice group of 8, 64 bins, one head, fp32, M = 1024: this
// kernel 13.3 -> 5.6 us, the decode step 23.9 -> 16.2; 64 slices x 1024 bins, 4 heads, read-only step 68 -> 42 us.
constexpr int kQcFewBins = 128;
template <bool BF16, int GT, int MODE>
__global__ __launch_bounds__(qc_threads(MODE != kPlain)) void attn_qc_few_kernel(Params P, const void* __restrict__ q,
                                                                float2* __restrict__ qc, float* __restrict__ pe,
                                                                int chunks, int passes, StepUpdate up) {
  constexpr int THREADS = qc_threads(MODE != kPlain);
  __shared__ float sm[qc_smem_floats(GT, MODE)];
  __shared__ v4f part[GT * THREADS];
  qc_body<BF16, GT, MODE, THREADS, kQcFewBins / 2>(P, q, qc, pe, chunks, passes, up, blockIdx.x, sm, part);
}

// ------------------------------------------------------------------------------------------ C
constexpr int kOutThreads = 256;
// Channels per block: 16, or 8 where 16 channels x 8 query heads of accumulators would leave one wave per SIMD.
// (8 query heads, update modes: 256 registers + spills at 16 channels; measured 11.8 -> 7.5 ms per write-back launch on
// 10240 slices x 1638 bins.  The read-only form is faster with 16.)
constexpr int out_dc(int GT, int MODE) {
  const bool upd = MODE == kUpdate1 || MODE == kUpdateN;
  return (GT == 8 && upd) ? 8 : 16;
}

// logical block: (slice * (128 / channels per block) + dchunk) * passes + pass.  Lane = two adjacent bins; a block walks all
// bins of its slice for 16 channels, so no cross-block reduction is needed.  Hardware block ids are
// dealt round-robin to the 8 XCDs; they are remapped so that the 8 channel chunks of a slice run on
// ONE XCD and fetch the slice's Pn rows into that XCD's L2 once instead of eight times.
// The coefficient loads are ordinary (cacheable) loads on purpose: what they leave in the
// memory-side cache is V state the next append reads first (measured: append 357 -> 326 us on the
// 32 x 8 x 2048-bin workload, this kernel +5 us).
// Update modes (fused decode step): every V coefficient absorbs the pending token(s) on its way through
// (written back, the updated value is what attention uses), so V coefficients are read once per step
// too.  There the state is touched once per step and nothing gains from caching it: streaming
// (non-temporal) loads and stores measured 195 -> 177 us.  kPlain with pending tokens: the output gets
// sum_j ps[j] v_j added at the end, and the loads stream as well (no append follows that could reuse them).
template <bool BF16, int GT, int MODE>
__global__ __launch_bounds__(kOutThreads) void attn_out_kernel(Params P, const float2* __restrict__ Pn,
                                                              void* __restrict__ out, const float* __restrict__ pe,
                                                              int passes, int per_xcd, int total, StepUpdate up) {
  constexpr bool UPD = MODE == kUpdate1 || MODE == kUpdateN;
  constexpr bool PLAIN = !UPD;
  constexpr bool STREAM = MODE != kPlain;  // nothing re-reads the V coefficients soon: bypass the caches
  constexpr int kOutDC = out_dc(GT, MODE);
  constexpr int V = kOutDC * GT;
  constexpr int VR = V > 64 ? 64 : V;  // values per reduction round
  __shared__ float red[kOutThreads / 64][V];
  uint32_t bid = (blockIdx.x & 7u) * (uint32_t)per_xcd + (blockIdx.x >> 3);
  if (bid >= (uint32_t)total) return;
  const int pass = bid % passes;
  bid /= passes;
  const int dc = bid % (kHeadDim / kOutDC);
  const int slice = bid / (kHeadDim / kOutDC);
  const int spl = P.batch * P.n_kv;
  const int layer = slice / spl;
  const int s = slice - layer * spl;
  const LayerInfo L = P.layers[layer];
  const int g0 = pass * GT;
  const int d0 = dc * kOutDC;
  const int64_t stride = L.Bp / 2;
  v4f* Fv = (v4f*)(P.FV + L.coef_off + ((int64_t)s * kHeadDim + d0) * L.Bp);
  const float2* Prow = Pn + L.ws_off + ((int64_t)s * P.G + g0) * L.Bp;

  float acc[V];
#pragma unroll
  for (int v = 0; v < V; ++v) acc[v] = 0.f;
  float xr[MODE == kUpdate1 ? kOutDC : 1];
  if constexpr (MODE == kUpdate1) {
#pragma unroll
    for (int dd = 0; dd < kOutDC; ++dd) xr[dd] = pend_elem<BF16>(P, up, true, slice, 0, d0 + dd);
  }
  __shared__ float xs[MODE == kUpdateN ? kMaxPend : 1][kOutDC];  // pending V rows, this block's channels
  if constexpr (MODE == kUpdateN) {
    for (int e = threadIdx.x; e < up.np * kOutDC; e += kOutThreads)
      xs[e / kOutDC][e % kOutDC] =
          pend_elem<BF16>(P, up, true, slice, e / kOutDC, d0 + (e % kOutDC));
    __syncthreads();
  }

  for (int i0 = threadIdx.x * 2; i0 < L.Bp; i0 += kOutThreads * 2) {
    v4f p[GT];
#pragma unroll
    for (int g = 0; g < GT; ++g)
      p[g] = (g0 + g < P.G) ? *(const v4f*)(Prow + (int64_t)g * L.Bp + i0) : (v4f)(0.f);
    v4f f[kOutDC];
#pragma unroll
    for (int dd = 0; dd < kOutDC; ++dd)
      f[dd] = STREAM ? __builtin_nontemporal_load(Fv + dd * stride + i0 / 2) : Fv[dd * stride + i0 / 2];
    if constexpr (MODE == kUpdateN) {
      if (i0 < L.nb) {  // padding entries are never written
        v4f t = (v4f)(0.f), w = (v4f)(0.f);
        const uint32_t k0 = (uint32_t)P.bins[L.bin_off + i0];
        const float2 a0 = cis_poly(mulmod(k0, up.tsh, P.M, P.Mmask), P.M), b0 = cis_poly(k0, P.M);
        t.x = a0.x, t.y = a0.y, w.x = b0.x, w.y = b0.y;
        if (i0 + 1 < L.nb) {
          const uint32_t k1 = (uint32_t)P.bins[L.bin_off + i0 + 1];
          const float2 a1 = cis_poly(mulmod(k1, up.tsh, P.M, P.Mmask), P.M), b1 = cis_poly(k1, P.M);
          t.z = a1.x, t.w = a1.y, w.z = b1.x, w.w = b1.y;
        }
        for (int j = 0; j < up.np; ++j) {
#pragma unroll
          for (int dd = 0; dd < kOutDC; ++dd) f[dd] += xs[j][dd] * t;
          t = cmul2(t, w);
        }
#pragma unroll
        for (int dd = 0; dd < kOutDC; ++dd) __builtin_nontemporal_store(f[dd], Fv + dd * stride + i0 / 2);
      }
    }
    if constexpr (MODE == kUpdate1) {
      if (i0 < L.nb) {  // padding entries are never written
        v4f tw = (v4f)(0.f);
        const float2 w0 = cis_poly(mulmod((uint32_t)P.bins[L.bin_off + i0], up.tsh, P.M, P.Mmask), P.M);
        tw.x = w0.x;
        tw.y = w0.y;
        if (i0 + 1 < L.nb) {
          const float2 w1 = cis_poly(mulmod((uint32_t)P.bins[L.bin_off + i0 + 1], up.tsh, P.M, P.Mmask), P.M);
          tw.z = w1.x;
          tw.w = w1.y;
        }
#pragma unroll
        for (int dd = 0; dd < kOutDC; ++dd) {
          f[dd] += xr[dd] * tw;
          __builtin_nontemporal_store(f[dd], Fv + dd * stride + i0 / 2);
        }
      }
    }
#pragma unroll
    for (int dd = 0; dd < kOutDC; ++dd)
#pragma unroll
      for (int g = 0; g < GT; ++g)
        acc[dd * GT + g] += f[dd].x * p[g].x - f[dd].y * p[g].y + f[dd].z * p[g].z - f[dd].w * p[g].w;
  }

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int r = 0; r < V / VR; ++r) {
    float part[VR];
#pragma unroll
    for (int v = 0; v < VR; ++v) part[v] = acc[r * VR + v];
    const float tot = wave_reduce_scatter<VR>(part, lane);
    constexpr int rep = 64 / VR;  // lanes holding the same value
    if ((lane % rep) == 0) red[wave][r * VR + lane / rep] = tot;
  }
  // Exact tokens (weights already divided by the softmax sum): every thread takes a share of the tokens for one
  // (channel, head) of the block, so that the rows are fetched side by side instead of one after the other.
  static_assert(V <= kOutThreads && kOutThreads % V == 0, "one or more threads per output value");
  constexpr int kParts = kOutThreads / V;
  __shared__ float exs[kOutThreads];
  const int E = P.S + P.R;
  const int np_plain = PLAIN ? up.np : 0;  // pending tokens of the deferred write-back: rows weighted by kernel B's ps
  if (E + np_plain > 0) {  // block-uniform
    const int v = threadIdx.x % V, part = threadIdx.x / V;
    const int dd = v / GT, g = v % GT;
    float a = 0.f;
    if (g0 + g < P.G) {
      const float* w = pe + ((int64_t)slice * P.G + g0 + g) * E;
      for (int e = part; e < E; e += kParts)
        a += w[e] * load_kv<BF16>(exact_row_step<BF16>(P, up, true, slice, e), d0 + dd);
      if constexpr (PLAIN) {
        const float* sj = up.ps + ((int64_t)slice * P.G + g0 + g) * kMaxPend;
        for (int j = part; j < np_plain; j += kParts) a += sj[j] * pend_elem<BF16>(P, up, true, slice, j, d0 + dd);
      }
    }
    exs[threadIdx.x] = a;
  }
  __syncthreads();
  for (int v = threadIdx.x; v < V; v += kOutThreads) {
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < kOutThreads / 64; ++w) tot += red[w][v];
    const int dd = v / GT, g = v % GT;
    if (g0 + g < P.G) {
      if (E + np_plain > 0) {
#pragma unroll
        for (int part = 0; part < kParts; ++part) tot += exs[part * V + v];
      }
      store_kv<BF16>(out, ((int64_t)slice * P.G + g0 + g) * kHeadDim + d0 + dd, tot);
    }
  }
  if constexpr (PLAIN) {
    if (up.np > 0 && pass == 0) pend_keep<BF16>(P, up, true, slice, d0, kOutDC);  // this block's 16 channels
  }
  if (up.nk && up.ring_slot >= 0 && pass == 0) {
    // The step's token takes the ring slot (K and V, this block's 16 channels) once every read of the old
    // content by this block is done; no other block touches these channels, and kernel A is long finished.
    __syncthreads();
    if (threadIdx.x < kOutDC) {
      const int64_t src = (int64_t)slice * kHeadDim + d0 + threadIdx.x;
      const int64_t dst = ((int64_t)slice * P.R + up.ring_slot) * kHeadDim + d0 + threadIdx.x;
      store_kv<BF16>(P.ringK, dst, load_kv<BF16>(up.nk, src));
      store_kv<BF16>(P.ringV, dst, load_kv<BF16>(up.nv, src));
    }
  }
}

// ------------------------------------------------------------------------------------- B (FFT)
// A value that all lanes share, in scalar registers.
__device__ __forceinline__ float2 wave_uniform(float2 v) {
  return make_float2(__uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v.x))),
                     __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v.y))));
}

// Scores at all M = D N tokens from the grid x (positions 16 t + m of the digit-reversed order) by interpolation, softmax, and the
// weights folded back onto the grid by the same taps (interp.h, time and frequency exchanged: 1 / W multiplies the bins):
//   s[m D + d] = sum_i w(d / D + 3 - i) y[m + i - 3],   z[m + i - 3] += w(d / D + 3 - i) p[m D + d],   i = 0 .. 7.
// A thread takes 16 grid points with the 7 around them, y and z in registers: a token costs 8 multiply-adds per head each way and no
// LDS trip; its eight weights are wave-uniform.  Maximum: a trigonometric polynomial of degree N / 4 is nowhere above the
// largest magnitude on 2 N points divided by cos(pi / 8) (H. Ehlich and K. Zeller, Math. Zeitschrift 86 (1964)), so the tokens d = 0 and D / 2 give it up to
// 0.083 max|s|; where that is more than 2^64 in the weights all tokens are looked at.
// Constants stay out of either direction, where their roundings would spread over the kept bins with those of N points only: the scores
// come in without their mean (the caller's bin 0), and what is folded back is e^s - level, the weight that a token at the mean has; the
// caller adds M level to bin 0.  Error against 64 bits, M = 65536, 1000 bins, flat scores 1.5e-7 -> 1.1e-7, beside a mean of 19 3.0e-7 ->
// 1.0e-7 (attn_fft_kernel: 1.4e-7, 1.6e-7), for two subtractions a token: a decode step of 32 x 8 slices of 131072 tokens 525 -> 530 us.
// Tokens m D + d_lo .. m D + d_hi - 1 enter the sums; the maximum is that of all tokens.
template <int LOGN>
__device__ __forceinline__ void low_softmax(const Params& P, float2* buf, const float* __restrict__ taps, int t, int d_lo,
                                            int d_hi, bool has1, float2 (&x)[16], float2& mx, float2& Z, float2& f, float2& level) {
  constexpr int N = 1 << LOGN, T = fft_threads(LOGN), NWV = T / 64;
  static_assert(T >= 64, "whole waves");
  __shared__ float4 lmax[NWV];
  const int D = (int)(P.M >> LOGN);
  const uint32_t n0 = sample_at<LOGN>(16 * t);
  __syncthreads();  // the last reads of the inverse transform
#pragma unroll
  for (int m = 0; m < 16; ++m) buf[fpad((int)n0 + sample_step<LOGN>(m))] = x[m];
  __syncthreads();
  float2 y[24];  // grid points 16 t - 4 .. 16 t + 19
  {
    const float4 *lo = (const float4*)(buf + 18 * ((t - 1) & (T - 1)) + 12), *own = (const float4*)(buf + 18 * t),
                 *hi = (const float4*)(buf + 18 * ((t + 1) & (T - 1)));
#pragma unroll
    for (int j = 0; j < 12; ++j) {
      const float4 v = j < 2 ? lo[j] : j < 10 ? own[j - 2] : hi[j - 10];
      y[2 * j] = make_float2(v.x, v.y);
      y[2 * j + 1] = make_float2(v.z, v.w);
    }
  }
  auto score = [&](const float (&w)[8], int m) {
    float2 s = make_float2(w[0] * y[m + 1].x, w[0] * y[m + 1].y);
#pragma unroll
    for (int i = 1; i < 8; ++i) s = make_float2(fmaf(w[i], y[m + 1 + i].x, s.x), fmaf(w[i], y[m + 1 + i].y, s.y));
    return s;
  };
  float2 lm = make_float2(-INFINITY, -INFINITY);
  float la = 0.f;
  auto scan = [&](int d) {
    float w[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = taps[8 * d + i];
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      const float2 s = score(w, m);
      lm = make_float2(fmaxf(lm.x, s.x), fmaxf(lm.y, s.y));
      la = fmaxf(la, fmaxf(fabsf(s.x), fabsf(s.y)));
    }
  };
  auto block_max = [&] {
    auto max2 = [](float a, float b) { return fmaxf(a, b); };
    lm = make_float2(wave_reduce(lm.x, max2), wave_reduce(lm.y, max2));
    la = wave_reduce(la, max2);
    if constexpr (NWV > 1) {
      if ((t & 63) == 0) lmax[t >> 6] = make_float4(lm.x, lm.y, la, 0.f);
      __syncthreads();
#pragma unroll
      for (int v = 0; v < NWV; ++v) {
        const float4 o = lmax[v];
        lm = make_float2(fmaxf(lm.x, o.x), fmaxf(lm.y, o.y));
        la = fmaxf(la, o.z);
      }
    }
  };
#pragma unroll 1
  for (int d = 0; d < D; d += D / 2) scan(d);
  block_max();
  if (!(0.083f * la <= 64.f)) {  // block-uniform
#pragma unroll 1
    for (int d = 0; d < D; ++d) scan(d);
    __syncthreads();
    block_max();
  }
  const float2 mn = make_float2(fmaxf(mx.x, lm.x), fmaxf(mx.y, lm.y));
  f = make_float2(__builtin_amdgcn_exp2f(mx.x - mn.x), __builtin_amdgcn_exp2f(mx.y - mn.y));
  mx = mn;
  level = wave_uniform(make_float2(__builtin_amdgcn_exp2f(-mn.x), has1 ? __builtin_amdgcn_exp2f(-mn.y) : 0.f));
  float2 z[23], ls = make_float2(0.f, 0.f);  // grid points 16 t - 3 .. 16 t + 19
#pragma unroll
  for (int j = 0; j < 23; ++j) z[j] = make_float2(0.f, 0.f);
#pragma unroll 1
  for (int d = d_lo; d < d_hi; ++d) {
    float w[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = taps[8 * d + i];
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      const float2 s = score(w, m);
      const float2 e = make_float2(__builtin_amdgcn_exp2f(s.x - mn.x), has1 ? __builtin_amdgcn_exp2f(s.y - mn.y) : 0.f);
      ls = cadd(ls, e);
      const float2 v = csub(e, level);
#pragma unroll
      for (int i = 0; i < 8; ++i) z[m + i] = make_float2(fmaf(w[i], v.x, z[m + i].x), fmaf(w[i], v.y, z[m + i].y));
    }
  }
  Z = make_float2(Z.x * f.x + ls.x, Z.y * f.y + ls.y);
  // Grid point g lies at position g + 3; the last seven belong to the next thread's sixteen.
#pragma unroll
  for (int m = 0; m < 16; ++m) x[m] = z[m];
  __syncthreads();  // one wave: its own barrier ahead of the overwriting
  write16(buf, t, x);
  __syncthreads();
  float2* nxt = buf + 18 * ((t + 1) & (T - 1));
#pragma unroll
  for (int j = 0; j < 7; ++j) nxt[j] = cadd(nxt[j], z[16 + j]);
  __syncthreads();
#pragma unroll
  for (int m = 0; m < 16; ++m) x[m] = buf[fpad(((int)n0 + sample_step<LOGN>(m) + 3) & (N - 1))];
  __syncthreads();  // the forward transform writes to other positions
}

// grid: slice * pairs + pair, attn_threads(LOGQ) threads.  Two query heads share one complex transform: head g0 travels in the real
// part, head g0 + 1 in the imaginary part (each head's spectrum is made Hermitian first, so its time-domain signal is
// real).  Time index a = Pb * a' + b: block b of Q = M / Pb samples comes from the spectrum folded modulo Q with twiddle
// e^{j 2 pi k b / M}; softmax runs online across the Pb blocks (MULTI).
// Folding uses no atomics: entries that share a slot are added in successive rounds (host-made schedule in P.fold), which
// also fixes the summation order.
// A thread's 16 scores leave the inverse transform in registers and enter the forward one from there, so that softmax costs
// one barrier (the maximum); the sum stays a partial sum per thread until the end.
// Weights: with one block they are normalised and written as the spectrum is gathered; MULTI keeps the running sums of the
// thread's NBT bins in registers, or (NBT = 0, more than 4096 kept bins) in the output rows themselves -- every bin belongs
// to one thread, which reads back its own earlier store.
// LOW: low frequencies only (see attn_low_kernel): one transform of a grid that carries them, low_softmax between it and the tokens.
// PART: `parts.n` workgroups per pair of heads take their share of the blocks (LOW: of the tokens behind every grid point) each and leave
// sums that are not normalised, see attn_parts.hip.
// The work of logical block `bid` (wave-uniform); buf: fft_lds(LOGQ) float2.
template <int LOGQ, int NBT, bool MULTI, bool LOW = false, bool PART = false>
__device__ __forceinline__ void fft_body(const Params& P, const float2* __restrict__ qc, float2* __restrict__ Pn,
                                         float* __restrict__ pe, float scale, int pairs, int np, uint32_t ptsh,
                                         float* __restrict__ ps, uint32_t bid, float2* buf,
                                         const float* __restrict__ taps = nullptr, const Parts& parts = Parts{}) {
  constexpr int Q = 1 << LOGQ, T = fft_threads(LOGQ), TB = attn_threads(LOGQ), NWV = TB / 64;
  constexpr bool kRegs = MULTI && NBT > 0;  // running sums in registers
  constexpr bool kKeep = kRegs && NBT > 4;  // with the register budget of one workgroup per CU: the inputs stay as well
  constexpr int U = kRegs ? NBT : 4;  // bins whose inputs are fetched together
  static_assert(MULTI || NBT == 0, "one block: nothing to keep");
  static_assert(!LOW || (!MULTI && TB == T), "");
  __shared__ float2 smax[NWV], ssum[NWV];
  __shared__ float pscr[NWV][2 * kMaxPend];
  const TabMem tab{P.tab + tab_base(LOGQ)};
  const int t = threadIdx.x, tx = t & (T - 1);  // TB > T: lanes T .. 63 run lane tx's part of the transforms beside it
  const uint32_t pid = PART ? bid / (uint32_t)parts.n : bid, part = PART ? bid - pid * (uint32_t)parts.n : 0u;
  const int pair = pid % pairs;
  const int slice = pid / pairs;
  const int spl = P.batch * P.n_kv;
  const int layer = slice / spl;
  const int s = slice - layer * spl;
  const LayerInfo L = layer_info(P, layer);
  const int g0 = pair * 2;
  const bool has1 = (g0 + 1) < P.G;
  const uint32_t Pb = MULTI ? (P.M >> LOGQ) : 1u;
  const float2* q0 = qc + L.ws_off + ((int64_t)s * P.G + g0) * L.Bp;
  const float2* q1 = has1 ? q0 + L.Bp : q0;
  float2* o0 = (PART ? parts.rows + (int64_t)part * parts.stride : Pn) + L.ws_off + ((int64_t)s * P.G + g0) * L.Bp;
  float2* o1 = o0 + L.Bp;  // written only if has1
  const int32_t* bins = P.bins + L.bin_off;
  const float* wts = P.weights + L.bin_off;
  const uint16_t* fold = P.fold + L.bin_off;
  // log2(e) is folded into the scores so that softmax can use the bare exp2 instruction;
  // 0.5: each bin is split into k and its mirror.
  const float gain = 0.5f * 1.44269504088896341f * scale * P.gain / (float)P.M;
  auto max2 = [](float a, float b) { return fmaxf(a, b); };
  auto add2 = [](float a, float b) { return a + b; };
  auto block_max = [&](float2 v) {  // other barriers separate its reads from its next writes
    v = make_float2(wave_reduce(v.x, max2), wave_reduce(v.y, max2));
    if constexpr (NWV > 1) {
      if ((t & 63) == 0) smax[t >> 6] = v;
      __syncthreads();
      v = smax[0];
#pragma unroll
      for (int w = 1; w < NWV; ++w) v = make_float2(fmaxf(v.x, smax[w].x), fmaxf(v.y, smax[w].y));
    }
    return v;
  };

  // Exact tokens open the online softmax: their raw scores q . k_e come from kernel A.
  float2 mx = make_float2(-INFINITY, -INFINITY), Z = make_float2(0.f, 0.f);  // Z: this thread's share
  const int E = PART ? 0 : P.S + P.R;
  float* pe0 = pe + ((int64_t)slice * P.G + g0) * E;
  float* pe1 = pe0 + E;
  const float escale = 1.44269504088896341f * scale;  // scores live in log2 units (exp2 softmax)
  if (E > 0) {
    float2 lm = mx;
    for (int e = t; e < E; e += TB) {
      lm.x = fmaxf(lm.x, pe0[e] * escale);
      if (has1) lm.y = fmaxf(lm.y, pe1[e] * escale);
    }
    mx = block_max(lm);
    for (int e = t; e < E; e += TB) {
      Z.x += __builtin_amdgcn_exp2f(pe0[e] * escale - mx.x);
      if (has1) Z.y += __builtin_amdgcn_exp2f(pe1[e] * escale - mx.y);
    }
  }

  // Weights of the output: normalised and with the bin weight; the share of the pending tokens of the fused decode step (not
  // yet inside F_V): token j adds v_j * Re sum_k e^{j theta_jk} Pn[k], summed here, where Pn is at hand.
  float iz0 = 0.f, iz1 = 0.f;
  float sp[2 * kMaxPend];  // [token][head g0, head g0 + 1]
  auto finish = [&](int i, uint32_t k, float2 a0, float2 a1) {
    float2 r0 = make_float2(0.f, 0.f), r1 = r0;  // padding entries are written as zeros: kernel C reads whole rows
    if (i < L.nb) {
      const float w = wts[i];
      r0 = make_float2(a0.x * (w * iz0), -a0.y * (w * iz0));
      r1 = make_float2(a1.x * (w * iz1), -a1.y * (w * iz1));
    }
    if (np > 0) {  // block-uniform
      // hardware sine / cosine (~1e-6 absolute): these are weights of value rows, far inside the tolerance.
      // u_n = Re(tw step^n r) for n = 0 .. np - 1 obeys u_{n+1} = 2 cos(phi) u_n - u_{n-1} (phi = the step's angle):
      // one multiply-add per token and head instead of a complex rotation.  The step's 1e-6 grow with n; the weights of up
      // to 15 tokens are off by 1.4e-6 .. 3.3e-6 (M = 512 .. 131072, fp32, relative 2-norm), against 5e-7 .. 2.1e-6 where
      // every step writes back
      const float2 tw = cis_fast((k * ptsh) & (P.M - 1u), P.M), step = cis_fast(k, P.M), t1 = cmul(tw, step);
      const float c2 = 2.f * step.x;
      float u0 = tw.x * r0.x - tw.y * r0.y, u1 = t1.x * r0.x - t1.y * r0.y;
      float v0 = tw.x * r1.x - tw.y * r1.y, v1 = t1.x * r1.x - t1.y * r1.y;
#pragma unroll
      for (int j = 0; j < kMaxPend; ++j) {
        if (j < np) {
          sp[2 * j] += u0;
          sp[2 * j + 1] += v0;
          const float u2 = c2 * u1 - u0, v2 = c2 * v1 - v0;
          u0 = u1, u1 = u2;
          v0 = v1, v1 = v2;
        }
      }
    }
    o0[i] = r0;
    if (has1) o1[i] = r1;
  };
  auto normalise = [&] {  // behind a barrier that publishes ssum
    float2 z = ssum[0];
#pragma unroll
    for (int w = 1; w < NWV; ++w) z = cadd(z, ssum[w]);
    Z = z;
    const float inv_M = P.gain / (float)P.M;
    iz0 = inv_M / Z.x;
    iz1 = has1 ? inv_M / Z.y : 0.f;
#pragma unroll
    for (int v = 0; v < 2 * kMaxPend; ++v) sp[v] = 0.f;
  };
  auto publish_sum = [&] {
    const float2 z = make_float2(wave_reduce(Z.x, add2), wave_reduce(Z.y, add2));
    if ((t & 63) == 0) ssum[t >> 6] = z;
  };

  float2 A0[kRegs ? NBT : 1], A1[kRegs ? NBT : 1];  // running sums over the blocks
  if constexpr (kRegs) {
#pragma unroll
    for (int j = 0; j < NBT; ++j) A0[j] = A1[j] = make_float2(0.f, 0.f);
  }

  uint32_t fr[U], kj[U];
  float2 y0[U], y1[U], wj[U];
  // Inputs of the bins i0 + T j of this thread: fold schedule (0xff: no round matches), then spectrum entries of the heads.
  auto load_fold = [&](int i0) {
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int i = i0 + j * TB;
      // LOW: no bin above a quarter of the grid, so that only the mirror of bin 0 shares a slot
      if constexpr (LOW) fr[j] = i >= L.nb ? 0xffffu : bins[i] ? 0u : 0xff00u;
      else fr[j] = i < L.nb ? (uint32_t)fold[i] : 0xffffu;
    }
  };
  auto load_in = [&](int i0) {
    float w[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int i = i0 + j * TB, ic = i < L.nb ? i : L.nb - 1;
      kj[j] = (uint32_t)bins[ic];
      w[j] = wts[ic] * gain;
      if constexpr (LOW) w[j] *= P.low_gain[kj[j]];
      y0[j] = q0[ic];
      y1[j] = q1[ic];
    }
#pragma unroll
    for (int j = 0; j < U; ++j) {
      y0[j] = make_float2(y0[j].x * w[j], y0[j].y * w[j]);
      y1[j] = has1 ? make_float2(y1[j].x * w[j], y1[j].y * w[j]) : make_float2(0.f, 0.f);
    }
  };
  auto load_tw = [&] {
#pragma unroll
    for (int j = 0; j < U; ++j) wj[j] = pair_twiddle<LOGQ>(tab.tab, kj[j] & (Q - 1));
  };
  if constexpr (kKeep) {
    load_fold(t);
    load_in(t);
    load_tw();
  }

  const uint32_t b_lo = PART && MULTI ? part * Pb / (uint32_t)parts.n : 0u;
  const uint32_t b_hi = PART && MULTI ? (part + 1) * Pb / (uint32_t)parts.n : Pb;
  // LOW: tokens d_lo .. d_hi - 1 behind every grid point
  const int D = LOW ? (int)(P.M >> LOGQ) : 0;
  const int d_lo = PART && LOW ? (int)part * D / parts.n : 0, d_hi = PART && LOW ? ((int)part + 1) * D / parts.n : D;
  for (uint32_t b = b_lo; b < b_hi; ++b) {
    // The thread index is made opaque per iteration so that the address arithmetic of the transforms is recomputed (a few
    // instructions) instead of being hoisted out of the block loop into long-lived registers.
    int lt = t;
    if (MULTI) asm volatile("" : "+v"(lt));
    const int lx = TB > T ? tx : lt;
    float2 x[16];
#pragma unroll
    for (int m = 0; m < 16; ++m) x[m] = make_float2(0.f, 0.f);
    write16(buf, lx, x);
    __syncthreads();
    auto fold_group = [&](int i0, int round) {
      if constexpr (!kKeep) {
        load_fold(i0);
        bool any = round == 0;
#pragma unroll
        for (int j = 0; j < U; ++j) any |= (fr[j] & 0xffu) == (uint32_t)round || (fr[j] >> 8) == (uint32_t)round;
        if (!any) return;  // few bins share a slot
        load_in(i0);
      }
#pragma unroll
      for (int j = 0; j < U; ++j) {
        float2 z0 = y0[j], z1 = y1[j];
        if (MULTI) {
          const float2 tw = cis_fast((kj[j] * b) & (P.M - 1u), P.M);
          z0 = cmul(z0, tw);
          z1 = cmul(z1, tw);
        }
        const int r = kj[j] & (Q - 1), rm = (Q - r) & (Q - 1);
        if ((fr[j] & 0xffu) == (uint32_t)round) {  //      z0  + j z1
          float2 v = make_float2(z0.x - z1.y, z0.y + z1.x);
          if (r == rm) v = LOW ? make_float2(0.f, 0.f) : make_float2(2.f * z0.x, 2.f * z1.x);  // ... plus the mirror term, same slot
          if (round) v = cadd(v, buf[fpad(r)]);
          buf[fpad(r)] = v;
        }
        if ((fr[j] >> 8) == (uint32_t)round) {     // conj z0  + j conj z1
          float2 v = make_float2(z0.x + z1.y, z1.x - z0.y);
          if (round) v = cadd(v, buf[fpad(rm)]);
          buf[fpad(rm)] = v;
        }
      }
    };
    for (int round = 0; round < (LOW ? 1 : L.fold_rounds); ++round) {
      if constexpr (kRegs) {
        fold_group(lt, round);
      } else {
        for (int i0 = lt; i0 < L.nb; i0 += U * TB) fold_group(i0, round);
      }
      __syncthreads();
    }
    fft_inverse<LOGQ>(buf, tab.tab, lx, x);

    // softmax: real part head g0, imaginary part head g0 + 1
    float2 f, level;
    if constexpr (LOW) {
      float2 mean = make_float2(0.f, 0.f);  // of the scores: bin 0, which the spectrum above leaves out
      if (bins[0] == 0) mean = wave_uniform(make_float2(2.f * gain * wts[0] * q0[0].x, has1 ? 2.f * gain * wts[0] * q1[0].x : 0.f));
      mx = csub(mx, mean);
      low_softmax<LOGQ>(P, buf, taps, lx, d_lo, d_hi, has1, x, mx, Z, f, level);
      mx = cadd(mx, mean);
    } else {
    float2 lm = x[0];
#pragma unroll
    for (int m = 1; m < 16; ++m) lm = make_float2(fmaxf(lm.x, x[m].x), fmaxf(lm.y, x[m].y));
    const float2 bm = block_max(lm);
    const float2 mn = make_float2(fmaxf(mx.x, bm.x), fmaxf(mx.y, bm.y));
    // exp2(-inf) = 0 the first time
    f = make_float2(__builtin_amdgcn_exp2f(mx.x - mn.x), __builtin_amdgcn_exp2f(mx.y - mn.y));
    mx = mn;
    float2 ls = make_float2(0.f, 0.f);
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      x[m] = make_float2(__builtin_amdgcn_exp2f(x[m].x - mn.x), has1 ? __builtin_amdgcn_exp2f(x[m].y - mn.y) : 0.f);
      ls = cadd(ls, x[m]);
    }
    if (TB > T && t >= T) ls = make_float2(0.f, 0.f);  // counted by lane tx
    Z = make_float2(Z.x * f.x + ls.x, Z.y * f.y + ls.y);
    }
    if constexpr (!MULTI) publish_sum();  // read behind the barriers of the transform

    auto fetch_bins = [&](int i0) {
#pragma unroll
      for (int j = 0; j < U; ++j) {
        const int i = i0 + j * TB;
        kj[j] = (uint32_t)bins[i < L.nb ? i : L.nb - 1];
      }
    };
    if constexpr (!kKeep) fetch_bins(pin_index(lt));
    fft_forward<LOGQ>(buf, tab, lx, x, [&](int pass) {  // the first bins' twiddles are fetched while the transform runs
      if constexpr (!kKeep) {
        if (pass == fft_np(LOGQ) - 1) load_tw();
      }
    });
    auto gather = [&](int j, float2& p0, float2& p1) {
      float2 w1, w2;
      spectrum_pair<LOGQ>(buf, kj[j] & (Q - 1), wj[j], w1, w2);
      p0 = make_float2(0.5f * (w1.x + w2.x), 0.5f * (w1.y - w2.y));
      p1 = make_float2(0.5f * (w1.y + w2.y), 0.5f * (w2.x - w1.x));
      if constexpr (LOW) {
        const float g = P.low_gain[kj[j]];
        p0 = make_float2(g * p0.x, g * p0.y);
        p1 = make_float2(g * p1.x, g * p1.y);
        if (kj[j] == 0) {
          const float tokens = PART ? (float)((uint32_t)(d_hi - d_lo) << LOGQ) : (float)P.M;
          p0.x = fmaf(tokens, level.x, p0.x);
          p1.x = fmaf(tokens, level.y, p1.x);
        }
      }
      if constexpr (MULTI) {
        const float2 twc = conjf2(cis_fast((kj[j] * b) & (P.M - 1u), P.M));
        p0 = cmul(twc, p0);
        p1 = cmul(twc, p1);
      }
    };
    if constexpr (kRegs) {
#pragma unroll
      for (int j = 0; j < NBT; ++j) {
        float2 p0, p1;
        gather(j, p0, p1);
        A0[j] = make_float2(fmaf(A0[j].x, f.x, p0.x), fmaf(A0[j].y, f.x, p0.y));
        A1[j] = make_float2(fmaf(A1[j].x, f.y, p1.x), fmaf(A1[j].y, f.y, p1.y));
      }
    } else {
      if constexpr (!MULTI && !PART) normalise();
      const int n = MULTI || PART ? L.nb : L.Bp;
      for (int i0 = lt; i0 < n; i0 += U * TB) {
        if (i0 >= U * TB) {
          fetch_bins(i0);
          load_tw();
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
          const int i = i0 + j * TB;
          if (i >= n) continue;
          float2 p0, p1;
          gather(j, p0, p1);
          if constexpr (!MULTI && !PART) {
            finish(i, kj[j], p0, p1);
          } else {
            if (b > b_lo) {  // this thread's own running sums, scaled to the new maximum
              const float2 a0 = o0[i];
              p0 = make_float2(a0.x * f.x + p0.x, a0.y * f.x + p0.y);
              if (has1) {
                const float2 a1 = o1[i];
                p1 = make_float2(a1.x * f.y + p1.x, a1.y * f.y + p1.y);
              }
            }
            o0[i] = p0;
            if (has1) o1[i] = p1;
          }
        }
      }
    }
    if (MULTI) __syncthreads();
  }

  if constexpr (PART) {
    if constexpr (MULTI) {
      publish_sum();
      __syncthreads();
    }
    if (t == 0) {
      float2 z = ssum[0];
#pragma unroll
      for (int w = 1; w < NWV; ++w) z = cadd(z, ssum[w]);
      parts.stats[bid] = make_float4(mx.x, mx.y, z.x, z.y);
    }
    if constexpr (kRegs) {
#pragma unroll
      for (int j = 0; j < NBT; ++j) {
        const int i = j * TB + t;
        if (i >= L.nb) continue;
        o0[i] = A0[j];
        if (has1) o1[i] = A1[j];
      }
    }
    return;
  }
  if constexpr (MULTI) {
    publish_sum();
    __syncthreads();
    normalise();
    const float2 none = make_float2(0.f, 0.f);
    if constexpr (kRegs) {
#pragma unroll
      for (int j = 0; j < NBT; ++j) {
        const int i = j * TB + t;
        if (i < L.Bp) finish(i, kj[j], A0[j], A1[j]);
      }
    } else {
      for (int i = t; i < L.Bp; i += TB) {
        const bool live = i < L.nb;
        finish(i, live ? (uint32_t)bins[i] : 0u, live ? o0[i] : none, live && has1 ? o1[i] : none);
      }
    }
  }
  if (np > 0) {
    // all 2 * kMaxPend sums over the wave at once: afterwards lane l holds the total of entry l / rep
    const float tot = wave_reduce_scatter<2 * kMaxPend>(sp, t & 63);
    constexpr int rep = 64 / (2 * kMaxPend);  // lanes that end up with the same total
    if ((t & 63) % rep == 0) pscr[t >> 6][(t & 63) / rep] = tot;
    __syncthreads();
    for (int v = t; v < 2 * np; v += TB) {
      float sum = 0.f;
      for (int w = 0; w < NWV; ++w) sum += pscr[w][v];
      const int jp = v >> 1, head = v & 1;
      if (head == 0 || has1) ps[((int64_t)slice * P.G + g0 + head) * kMaxPend + jp] = sum;
    }
  }
  for (int e = t; e < E; e += TB) {  // raw scores -> weights p_e / Z (same thread, same entry)
    pe0[e] = __builtin_amdgcn_exp2f(pe0[e] * escale - mx.x) / Z.x;
    if (has1) pe1[e] = __builtin_amdgcn_exp2f(pe1[e] * escale - mx.y) / Z.y;
  }
}

template <int LOGQ, int NBT, bool MULTI>
__global__ __launch_bounds__(attn_threads(LOGQ), NBT > 4 ? 2 : 4) void attn_fft_kernel(Params P, const float2* __restrict__ qc,
                                                                       float2* __restrict__ Pn, float* __restrict__ pe,
                                                                       float scale, int pairs, int np, uint32_t ptsh,
                                                                       float* __restrict__ ps) {
  extern __shared__ __attribute__((aligned(16))) float2 smem[];
  fft_body<LOGQ, NBT, MULTI>(P, qc, Pn, pe, scale, pairs, np, ptsh, ps, blockIdx.x, smem);
}
// Several workgroups per pair of heads (attn_parts.hip); LOW: as attn_low_kernel.
template <int LOGQ, int NBT, bool LOW>
__global__ __launch_bounds__(attn_threads(LOGQ), NBT > 4 ? 2 : 4) void attn_part_kernel(Params P, const float2* __restrict__ qc,
                                                                        float scale, int pairs, Parts parts) {
  extern __shared__ __attribute__((aligned(16))) float2 smem[];
  fft_body<LOGQ, NBT, !LOW, LOW, true>(P, qc, nullptr, nullptr, scale, pairs, 0, 0u, nullptr, blockIdx.x, smem, P.low_taps, parts);
}

// Long contexts that keep low frequencies only, |k| <= N / 4 on a grid of N = 2^LOGN points, D = M / N tokens apart: see low_softmax.
// What bounds it is the vector ALU, 50 instructions a token and pair of heads (32 of them the multiply-adds), beside the transforms of one
// workgroup per CU.  32 x 8 slices of 131072 tokens, 4096 bins, 4 heads: 300 (attn_fft_kernel, 16 pairs of 8192-point transforms each) -> 150 us, a
// read-only decode step 683 -> 524.
template <int LOGN>
__global__ __launch_bounds__(attn_threads(LOGN), 4) void attn_low_kernel(Params P, const float2* __restrict__ qc,
                                                                        float2* __restrict__ Pn, float* __restrict__ pe,
                                                                        float scale, int pairs, int np, uint32_t ptsh,
                                                                        float* __restrict__ ps,
                                                                        const float* __restrict__ taps) {
  extern __shared__ __attribute__((aligned(16))) float2 smem[];
  fft_body<LOGN, 0, false, true>(P, qc, Pn, pe, scale, pairs, np, ptsh, ps, blockIdx.x, smem, taps);
}

// ----------------------------------------------------------------------------------- A + B
// Kernel-A blocks of one group of slices and kernel-B blocks of ANOTHER group in one launch, dealt to the CUs
// side by side: B's transforms run on the vector ALU while A's blocks wait on HBM.  Nothing inside a launch
// depends on anything else inside it -- the host walks the groups as a pipeline, launch i = A(group i) next to
// B(group i - 1), so B always reads qc rows that an earlier launch on the same stream completed.
// Hardware block ids go round-robin to the 8 XCDs; the role is a function of the per-XCD sequence number, so
// every XCD sees the same even mix (nA8 / nB8 = blocks of either role per XCD, rounded up).
// A runs in its read-only form with 512 threads (1024 bins per block).
constexpr int kAbThreads = fft_threads(kFftMaxLogQ);
template <bool BF16, int GT, int NBT>
__global__ __launch_bounds__(kAbThreads, NBT > 4 ? 2 : 4) void attn_ab_kernel(
    Params P, const void* __restrict__ q, float2* __restrict__ qc, float* __restrict__ pe, int chunks, StepUpdate up,
    float2* __restrict__ Pn, float scale, int pairs, int np, float* __restrict__ ps, uint32_t baseA, uint32_t nA,
    uint32_t nA8, uint32_t baseB, uint32_t nB, uint32_t nB8) {
  extern __shared__ __attribute__((aligned(16))) float2 smem[];
  const uint32_t seq = blockIdx.x >> 3, xcd = blockIdx.x & 7u, tot = nA8 + nB8;
  const uint32_t cb = (uint32_t)(((uint64_t)seq * nB8) / tot), cb1 = (uint32_t)(((uint64_t)(seq + 1) * nB8) / tot);
  if (cb1 > cb) {
    const uint32_t id = (uint32_t)__builtin_amdgcn_readfirstlane((int)(cb * 8 + xcd));
    if (id < nB) fft_body<kFftMaxLogQ, NBT, true>(P, qc, Pn, pe, scale, pairs, np, up.tsh, ps, baseB + id, smem);
  } else {
    const uint32_t id = (uint32_t)__builtin_amdgcn_readfirstlane((int)((seq - cb) * 8 + xcd));
    if (id < nA) qc_body<BF16, GT, kPlain, kAbThreads>(P, q, qc, pe, chunks, 1, up, baseA + id, (float*)smem);
  }
}

// ---------------------------------------------------------------------------------- B (direct)
constexpr int kDirThreads = 256;
constexpr int kDirStage = 1024;

// grid: slice * G + g.  Evaluates the score and weight sums term by term; O(M |B|) per head.
__global__ __launch_bounds__(kDirThreads) void attn_direct_kernel(Params P, const float2* __restrict__ qc,
                                                                 float2* __restrict__ Pn, float* __restrict__ pe,
                                                                 float scale, float* __restrict__ scores) {
  __shared__ float2 Ys[kDirStage];
  __shared__ uint32_t ks[kDirStage];
  __shared__ float redf[kDirThreads / 64];
  const int tid = threadIdx.x;
  const int g = blockIdx.x % P.G;
  const int slice = blockIdx.x / P.G;
  const int spl = P.batch * P.n_kv;
  const int layer = slice / spl;
  const int s = slice - layer * spl;
  const LayerInfo L = P.layers[layer];
  const float2* qrow = qc + L.ws_off + ((int64_t)s * P.G + g) * L.Bp;
  float* sc = scores + (int64_t)blockIdx.x * P.M;
  const float gain = scale * P.gain / (float)P.M;

  for (int c0 = 0; c0 < L.nb; c0 += kDirStage) {
    const int cn = min(kDirStage, L.nb - c0);
    __syncthreads();
    for (int e = tid; e < cn; e += kDirThreads) {
      const float w = P.weights[L.bin_off + c0 + e] * gain;
      const float2 a = qrow[c0 + e];
      Ys[e] = make_float2(a.x * w, a.y * w);
      ks[e] = (uint32_t)P.bins[L.bin_off + c0 + e];
    }
    __syncthreads();
    for (uint32_t a = tid; a < P.M; a += kDirThreads) {
      float acc = c0 ? sc[a] : 0.f;
      for (int e = 0; e < cn; ++e) {
        const float2 w = cis(mulmod(ks[e], a, P.M, P.Mmask), P.M);
        acc += Ys[e].x * w.x - Ys[e].y * w.y;
      }
      sc[a] = acc;
    }
  }
  __syncthreads();
  const int E = P.S + P.R;
  float* per = pe + ((int64_t)slice * P.G + g) * E;  // raw q . k_e from kernel A
  float lm = -INFINITY;
  for (uint32_t a = tid; a < P.M; a += kDirThreads) lm = fmaxf(lm, sc[a]);
  for (int e = tid; e < E; e += kDirThreads) lm = fmaxf(lm, per[e] * scale);
  lm = wave_max(lm);
  if ((tid & 63) == 0) redf[tid >> 6] = lm;
  __syncthreads();
  float mx = redf[0];
  for (int w = 1; w < kDirThreads / 64; ++w) mx = fmaxf(mx, redf[w]);
  __syncthreads();
  float lsum = 0.f;
  for (uint32_t a = tid; a < P.M; a += kDirThreads) {
    const float p = expf(sc[a] - mx);
    sc[a] = p;
    lsum += p;
  }
  for (int e = tid; e < E; e += kDirThreads) lsum += expf(per[e] * scale - mx);
  lsum = wave_sum(lsum);
  if ((tid & 63) == 0) redf[tid >> 6] = lsum;
  __syncthreads();
  float Z = 0.f;
  for (int w = 0; w < kDirThreads / 64; ++w) Z += redf[w];

  for (int e = tid; e < E; e += kDirThreads) per[e] = expf(per[e] * scale - mx) / Z;  // weights p_e / Z
  float2* orow = Pn + L.ws_off + ((int64_t)s * P.G + g) * L.Bp;
  const float inv_M = P.gain / (float)P.M;
  for (int i = tid; i < L.Bp; i += kDirThreads) {
    float2 r = make_float2(0.f, 0.f);
    if (i < L.nb) {
      const uint32_t k = (uint32_t)P.bins[L.bin_off + i];
      float re = 0.f, im = 0.f;
      uint32_t ph = 0;
      for (uint32_t a = 0; a < P.M; ++a) {
        const float2 w = cis(ph, P.M);
        const float p = sc[a];
        re += p * w.x;
        im += p * w.y;  // conj of sum p e^{-j..} = sum p e^{+j..}
        ph += k;
        if (ph >= P.M) ph -= P.M;
      }
      const float c = P.weights[L.bin_off + i] * inv_M / Z;
      r = make_float2(re * c, im * c);
    }
    orow[i] = r;
  }
}

// --------------------------------------------------------------------------------------- host
// Most blocks of attn_qc_few_kernel: beyond these the wider rows of attn_qc_kernel stream better.  Decode step of 64 .. 1024 slices and
// 64 .. 2048 bins against attn_qc_kernel, by blocks: update modes 512: 0.67 .. 0.95, 1024: 0.94 .. 1.04; read-only, 1 or 2 heads 512:
// 0.82 .. 0.96, 1024: 0.97 .. 1.07; 4 heads 2048: 0.91 .. 0.96, 4096: 1.03; 8 heads 1024: 0.81 .. 0.94, 2048: 1.00 .. 1.06.
constexpr uint64_t qc_few_blocks(int GT, bool upd) { return upd || GT <= 2 ? 512 : GT == 4 ? 2048 : 1024; }
constexpr uint32_t kAbMinB = 1024, kAbMaxGroups = 8;  // fewest B blocks per group of slices, most groups
static int heads_per_pass(int G);
static bool attn_is_low(const Params& P) { return P.low_logN != 0; }
bool attn_pipelines(const Params& P, bool use_fft) {
  const int GT = heads_per_pass(P.G);
  const int per_thread = (P.max_Bp + kAbThreads - 1) / kAbThreads;
  return use_fft && !attn_is_low(P) && P.G <= GT && (GT == 4 || GT == 8) && P.M >= 16384u && per_thread > 2 && per_thread <= 8 &&
         (uint64_t)P.n_slices * ((P.G + 1) / 2) >= 2 * kAbMinB && !P.serial_phases;
}
static int heads_per_pass(int G) { return G <= 2 ? G : (G <= 4 ? 4 : 8); }  // 1, 2, 4 or 8; heads beyond G are masked

// up / mode: the fused decode step's pending tokens and what kernels A and C do with them (see StepUpdate).
template <bool BF16>
static hipError_t launch_attn_t(const Params& P, const void* q, void* out, float scale, float2* qc,
                                float2* Pn, float* pe, float* direct_scratch, bool use_fft,
                                const StepUpdate* up, int mode, const Parts& parts, const PhaseEvents* marks, hipStream_t st) {
  const int GT = heads_per_pass(P.G);
  const int passes = (P.G + GT - 1) / GT;
  const StepUpdate u = up ? *up : StepUpdate{nullptr, nullptr, 0, 0, 0, nullptr, nullptr, nullptr, -1};
  const int kQcThreads = qc_threads(mode != kPlain), kQcBins = qc_bins(mode != kPlain);
  const int chunks = (P.max_Bp + kQcBins - 1) / kQcBins;
  const uint64_t gridA = (uint64_t)P.n_slices * chunks * passes;
  const int dcC = out_dc(GT, mode == kPlain && u.np > 0 ? kPlainStream : mode);
  const uint64_t gridC = (uint64_t)P.n_slices * (kHeadDim / dcC) * passes;
  const uint64_t gridBd = (uint64_t)P.n_slices * P.G;
  if (gridA > 0x7fffffffull || gridC > 0x7fffffffull || gridBd > 0x7fffffffull)
    return hipErrorInvalidConfiguration;

#define IWDFT_GT_SWITCH1(KERNEL, MODE, GRID, THREADS, ...)                                               \
  switch (GT) {                                                                                          \
    case 1: KERNEL<BF16, 1, MODE><<<dim3((uint32_t)(GRID)), dim3(THREADS), 0, st>>>(__VA_ARGS__); break;  \
    case 2: KERNEL<BF16, 2, MODE><<<dim3((uint32_t)(GRID)), dim3(THREADS), 0, st>>>(__VA_ARGS__); break;  \
    case 4: KERNEL<BF16, 4, MODE><<<dim3((uint32_t)(GRID)), dim3(THREADS), 0, st>>>(__VA_ARGS__); break;  \
    default: KERNEL<BF16, 8, MODE><<<dim3((uint32_t)(GRID)), dim3(THREADS), 0, st>>>(__VA_ARGS__); break; \
  }
#define IWDFT_GT_SWITCH(KERNEL, GRID, THREADS, ...)                                              \
  if (mode == kUpdate1) { IWDFT_GT_SWITCH1(KERNEL, kUpdate1, GRID, THREADS, __VA_ARGS__) }       \
  else if (mode == kUpdateN) { IWDFT_GT_SWITCH1(KERNEL, kUpdateN, GRID, THREADS, __VA_ARGS__) }  \
  else { IWDFT_GT_SWITCH1(KERNEL, kPlain, GRID, THREADS, __VA_ARGS__) }

  if (u.np > 0 && passes != 1) return hipErrorInvalidValue;  // the fused step needs all heads in one pass
  if (u.np > kMaxPend || (mode == kUpdate1 && u.np != 1) || (mode != kPlain && u.np < 1) ||
      (u.np > 0 && mode == kPlain && (!(use_fft || P.chirp) || !u.ps)))
    return hipErrorInvalidValue;
  const int np_plain = mode == kPlain ? u.np : 0;  // pending tokens kernel B has to weigh
  hipError_t e = hipSuccess;
#define IWDFT_MARK(I)                                            \
  if (marks && (e = hipEventRecord(marks->ev[I], st)) != hipSuccess) return e;
  // Long contexts with many slices: A and B run as a pipeline over groups of slices, each launch holding the
  // A blocks of one group next to the B blocks of the group before (attn_ab_kernel).  Worth it when B is a
  // large share of the step and a group still fills the chip: M >= 16384 and at least kAbMinB B blocks per group;
  // measured (A + B, all slices, ms): 2048 slices x 4096 bins, M = 32768: 2.36 -> 1.9; 10240 x 1638, M = 16384:
  // 6.3 -> 5.5; no gain at M = 8192 (B is 30 us) or with 512 B blocks in all (M = 131072, 256 slices).
  const int pairsB = (P.G + 1) / 2;
  const int per_thread_ab = (P.max_Bp + kAbThreads - 1) / kAbThreads;
  const uint64_t nB_all = (uint64_t)P.n_slices * pairsB;
  const bool pipeline_ab = mode == kPlain && attn_pipelines(P, use_fft);
  if (use_fft && passes == 1 && attn_slice_fits(P, u.np, mode != kPlain)) {
    IWDFT_MARK(0)
    e = launch_attn_slice(P, q, out, scale, u, mode != kPlain, st);
    if (e != hipSuccess) return e;
    IWDFT_MARK(1)
    IWDFT_MARK(2)
    IWDFT_MARK(3)
    return hipSuccess;
  }
  if (pipeline_ab) {
    IWDFT_MARK(0)
    const size_t lds = sizeof(float2) * (size_t)fft_lds(kFftMaxLogQ);
    const int chunksA = (P.max_Bp + 2 * kAbThreads - 1) / (2 * kAbThreads);
    uint32_t groups = (uint32_t)(nB_all / kAbMinB);
    if (groups > kAbMaxGroups) groups = kAbMaxGroups;
    const uint32_t spg = ((uint32_t)P.n_slices + groups - 1) / groups;  // slices per group
    for (uint32_t i = 0; i <= groups; ++i) {
      // A: group i, B: group i - 1
      const uint32_t a0 = i * spg, a1 = i < groups ? (a0 + spg < (uint32_t)P.n_slices ? a0 + spg : (uint32_t)P.n_slices) : a0;
      const uint32_t b0 = i ? (i - 1) * spg : 0, b1 = i ? (b0 + spg < (uint32_t)P.n_slices ? b0 + spg : (uint32_t)P.n_slices) : 0;
      const uint32_t sa = a1 > a0 ? a1 - a0 : 0, sb = b1 > b0 ? b1 - b0 : 0;
      const uint32_t nA = sa * chunksA, nB = sb * pairsB;
      if (nA + nB == 0) continue;
      const uint32_t nA8 = (nA + 7) / 8, nB8 = (nB + 7) / 8;
      const uint32_t grid = (nA8 + nB8) * 8;
#define IWDFT_AB_CASE(GTV, NBT)                                                                          \
  {                                                                                                             \
    static LdsLimit lim;                                                                                        \
    e = lim.ensure((const void*)attn_ab_kernel<BF16, GTV, NBT>, (int)lds);                  \
    if (e != hipSuccess) return e;                                                                              \
    attn_ab_kernel<BF16, GTV, NBT><<<dim3(grid), dim3(kAbThreads), lds, st>>>(             \
        P, q, qc, pe, chunksA, u, Pn, scale, pairsB, np_plain, u.ps, a0 * chunksA, nA, nA8, b0 * pairsB, nB,    \
        nB8);                                                                                                   \
  }
      if (GT == 4) {
        if (per_thread_ab <= 4) IWDFT_AB_CASE(4, 4) else IWDFT_AB_CASE(4, 8)
      } else {
        if (per_thread_ab <= 4) IWDFT_AB_CASE(8, 4) else IWDFT_AB_CASE(8, 8)
      }
#undef IWDFT_AB_CASE
      e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    IWDFT_MARK(1)  // the marks cannot separate A from B here: phase A = the pipeline, phase B = nothing
    IWDFT_MARK(2)
  } else {
  IWDFT_MARK(0)
  const int few = (P.max_Bp + kQcFewBins - 1) / kQcFewBins;
  if ((uint64_t)P.n_slices * few * passes <= qc_few_blocks(GT, mode != kPlain)) {
    IWDFT_GT_SWITCH(attn_qc_few_kernel, (uint64_t)P.n_slices * few * passes, kQcThreads, P, q, qc, pe, few, passes, u)
  } else {
    IWDFT_GT_SWITCH(attn_qc_kernel, gridA, kQcThreads, P, q, qc, pe, chunks, passes, u)
  }
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  IWDFT_MARK(1)
  }

  if (pipeline_ab) {
  } else if (use_fft) {
    int logM = 0;
    while ((1u << logM) < P.M) ++logM;
    const int logQ = logM < kFftMaxLogQ ? logM : kFftMaxLogQ;
    const int pairs = (P.G + 1) / 2;
    const uint32_t gridB = (uint32_t)((uint64_t)P.n_slices * pairs);
#define IWDFT_FFT_CASE(LQ, NBT, MULTI)                                                                    \
  {                                                                                                       \
    constexpr int lds = (int)sizeof(float2) * fft_lds(LQ);                                                \
    static LdsLimit lim;                                                                                  \
    e = lim.ensure((const void*)attn_fft_kernel<LQ, NBT, MULTI>, lds);                                    \
    if (e != hipSuccess) return e;                                                                        \
    attn_fft_kernel<LQ, NBT, MULTI><<<dim3(gridB), dim3(attn_threads(LQ)), lds, st>>>(                     \
        P, qc, Pn, pe, scale, pairs, np_plain, u.tsh, u.ps);                                              \
  }
#define IWDFT_PART_CASE(LQ, NBT, LOW)                                                                     \
  {                                                                                                       \
    constexpr int lds = (int)sizeof(float2) * fft_lds(LQ);                                                \
    static LdsLimit lim;                                                                                  \
    e = lim.ensure((const void*)attn_part_kernel<LQ, NBT, LOW>, lds);                                     \
    if (e != hipSuccess) return e;                                                                        \
    attn_part_kernel<LQ, NBT, LOW><<<dim3(gridB * (uint32_t)parts.n), dim3(attn_threads(LQ)), lds, st>>>( \
        P, qc, scale, pairs, parts);                                                                      \
  }
    if (parts.n > 1) {
      const int per_thread = (P.max_Bp + fft_threads(kFftMaxLogQ) - 1) / fft_threads(kFftMaxLogQ);
      if (attn_is_low(P)) {
        if (P.low_logN == 12) IWDFT_PART_CASE(12, 0, true)
        else if (P.low_logN == 13) IWDFT_PART_CASE(13, 0, true)
        else if (P.low_logN == 14) IWDFT_PART_CASE(14, 0, true)
        else return hipErrorInvalidValue;
      } else if (per_thread <= 2) IWDFT_PART_CASE(kFftMaxLogQ, 2, false)
      else if (per_thread <= 4) IWDFT_PART_CASE(kFftMaxLogQ, 4, false)
      else if (per_thread <= 8) IWDFT_PART_CASE(kFftMaxLogQ, 8, false)
      else IWDFT_PART_CASE(kFftMaxLogQ, 0, false)
      e = hipGetLastError();
      if (e == hipSuccess) e = launch_merge(P, parts, Pn, pe, scale, np_plain, u.tsh, u.ps, st);
      if (e != hipSuccess) return e;
    } else if (attn_is_low(P)) {
#define IWDFT_LOW_CASE(LN)                                                                                \
  case LN: {                                                                                              \
    constexpr int lds = (int)sizeof(float2) * fft_lds(LN);                                                \
    static LdsLimit lim;                                                                                  \
    e = lim.ensure((const void*)attn_low_kernel<LN>, lds);                                                \
    if (e != hipSuccess) return e;                                                                        \
    attn_low_kernel<LN><<<dim3(gridB), dim3(attn_threads(LN)), lds, st>>>(                                \
        P, qc, Pn, pe, scale, pairs, np_plain, u.tsh, u.ps, P.low_taps);                                  \
    break;                                                                                                \
  }
      switch (P.low_logN) {
        IWDFT_LOW_CASE(12)
        IWDFT_LOW_CASE(13)
        IWDFT_LOW_CASE(14)
        default: return hipErrorInvalidValue;
      }
#undef IWDFT_LOW_CASE
#undef IWDFT_PART_CASE
    } else if (logM > logQ) {
      const int per_thread = (P.max_Bp + fft_threads(kFftMaxLogQ) - 1) / fft_threads(kFftMaxLogQ);
      if (per_thread <= 2) IWDFT_FFT_CASE(kFftMaxLogQ, 2, true)
      else if (per_thread <= 4) IWDFT_FFT_CASE(kFftMaxLogQ, 4, true)
      else if (per_thread <= 8) IWDFT_FFT_CASE(kFftMaxLogQ, 8, true)
      else IWDFT_FFT_CASE(kFftMaxLogQ, 0, true)
    } else switch (logQ) {
      case 8: IWDFT_FFT_CASE(8, 0, false) break;
      case 9: IWDFT_FFT_CASE(9, 0, false) break;
      case 10: IWDFT_FFT_CASE(10, 0, false) break;
      case 11: IWDFT_FFT_CASE(11, 0, false) break;
      case 12: IWDFT_FFT_CASE(12, 0, false) break;
      default: IWDFT_FFT_CASE(13, 0, false) break;
    }
#undef IWDFT_FFT_CASE
  } else if (P.chirp) {
    e = launch_attn_chirp(P, qc, Pn, pe, scale, np_plain, u.tsh, u.ps, parts, st);
    if (e != hipSuccess) return e;
  } else {
    attn_direct_kernel<<<dim3((uint32_t)gridBd), dim3(kDirThreads), 0, st>>>(P, qc, Pn, pe, scale, direct_scratch);
  }
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (!pipeline_ab) { IWDFT_MARK(2) }

  const int per_xcd = (int)((gridC + 7) / 8);
  if (mode == kPlain && u.np > 0) {  // deferred write-back: no append follows that could reuse cached V state
    IWDFT_GT_SWITCH1(attn_out_kernel, kPlainStream, (uint64_t)per_xcd * 8, kOutThreads, P, Pn, out, pe, passes, per_xcd,
                     (int)gridC, u)
  } else {
    IWDFT_GT_SWITCH(attn_out_kernel, (uint64_t)per_xcd * 8, kOutThreads, P, Pn, out, pe, passes, per_xcd, (int)gridC, u)
  }
#undef IWDFT_GT_SWITCH
#undef IWDFT_GT_SWITCH1
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  IWDFT_MARK(3)
#undef IWDFT_MARK
  return hipSuccess;
}

hipError_t launch_attn(const Params& P, const void* q, void* out, float scale, float2* qc, float2* Pn,
                       float* pe, float* direct_scratch, bool use_fft, const Parts& parts, const PhaseEvents* marks,
                       hipStream_t st) {
  return P.kv_dtype == 1
             ? launch_attn_t<true>(P, q, out, scale, qc, Pn, pe, direct_scratch, use_fft, nullptr, kPlain, parts, marks, st)
             : launch_attn_t<false>(P, q, out, scale, qc, Pn, pe, direct_scratch, use_fft, nullptr, kPlain, parts, marks, st);
}

bool heads_fit_one_pass(int G) { return (G + heads_per_pass(G) - 1) / heads_per_pass(G) == 1; }
bool step_can_fuse(const Params& P) { return heads_fit_one_pass(P.G); }

hipError_t launch_step(const Params& P, const void* tok_k, const void* tok_v, const void* q, void* out,
                       float scale, float2* qc, float2* Pn, float* pe, void* pend_k, void* pend_v, float* ps,
                       float* direct_scratch, bool use_fft, uint32_t tsh0, uint32_t ring_pos, int pend_before,
                       int write_every, const Parts& parts, const PhaseEvents* marks, hipStream_t st) {
  if (write_every < 1 || write_every > kMaxPend || pend_before < 0 || pend_before >= write_every)
    return hipErrorInvalidValue;
  StepUpdate up{tok_k, tok_v, kHeadDim, tsh0, pend_before + 1, ps, nullptr, nullptr, -1};
  if (P.R > 0 || write_every > 1) {  // the kernels file the step's token themselves (see StepUpdate)
    up.xk = pend_k;
    up.xv = pend_v;
    up.stride = (int64_t)write_every * kHeadDim;
    up.nk = tok_k;
    up.nv = tok_v;
    up.ring_slot = P.R > 0 ? (int)ring_pos : -1;
  }
  const int mode = up.np < write_every ? kPlain : (write_every == 1 ? kUpdate1 : kUpdateN);
  return P.kv_dtype == 1
             ? launch_attn_t<true>(P, q, out, scale, qc, Pn, pe, direct_scratch, use_fft, &up, mode, parts, marks, st)
             : launch_attn_t<false>(P, q, out, scale, qc, Pn, pe, direct_scratch, use_fft, &up, mode, parts, marks, st);
}

}  // namespace iwdft
