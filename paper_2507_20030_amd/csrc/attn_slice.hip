// Decode attention of short contexts in one launch: a workgroup runs the three phases of attn.hip (scores in the frequency domain,
// softmax through transforms in LDS, output from the V coefficients) for all query heads of one slice, the fused decode step
// included.  Scores, weights and their spectra never leave the workgroup.
#include "attn_step.h"
#include "fft_core.h"

namespace iwdft {
namespace {

constexpr int kThreads = 512;
constexpr int kRows = 8;  // coefficient rows in flight
constexpr int kSliceMany = 96, kCus = 256;
constexpr int slice_pairs(int GT) { return (GT + 1) / 2; }
// Float2 of the transforms' buffers; the partial sums of the scores lie over them.
constexpr int slice_buf(int GT, int logQ) {
  const int b = slice_pairs(GT) * fft_lds(logQ), part = 2 * GT * kThreads;
  return b > part ? b : part;
}
int slice_lds(int GT, int logQ, int np, int E) {
  return (int)sizeof(float2) * slice_buf(GT, logQ) + (int)sizeof(float) * (GT * kHeadDim + 2 * np * kHeadDim + GT * E);
}

// N = 4 or 8 adjacent channels of a token row.
template <int N>
__device__ __forceinline__ void load_channels(bool bf16, const void* row, int c, float (&v)[N]) {
  if (bf16) {
#pragma unroll
    for (int j = 0; j < N; j += 4) {
      const uint2 w = *(const uint2*)((const uint16_t*)row + c + j);
      v[j] = __uint_as_float(w.x << 16), v[j + 1] = __uint_as_float(w.x & 0xffff0000u);
      v[j + 2] = __uint_as_float(w.y << 16), v[j + 3] = __uint_as_float(w.y & 0xffff0000u);
    }
  } else {
#pragma unroll
    for (int j = 0; j < N; j += 4) {
      const float4 a = *(const float4*)((const float*)row + c + j);
      v[j] = a.x, v[j + 1] = a.y, v[j + 2] = a.z, v[j + 3] = a.w;
    }
  }
}
__device__ __forceinline__ const void* exact_row_any(bool bf16, const Params& P, const StepUpdate& up, bool value, int slice,
                                                     int e) {
  return bf16 ? exact_row_step<true>(P, up, value, slice, e) : exact_row_step<false>(P, up, value, slice, e);
}

// What bounds it: few slices, the chain of dependent steps of one workgroup (load, sum, transform, weigh, load, sum); many, HBM and the vector
// ALU side by side, since slices in different phases share a compute unit -- which is what the three kernels cannot do, and why 512 threads and at most
// 128 registers (two workgroups per compute unit).  The next rows are on their way while one set is added; sums over the waves go through
// LDS that the transforms take over, the weights take the place of the spectra.  Decode step, three kernels / this one, us: 8 slices of 1024 tokens,
// 64 bins, one head, fp32 15.9 / 12.1; 1024 slices, 128 bins, 4 heads, bf16, written back 154 / 93, read-only 104 / 60.
//
// grid: one workgroup per slice.  rlog: log2 of the lanes along the bins in phase A (two bins each, 32 .. 512, all of a row), the
// other lanes split the channels.  UPD: the np tokens are added to every coefficient, which is written back; otherwise they enter
// through their shares (see attn.hip).  Needs one fold round per layer, rows of up to 2^LOGQ / 4 bins, all heads in one pass.
template <int LOGQ, int GT, bool UPD>
__global__ __launch_bounds__(kThreads, 4) void attn_slice_kernel(Params P, const void* __restrict__ q, void* __restrict__ out,
                                                                float scale, int rlog, StepUpdate up) {
  constexpr int Q = 1 << LOGQ, T = fft_threads(LOGQ), TB = attn_threads(LOGQ), NWV = TB / 64, PAIRS = slice_pairs(GT);
  constexpr bool kAhead = GT < 8;  // two times kRows rows in flight, as far as the registers go
  constexpr int FB = fft_lds(LOGQ), BPT = Q / 4 / TB > 0 ? Q / 4 / TB : 1;  // kept bins of a thread at most
  static_assert(PAIRS * TB <= kThreads, "");
  extern __shared__ __attribute__((aligned(16))) float2 smem[];
  __shared__ float2 smax[PAIRS][NWV], ssum[PAIRS][NWV];
  __shared__ float dq[kMaxPend][GT];
  __shared__ float pscr[PAIRS][NWV][2 * kMaxPend];
  const bool bf16 = P.kv_dtype == 1;
  const int np = up.np, E = P.S + P.R;
  float (*qs)[kHeadDim] = (float (*)[kHeadDim])(smem + slice_buf(GT, LOGQ));  // [GT]
  float (*xk)[kHeadDim] = qs + GT;                                            // pending rows
  float (*xv)[kHeadDim] = xk + np;
  float* pe = (float*)(xv + np);                                              // [GT][E]
  const int tid = threadIdx.x, wave = tid >> 6, ln = tid & 63;
  const int slice = blockIdx.x;
  const int spl = P.batch * P.n_kv;
  const int layer = slice / spl;
  const int s = slice - layer * spl;
  const LayerInfo L = layer_info(P, layer);
  const int32_t* bins = P.bins + L.bin_off;
  const float* wts = P.weights + L.bin_off;
  const int64_t stride = L.Bp / 2;

  // ---- A
  const int RL = 1 << rlog, groups = kThreads >> rlog, cpg = RL / 4;  // channels of a group of lanes
  const int i0 = (tid & (RL - 1)) * 2, grp = tid >> rlog;
  const bool cols = i0 < L.Bp, live = i0 < L.nb;
  // bins i, i + 1 of a lane; any where there is none
  auto lane_bins = [&](int i, uint32_t (&k)[2]) {
    k[0] = (uint32_t)bins[i < L.nb ? i : L.nb - 1];
    k[1] = (uint32_t)bins[i + 1 < L.nb ? i + 1 : L.nb - 1];
  };
  // e^{j 2 pi k p / M} of a lane's bins, 0 where there is none: padding entries stay zero.  As in the three kernels, K takes them from `cis` and V
  // from the polynomial: a step's error comes back in every later token of the chain, M = 1024, 16 tokens, all bins: with `cis` 2.1e-7 rms, 7.4e-7
  // at most (there, two chains of eight: 2.2e-7, 7.2e-7), with the polynomial 3.0e-7, 1.5e-6.
  auto lane_tw = [&](auto turn, int i, const uint32_t (&k)[2], uint32_t p) {
    const float2 a = turn((k[0] * p) & (Q - 1u)), b = turn((k[1] * p) & (Q - 1u));
    v4f t = (v4f)(0.f);
    if (i < L.nb) t.x = a.x, t.y = a.y;
    if (i + 1 < L.nb) t.z = b.x, t.w = b.y;
    return t;
  };
  auto turn_k = [](uint32_t p) { return cis(p, Q); };
  auto turn_v = [](uint32_t p) { return cis_poly2(p, Q); };
  uint32_t kA[2];
  lane_bins(i0, kA);
  v4f* rowK = (v4f*)(P.FK + L.coef_off + ((int64_t)s * kHeadDim + grp * cpg) * L.Bp + i0);
  v4f f[kRows];
#pragma unroll
  for (int u = 0; u < kRows; ++u) f[u] = cols ? rowK[u * stride] : (v4f)(0.f);

  for (int e = tid; e < GT * kHeadDim; e += kThreads) {
    const int64_t at = ((int64_t)slice * P.G + e / kHeadDim) * kHeadDim + (e % kHeadDim);
    qs[e / kHeadDim][e % kHeadDim] = e / kHeadDim >= P.G ? 0.f : bf16 ? load_kv<true>(q, at) : load_kv<false>(q, at);
  }
  for (int e = tid; e < np * kHeadDim; e += kThreads) {
    const int j = e / kHeadDim, c = e % kHeadDim;
    xk[j][c] = bf16 ? pend_elem<true>(P, up, false, slice, j, c) : pend_elem<false>(P, up, false, slice, j, c);
    xv[j][c] = bf16 ? pend_elem<true>(P, up, true, slice, j, c) : pend_elem<false>(P, up, true, slice, j, c);
  }
  v4f tw = (v4f)(0.f), tw1 = (v4f)(0.f);  // of this lane's bins: the oldest pending token, one slot further
  if (np > 0) {
    tw = lane_tw(turn_k, i0, kA, up.tsh);
    if (np > 1) tw1 = lane_tw(turn_k, i0, kA, 1u);
  }
  __syncthreads();
  if (!UPD && up.nk && tid < 2 * kHeadDim) {  // the newest pending token is kept for the steps to come
    const int c = tid & (kHeadDim - 1);
    const int64_t at = (int64_t)slice * up.stride + (int64_t)(np - 1) * kHeadDim + c;
    void* dst = const_cast<void*>(tid < kHeadDim ? up.xk : up.xv);
    const float x = (tid < kHeadDim ? xk : xv)[np - 1][c];
    if (bf16) store_kv<true>(dst, at, x);
    else store_kv<false>(dst, at, x);
  }
  if (E > 0) {  // raw scores of the exact tokens, eight lanes a token
    constexpr int kLanes = 8, kCh = kHeadDim / kLanes;
    const int c = (tid % kLanes) * kCh;
    for (int e0 = 0; e0 < E; e0 += kThreads / kLanes) {
      const int e = e0 + tid / kLanes;
      float v[kCh];
      const void* kr = exact_row_any(bf16, P, up, false, slice, e < E ? e : E - 1);
#pragma unroll
      for (int j = 0; j < kCh; j += 8) load_channels<8>(bf16, kr, c + j, (float(&)[8])v[j]);
#pragma unroll
      for (int g = 0; g < GT; ++g) {
        float dot = 0.f;
#pragma unroll
        for (int j = 0; j < kCh; ++j) dot = fmaf(qs[g][c + j], v[j], dot);
#pragma unroll
        for (int o = kLanes / 2; o >= 1; o >>= 1) dot += __shfl_xor(dot, o);
        if (e < E && tid % kLanes == 0) pe[g * E + e] = dot;
      }
    }
  }
  if (!UPD && np > 0) {  // q . x_j, four lanes each
    static_assert(GT * kMaxPend * 4 <= kThreads, "");
    const int j = (tid >> 2) / GT, g = (tid >> 2) % GT;
    float dot = 0.f;
    if (j < np) {
#pragma unroll
      for (int c = 0; c < kHeadDim; c += 16) {
        const float4 a = *(const float4*)&qs[g][c + 4 * (tid & 3)], b = *(const float4*)&xk[j][c + 4 * (tid & 3)];
        dot = fmaf(a.x, b.x, fmaf(a.y, b.y, fmaf(a.z, b.z, fmaf(a.w, b.w, dot))));
      }
    }
    dot += __shfl_xor(dot, 1);
    dot += __shfl_xor(dot, 2);
    if ((tid & 3) == 0 && j < np) dq[j][g] = dot;
    __syncthreads();
  }
  v4f acc[GT];
#pragma unroll
  for (int g = 0; g < GT; ++g) acc[g] = (v4f)(0.f);
  if (!UPD && np > 0 && live && grp == 0) {  // the pending tokens' share
    v4f t = tw;
    for (int j = 0; j < np; ++j) {
#pragma unroll
      for (int g = 0; g < GT; ++g) acc[g] += dq[j][g] * t;
      if (np > 1) t = cmul2(t, tw1);
    }
  }
#pragma unroll 1
  for (int r = 0; r < cpg; r += kRows) {
    const int d = grp * cpg + r;
    v4f x[kRows];
    if (!kAhead && r > 0) {
#pragma unroll
      for (int u = 0; u < kRows; ++u) f[u] = cols ? rowK[(r + u) * stride] : (v4f)(0.f);
    }
#pragma unroll
    for (int u = 0; u < kRows; ++u) x[u] = f[u];
    if (kAhead && r + kRows < cpg) {  // the next rows
#pragma unroll
      for (int u = 0; u < kRows; ++u) f[u] = cols ? rowK[(r + kRows + u) * stride] : (v4f)(0.f);
    }
    if constexpr (UPD) {
      v4f t = tw;
      for (int j = 0; j < np; ++j) {
#pragma unroll
        for (int u = 0; u < kRows; ++u) x[u] += xk[j][d + u] * t;
        if (np > 1) t = cmul2(t, tw1);
      }
      if (live) {
#pragma unroll
        for (int u = 0; u < kRows; ++u) rowK[(r + u) * stride] = x[u];
      }
    }
#pragma unroll
    for (int u = 0; u < kRows; ++u)
#pragma unroll
      for (int g = 0; g < GT; ++g) acc[g] += qs[g][d + u] * x[u];
  }
  // sums over the groups; then one thread holds two bins of both heads of a pair
  v4f s0[PAIRS], s1[PAIRS];
  if (groups > 1) {
    v4f* part = (v4f*)smem;
#pragma unroll
    for (int g = 0; g < GT; ++g) part[g * kThreads + tid] = acc[g];
    __syncthreads();
#pragma unroll
    for (int it = 0; it < PAIRS; ++it) {
      const int e = it * kThreads + tid, pair = e >> rlog, l = e & (RL - 1);
      s0[it] = s1[it] = (v4f)(0.f);
      if (pair < PAIRS) {
        for (int k = 0; k < groups; ++k) {
          s0[it] += part[2 * pair * kThreads + (k << rlog) + l];
          if constexpr (GT > 1) s1[it] += part[(2 * pair + 1) * kThreads + (k << rlog) + l];
        }
      }
    }
  } else {
#pragma unroll
    for (int it = 0; it < PAIRS; ++it) s0[it] = acc[2 * it], s1[it] = GT > 1 ? acc[GT > 1 ? 2 * it + 1 : 0] : (v4f)(0.f);
  }
  __syncthreads();
  for (int i = tid; i < PAIRS * FB / 2; i += kThreads) ((v4f*)smem)[i] = (v4f)(0.f);
  __syncthreads();
  // log2(e) is folded into the scores (exp2 softmax); 0.5: each bin is split into k and its mirror
  const float gain = 0.5f * 1.44269504088896341f * scale * P.gain / (float)Q;
#pragma unroll
  for (int it = 0; it < PAIRS; ++it) {
    const int e = it * kThreads + tid, pair = e >> rlog, i = (e & (RL - 1)) * 2;
    if (pair >= PAIRS) continue;
    float2* buf = smem + pair * FB;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if (i + b >= L.nb) continue;
      const uint32_t k = (uint32_t)bins[i + b], km = (Q - k) & (Q - 1);
      const float w = wts[i + b] * gain;
      const float2 z0 = b ? make_float2(s0[it].z * w, s0[it].w * w) : make_float2(s0[it].x * w, s0[it].y * w);
      const float2 z1 = b ? make_float2(s1[it].z * w, s1[it].w * w) : make_float2(s1[it].x * w, s1[it].y * w);
      if (k == km) {
        buf[fpad((int)k)] = make_float2(2.f * z0.x, 2.f * z1.x);
      } else {
        buf[fpad((int)k)] = make_float2(z0.x - z1.y, z0.y + z1.x);   //      z0 + j z1
        buf[fpad((int)km)] = make_float2(z0.x + z1.y, z1.x - z0.y);  // conj z0 + j conj z1
      }
    }
  }
  __syncthreads();

  // ---- C takes 16 channels a wave, R at a time, 128 bins at a time: R rows of step 0 .. 16 / R * chunks - 1
  constexpr int R = GT * (UPD ? 2 : 1) > 4 ? 4 : 8;
  const int c0 = wave * 16, j0 = ln * 2, chunks = (L.Bp + 127) / 128;
  v4f* rowV = (v4f*)(P.FV + L.coef_off + ((int64_t)s * kHeadDim + c0) * L.Bp + j0);
  v4f fv[R];
  uint32_t kV[2];
  auto fetch_v = [&](int h, int ch) {
#pragma unroll
    for (int u = 0; u < R; ++u) fv[u] = ch * 128 + j0 < L.Bp ? rowV[(h * R + u) * stride + ch * 64] : (v4f)(0.f);
    if constexpr (UPD) lane_bins(ch * 128 + j0, kV);
  };

  // ---- B: TB threads per pair of heads, head 2 pair in the real part, 2 pair + 1 in the imaginary one
  const int pair = tid / TB;  // wave-uniform
  const int t = tid % TB, tx = t & (T - 1), bw = t >> 6;
  const int g0 = 2 * pair;
  float2 r[BPT][2];
  if (pair < PAIRS) {
    constexpr int G1 = GT > 1 ? 1 : 0;
    float2* buf = smem + pair * FB;
    const TabMem tab{P.tab + tab_base(LOGQ)};
    float *pe0 = pe + g0 * E, *pe1 = pe0 + G1 * E;
    const float escale = 1.44269504088896341f * scale;
    auto max2 = [](float a, float b) { return fmaxf(a, b); };
    auto add2 = [](float a, float b) { return a + b; };
    float2 x[16];
    fft_inverse<LOGQ>(buf, tab.tab, tx, x);
    float2 mx = x[0];
#pragma unroll
    for (int m = 1; m < 16; ++m) mx = make_float2(fmaxf(mx.x, x[m].x), fmaxf(mx.y, x[m].y));
    for (int e = t; e < E; e += TB) mx = make_float2(fmaxf(mx.x, pe0[e] * escale), fmaxf(mx.y, pe1[e] * escale));
    mx = make_float2(wave_reduce(mx.x, max2), wave_reduce(mx.y, max2));
    if (NWV > 1 && (t & 63) == 0) smax[pair][bw] = mx;
    __syncthreads();  // (1)
    if constexpr (NWV > 1) {
#pragma unroll
      for (int w = 0; w < NWV; ++w) mx = make_float2(fmaxf(mx.x, smax[pair][w].x), fmaxf(mx.y, smax[pair][w].y));
    }
    float2 Z = make_float2(0.f, 0.f);
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      x[m] = make_float2(__builtin_amdgcn_exp2f(x[m].x - mx.x), G1 ? __builtin_amdgcn_exp2f(x[m].y - mx.y) : 0.f);
      Z = cadd(Z, x[m]);
    }
    if (TB > T && t >= T) Z = make_float2(0.f, 0.f);  // counted by lane tx
    for (int e = t; e < E; e += TB) {
      pe0[e] = __builtin_amdgcn_exp2f(pe0[e] * escale - mx.x);
      Z.x += pe0[e];
      if (G1) {
        pe1[e] = __builtin_amdgcn_exp2f(pe1[e] * escale - mx.y);
        Z.y += pe1[e];
      }
    }
    Z = make_float2(wave_reduce(Z.x, add2), wave_reduce(Z.y, add2));
    if ((t & 63) == 0) ssum[pair][bw] = Z;
    uint32_t kj[BPT];
    float2 wj[BPT];
#pragma unroll
    for (int j = 0; j < BPT; ++j) {
      const int i = t + j * TB;
      kj[j] = (uint32_t)bins[i < L.nb ? i : L.nb - 1];
    }
    fft_forward<LOGQ>(buf, tab, tx, x, [&](int pass) {
      if (pass == fft_np(LOGQ) - 1) {
#pragma unroll
        for (int j = 0; j < BPT; ++j) wj[j] = pair_twiddle<LOGQ>(tab.tab, kj[j]);
      }
    });
    Z = ssum[pair][0];
#pragma unroll
    for (int w = 1; w < NWV; ++w) Z = cadd(Z, ssum[pair][w]);
    const float iz0 = P.gain / (float)Q / Z.x, iz1 = G1 ? P.gain / (float)Q / Z.y : 0.f;
    float sp[2 * kMaxPend];  // shares of the pending tokens: [token][head g0, g0 + 1]
#pragma unroll
    for (int v = 0; v < 2 * kMaxPend; ++v) sp[v] = 0.f;
#pragma unroll
    for (int j = 0; j < BPT; ++j) {
      const int i = t + j * TB;
      r[j][0] = r[j][1] = make_float2(0.f, 0.f);
      if (i < L.nb) {
        float2 w1, w2;
        spectrum_pair<LOGQ>(buf, kj[j], wj[j], w1, w2);
        const float w = 0.5f * wts[i];
        r[j][0] = make_float2((w1.x + w2.x) * (w * iz0), (w2.y - w1.y) * (w * iz0));
        if (G1) r[j][1] = make_float2((w1.y + w2.y) * (w * iz1), (w1.x - w2.x) * (w * iz1));
        if (!UPD && np > 0) {  // as in attn_fft_kernel
          const float2 a = cis_fast((kj[j] * up.tsh) & (Q - 1u), Q), step = cis_fast(kj[j], Q), b = cmul(a, step);
          const float c2 = 2.f * step.x;
          float u0 = a.x * r[j][0].x - a.y * r[j][0].y, u1 = b.x * r[j][0].x - b.y * r[j][0].y;
          float v0 = a.x * r[j][1].x - a.y * r[j][1].y, v1 = b.x * r[j][1].x - b.y * r[j][1].y;
#pragma unroll
          for (int n = 0; n < kMaxPend; ++n) {
            if (n < np) {
              sp[2 * n] += u0;
              sp[2 * n + 1] += v0;
              const float u2 = c2 * u1 - u0, v2 = c2 * v1 - v0;
              u0 = u1, u1 = u2;
              v0 = v1, v1 = v2;
            }
          }
        }
      }
    }
    if (!UPD && np > 0) {
      const float tot = wave_reduce_scatter<2 * kMaxPend>(sp, t & 63);
      constexpr int rep = 64 / (2 * kMaxPend);
      if ((t & 63) % rep == 0) pscr[pair][bw][(t & 63) / rep] = tot;
    }
    for (int e = t; e < E; e += TB) {
      pe0[e] *= 1.f / Z.x;
      if (G1) pe1[e] *= 1.f / Z.y;
    }
    fetch_v(0, 0);
  } else {
    fetch_v(0, 0);
#pragma unroll 1
    for (int i = 0; i < fft_inverse_barriers(LOGQ) + 1 + fft_forward_barriers(LOGQ); ++i) __syncthreads();  // (1) and the transforms'
  }
  __syncthreads();  // the weights take the place of the spectra
  if (pair < PAIRS) {
    float2* Pw = smem + pair * FB;  // [2][Bp]
#pragma unroll
    for (int j = 0; j < BPT; ++j) {
      const int i = t + j * TB;
      if (i < L.Bp) {
        Pw[i] = r[j][0];
        if (GT > 1) Pw[L.Bp + i] = r[j][1];
      }
    }
  }
  __syncthreads();

  // ---- C
  constexpr int V = R * GT;
#pragma unroll 1
  for (int h = 0; h < 16 / R; ++h) {
    const int c = c0 + h * R;
    float a[V];
#pragma unroll
    for (int v = 0; v < V; ++v) a[v] = 0.f;
#pragma unroll 1
    for (int ch = 0; ch < chunks; ++ch) {
      const int j = ch * 128 + j0;
      v4f x[R];
#pragma unroll
      for (int u = 0; u < R; ++u) x[u] = fv[u];
      const uint32_t k[2] = {kV[0], kV[1]};
      const bool row_end = ch + 1 == chunks;
      if (!row_end || h + 1 < 16 / R) fetch_v(h + row_end, row_end ? 0 : ch + 1);  // the next step's rows
      if constexpr (UPD) {
        if (j < L.nb) {
          v4f t = lane_tw(turn_v, j, k, up.tsh), w = (v4f)(0.f);
          if (np > 1) w = lane_tw(turn_v, j, k, 1u);
          for (int n = 0; n < np; ++n) {
#pragma unroll
            for (int u = 0; u < R; ++u) x[u] += xv[n][c + u] * t;
            if (np > 1) t = cmul2(t, w);
          }
#pragma unroll
          for (int u = 0; u < R; ++u) rowV[(h * R + u) * stride + ch * 64] = x[u];
        }
      }
      const int jc = j < L.Bp ? j : 0;
#pragma unroll
      for (int g = 0; g < GT; ++g) {
        const v4f p = *(const v4f*)(smem + (g >> 1) * FB + (g & 1) * L.Bp + jc);
#pragma unroll
        for (int u = 0; u < R; ++u)
          a[u * GT + g] += x[u].x * p.x - x[u].y * p.y + x[u].z * p.z - x[u].w * p.w;
      }
    }
    for (int e = ln; e < E; e += 64) {  // exact tokens, one per lane
      float v[R];
      load_channels<R>(bf16, exact_row_any(bf16, P, up, true, slice, e), c, v);
#pragma unroll
      for (int g = 0; g < GT; ++g) {
        const float w = g < P.G ? pe[g * E + e] : 0.f;
#pragma unroll
        for (int u = 0; u < R; ++u) a[u * GT + g] = fmaf(w, v[u], a[u * GT + g]);
      }
    }
    if (!UPD && ln < np) {  // pending tokens, one per lane
#pragma unroll
      for (int g = 0; g < GT; ++g) {
        float w = 0.f;
#pragma unroll
        for (int i = 0; i < NWV; ++i) w += pscr[g >> 1][i][2 * ln + (g & 1)];
#pragma unroll
        for (int u = 0; u < R; ++u) a[u * GT + g] = fmaf(w, xv[ln][c + u], a[u * GT + g]);
      }
    }
    const float tot = wave_reduce_scatter<V>(a, ln);
    constexpr int rep = 64 / V;  // lanes that end up with the same total
    const int v = ln / rep, g = v % GT;
    if (ln % rep == 0 && g < P.G) {
      const int64_t at = ((int64_t)slice * P.G + g) * kHeadDim + c + v / GT;
      if (bf16) store_kv<true>(out, at, tot);
      else store_kv<false>(out, at, tot);
    }
  }
  if (up.nk && up.ring_slot >= 0) {  // the step's token takes its ring slot behind the last read of what was there
    __syncthreads();
    if (tid < 2 * kHeadDim) {
      const int c = tid & (kHeadDim - 1);
      const int64_t src = (int64_t)slice * kHeadDim + c, dst = ((int64_t)slice * P.R + up.ring_slot) * kHeadDim + c;
      void* ring = tid < kHeadDim ? P.ringK : P.ringV;
      const void* tok = tid < kHeadDim ? up.nk : up.nv;
      if (bf16) ((uint16_t*)ring)[dst] = ((const uint16_t*)tok)[src];
      else ((float*)ring)[dst] = ((const float*)tok)[src];
    }
  }
}

}  // namespace

// Where one workgroup per slice beats the three kernels, whether the coefficients come from the caches or from memory.  Figures: how many times
// as fast, three states in turn; where there are two, the second behind other data in the caches.
// - Few slices save two launches and pay with one compute unit's share of the bandwidth.  8 slices, written back, one head: 128 bins 1.41, 1.23; 160 1.11,
//   1.02; 192 1.10, 0.94; 256 1.09, 0.88; four heads, 128 1.18, 1.08, 256 19.9 us / 23.0.  Read only, 256 bins: one head 1.30, 1.01, four 1.14,
//   1.09; eight heads, 128 bins 1.20, 1.15.
// - From kSliceMany slices on the phases of different slices run side by side; long rows want more of them.  Four heads, written back: 512
//   bins, 96 slices 0.80, 128 0.90, 160 1.08, 192 1.05 (256 bins, 96 1.20).  Attention alone behind the append: 512 bins, 112 0.98,
//   128 0.96, 144 1.01; 768, 112 0.93, 144 1.04.  Steps with pending tokens, which follow each other: 768 bins, 96 1.13, 0.96; 1024, 96
//   1.11, 0.87, 128 1.11, 0.98.
// - Written back, states that the caches do not hold gain by short rows only (one head: 384 slices of 512 bins 159 us / 165, 2048 of 150 311 / 311; four
//   heads, 1024 of 1024 784 / 840).
// - Read only, a compute unit holds two workgroups, and where the last round of 2 kCus is nearly empty long rows wait for its bandwidth.  1024 bins,
//   one head: 256 slices 1.11, 320 0.91, 512 1.09, 576 0.93, 1024 1.02.  768 bins, four heads, pending tokens: 272 0.91, 320 0.96, 384 1.08.
//   256 bins, one head, pending tokens: 512 1.28, 576 0.98, 640 0.93, 768 0.94 (two heads 1.03), 896 1.00; 512 bins 512 1.02, 576 0.95, 896 1.02.
bool attn_slice_fits(const Params& P, int np, bool update) {
  if (!P.one_fold || P.M > 4096u || P.G > 8 || P.serial_phases) return false;
  const int GT = P.G <= 2 ? P.G : (P.G <= 4 ? 4 : 8), S = P.n_slices, row = P.max_Bp;
  int logQ = 8;
  while ((1u << logQ) < P.M) ++logQ;
  if ((GT == 8 && logQ == 12) || slice_lds(GT, logQ, np, P.S + P.R) > kSliceMaxLds) return false;
  if (S < kSliceMany) return update ? GT < 8 && row <= 160 && row * GT <= 512 : row <= 256 && row * GT <= 1024;
  if (update) return row <= (GT == 1 ? 160 : 256) || ((row <= 256 || S >= 160) && (int64_t)S * row <= 131072);
  if ((row > 384 && np == 0 && S < 144) || (row > 768 && S < 128)) return false;
  const int slots = 2 * kCus, rounds = (S + slots - 1) / slots;
  const int least = S <= kCus ? 0 : row > 768 ? 85 : row > 512 ? 60 : row > 192 && GT <= 2 && np > 0 && S > slots ? (GT == 1 ? 80 : 70) : 0;
  return S * 100LL >= (int64_t)least * rounds * slots;  // least per cent of the slots filled
}

hipError_t launch_attn_slice(const Params& P, const void* q, void* out, float scale, const StepUpdate& up, bool update,
                             hipStream_t st) {
  const int GT = P.G <= 2 ? P.G : (P.G <= 4 ? 4 : 8);
  int logQ = 8, rlog = 5;
  while ((1u << logQ) < P.M) ++logQ;
  while ((2 << rlog) < P.max_Bp) ++rlog;
  const int lds = slice_lds(GT, logQ, up.np, P.S + P.R);
  hipError_t e = hipSuccess;
#define IWDFT_SLICE1(LQ, GTV, UPD)                                                                       \
  {                                                                                                      \
    static LdsLimit lim;                                                                                 \
    e = lim.ensure((const void*)attn_slice_kernel<LQ, GTV, UPD>, kSliceMaxLds);                          \
    if (e != hipSuccess) return e;                                                                       \
    attn_slice_kernel<LQ, GTV, UPD><<<dim3((uint32_t)P.n_slices), dim3(kThreads), (size_t)lds, st>>>(    \
        P, q, out, scale, rlog, up);                                                                         \
  }
#define IWDFT_SLICE(LQ, GTV)             \
  {                                      \
    if (update) IWDFT_SLICE1(LQ, GTV, true) else IWDFT_SLICE1(LQ, GTV, false) \
  }                                      \
  break;
#define IWDFT_SLICE_Q(LQ)                  \
  case LQ:                                 \
    switch (GT) {                          \
      case 1: IWDFT_SLICE(LQ, 1)           \
      case 2: IWDFT_SLICE(LQ, 2)           \
      case 4: IWDFT_SLICE(LQ, 4)           \
      default: IWDFT_SLICE(LQ, 8)          \
    }                                      \
    break;
  switch (logQ) {
    IWDFT_SLICE_Q(8)
    IWDFT_SLICE_Q(9)
    IWDFT_SLICE_Q(10)
    IWDFT_SLICE_Q(11)
    default:
      switch (GT) {
        case 1: IWDFT_SLICE(12, 1)
        case 2: IWDFT_SLICE(12, 2)
        case 4: IWDFT_SLICE(12, 4)
        default: return hipErrorInvalidValue;
      }
  }
#undef IWDFT_SLICE_Q
#undef IWDFT_SLICE
#undef IWDFT_SLICE1
  return hipGetLastError();
}

}  // namespace iwdft
