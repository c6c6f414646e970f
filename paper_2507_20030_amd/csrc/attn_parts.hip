// Decode attention of few slices with a long context: several workgroups share the softmax of a pair of query heads (kernel B), each
// over its own blocks or tokens (attn_part_kernel, attn_chirp_kernel), and leave sums relative to their own maximum; here these become
// the weights of the output, the exact tokens and the tokens of a fused step with them.
#include "attn_step.h"
#include "chirp.h"

namespace iwdft {

// grid: slice * pairs + pair.  What bounds it is latency: a launch, and one trip to memory per kRows parts of a thread's bins; what it
// saves is the serial chain of a whole context in one workgroup.
// POW2: M = 2^m, where the phases of the pending tokens come from the hardware sine and cosine and their weights from a recurrence, as in
// attn_fft_kernel; otherwise as in attn_chirp_kernel.
constexpr int kMergeThreads = 1024;
template <bool POW2>
__global__ __launch_bounds__(kMergeThreads) void attn_merge_kernel(Params P, Parts parts, float2* __restrict__ Pn,
                                                                   float* __restrict__ pe, float scale, int pairs, int np,
                                                                   uint32_t ptsh, float* __restrict__ ps) {
  constexpr int NWV = kMergeThreads / 64, kRows = 4;
  __shared__ float2 smax[NWV], ssum[NWV], fac[kMaxParts];
  __shared__ float pscr[NWV][2 * kMaxPend];
  const int t = threadIdx.x, wave = t >> 6, n = parts.n;
  const int pair = blockIdx.x % pairs, slice = blockIdx.x / pairs;
  const int spl = P.batch * P.n_kv;
  const int layer = slice / spl;
  const int s = slice - layer * spl;
  const LayerInfo L = layer_info(P, layer);
  const int g0 = pair * 2;
  const bool has1 = (g0 + 1) < P.G;
  const int64_t at = L.ws_off + ((int64_t)s * P.G + g0) * L.Bp;
  const int32_t* bins = P.bins + L.bin_off;
  const float* wts = P.weights + L.bin_off;
  auto max2 = [](float a, float b) { return fmaxf(a, b); };
  auto add2 = [](float a, float b) { return a + b; };

  const float4* __restrict__ st = parts.stats + (int64_t)blockIdx.x * n;
  float2 mx = make_float2(-INFINITY, -INFINITY);
  for (int p = 0; p < n; ++p) mx = make_float2(fmaxf(mx.x, st[p].x), fmaxf(mx.y, st[p].y));
  const int E = P.S + P.R;
  float* pe0 = pe + ((int64_t)slice * P.G + g0) * E;
  float* pe1 = pe0 + E;
  const float escale = 1.44269504088896341f * scale;
  float2 Z = make_float2(0.f, 0.f);
  static_assert(kMergeThreads >= 1024, "an exact token per thread");
  float2 raw = mx;  // this thread's exact token
  if (E > 0) {
    if (t < E) raw = make_float2(pe0[t] * escale, has1 ? pe1[t] * escale : 0.f);
    mx = make_float2(wave_reduce(fmaxf(mx.x, raw.x), max2), wave_reduce(has1 ? fmaxf(mx.y, raw.y) : mx.y, max2));
    if ((t & 63) == 0) smax[wave] = mx;
    __syncthreads();
    for (int w = 0; w < NWV; ++w) mx = make_float2(fmaxf(mx.x, smax[w].x), fmaxf(mx.y, smax[w].y));
    raw = t < E ? make_float2(__builtin_amdgcn_exp2f(raw.x - mx.x), has1 ? __builtin_amdgcn_exp2f(raw.y - mx.y) : 0.f)
                : make_float2(0.f, 0.f);
    const float2 z = make_float2(wave_reduce(raw.x, add2), wave_reduce(raw.y, add2));
    if ((t & 63) == 0) ssum[wave] = z;
    __syncthreads();
    for (int w = 0; w < NWV; ++w) Z = cadd(Z, ssum[w]);
  }
  for (int p = 0; p < n; ++p) {
    const float4 v = st[p];
    Z = make_float2(fmaf(v.z, __builtin_amdgcn_exp2f(v.x - mx.x), Z.x), fmaf(v.w, __builtin_amdgcn_exp2f(v.y - mx.y), Z.y));
  }
  if (t < n) {  // what a part's rows are multiplied by
    const float4 v = st[t];
    const float inv_M = P.gain / (float)P.M;
    fac[t] = make_float2(inv_M / Z.x * __builtin_amdgcn_exp2f(v.x - mx.x),
                         has1 ? inv_M / Z.y * __builtin_amdgcn_exp2f(v.y - mx.y) : 0.f);
  }
  __syncthreads();

  const double inv_Md = 1.0 / (double)P.M;
  float sp[2 * kMaxPend];
#pragma unroll
  for (int v = 0; v < 2 * kMaxPend; ++v) sp[v] = 0.f;
  for (int i = t; i < L.Bp; i += kMergeThreads) {
    float2 r0 = make_float2(0.f, 0.f), r1 = r0;  // padding entries are written as zeros
    if (i < L.nb) {
      const float2* __restrict__ row = parts.rows + at + i;
      for (int p0 = 0; p0 < n; p0 += kRows) {
        float2 a0[kRows], a1[kRows];
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
          const float2* __restrict__ x = row + (int64_t)(p0 + u < n ? p0 + u : n - 1) * parts.stride;
          a0[u] = x[0];
          a1[u] = has1 ? x[L.Bp] : make_float2(0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
          if (p0 + u >= n) continue;
          const float2 f = fac[p0 + u];
          r0 = make_float2(fmaf(a0[u].x, f.x, r0.x), fmaf(a0[u].y, -f.x, r0.y));
          r1 = make_float2(fmaf(a1[u].x, f.y, r1.x), fmaf(a1[u].y, -f.y, r1.y));
        }
      }
      const float w = wts[i];
      r0 = make_float2(r0.x * w, r0.y * w);
      r1 = make_float2(r1.x * w, r1.y * w);
      if (np > 0) {  // block-uniform
        const uint32_t k = (uint32_t)bins[i];
        if constexpr (POW2) {
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
        } else {
          const float2 step = cis_exact(k, 1u, P.M, inv_Md);
          float2 tw = cis_exact(k, ptsh, P.M, inv_Md);
#pragma unroll
          for (int j = 0; j < kMaxPend; ++j) {
            if (j < np) {
              sp[2 * j] += tw.x * r0.x - tw.y * r0.y;
              sp[2 * j + 1] += tw.x * r1.x - tw.y * r1.y;
              tw = cmul(tw, step);
            }
          }
        }
      }
    }
    Pn[at + i] = r0;
    if (has1) Pn[at + L.Bp + i] = r1;
  }
  if (np > 0) {
    const float tot = wave_reduce_scatter<2 * kMaxPend>(sp, t & 63);
    constexpr int rep = 64 / (2 * kMaxPend);  // lanes that end up with the same total
    if ((t & 63) % rep == 0) pscr[wave][(t & 63) / rep] = tot;
    __syncthreads();
    if (t < 2 * np) {
      float sum = 0.f;
      for (int w = 0; w < NWV; ++w) sum += pscr[w][t];
      if ((t & 1) == 0 || has1) ps[((int64_t)slice * P.G + g0 + (t & 1)) * kMaxPend + (t >> 1)] = sum;
    }
  }
  if (t < E) {  // raw scores -> weights p_e / Z
    pe0[t] = raw.x / Z.x;
    if (has1) pe1[t] = raw.y / Z.y;
  }
}

hipError_t launch_merge(const Params& P, const Parts& parts, float2* Pn, float* pe, float scale, int np, uint32_t ptsh, float* ps,
                        hipStream_t st) {
  const int pairs = (P.G + 1) / 2;
  const uint64_t grid = (uint64_t)P.n_slices * pairs;
  if (parts.n > kMaxParts || grid > 0x7fffffffull) return hipErrorInvalidConfiguration;
  if (P.Mmask)
    attn_merge_kernel<true><<<dim3((uint32_t)grid), dim3(kMergeThreads), 0, st>>>(P, parts, Pn, pe, scale, pairs, np, ptsh, ps);
  else
    attn_merge_kernel<false><<<dim3((uint32_t)grid), dim3(kMergeThreads), 0, st>>>(P, parts, Pn, pe, scale, pairs, np, ptsh, ps);
  return hipGetLastError();
}

}  // namespace iwdft
