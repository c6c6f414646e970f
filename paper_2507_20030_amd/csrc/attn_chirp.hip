// Kernel B of the decode attention (see attn.hip) for M that is not a power of two (e.g. M = context - sink - recent,
// Sec. 4.2.1, which is a power of two only by arrangement): scores, softmax and weights through chirp-z transforms (chirp.h).
#include "chirp.h"
#include "interp.h"

namespace iwdft {

// One workgroup of N / 16 threads, a wave at least, per (slice, pair of query heads: real and imaginary part of one signal).  Q = M up to 8192.
// Longer M run Pb = M / Q blocks (Pb the smallest divisor of M that brings Q down to 8192): time index a = Pb a' + b, block b
// comes from the spectrum folded modulo Q with twiddle e^{j 2 pi k b / M}, softmax runs online across the blocks and the
// running sums of the weights live in the output rows (every bin belongs to one thread, which reads back its own earlier
// store).
// What bounds it is vector arithmetic and the barriers of four N-point transforms per block: half of every input is zero and
// half of every output is not wanted, so the wide stages run on registers, and scores, softmax and weights never leave them.
// 32 x 8 slices, 4 query heads each, M = 8132, 2033 bins: 75 us (134 with one transform of 16384 points by 512 threads, every
// pass through LDS); with the write-back deferred a decode step takes 286 us instead of 510.
// Pending tokens of the deferred write-back enter as in attn_fft_kernel (np, ptsh, ps).  PART: several workgroups share the blocks, see
// attn_parts.hip.
//
// GRID (M <= 2^LOGN, all |frequencies| < 2^LOGN / 4): two transforms of half the length in place of four.  The scores are interpolated from a grid of N points
// and the weights folded back onto it by the same eight taps (interp.h: bins in the place of samples, tokens in that of frequencies; the
// way back is its transpose, gathered per grid point from tables of its own).  The decode step above: 286 -> 250 us.
template <int LOGN, bool GRID, bool PART = false>
__global__ __launch_bounds__(attn_threads(LOGN), 4) void attn_chirp_kernel(Params P, const float2* __restrict__ qc,
                                                                      float2* __restrict__ Pn, float* __restrict__ pe,
                                                                      float scale, int pairs, int np, uint32_t ptsh,
                                                                      float* __restrict__ ps, Parts parts) {
  constexpr int T = fft_threads(LOGN), TB = attn_threads(LOGN), NWV = TB / 64;
  constexpr int SP = T + T / 8;  // distance in LDS of entries T apart
  extern __shared__ __attribute__((aligned(16))) float2 buf[];
  __shared__ float2 smax[NWV], ssum[NWV];
  __shared__ float pscr[NWV][2 * kMaxPend];
  const TabMem tab{P.tab + tab_base(LOGN)};
  const float4* __restrict__ H = P.chirpW;
  const int tid = threadIdx.x, t = tid & (T - 1);  // TB > T: lanes T .. 63 run lane t's part of the transforms beside it
  const uint32_t pid = PART ? blockIdx.x / (uint32_t)parts.n : blockIdx.x, part = PART ? blockIdx.x - pid * (uint32_t)parts.n : 0u;
  const int pair = pid % pairs;
  const int slice = pid / pairs;
  const int spl = P.batch * P.n_kv;
  const int layer = slice / spl;
  const int s = slice - layer * spl;
  const LayerInfo L = layer_info(P, layer);
  const int g0 = pair * 2;
  const bool has1 = (g0 + 1) < P.G;
  const uint32_t M = P.M, Q = GRID ? P.M : P.any_Q, Pb = GRID ? 1u : M / Q;
  const float2* q0 = qc + L.ws_off + ((int64_t)s * P.G + g0) * L.Bp;
  const float2* q1 = has1 ? q0 + L.Bp : q0;
  float2* o0 = (PART ? parts.rows + (int64_t)part * parts.stride : Pn) + L.ws_off + ((int64_t)s * P.G + g0) * L.Bp;
  float2* o1 = o0 + L.Bp;  // written only if has1
  const int32_t* bins = P.bins + L.bin_off;
  const float* wts = P.weights + L.bin_off;
  const uint16_t* fold = P.fold + L.bin_off;
  const float gain = 0.5f * 1.44269504088896341f * scale * P.gain / (float)M;  // log2 units; 0.5: bin + mirror
  const float inv_Mf = 1.0f / (float)M, inv_Q = 1.0f / (float)Q;
  float2* own = buf + fpad(t);  // this thread's entries t + T i at i * SP

  auto wave_op = [&](float v, auto op) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = op(v, __shfl_xor(v, o));
    return v;
  };
  auto max2 = [](float a, float b) { return fmaxf(a, b); };
  auto add2 = [](float a, float b) { return a + b; };
  // Over the workgroup; the barrier of the one separates the reads of the other from its next writes.
  auto block_max = [&](float2 v) {
    v = make_float2(wave_op(v.x, max2), wave_op(v.y, max2));
    if ((tid & 63) == 0) smax[tid >> 6] = v;
    __syncthreads();
    v = smax[0];
    for (int w = 1; w < NWV; ++w) v = make_float2(fmaxf(v.x, smax[w].x), fmaxf(v.y, smax[w].y));
    return v;
  };
  auto block_sum = [&](float2 v) {
    v = make_float2(wave_op(v.x, add2), wave_op(v.y, add2));
    if ((tid & 63) == 0) ssum[tid >> 6] = v;
    __syncthreads();
    v = ssum[0];
    for (int w = 1; w < NWV; ++w) v = cadd(v, ssum[w]);
    return v;
  };

  float2 c[GRID ? 1 : 8];  // chirp of the thread's entries, 0 from Q on
#pragma unroll
  for (int i = 0; i < (GRID ? 0 : 8); ++i) c[i] = (uint32_t)(t + T * i) < Q ? P.chirp[t + T * i] : make_float2(0.f, 0.f);

  // Exact tokens open the softmax (raw scores q . k_e from kernel A).
  float2 mx = make_float2(-INFINITY, -INFINITY), Z = make_float2(0.f, 0.f);
  const int E = PART ? 0 : P.S + P.R;
  float* pe0 = pe + ((int64_t)slice * P.G + g0) * E;
  float* pe1 = pe0 + E;
  const float escale = 1.44269504088896341f * scale;
  if (E > 0) {
    float2 lm = mx;
    for (int e = tid; e < E; e += TB) {
      lm.x = fmaxf(lm.x, pe0[e] * escale);
      if (has1) lm.y = fmaxf(lm.y, pe1[e] * escale);
    }
    mx = block_max(lm);
    float2 ls = make_float2(0.f, 0.f);
    for (int e = tid; e < E; e += TB) {
      ls.x += __builtin_amdgcn_exp2f(pe0[e] * escale - mx.x);
      if (has1) ls.y += __builtin_amdgcn_exp2f(pe1[e] * escale - mx.y);
    }
    Z = block_sum(ls);
  }

  constexpr int U = 4;  // bins whose inputs are fetched together
  const uint32_t b_lo = PART ? part * Pb / (uint32_t)parts.n : 0u, b_hi = PART ? (part + 1) * Pb / (uint32_t)parts.n : Pb;
  for (uint32_t b = b_lo; b < b_hi; ++b) {
    auto block_tw = [&](uint32_t k) {  // e^{j 2 pi k b / M}
      return Pb == 1 ? make_float2(1.f, 0.f) : cis_rev((float)mod_small(k * b, M, inv_Mf) * inv_Mf);
    };
    // Where the entry of slot r lies; GRID: frequency f = r or r - M as sample -f of N, padded so that both consecutive samples and those
    // that consecutive threads transform, 4 or 8 apart, fall into distinct banks.
    auto grid_pad = [](uint32_t n) { return (int)(n + (n >> 3)); };
    auto entry = [&](uint32_t r) {
      if constexpr (GRID) return grid_pad((r <= M / 2 ? 0u - r : M - r) & ((1u << LOGN) - 1u));
      else return fpad((int)r);
    };
    auto slot_of = [&](uint32_t k) { return Pb == 1 ? k : mod_small(k, Q, inv_Q); };
    if constexpr (GRID) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (i < 4 || i >= 12) buf[grid_pad((uint32_t)(t + T * i))] = make_float2(0.f, 0.f);  // the quarters that hold frequencies
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) own[i * SP] = make_float2(0.f, 0.f);
    }
    __syncthreads();
    // Hermitian spectrum of both heads (head g0 real, head g0 + 1 imaginary in time), folded modulo Q.  A slot can receive
    // several terms: successive rounds (host-made schedule).
    for (int round = 0; round < L.fold_rounds; ++round) {
      for (int i0 = tid; i0 < L.nb; i0 += U * TB) {
        uint32_t k[U], fr[U];
        float w[U];
        float2 y0[U], y1[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
          const int i = i0 + j * TB, ic = i < L.nb ? i : L.nb - 1;
          k[j] = (uint32_t)bins[ic];
          fr[j] = i < L.nb ? (uint32_t)fold[ic] : 0xffffu;  // 0xff: no round matches
          w[j] = wts[ic] * gain;
          if constexpr (GRID) w[j] *= P.low_gain[k[j] <= M / 2 ? k[j] : M - k[j]];
          y0[j] = q0[ic];
          y1[j] = q1[ic];
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
          const bool direct = (fr[j] & 0xffu) == (uint32_t)round, mirror = (fr[j] >> 8) == (uint32_t)round;
          if (!direct && !mirror) continue;
          const float2 tw = block_tw(k[j]);
          const float2 z0 = cmul(make_float2(y0[j].x * w[j], y0[j].y * w[j]), tw);
          const float2 z1 = has1 ? cmul(make_float2(y1[j].x * w[j], y1[j].y * w[j]), tw) : make_float2(0.f, 0.f);
          const uint32_t r = slot_of(k[j]), rm = r ? Q - r : 0u;
          if (direct) {  //      z0  + j z1
            float2 v = make_float2(z0.x - z1.y, z0.y + z1.x);
            if (r == rm) v = make_float2(2.f * z0.x, 2.f * z1.x);  // ... plus the mirror term, same slot
            if (round) v = cadd(v, buf[entry(r)]);
            buf[entry(r)] = v;
          }
          if (mirror) {  // conj z0  + j conj z1
            float2 v = make_float2(z0.x + z1.y, z1.x - z0.y);
            if (round) v = cadd(v, buf[entry(rm)]);
            buf[entry(rm)] = v;
          }
        }
      }
      __syncthreads();
    }
    // scores of slot a < Q of this block: real part head g0, imaginary part head g0 + 1; v[i]: slot t + T i, or (GRID) v[2 i] and
    // v[2 i + 1]: tokens t + T i and M - (t + T i)
    constexpr int V = GRID ? 16 : 8;
    float2 v[V];
    auto live = [&](int i) {
      const uint32_t a = (uint32_t)(t + T * (GRID ? i >> 1 : i));
      if constexpr (GRID) return (i & 1) ? a > 0 && 2 * a < M : 2 * a <= M;
      else return a < Q;
    };
    if constexpr (GRID) {
      float2 x[16];
      const uint32_t n0 = sample_at<LOGN>(16 * t);
#pragma unroll
      for (int i = 0; i < 8; ++i)
        x[wing_position(i)] = buf[grid_pad((n0 + ((uint32_t)(i < 4 ? i : i - 8) << (LOGN - 4))) & ((1u << LOGN) - 1u))];
      __syncthreads();
      grid_forward<LOGN>(buf, tab, t, x, 1 << LOGN);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        v[2 * i] = v[2 * i + 1] = make_float2(0.f, 0.f);
        if (live(2 * i)) {
          const uint32_t r = (uint32_t)pin_index(t + T * i);  // keeps the taps of one or two items in registers, not of all
          grid_at(buf, 1 << LOGN, load_taps((const float4*)P.low_taps, r, M), v[2 * i], v[2 * i + 1]);
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = cmul(own[i * SP], c[i]);
      chirp_convolve<LOGN, false>(buf, tab, H, t, v);
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = cmul(v[i], c[i]);
    }
    float2 lm = make_float2(-INFINITY, -INFINITY);
#pragma unroll
    for (int i = 0; i < V; ++i) {
      if (live(i)) {
        lm.x = fmaxf(lm.x, v[i].x);
        lm.y = fmaxf(lm.y, v[i].y);
      }
    }
    const float2 bm = block_max(lm);
    const float2 mn = make_float2(fmaxf(mx.x, bm.x), fmaxf(mx.y, bm.y));
    // exp2(-inf) = 0 the first time
    const float2 f = make_float2(__builtin_amdgcn_exp2f(mx.x - mn.x), __builtin_amdgcn_exp2f(mx.y - mn.y));
    mx = mn;
    float2 ls = make_float2(0.f, 0.f);
#pragma unroll
    for (int i = 0; i < V; ++i) {
      float2 p = make_float2(0.f, 0.f);
      if (live(i))
        p = make_float2(__builtin_amdgcn_exp2f(v[i].x - mn.x), has1 ? __builtin_amdgcn_exp2f(v[i].y - mn.y) : 0.f);
      if (TB == T || tid < T) ls = cadd(ls, p);  // else counted by lane t
      if constexpr (GRID) {
        if (live(i)) {  // the grid was last read ahead of block_max's barrier
          const uint32_t a = (i & 1) ? M - (uint32_t)(t + T * (i >> 1)) : (uint32_t)(t + T * (i >> 1));
          buf[kHalo + a] = p;
          if (a < (uint32_t)kHalo) buf[kHalo + M + a] = p;
          if (a + kHalo >= M) buf[kHalo + a - M] = p;
        }
      } else {
        v[i] = cmul(p, conjf2(c[i]));
      }
    }
    const float2 bs = block_sum(ls);
    Z = make_float2(Z.x * f.x + bs.x, Z.y * f.y + bs.y);
    if constexpr (GRID) {
      constexpr int N = 1 << LOGN;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        float2 &u = v[2 * i], &d = v[2 * i + 1];
        grid_at<true>(buf, (int)M, load_taps(P.grid_taps, (uint32_t)pin_index(t + T * i), N), u, d);
        asm volatile("" : "+v"(u.x), "+v"(u.y), "+v"(d.x), "+v"(d.y));  // one item after the other: 300 registers spilled otherwise
      }
      float2 top = make_float2(0.f, 0.f), unused;
      if (t == 0) grid_at<true>(buf, (int)M, load_taps(P.grid_taps, N / 2, N), top, unused);
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int r = t + T * i;
        buf[fpad(r)] = v[2 * i];
        if (r) buf[fpad(N - r)] = v[2 * i + 1];
      }
      if (t == 0) buf[fpad(N / 2)] = top;
      __syncthreads();
      float2 x[16];
      fft_inverse<LOGN>(buf, tab.tab, t, x);  // entry f of the forward transform is entry -f of the inverse one
      const uint32_t n0 = sample_at<LOGN>(16 * t);
      __syncthreads();
#pragma unroll
      for (int m = 0; m < 16; ++m) {
        const int n = (int)n0 + sample_step<LOGN>(m);
        if (sample_step<LOGN>(m) < N / 4 || sample_step<LOGN>(m) >= 3 * (N / 4)) buf[grid_pad((uint32_t)n)] = x[m];
      }
    } else {
      chirp_convolve<LOGN, true>(buf, tab, H, t, v);
#pragma unroll
      for (int i = 0; i < 8; ++i) own[i * SP] = cmul(v[i], conjf2(c[i]));
    }
    __syncthreads();

    for (int i0 = tid; i0 < L.nb; i0 += U * TB) {
      uint32_t k[U];
#pragma unroll
      for (int j = 0; j < U; ++j) {
        const int i = i0 + j * TB;
        k[j] = (uint32_t)bins[i < L.nb ? i : L.nb - 1];
      }
#pragma unroll
      for (int j = 0; j < U; ++j) {
        const int i = i0 + j * TB;
        if (i >= L.nb) continue;
        const uint32_t r = slot_of(k[j]), rm = r ? Q - r : 0u;
        float2 w1 = buf[entry(r)], w2 = buf[entry(rm)];
        float half = 0.5f;
        if constexpr (GRID) {
          half *= P.low_gain[r <= M / 2 ? r : M - r];
        }
        float2 p0 = make_float2(half * (w1.x + w2.x), half * (w1.y - w2.y));
        float2 p1 = make_float2(half * (w1.y + w2.y), half * (w2.x - w1.x));
        if (Pb > 1) {
          const float2 twc = conjf2(block_tw(k[j]));
          p0 = cmul(twc, p0);
          p1 = cmul(twc, p1);
          if (b > b_lo) {  // this thread's own running sums, scaled to the new maximum
            const float2 a0 = o0[i];
            p0 = make_float2(a0.x * f.x + p0.x, a0.y * f.x + p0.y);
            if (has1) {
              const float2 a1 = o1[i];
              p1 = make_float2(a1.x * f.y + p1.x, a1.y * f.y + p1.y);
            }
          }
        }
        o0[i] = p0;
        if (has1) o1[i] = p1;
      }
    }
    __syncthreads();
  }

  if constexpr (PART) {
    if (tid == 0) parts.stats[blockIdx.x] = make_float4(mx.x, mx.y, Z.x, Z.y);
    return;
  }
  const float inv_M = P.gain / (float)M;
  const float iz0 = inv_M / Z.x, iz1 = has1 ? inv_M / Z.y : 0.f;
  const double inv_Md = 1.0 / (double)M;
  float sp[2 * kMaxPend];  // [token][head g0, head g0 + 1]: Re sum_k e^{j theta_jk} Pn[k] of the pending tokens
#pragma unroll
  for (int j = 0; j < 2 * kMaxPend; ++j) sp[j] = 0.f;
  for (int i = tid; i < L.Bp; i += TB) {  // padding entries are written as zeros: kernel C reads whole rows
    float2 r0 = make_float2(0.f, 0.f), r1 = r0;
    if (i < L.nb) {
      const float w = wts[i];
      const float2 a0 = o0[i];
      r0 = make_float2(a0.x * (w * iz0), -a0.y * (w * iz0));
      if (has1) {
        const float2 a1 = o1[i];
        r1 = make_float2(a1.x * (w * iz1), -a1.y * (w * iz1));
      }
      if (np > 0) {  // block-uniform
        // exact first phase and step, one rotation per token: a token's weight is off by less than 16 roundings, as where the
        // coefficients themselves take the tokens up (kernel A's and C's update modes)
        const uint32_t k = (uint32_t)bins[i];
        const float2 step = cis_exact(k, 1u, M, inv_Md);
        float2 tw = cis_exact(k, ptsh, M, inv_Md);
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
    o0[i] = r0;
    if (has1) o1[i] = r1;
  }
  if (np > 0) {
#pragma unroll
    for (int j = 0; j < 2 * kMaxPend; ++j) {
      if (j < 2 * np) {
        const float tot = wave_op(sp[j], add2);
        if ((tid & 63) == 0) pscr[tid >> 6][j] = tot;
      }
    }
    __syncthreads();
    for (int e = tid; e < 2 * np; e += TB) {
      float sum = 0.f;
      for (int w = 0; w < NWV; ++w) sum += pscr[w][e];
      if ((e & 1) == 0 || has1) ps[((int64_t)slice * P.G + g0 + (e & 1)) * kMaxPend + (e >> 1)] = sum;
    }
  }
  for (int e = tid; e < E; e += TB) {  // raw scores -> weights p_e / Z
    pe0[e] = __builtin_amdgcn_exp2f(pe0[e] * escale - mx.x) / Z.x;
    if (has1) pe1[e] = __builtin_amdgcn_exp2f(pe1[e] * escale - mx.y) / Z.y;
  }
}

hipError_t launch_attn_chirp(const Params& P, const float2* qc, float2* Pn, float* pe, float scale, int np, uint32_t ptsh,
                             float* ps, const Parts& parts, hipStream_t st) {
  const int pairs = (P.G + 1) / 2;
  const uint64_t grid = (uint64_t)P.n_slices * pairs;
  if (grid > 0x7fffffffull || np > kMaxPend) return hipErrorInvalidConfiguration;
#define IWDFT_CHIRP_CASE(LN, GRID)                                                                                            \
  case LN: {                                                                                                                  \
    constexpr int bytes = (int)sizeof(float2) * (GRID ? grid_lds(LN) : fft_lds(LN));                                          \
    static LdsLimit lim;                                                                                                      \
    const hipError_t e = lim.ensure((const void*)attn_chirp_kernel<LN, GRID>, bytes);                                         \
    if (e != hipSuccess) return e;                                                                                            \
    attn_chirp_kernel<LN, GRID><<<dim3((uint32_t)grid), dim3(attn_threads(LN)), bytes, st>>>(P, qc, Pn, pe, scale, pairs, np, \
                                                                                           ptsh, ps, parts);                 \
  } break;
#define IWDFT_CHIRP_PART(LN)                                                                                                  \
  case LN: {                                                                                                                  \
    constexpr int bytes = (int)sizeof(float2) * fft_lds(LN);                                                                  \
    static LdsLimit lim;                                                                                                      \
    const hipError_t e = lim.ensure((const void*)attn_chirp_kernel<LN, false, true>, bytes);                                  \
    if (e != hipSuccess) return e;                                                                                            \
    attn_chirp_kernel<LN, false, true><<<dim3((uint32_t)grid * (uint32_t)parts.n), dim3(attn_threads(LN)), bytes, st>>>(      \
        P, qc, Pn, pe, scale, pairs, np, ptsh, ps, parts);                                                                    \
  } break;
  if (parts.n > 1) {
    switch (P.any_logN) {
      IWDFT_CHIRP_PART(8)
      IWDFT_CHIRP_PART(9)
      IWDFT_CHIRP_PART(10)
      IWDFT_CHIRP_PART(11)
      IWDFT_CHIRP_PART(12)
      IWDFT_CHIRP_PART(13)
      IWDFT_CHIRP_PART(14)
      default: return hipErrorInvalidValue;
    }
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? launch_merge(P, parts, Pn, pe, scale, np, ptsh, ps, st) : e;
  }
  if (P.low_logN) {
    switch (P.low_logN) {
      IWDFT_CHIRP_CASE(12, true)
      IWDFT_CHIRP_CASE(13, true)
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  switch (P.any_logN) {
    IWDFT_CHIRP_CASE(8, false)
    IWDFT_CHIRP_CASE(9, false)
    IWDFT_CHIRP_CASE(10, false)
    IWDFT_CHIRP_CASE(11, false)
    IWDFT_CHIRP_CASE(12, false)
    IWDFT_CHIRP_CASE(13, false)
    IWDFT_CHIRP_CASE(14, false)
    default: return hipErrorInvalidValue;
  }
#undef IWDFT_CHIRP_CASE
#undef IWDFT_CHIRP_PART
  return hipGetLastError();
}

}  // namespace iwdft
