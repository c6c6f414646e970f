// Parts that the decode attention kernels share (attn.hip, attn_slice.hip): reductions over a wave, the exact tokens, the
// tokens of a fused step that the stored coefficients do not hold yet.
#pragma once
#include "common.h"

namespace iwdft {

typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// Row e of the exact tokens of a slice: sink tokens first, then the recent ring (slot order; the
// order is irrelevant to softmax attention as long as K and V use the same one).
template <bool BF16>
__device__ __forceinline__ const void* exact_row(const Params& P, bool value, int slice, int e) {
  constexpr int kElem = BF16 ? 2 : 4;
  const char* base;
  int64_t row;
  if (e < P.S) {
    base = (const char*)(value ? P.sinkV : P.sinkK);
    row = (int64_t)slice * P.S + e;
  } else {
    base = (const char*)(value ? P.ringV : P.ringK);
    row = (int64_t)slice * P.R + (e - P.S);
  }
  return base + row * kHeadDim * kElem;
}

// Tokens of the fused decode step that the stored coefficients do not hold yet (see launch_step):
// row j of a slice is x[slice * stride + j * 128 + channel], j < np, and token j has the slot shift
// (tsh + j) mod M.  The kernels come in three modes:
//   kPlain  : coefficients are only read; the np pending tokens (possibly none) enter the result
//             through rank-np corrections -- F + sum_j x_j e^{j theta_j} is what attention sees,
//   kUpdate1: np == 1, the token is added to every coefficient on its way through, written back,
//   kUpdateN: the same for np <= kMaxPend tokens at once (the deferred write-back of several steps).
constexpr int kPlain = 0, kUpdate1 = 1, kUpdateN = 2;
constexpr int kPlainStream = 3;  // kernel C only: kPlain with streaming (non-temporal) coefficient loads
struct StepUpdate {
  const void* xk;
  const void* xv;
  int64_t stride;
  uint32_t tsh;
  int np;
  float* ps;  // kPlain with np > 0: [slice][query head][kMaxPend], Re sum_k e^{j theta_jk} Pn[k] (from kernel B)
  // Non-null: the step's token has not been filed yet; it is still in the caller's tensors ([slice][128])
  // and the kernels do the filing themselves.  Without a recent window (ring_slot < 0) the token is the
  // newest pending row (np - 1).  With one, the newest pending row is the token that ages out of the
  // window -- still in ring slot `ring_slot` -- and the step's token stands in for that slot among the
  // exact tokens; kernel C writes it there at its end.  In kPlain mode kernel A stores the K row and
  // kernel C the V row of the newest pending token into the pending rows for the steps to come.
  const void* nk;
  const void* nv;
  int ring_slot;
};

// Element `c` of pending row j of a slice (K: value = false, V: value = true).
template <bool BF16>
__device__ __forceinline__ float pend_elem(const Params& P, const StepUpdate& up, bool value, int slice, int j,
                                           int c) {
  if (up.nk && j == up.np - 1) {
    if (up.ring_slot >= 0)
      return load_kv<BF16>(value ? P.ringV : P.ringK, ((int64_t)slice * P.R + up.ring_slot) * kHeadDim + c);
    return load_kv<BF16>(value ? up.nv : up.nk, (int64_t)slice * kHeadDim + c);
  }
  return load_kv<BF16>(value ? up.xv : up.xk, (int64_t)slice * up.stride + j * kHeadDim + c);
}
// Keeps the newest pending token for later steps: row np - 1, channels [c0, c0 + n), one per thread.
template <bool BF16>
__device__ __forceinline__ void pend_keep(const Params& P, const StepUpdate& up, bool value, int slice, int c0,
                                          int n) {
  if (!up.nk || (int)threadIdx.x >= n) return;
  const int c = c0 + threadIdx.x;
  const float x = pend_elem<BF16>(P, up, value, slice, up.np - 1, c);  // exact: a storage-dtype value
  store_kv<BF16>(const_cast<void*>(value ? up.xv : up.xk),
                 (int64_t)slice * up.stride + (int64_t)(up.np - 1) * kHeadDim + c, x);
}
// Row e of the exact tokens during a fused step: the step's token stands in for the ring slot it is
// about to take.
template <bool BF16>
__device__ __forceinline__ const void* exact_row_step(const Params& P, const StepUpdate& up, bool value, int slice,
                                                      int e) {
  if (up.nk && up.ring_slot >= 0 && e == P.S + up.ring_slot)
    return (const char*)(value ? up.nv : up.nk) + (int64_t)slice * kHeadDim * (BF16 ? 2 : 4);
  return exact_row<BF16>(P, value, slice, e);
}

// (a.xy, a.zw) * (b.xy, b.zw): two complex products side by side.
__device__ __forceinline__ v4f cmul2(v4f a, v4f b) {
  v4f r;
  r.x = a.x * b.x - a.y * b.y;
  r.y = a.x * b.y + a.y * b.x;
  r.z = a.z * b.z - a.w * b.w;
  r.w = a.z * b.w + a.w * b.z;
  return r;
}

// Twiddles of a lane's two adjacent bins i0, i0 + 1 for slot shift p: (e^{j 2 pi k0 p / M}, e^{j 2 pi k1 p / M});
// a bin beyond the layer's list gets 0, which keeps padding entries at zero.
__device__ __forceinline__ v4f lane_twiddles(const Params& P, const LayerInfo& L, int i0, uint32_t p) {
  v4f tw = (v4f)(0.f);
  if (i0 < L.nb) {
    const float2 w0 = cis(mulmod((uint32_t)P.bins[L.bin_off + i0], p, P.M, P.Mmask), P.M);
    tw.x = w0.x;
    tw.y = w0.y;
    if (i0 + 1 < L.nb) {
      const float2 w1 = cis(mulmod((uint32_t)P.bins[L.bin_off + i0 + 1], p, P.M, P.Mmask), P.M);
      tw.z = w1.x;
      tw.w = w1.y;
    }
  }
  return tw;
}

// Sum V values per lane over the whole wave; on return lane L holds the total of value
// L >> (6 - log2 V)  (V <= 64, power of two).  Each step halves the number of live values.
template <int CNT, int OFF, int V>
__device__ __forceinline__ void wave_reduce_step(float (&v)[V], int lane) {
  if constexpr (OFF >= 1) {
    if constexpr (CNT > 1) {
      constexpr int half = CNT / 2;
      const bool upper = (lane & OFF) != 0;
#pragma unroll
      for (int i = 0; i < half; ++i) {
        const float send = upper ? v[i] : v[i + half];
        const float keep = upper ? v[i + half] : v[i];
        v[i] = keep + __shfl_xor(send, OFF);
      }
      wave_reduce_step<half, OFF / 2, V>(v, lane);
    } else {
      v[0] += __shfl_xor(v[0], OFF);
      wave_reduce_step<1, OFF / 2, V>(v, lane);
    }
  }
}
template <int V>
__device__ __forceinline__ float wave_reduce_scatter(float (&v)[V], int lane) {
  wave_reduce_step<V, 32, V>(v, lane);
  return v[0];
}

// exp(+j 2 pi p / M) through the hardware sine / cosine (argument in revolutions, exact for the power-of-two M of this
// path; ~1e-6 absolute error: block twiddles of the scores and weights, where 1e-6 is far below the output tolerance).
__device__ __forceinline__ float2 cis_fast(uint32_t p, uint32_t M) {
  const float f = (float)p * rcp_pow2(M);
  return make_float2(__builtin_amdgcn_cosf(f), __builtin_amdgcn_sinf(f));
}
template <typename Op>
__device__ __forceinline__ float wave_reduce(float v, Op op) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = op(v, __shfl_xor(v, o));
  return v;
}

// Decode attention of short contexts, all three phases of a slice in one workgroup (attn_slice.hip).
constexpr int kSliceMaxLds = 152 << 10;
hipError_t launch_attn_slice(const Params& P, const void* q, void* out, float scale, const StepUpdate& up, bool update,
                             hipStream_t st);

}  // namespace iwdft
