// Device-side pieces of the token assignment that more than one translation unit uses (hipcc only).
#pragma once
#include "si_internal.h"

namespace si {

__device__ inline bool route_better(float v, int i, float ov, int oi) {
  // true when (ov, oi) should replace (v, i): larger logit, or equal logit and lower index
  return ov > v || (ov == v && oi < i);
}

// order-preserving map of a float to an unsigned integer; -0 and +0 map to the same key.  A total order, so that exactly
// k lanes get a rank below k whatever the bits are.
__device__ inline uint32_t route_key(float v) {
  const uint32_t u = v == 0.f ? 0u : __float_as_uint(v);
  return (u & 0x80000000u) ? ~u : u | 0x80000000u;
}

// One wave selects the top-k experts of one token (Section II-A: the gating function) on the raw logits, ties to the
// lower expert index, then the softmax over the k selected logits.  E <= 256.  sel (LDS, >= k floats) receives the k
// logits, sel_idx (LDS or global, >= k ints) their experts; both are complete for the wave when the call returns.
// Up to 64 experts: one logit per lane, whose rank is the number of logits before it in the order; E compare-and-count
// steps on a broadcast logit (about 5 instructions each) instead of k butterfly reductions of 12 dependent lane exchanges
// (64 experts, top-8, 2011 tokens: 9.8 -> 6.5 us).  More experts: k rounds of a butterfly arg-max.
__device__ inline void topk_token(const float* __restrict__ l, int E, int k, int lane, int32_t* sel_idx, float* __restrict__ w_out,
                                  float* sel) {
  constexpr int WAVE = 64;
  if (E <= WAVE) {
    const float v = lane < E ? l[lane] : 0.f;
    const uint32_t key = route_key(v);
    int rank = 0;
    for (int j = 0; j < E; ++j) {
      const uint32_t kj = __builtin_amdgcn_readlane(key, j);
      rank += kj > key || (kj == key && j < lane) ? 1 : 0;
    }
    if (lane < E && rank < k) { sel_idx[rank] = lane; sel[rank] = v; }
  } else {
    float v[4];
    unsigned taken = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      int e = lane + WAVE * i;
      v[i] = e < E ? l[e] : 0.f;
      if (e >= E) taken |= 1u << i;
    }
    for (int s = 0; s < k; ++s) {
      float bv = 0.f;
      int bi = 0x7fffffff;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (!(taken & (1u << i))) {
          int e = lane + WAVE * i;
          if (bi == 0x7fffffff || route_better(bv, bi, v[i], e)) { bv = v[i]; bi = e; }
        }
      }
#pragma unroll
      for (int d = 1; d < WAVE; d <<= 1) {
        float ov = __shfl_xor(bv, d, WAVE);
        int oi = __shfl_xor(bi, d, WAVE);
        bool take = (oi != 0x7fffffff) && (bi == 0x7fffffff || route_better(bv, bi, ov, oi));
        if (take) { bv = ov; bi = oi; }
      }
      // every lane now holds the same winner
      if ((bi & (WAVE - 1)) == lane) taken |= 1u << (bi / WAVE);
      if (lane == 0) { sel_idx[s] = bi; sel[s] = bv; }
    }
  }
  // (LDS operations of a wave complete in order: the lanes below read what the lanes above wrote)
  __builtin_amdgcn_wave_barrier();
  __threadfence_block();
  // softmax over the k selected logits; sel[0] is the maximum.  Every slot's lane forms the sum in slot order.
  for (int s = lane; s < k; s += WAVE) {
    const float l0 = sel[0];
    float sum = 0.f;
    for (int i = 0; i < k; ++i) sum += expf(sel[i] - l0);
    w_out[s] = expf(sel[s] - l0) / sum;
  }
}

}  // namespace si
