// Device-side pieces of the token assignment that more than one translation unit uses (hipcc only).
#pragma once
#include "si_internal.h"

#include <type_traits>

namespace si {

// order-preserving map of a float to an unsigned integer; -0 and +0 map to the same key.  A total order, so that exactly
// k lanes get a rank below k whatever the bits are.
__device__ inline uint32_t route_key(float v) {
  const uint32_t u = v == 0.f ? 0u : __float_as_uint(v);
  return (u & 0x80000000u) ? ~u : u | 0x80000000u;
}

__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  auto dpp = [](uint32_t x, auto ctrl) { return max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, x, decltype(ctrl)::value, 0xf, 0xf, false)); };
  v = dpp(v, std::integral_constant<int, 0x121>{});  // rotations of rows of 16 lanes by 1, 2, 4, 8
  v = dpp(v, std::integral_constant<int, 0x122>{});
  v = dpp(v, std::integral_constant<int, 0x124>{});
  v = dpp(v, std::integral_constant<int, 0x128>{});
  const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = max(r[0], r[1]);
  const auto q = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return max(q[0], q[1]);
}

// k rounds: the largest key of the wave, then the lowest expert that has it.  N: logits per lane (expert lane + 64 i).  Lane s
// (of group s / 64, in sel_v[s / 64]) gets the s-th.
template <int N> __device__ __forceinline__ void select_rounds(const float* __restrict__ l, int E, int k, int lane, float (&sel_v)[N], int (&sel_e)[N]) {
  float v[N];
  uint32_t key[N];
  unsigned long long open[N];  // lanes whose i-th logit is not taken yet
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const bool in = lane + 64 * i < E;
    v[i] = in ? l[lane + 64 * i] : 0.f;
    key[i] = in ? route_key(v[i]) : 0u;
    open[i] = __ballot(in);
    sel_v[i] = 0.f; sel_e[i] = 0;
  }
  for (int s = 0; s < k; ++s) {
    uint32_t m = key[0];
#pragma unroll
    for (int i = 1; i < N; ++i) m = max(m, key[i]);
    m = wave_max(m);
    bool found = false;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const unsigned long long c = __ballot(key[i] == m) & open[i];
      if (!found && c) {
        const int w = __builtin_ctzll(c);
        const float wv = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v[i]), w));
#pragma unroll
        for (int g = 0; g < N; ++g)
          if (lane + 64 * g == s) { sel_v[g] = wv; sel_e[g] = w + 64 * i; }
        if (lane == w) key[i] = 0u;
        open[i] &= ~(1ull << w);
        found = true;
      }
    }
  }
}

// One wave selects the top-k experts of one token (Section II-A: the gating function) on the raw logits, ties to the
// lower expert index, then the softmax over the k selected logits, summed in slot order.  E <= 256.  put(slot, expert, weight) is
// called by one lane per slot.  All in registers: a round is six lane exchanges inside the vector unit, a comparison and scalar
// work, about 130 cycles whatever E is.  Ranks by E compare-and-count steps (112 cycles each) and exponentials one after the
// other from LDS took 4.5 us of the 9.5 of an assignment of 4 tokens, top-8 of 64, and more where several waves share a SIMD.  A launch for
// 1000 tokens, top-8 of 64: 7.0 -> 4.8 us.
template <int N, class F> __device__ __forceinline__ void topk_rounds(const float* __restrict__ l, int E, int k, int lane, F put) {
  float v[N];
  int e[N];
  select_rounds<N>(l, E, k, lane, v, e);
  const float l0 = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v[0])));
  float x[N], sum = 0.f;
#pragma unroll
  for (int g = 0; g < N; ++g) {
    x[g] = expf(v[g] - l0);
    for (int i = 0; i < min(k - 64 * g, 64); ++i) sum += __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x[g]), i));
  }
#pragma unroll
  for (int g = 0; g < N; ++g)
    if (lane + 64 * g < k) put(lane + 64 * g, e[g], x[g] / sum);
}
template <class F> __device__ __forceinline__ void topk_token(const float* __restrict__ l, int E, int k, int lane, F put) {
  if (E <= 64) topk_rounds<1>(l, E, k, lane, put);
  else topk_rounds<4>(l, E, k, lane, put);
}

// Up to 64 pairs, one per lane of a wave: a ballot per bit of the expert index (E <= 256).
struct FewPairs {
  unsigned long long all, bits[8];
  __device__ __forceinline__ FewPairs(int e, bool valid) : all(__ballot(valid)) {
#pragma unroll
    for (int b = 0; b < 8; ++b) bits[b] = __ballot((e >> b) & 1);
  }
  // number of the pairs in `of` whose expert is below ex; own: those of ex
  __device__ __forceinline__ int below(int ex, unsigned long long of, unsigned long long& own) const {
    int n = 0;
    own = of;
#pragma unroll
    for (int b = 7; b >= 0; --b) {
      const bool one = (ex >> b) & 1;
      if (one) n += __popcll(own & ~bits[b]);
      own &= one ? bits[b] : ~bits[b];
    }
    return n;
  }
};

}  // namespace si
