// Device-side pieces that the generation-phase kernels of both storage forms use (hipcc only).
#pragma once
#include "si_internal.h"

namespace si {

__device__ inline float silu_f(float z) { return z / (1.f + __expf(-z)); }

// Sums of N values over the lanes of a wave, value i in the lanes whose bits 5 and 4 are `i's place`: the first two steps of a
// butterfly (lanes 32 and 16 apart) halve the values, one swap instruction and one addition for two of them, instead of exchanging
// all; the last ones add rotated rows of 16 lanes (DPP).  The additions are those of the butterfly, pair for pair.  Result for value
// i = 4 g + 2 a + b (N >= 4): v[g], in the lanes 32 b + 16 a .. + 15 (every lane of them; LAST: down to LAST lanes apart, lanes below
// that distance keep sums of their own).  24 shuffles through LDS and as many additions per 4 values took the epilogue of a 16-column
// block with 4 rows, 32 values a wave, 4.4 us longer (gate/up launch of a small dense split part 9.2 -> 4.8 us, of a 60-expert layer with 4
// tokens 138.9 -> 134.5 us).
template <int CTRL> __device__ __forceinline__ float dpp_add(float v) {
  return v + __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), CTRL, 0xf, 0xf, false));
}
template <int N, int LAST = 1> __device__ __forceinline__ void wave_sums(float (&v)[N]) {
  static_assert(N % 4 == 0, "groups of four");
#pragma unroll
  for (int g = 0; g < N / 4; ++g) {
    float s[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[4 * g + 2 * a]), __float_as_uint(v[4 * g + 2 * a + 1]), false, false);
      s[a] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(s[0]), __float_as_uint(s[1]), false, false);
    float t = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    t = dpp_add<0x128>(t);                        // row_ror:8
    if constexpr (LAST <= 4) t = dpp_add<0x124>(t);
    if constexpr (LAST <= 2) t = dpp_add<0x122>(t);
    if constexpr (LAST <= 1) t = dpp_add<0x121>(t);
    v[g] = t;
  }
}

// expert handled by this block and its row range; returns false when there is nothing to do
// (slot < 0: the shared expert, entry n_routed, of a launch that covers it along with the routed ones)
__device__ inline bool block_rows(const Plan& p, int expert_sel, int x2_only, int slot, int& e, int& r0, int& r1) {
  if (slot < 0) {
    e = p.n_routed;
  } else if (expert_sel >= 0) {
    e = expert_sel;
  } else {
    // one trip to memory for the expert and its rows: the number of experts, their indices and their offsets one after the other
    // were three, before the first weight could be asked for.  (slot < entries of the table: the grid has no more)
    const int32_t* rec = reinterpret_cast<const int32_t*>(p.touched);
    const int n = table(p.n_touched, 0);
    e = table(rec, 4 * slot);
    r0 = table(rec, 4 * slot + 1);
    r1 = table(rec, 4 * slot + 2);
    if (slot >= n || e >= p.n_routed) return false;
    if (x2_only) r0 += table(p.count1, e);
    return r1 > r0;
  }
  r0 = row_begin(p, e, x2_only);
  r1 = row_end(p, e);
  return r1 > r0;
}

}  // namespace si
