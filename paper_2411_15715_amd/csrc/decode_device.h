// Device-side pieces that the generation-phase kernels of both storage forms use (hipcc only).
#pragma once
#include "si_internal.h"

namespace si {

__device__ inline float silu_f(float z) { return z / (1.f + __expf(-z)); }

// expert handled by this block and its row range; returns false when there is nothing to do
// (slot < 0: the shared expert, entry n_routed, of a launch that covers it along with the routed ones)
__device__ inline bool block_rows(const Plan& p, int expert_sel, int x2_only, int slot, int& e, int& r0, int& r1) {
  if (slot < 0) {
    e = p.n_routed;
  } else if (expert_sel >= 0) {
    e = expert_sel;
  } else {
    if (slot >= *p.n_touched) return false;
    e = p.touched[slot];
    if (e >= p.n_routed) return false;
  }
  r0 = row_begin(p, e, x2_only);
  r1 = row_end(p, e);
  return r1 > r0;
}

}  // namespace si
