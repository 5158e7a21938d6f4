// Token assignment (Section II-A: a gating function assigns tokens to their experts).
// top-k on raw logits (ties -> lower index), softmax over the selected k, per-expert histogram,
// exclusive prefix sum, stable expert-sorted permutation, and the launch tables derived from them.
// Everything that decides an index is integer or an exact fp32 comparison, so the result does not
// depend on scheduling.
#include "si_internal.h"
#include "route_device.h"

#include <algorithm>

namespace si {

namespace {

constexpr int WAVE = 64;
constexpr int ROUTE_WAVES = ROUTE_THREADS / WAVE;

// The caller's idx / w are written along with the plan's.
__device__ __forceinline__ void put_choice(const Plan& p, const RouteOut& u, size_t q, int e, float w) {
  p.idx[q] = e; p.w[q] = w;
  if (u.idx) u.idx[q] = e;
  if (u.w) u.w[q] = w;
}

// One wave per token.
__global__ __launch_bounds__(256) void k_topk(const float* __restrict__ logits, int T, int E, int k, Plan p, RouteOut u) {
  const int wv = threadIdx.x / WAVE, lane = threadIdx.x % WAVE;
  const int t = blockIdx.x * 4 + wv;
  if (t >= T) return;
  topk_token(logits + (size_t)t * E, E, k, lane, [&](int s, int e, float w) { put_choice(p, u, (size_t)t * k + s, e, w); });
}

struct AssignLds {
  int tot[MAX_EXPERTS + 2];     // pairs of each expert
  int tot1[MAX_EXPERTS + 2];    // of those, pairs of X1 tokens
  int base[MAX_EXPERTS + 2];    // pairs before this block's, then before the current pass
  int off[MAX_EXPERTS + 3];     // exclusive prefix of tot
  int tile[4][MAX_EXPERTS + 3]; // exclusive prefixes over the routed experts: spill tiles, other row tiles; the same of the X2 rows
  int touch[MAX_EXPERTS + 3];   // exclusive prefix of "has pairs"
  int multi[2];                 // some routed expert has more than one row tile
  int wcnt[ROUTE_WAVES][MAX_EXPERTS];
};

// exclusive prefix sum of f(0..n-1) into out[0..n] by one wave
template <class F> __device__ __forceinline__ void wave_scan(int n, int lane, int* out, F f) {
  int carry = 0;
  for (int b = 0; b < n; b += WAVE) {
    const int e = b + lane, v = e < n ? f(e) : 0;
    int x = v;
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);  // lanes of a row of 16: from 1, 2, 4, 8 below
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);
    const int r0 = __builtin_amdgcn_readlane(x, 15), r1 = r0 + __builtin_amdgcn_readlane(x, 31), r2 = r1 + __builtin_amdgcn_readlane(x, 47);
    x += lane < 16 ? 0 : lane < 32 ? r0 : lane < 48 ? r1 : r2;
    if (e < n) out[e] = carry + x - v;
    carry += __builtin_amdgcn_readlane(x, WAVE - 1);
  }
  if (lane == 0) out[n] = carry;
}

// Positions of the pairs [q_begin, q_end) and, by the first block, the launch tables.  Every block counts all pairs (16
// bytes of idx per load, LDS atomics), so that one launch after the selection suffices and no table has to be shared
// between blocks; the prefix sums run in parallel (one wave each), and a pair's rank among the equal experts of its wave
// comes from one ballot per bit of the expert index.  A single block with serial prefix sums and a ballot per distinct
// expert took 91 us for 16088 pairs over 64 experts and 25 us for 8192 over 8; this takes 10.5 and 7.0 us.
__device__ __forceinline__ void assign_body(AssignLds& s, int T, int E, int k, int has_shared, int n_x1, const Plan& p,
                                            const RouteOut& u, int q_begin, int q_end, bool first_block) {
  const int tid = threadIdx.x, lane = tid % WAVE, wv = tid / WAVE;
  const int EX = E + (has_shared ? 1 : 0);
  const int n_pairs = T * k, q_x1 = n_x1 * k;
  for (int e = tid; e < EX; e += ROUTE_THREADS) { s.tot[e] = 0; s.tot1[e] = 0; s.base[e] = 0; }
  if (tid < 2) s.multi[tid] = 0;
  __syncthreads();
  auto count = [&](int q, int e) {
    atomicAdd(&s.tot[e], 1);
    if (q_x1 < n_pairs && q < q_x1) atomicAdd(&s.tot1[e], 1);
    if (q < q_begin) atomicAdd(&s.base[e], 1);
  };
  {
    const bool wide = (reinterpret_cast<uintptr_t>(p.idx) & 15) == 0;
    const int n4 = wide ? n_pairs / 4 : 0;
    for (int i = tid; i < n4; i += ROUTE_THREADS) {
      const int4 v = reinterpret_cast<const int4*>(p.idx)[i];
      count(4 * i, v.x); count(4 * i + 1, v.y); count(4 * i + 2, v.z); count(4 * i + 3, v.w);
    }
    for (int q = 4 * n4 + tid; q < n_pairs; q += ROUTE_THREADS) count(q, p.idx[q]);
  }
  __syncthreads();
  if (q_x1 >= n_pairs)  // no X2 tokens: every pair is an X1 pair
    for (int e = tid; e < E; e += ROUTE_THREADS) s.tot1[e] = s.tot[e];
  if (has_shared && tid == 0) { s.tot[E] = T; s.tot1[E] = n_x1; }
  __syncthreads();
  if (wv == 0) wave_scan(EX, lane, s.off, [&](int e) { return s.tot[e]; });
  if (first_block) {
    if (wv < 4) wave_scan(E, lane, s.tile[wv], [&](int e) {
      const int rows = s.tot[e] - (wv >= 2 ? s.tot1[e] : 0), n = n_row_tiles(rows), spill = has_spill_tile(rows);
      if (n > 1) s.multi[wv / 2] = 1;
      return wv % 2 ? n - spill : spill;
    });
    if (wv == 4) wave_scan(EX, lane, s.touch, [&](int e) { return s.tot[e] > 0 ? 1 : 0; });
  }
  __syncthreads();
  if (first_block) {
    for (int e = tid; e < EX; e += ROUTE_THREADS) {
      if (p.count) p.count[e] = s.tot[e];
      if (p.count1) p.count1[e] = s.tot1[e];
      if (p.off) p.off[e] = s.off[e];
      if (p.touched && s.tot[e] > 0) p.touched[s.touch[e]] = make_int4(e, s.off[e], s.off[e] + s.tot[e], 0);
      if (e < E) {
        if (u.count) u.count[e] = s.tot[e];
        if (u.off) u.off[e] = s.off[e];
      }
    }
    if (p.tile_e)
      for (int i = tid; i < 4 * E; i += ROUTE_THREADS) {
        const int l = i / E, e = i % E, n = s.tile[l][e + 1] - s.tile[l][e];
        const int pos = s.tile[l][e] + (l % 2 ? s.tile[l - 1][E] : 0);            // the spill tiles are listed first
        const int r0 = l % 2 ? 0 : s.tile[l + 1][e + 1] - s.tile[l + 1][e];        // ... and each is the last of its expert
        int32_t *te = l < 2 ? p.tile_e : p.tile_e_x2, *tr = l < 2 ? p.tile_r : p.tile_r_x2;
        for (int r = 0; r < n; ++r) {
          te[pos + r] = e + n * (TILE_E_MASK + 1);
          tr[pos + r] = r0 + r;
        }
        if (e == 0 && l % 2) {
          // (of the routed experts only: the shared one, entry E, is found through its offset)
          int32_t* nt = p.n_tiles + (l < 2 ? 0 : 3);
          nt[0] = s.tile[l - 1][E] + s.tile[l][E];
          nt[1] = s.tile[l - 1][E];
          nt[2] = !s.multi[l / 2];
        }
      }
    if (tid == 0) {
      if (p.off) p.off[EX] = s.off[EX];
      if (u.off) u.off[E] = s.off[E];
      if (p.n_touched) *p.n_touched = s.touch[EX];
    }
  }
  // stable positions: pairs in ascending q, ROUTE_THREADS at a time
  for (int base = q_begin; base < q_end; base += ROUTE_THREADS) {
    for (int i = tid; i < ROUTE_WAVES * MAX_EXPERTS; i += ROUTE_THREADS) (&s.wcnt[0][0])[i] = 0;
    __syncthreads();
    const int q = base + tid;
    const bool valid = q < q_end;
    const int e = valid ? p.idx[q] : 0;
    unsigned long long peers = __ballot(valid);
    for (int bit = 1; bit < E; bit <<= 1) {
      const unsigned long long m = __ballot((e & bit) != 0);
      peers &= (e & bit) ? m : ~m;
    }
    const int rank = __popcll(peers & ((1ull << lane) - 1));
    if (valid && rank == 0) s.wcnt[wv][e] = __popcll(peers);
    __syncthreads();
    if (valid) {
      int pos = s.base[e] + rank;
      for (int w2 = 0; w2 < wv; ++w2) pos += s.wcnt[w2][e];
      const int row = s.off[e] + pos;
      if (p.perm) p.perm[row] = q;
      if (p.inv) p.inv[q] = row;
      if (u.perm) u.perm[row] = q;
      if (u.inv) u.inv[q] = row;
      if (p.row_token) p.row_token[row] = q / k;
    }
    if (base + ROUTE_THREADS < q_end) {
      __syncthreads();
      for (int e2 = tid; e2 < E; e2 += ROUTE_THREADS) {
        int add = 0;
        for (int w2 = 0; w2 < ROUTE_WAVES; ++w2) add += s.wcnt[w2][e2];
        s.base[e2] += add;
      }
      __syncthreads();
    }
  }
  if (has_shared && p.row_token)
    for (int q = q_begin + tid; q < q_end; q += ROUTE_THREADS)
      if (q % k == 0) p.row_token[n_pairs + q / k] = q / k;
}

// grid: one block per `span` pairs (a multiple of ROUTE_THREADS)
__global__ __launch_bounds__(ROUTE_THREADS) void k_assign(int T, int E, int k, int has_shared, int n_x1, int span,
                                                          Plan p, RouteOut u) {
  __shared__ AssignLds s;
  const int q0 = blockIdx.x * span;
  assign_body(s, T, E, k, has_shared, n_x1, p, u, q0, min(q0 + span, T * k), blockIdx.x == 0);
}

// A dense layer (one expert, weight 1): every table is known without looking at anything.  Launched only for a caller who asks
// for them: the kernels of the call know them too (Plan::dense_T).
__global__ __launch_bounds__(256) void k_dense_assign(int T, int n_x1, Plan p, RouteOut u) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t < T) {
    p.idx[t] = 0; p.w[t] = 1.f;
    if (p.perm) p.perm[t] = t;
    if (p.inv) p.inv[t] = t;
    if (p.row_token) p.row_token[t] = t;
    if (u.idx) u.idx[t] = 0;
    if (u.w) u.w[t] = 1.f;
    if (u.perm) u.perm[t] = t;
    if (u.inv) u.inv[t] = t;
  }
  if (t == 0) {
    if (p.count) p.count[0] = T;
    if (p.count1) p.count1[0] = n_x1;
    if (p.off) { p.off[0] = 0; p.off[1] = T; }
    if (p.touched) p.touched[0] = make_int4(0, 0, T, 0);
    if (p.n_touched) *p.n_touched = 1;
    if (u.count) u.count[0] = T;
    if (u.off) { u.off[0] = 0; u.off[1] = T; }
  }
}

// Few pairs (generation phase, small batches): selection by a wave per token, then everything else by the first wave without
// another barrier: one ballot per bit of the expert index gives, for a lane's pair or a lane's expert, the number of pairs of smaller
// experts and the mask of its own.  No expert has more than one row tile.  In the general kernel the assignment, with ten barriers and
// a reload of the choices, is 4.3 us.  Launches, with the faster selection: 4 tokens, top-8 of 64 experts 11.4 -> 5.2 us; 24 tokens,
// top-2 of 8 9.1 -> 5.5 (45 tokens, top-3 of 60, in the general kernel: 20.0 -> 9.2).
constexpr int FEW_PAIRS = WAVE;
__global__ __launch_bounds__(ROUTE_THREADS) void k_route_few(const float* __restrict__ logits, int T, int E, int k, int has_shared,
                                                             int n_x1, Plan p, RouteOut u) {
  __shared__ int32_t s_idx[FEW_PAIRS];
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE), lane = threadIdx.x % WAVE;
  const int n_pairs = T * k, EX = E + (has_shared ? 1 : 0);
  for (int t = wv; t < T; t += blockDim.x / WAVE)
    topk_token(logits + (size_t)t * E, E, k, lane, [&](int s, int e, float w) {
      s_idx[t * k + s] = e;
      put_choice(p, u, (size_t)t * k + s, e, w);
    });
  // (the barrier waits for LDS only, not for the tables on their way)
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  if (wv != 0) return;
  const bool valid = lane < n_pairs;
  const int e = valid ? s_idx[lane] : 0;
  const FewPairs few(e, valid);
  const unsigned long long x1 = __ballot(lane < n_x1 * k), lt = (1ull << lane) - 1;
  {
    unsigned long long own;
    const int row = few.below(e, few.all, own) + __popcll(own & lt);
    if (valid) {
      if (p.perm) p.perm[row] = lane;
      if (p.inv) p.inv[lane] = row;
      if (u.perm) u.perm[row] = lane;
      if (u.inv) u.inv[lane] = row;
      if (p.row_token) p.row_token[row] = lane / k;
    }
    if (has_shared && p.row_token && lane < T) p.row_token[n_pairs + lane] = lane;
  }
  int n_touched = 0, n_tiles = 0, n_x2 = 0;
  for (int e0 = 0; e0 < EX; e0 += WAVE) {
    const int ex = e0 + lane;
    const bool in = ex < EX, routed = ex < E;
    unsigned long long own;
    const int below = few.below(ex, few.all, own), c = routed ? __popcll(own) : T, c1 = routed ? __popcll(own & x1) : n_x1;
    const bool t_in = in && c > 0, r_in = routed && c > 0, x2_in = routed && c > c1;
    const unsigned long long mt = __ballot(t_in), mr = __ballot(r_in), mx = __ballot(x2_in);
    if (in) {
      const int off = routed ? below : n_pairs;
      if (p.count) p.count[ex] = c;
      if (p.count1) p.count1[ex] = c1;
      if (p.off) p.off[ex] = off;
      if (routed && u.count) u.count[ex] = c;
      if (routed && u.off) u.off[ex] = off;
    }
    if (p.touched && t_in) {
      const int off = routed ? below : n_pairs;
      p.touched[n_touched + __popcll(mt & lt)] = make_int4(ex, off, off + c, 0);
    }
    if (p.tile_e) {
      if (r_in) { const int i = n_tiles + __popcll(mr & lt); p.tile_e[i] = ex + TILE_E_MASK + 1; p.tile_r[i] = 0; }
      if (x2_in) { const int i = n_x2 + __popcll(mx & lt); p.tile_e_x2[i] = ex + TILE_E_MASK + 1; p.tile_r_x2[i] = 0; }
    }
    n_touched += __popcll(mt);
    n_tiles += __popcll(mr);
    n_x2 += __popcll(mx);
  }
  if (lane == 0) {
    if (p.off) p.off[EX] = n_pairs + (has_shared ? T : 0);
    if (u.off) u.off[E] = n_pairs;
    if (p.n_touched) *p.n_touched = n_touched;
    if (p.tile_e) {
      p.n_tiles[0] = n_tiles; p.n_tiles[1] = 0; p.n_tiles[2] = 1;
      p.n_tiles[3] = n_x2; p.n_tiles[4] = 0; p.n_tiles[5] = 1;
    }
  }
}

// Up to 64 tokens: selection and assignment in one launch.  Wave v of the block takes
// tokens v, v + 16, ...; the assignment then runs on the whole block.
__global__ __launch_bounds__(ROUTE_THREADS) void k_route_small(const float* __restrict__ logits, int T, int E, int k,
                                                               int has_shared, int n_x1, Plan p, RouteOut u) {
  __shared__ AssignLds s;
  const int wv = threadIdx.x / WAVE, lane = threadIdx.x % WAVE;
  if (logits) {
    for (int t = wv; t < T; t += ROUTE_WAVES)
      topk_token(logits + (size_t)t * E, E, k, lane, [&](int i, int e, float w) { put_choice(p, u, (size_t)t * k + i, e, w); });
  } else {
    for (int t = threadIdx.x; t < T; t += ROUTE_THREADS) {
      p.idx[t] = 0; p.w[t] = 1.f;
      if (u.idx) u.idx[t] = 0;
      if (u.w) u.w[t] = 1.f;
    }
  }
  __syncthreads();
  assign_body(s, T, E, k, has_shared, n_x1, p, u, 0, T * k, true);
}

// (rows of x are multiples of 128 bytes, x and the pinned buffer aligned to 16)
__global__ __launch_bounds__(256) void k_handoff(Plan p, const uint4* __restrict__ x, uint4* __restrict__ hx, int n16, int n_pairs,
                                                 int EX, int32_t* __restrict__ hidx, float* __restrict__ hw,
                                                 int32_t* __restrict__ hcount) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n16) hx[i] = x[i];
  if (i < n_pairs) { hidx[i] = p.idx[i]; hw[i] = p.w[i]; }
  if (i < EX) { hcount[i] = p.count[i]; hcount[EX + i] = p.count1[i]; }
}

}  // namespace

hipError_t launch_handoff(const Plan& plan, const uint16_t* x, size_t x_bytes, int n_pairs, int EX, uint16_t* hx, int32_t* hidx,
                          float* hw, int32_t* hcount, hipStream_t stream) {
  const int n16 = (int)(x_bytes / 16), n = std::max(std::max(n16, n_pairs), EX);
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_handoff, dim3((n + 255) / 256), dim3(256), 0, stream, plan, reinterpret_cast<const uint4*>(x),
                     reinterpret_cast<uint4*>(hx), n16, n_pairs, EX, hidx, hw, hcount);
  return hipGetLastError();
}

hipError_t launch_route(const float* logits, int T, int E, int k, int has_shared, int n_g,
                        const Plan& plan, const RouteOut& user, hipStream_t stream) {
  if (T <= 0) return hipSuccess;
  const int n_x1 = T - n_g;
  if (!logits && E == 1 && !has_shared) {
    hipLaunchKernelGGL(k_dense_assign, dim3((T + 255) / 256), dim3(256), 0, stream, T, n_x1, plan, user);
    return hipGetLastError();
  }
  if (logits && T * k <= FEW_PAIRS) {
    hipLaunchKernelGGL(k_route_few, dim3(1), dim3(WAVE * std::min(T, ROUTE_WAVES)), 0, stream, logits, T, E, k, has_shared, n_x1, plan, user);
    return hipGetLastError();
  }
  if (T <= 64 || !logits) {
    hipLaunchKernelGGL(k_route_small, dim3(1), dim3(ROUTE_THREADS), 0, stream, logits, T, E, k, has_shared, n_x1, plan, user);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_topk, dim3((T + 3) / 4), dim3(256), 0, stream, logits, T, E, k, plan, user);
  // at most 64 blocks: each counts all pairs
  const int n_pairs = T * k, per_block = (n_pairs + 63) / 64;
  const int span = (per_block + ROUTE_THREADS - 1) / ROUTE_THREADS * ROUTE_THREADS;
  hipLaunchKernelGGL(k_assign, dim3((n_pairs + span - 1) / span), dim3(ROUTE_THREADS), 0, stream, T, E, k, has_shared, n_x1, span, plan, user);
  return hipGetLastError();
}

}  // namespace si
