// Prompt-phase grouped GEMMs on the bf16 matrix cores (v_mfma_f32_16x16x32_bf16), fp32 accumulate.
//   gateup : Hact[row][j] = SiLU(X_e . Wg_e[j]) * (X_e . Wu_e[j])   (FC1 + activation, Eq. 1)
//   down   : Yp[row][m] (+)= Hact[row][:] . Wd_e[:, m]              (FC2, one term of Eq. 2)
//   combine: y[t] = sum_s w[t][s] Yp[row(t,s)] (+ shared expert row) (+ Y^CC for X1 rows)
// Rows are the expert-sorted (token, slot) pairs of the token assignment; a row tile never
// crosses an expert.  The gather of x rows is fused into the A-operand load of the first GEMM.
//
// Both GEMMs: one 512-thread block (8 waves, 2 per SIMD) per compute unit, which takes tile after tile of BM x 256 outputs
// (TileQueues), BK = 64, rings of LDS stages filled by direct global->LDS loads (global_load_lds_dwordx4, no VGPR staging), wave
// tile (BM/2) x 64.  A row tile holds up to 256 rows, the last one of an expert up to 320 (si_internal.h: n_row_tiles);
// the block runs the body instantiated for the next multiple of 32 rows that covers the tile's (4-bit: up to 256, the rows beyond in
// a second pass).
// The main loop is a ping-pong of two wave groups on v_mfma_f32_16x16x32_bf16 (gemm_pingpong; gemm_q4 converts 4-bit weights
// in the registers of the wave that multiplies them).
// LDS rows hold 64 contraction elements (128 bytes); the 16-byte piece c of row r sits at piece
// c ^ ((r >> 1) & 7): gfx950's LDS has 64 banks, so 16 consecutive rows x 16 bytes must cover 256
// distinct bytes of bank space for the 128-bit MFMA operand reads to be conflict free (measured:
// SQ_LDS_BANK_CONFLICT = 0).
#include "si_internal.h"

#include <type_traits>

namespace si {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
#define SI_LPTR(p) ((void __attribute__((address_space(3)))*)(p))

constexpr int WAVE = 64;
constexpr int THREADS = 512;
constexpr int BN = 256;  // B rows per tile: 128 hidden columns (gate+up) or 256 output columns
constexpr int BK = 64;
constexpr int B_BYTES = BN * BK * 2;  // 32 KB
constexpr int KERNEL_LDS = 160 * 1024 - 16;  // the largest body
constexpr int NEXT_LDS = 16;            // after it: the block's next item (run_items)

// z / (1 + exp(-z)), the division by one residual step on the reciprocal instruction, whose own error is up to 1 ulp and whose
// denormal results are flushed (hence the factor 1/4).  Equal to the division bit for bit on 4 M arguments in [-100, 100] and
// on infinities and NaN.  Against the bare reciprocal it costs 0.2 to 0.5 % of a call, 1.4 % where the k-loop is short (16
// experts of 6400 columns, d_model 1280, top-4, 3000 tokens: 570 -> 578 us; 8x22B-shaped prompt of 4096 tokens: 3925 -> 3945);
// the compiler's division 1 % of the Qwen-shaped prompt (1771 -> 1790 us, this 1774).
__device__ inline float silu_f(float z) {
  const float d4 = __builtin_fmaf(0.25f, __expf(-z), 0.25f), z4 = 0.25f * z, r = __builtin_amdgcn_rcpf(d4), q = z4 * r;
  return __builtin_amdgcn_div_fixupf(__builtin_fmaf(__builtin_fmaf(-q, d4, z4), r, q), d4, z4);
}

// two floats -> two bf16 (round to nearest even) in one register, a in the low half
__device__ inline uint32_t pack_bf16(float a, float b) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
}

__device__ inline bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// thread index, opaque, so that what a body derives from it is formed per tile: hoisted out of the loop over the tiles the lane
// offsets of all bodies are live through every main loop (9 registers spilled)
__device__ __forceinline__ int thread_of_item() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// the same for uniform values (the conditions on the number of k-tiles of all bodies filled the scalar registers)
__device__ __forceinline__ int scalar_of_item(int v) {
  asm volatile("" : "+s"(v));
  return v;
}

// direct global -> LDS load of 16 bytes per lane: uniform base (scalar registers) + 32-bit byte offset of the lane
__device__ inline void load_lds16(const void* base, uint32_t& off, unsigned char* l) {
  typedef const unsigned char __attribute__((address_space(1))) gchar;
  // (both opaque, so that no 64-bit address or zero-extended offset per lane is kept through the loop instead)
  asm volatile("" : "+s"(base), "+v"(off));
  __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)((gchar*)base + off), SI_LPTR(l), 16, 0, 0);
}

// swizzled byte offset of 16-byte piece c of row r in a [rows][64] bf16 tile
__device__ inline int swz(int r, int c) { return r * 128 + ((c ^ ((r >> 1) & 7)) << 4); }

// s_waitcnt vmcnt(n) only (lgkmcnt / expcnt untouched); n < 64
template <int N> __device__ inline void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt(0x0f70 | (N & 0xf) | (((N >> 4) & 3) << 14));
}

__device__ inline void wait_lgkmcnt0() { __builtin_amdgcn_s_waitcnt(0xc07f); }  // lgkmcnt(0) only

// Workgroup barrier WITHOUT the memory fence of __syncthreads(): the fence would drain every outstanding
// global->LDS load (s_waitcnt vmcnt(0)) and so defeat the multi-stage ring.  What has to be visible
// after the barrier is (a) each wave's own direct-to-LDS loads of the tile about to be read, which the
// wave itself waited for with wait_vmcnt<> just before, and (b) nothing else: fragments read from the
// slot about to be refilled were consumed by MFMAs earlier in program order.
__device__ inline void block_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// se: index of the expert inside the launch's weight storage; sh: the shared expert in a launch that covers it as well
// row_t0: row r is token r - row_t0 (the shared expert, a single routed one), -1: look it up
struct TileInfo { int e, row0, row_end, se, sh, row_t0; };

// The tiles of a launch, in one queue per XCD (hardware block ids go round-robin over the 8 XCDs).
//  * Three lists of ids: the shared expert's tiles, in a launch that covers it along with the routed ones (its tiles are the
//    longest of the down projection); the routed experts' spill tiles (the last tile of an expert where it has more than
//    TILE_ROWS rows), longer than all others; their other tiles in the order expert, inner index, row tile.  In a launch over one
//    expert whose last tile is a short one the second list is of its full tiles, the third of the last.  A queue holds an eighth of
//    each list, in this order: the longest tiles start first, the last round is of the shortest, and in between different
//    XCDs work on experts of different sizes (sorted by rows altogether, the tiles bound by the matrix cores came first and
//    those bound by the weights after them: 2011 tokens, 64 experts of 2560 columns, top-8, 1690 -> 1775 us).
//    The eighth is a range, so that the row tiles that read the same weights share an L2; when no expert of the launch has more
//    than one row tile nothing is shared but the few rows of x, and the ids are dealt one by one: every XCD gets the same mix.
//  * One block per compute unit takes tile after tile from the queue of its XCD and, when that is empty, from the fullest other
//    one: with ranges alone a launch took the time of the XCD with the fullest experts.
//  * Where the last round of a queue (a tile per compute unit) is at most half full its tiles are cut in two.
// A launch has 3 to 20 rounds, so a tile more than the mean is 5 to 30 %.  One block per tile in ranges of ids per XCD, tiles
// computed for 64, 128, 192, 256 or 320 rows, against this: 2011 tokens, 64 experts of 2560 columns, top-8, a shared one of 20480:
// 1757 -> 1694 us; 4096 tokens, 8 experts of 16384, d_model 6144, top-2: 3907 -> 3676 (3747 with the spill tiles in their place);
// 512 tokens, 8 experts of 14336: 543 -> 530; dense 6656 x 1152, 20 tokens (9 tiles cut along their columns): 65 -> 45.
constexpr int N_XCD = 8, XCD_CU = 32;  // XCDs, compute units of one
constexpr int SHORT_ROWS = 128;        // a last tile up to here is a short one
// a / b and the remainder of uniform numbers, 0 <= a < 2^24, b > 0: a tenth of the general division's instructions.  A launch
// starts with cold instruction caches; 2 KB less code before the first load are 1 to 2 us.
__device__ __forceinline__ int small_div(int a, int b, int& rem) {
  int q = (int)((float)a * __builtin_amdgcn_rcpf((float)b));  // at most 1 off
  int r = a - q * b;
  if (r < 0) { --q; r += b; }
  if (r >= b) { ++q; r -= b; }
  rem = __builtin_amdgcn_readfirstlane(r);
  return __builtin_amdgcn_readfirstlane(q);
}

struct TileQueues {
  unsigned n0, n1, n2;        // ids of each list
  int rows0, rows1, rows2;    // row tiles of an inner index in it (launch over one expert) or of all experts
  int deal;
  __device__ __forceinline__ int rows(int list) const { return rows0 * (list == 0) + rows1 * (list == 1) + rows2 * (list == 2); }
  static __device__ __forceinline__ unsigned first(unsigned n, unsigned q) { return n * q / N_XCD; }
  __device__ __forceinline__ unsigned count0(unsigned q) const { return first(n0, q + 1) - first(n0, q); }
  __device__ __forceinline__ unsigned count(unsigned n, unsigned q) const { return deal ? (n + N_XCD - 1 - q) / N_XCD : first(n, q + 1) - first(n, q); }
  __device__ __forceinline__ unsigned tiles(unsigned q) const { return count0(q) + count(n1, q) + count(n2, q); }
  __device__ __forceinline__ unsigned most_tiles() const { return (n0 + 7) / N_XCD + (n1 + 7) / N_XCD + (n2 + 7) / N_XCD; }  // >= any tiles(q)
  __device__ __forceinline__ unsigned cut(unsigned tiles) const { const unsigned r = tiles % XCD_CU; return 2 * r > XCD_CU ? 0 : r; }
  __device__ __forceinline__ int items(unsigned q) const { const unsigned t = tiles(q); return t + cut(t); }
  // item of queue q -> list and id in it, and which half of a cut tile (halves 2)
  __device__ __forceinline__ int find(unsigned q, unsigned item, int& list, int& half, int& halves) const {
    const unsigned t = tiles(q), whole = t - cut(t);
    halves = item < whole ? 1 : 2;
    half = item < whole ? 0 : (item - whole) & 1;
    const unsigned i = item < whole ? item : whole + (item - whole) / 2, c0 = count0(q), c1 = c0 + count(n1, q);
    list = i < c0 ? 0 : i < c1 ? 1 : 2;
    const unsigned k = i - (list == 0 ? 0 : list == 1 ? c0 : c1), f0 = first(n0, q), f1 = first(n1, q), f2 = first(n2, q);
    return list && deal ? k * N_XCD + q : (list == 0 ? f0 : list == 1 ? f1 : f2) + k;
  }
};

__device__ __forceinline__ TileQueues tile_queues(const Plan& p, int expert_sel, int x2_only, int n_inner, int n_inner_s, bool deal) {
  TileQueues t;
  t.rows0 = n_inner_s ? n_row_tiles(table(p.off, p.n_routed + 1) - table(p.off, p.n_routed)) : 0;
  int multi, n;
  if (expert_sel >= 0) {
    const int rows = p.dense_T ? p.dense_T - (x2_only ? p.dense_x1 : 0)
                               : table(p.off, expert_sel + 1) - table(p.off, expert_sel) - (x2_only ? table(p.count1, expert_sel) : 0);
    const int last = rows & (TILE_ROWS - 1);
    n = n_row_tiles(rows);
    multi = n > 1;
    t.rows1 = has_spill_tile(rows) ? 1 : multi && last && last <= SHORT_ROWS ? n - 1 : 0;
  } else {
    const int32_t* nt = p.n_tiles + 3 * x2_only;
    n = table(nt, 0);
    t.rows1 = table(nt, 1);
    multi = !table(nt, 2);
  }
  t.rows2 = n - t.rows1;
  t.deal = deal && !multi;
  t.n0 = t.rows0 * n_inner_s;
  t.n1 = t.rows1 * n_inner;
  t.n2 = t.rows2 * n_inner;
  return t;
}

// item -> expert, inner index, rows
__device__ __forceinline__ void item_tile(const TileQueues& tq, const Plan& p, int expert_sel, int x2_only, int q, int item, int n_inner,
                                          int& inner, TileInfo& ti, int& half, int& halves) {
  int list;
  const int id = tq.find(q, item, list, half, halves);
  ti.sh = list == 0;
  // the group of row tiles that share an inner index: id inside it, its size, its first row tile
  int in_group = id, size, r0 = 0, rem;
  if (ti.sh || expert_sel >= 0) {
    ti.e = ti.sh ? p.n_routed : expert_sel;
    size = tq.rows(list);
  } else {
    const int t = small_div(id, n_inner, rem), at = t + (list == 2 ? tq.rows1 : 0);
    const int32_t *te = x2_only ? p.tile_e_x2 : p.tile_e, *tr = x2_only ? p.tile_r_x2 : p.tile_r;
    const unsigned e = table(te, at);
    const int first = table(tr, at);
    ti.e = e & TILE_E_MASK;
    size = e / (TILE_E_MASK + 1);
    in_group = rem;
    if (list == 1) r0 = first;
    else in_group += first * n_inner;
  }
  const int off = p.dense_T ? 0 : table(p.off, ti.e), start = off + (!x2_only ? 0 : p.dense_T ? p.dense_x1 : table(p.count1, ti.e));
  const int rows = (p.dense_T ? p.dense_T : table(p.off, ti.e + 1)) - start, n = n_row_tiles(rows);
  // one expert: the spill tile (list 1) or the short last tile (list 2) is the last one
  if (expert_sel >= 0 && (has_spill_tile(rows) ? list == 1 : list == 2)) r0 = n - size;
  inner = small_div(in_group, size, rem);
  const int r = r0 + rem;
  // (uniform, but partly formed in vector registers)
  ti.sh = __builtin_amdgcn_readfirstlane(ti.sh);
  ti.e = __builtin_amdgcn_readfirstlane(ti.e);
  half = __builtin_amdgcn_readfirstlane(half);
  ti.row_t0 = ti.e == p.n_routed || p.n_routed == 1 ? off : -1;
  ti.row0 = start + r * TILE_ROWS;
  ti.row_end = r == n - 1 ? start + rows : ti.row0 + TILE_ROWS;
}

// Takes items until all queues are empty.  The first item of a block is given (block b: item b / 8 of queue b % 8), further ones
// come from a counter per queue, which the kernel before this one on the stream has cleared (it clears the other launch's).
//   body(queue, item, take): processes the item and calls take() once, when its last loads have been waited for: the answer of
//   the counter then arrives under the epilogue.
// Every block ends: a queue's counter never falls, so each of the 8 queues refuses a block at most once.
template <class F>
__device__ __forceinline__ void run_items(const TileQueues& tq, int32_t* head, int32_t* clear, unsigned char* lds, F body) {
  volatile int __attribute__((address_space(3)))* s_next = (volatile int __attribute__((address_space(3)))*)SI_LPTR(lds + KERNEL_LDS);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  constexpr int first = XCD_CU;
  if (blockIdx.x == 0 && threadIdx.x < N_XCD) clear[threadIdx.x * QUEUE_STRIDE] = 0;
  const bool more = tq.most_tiles() > XCD_CU;  // some items are not given to a block (a cut round is at most full)
  int q = blockIdx.x % N_XCD, cand = blockIdx.x / N_XCD, par = 0;
  bool given = cand < tq.items(q);
  for (;;) {
    if (!given) {
      if (!more) return;
      if (w == 0) {
        const int lane = thread_of_item();
        cand = __builtin_amdgcn_readfirstlane(cand);
        while (cand >= tq.items(q)) {
          int best = 0;  // items left * 8 + queue
          if (lane < N_XCD) best = max(0, tq.items(lane) - first - __hip_atomic_load(head + lane * QUEUE_STRIDE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) * N_XCD + lane;
#pragma unroll
          for (int d = 1; d < N_XCD; d <<= 1) best = max(best, __shfl_xor(best, d, WAVE));
          best = __builtin_amdgcn_readfirstlane(best);
          if (best < N_XCD) { q = -1; break; }
          q = best % N_XCD;
          int got = 0;
          if (lane == 0) got = first + __hip_atomic_fetch_add(head + q * QUEUE_STRIDE, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          cand = __builtin_amdgcn_readfirstlane(got);
        }
        if (lane == 0) s_next[par] = q < 0 ? -1 : cand * N_XCD + q;
        wait_lgkmcnt0();
      }
      block_barrier();
      const int v = __builtin_amdgcn_readfirstlane(s_next[par]);
      if (v < 0) return;
      q = v % N_XCD;
      cand = v / N_XCD;
      par ^= 1;
    }
    given = false;
    body(__builtin_amdgcn_readfirstlane(q), __builtin_amdgcn_readfirstlane(cand), [&]() {
      if (more && thread_of_item() == 0) cand = first + __hip_atomic_fetch_add(head + q * QUEUE_STRIDE, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    });
  }
}

// the rows of half a tile; false: none (of few rows the first half takes all; 4-bit, dense 7424 x 8128, 114 tokens: cut 141 us,
// whole 163)
__device__ __forceinline__ bool half_rows(TileInfo& ti, int half) {
  const int rows = ti.row_end - ti.row0;
  if (rows <= 64) return half == 0;
  const int hs = ((rows + 1) / 2 + 31) / 32 * 32;
  ti.row0 += half * hs;
  ti.row_end = min(ti.row_end, ti.row0 + hs);
  return ti.row0 < ti.row_end;
}

// ---------------------------------------------------------------------------------------------
// Main loop of the tiles: ping-pong of two wave groups.
// 8 waves as 2 (row groups) x 4 (B-row quarters of 64), wave tile (16 FA) x 64 in v_mfma_f32_16x16x32_bf16 tiles, FA = 1 .. 10
// fragments of 16 rows: a tile is computed for the next multiple of 32 rows.  Waves w and w + 4 share a SIMD; the second row
// group runs one barrier behind the first, so that in every slot between two barriers one wave of each SIMD issues matrix
// instructions and nothing else while the other reads its next fragments from LDS, issues tile loads and waits.  A k-tile of
// 64 is cut into phases of up to 4 fragments per group (32 matrix instructions of 16 cycles); B is read in the first phase and
// kept in registers.  A region (the A rows of one phase; B) is free once both groups have read it, i.e. one phase later, and is
// refilled then with the tile NA (A) or NB (B) further on: with 256 rows a load has three phases = 3072 matrix cycles to land.
// What bounds it: the power limit.  Counters of a 1024 x 65536 x 8192 product: matrix cores busy 0.90 of the time at a
// shader clock of 1.68 GHz (the loop with one barrier per k-tile that it replaces: 0.65 at 1.84 GHz): 1461 TFLOP/s against
// 1181.  The 16 x 16 x 32 instruction is part of it: register-resident on random operands it sustains 2.06 PFLOP/s under
// the power limit where the 32 x 32 x 16 one sustains 1.81 (its accumulators cost twice the register traffic).  Four
// phases of 16 matrix instructions (64 x 32 quadrants) measured 1378, one wave per SIMD with 128 x 128 tiles 1064.
// ---------------------------------------------------------------------------------------------
template <int FAV, int NJV> struct Ring {
  static constexpr int FA = FAV;
  static constexpr int NJ = NJV;                                   // B fragments (16 rows) of a wave: 4, or 2 of a tile cut in two
  static constexpr int BM = 32 * FA;                               // rows of the tile
  static constexpr int BNW = 64 * NJ;                              // B rows
  static constexpr int NP = FA <= 4 ? 1 : FA <= 8 ? 2 : 3;         // phases per k-tile
  // LDS stages of A and B.  Tiles of 65 to 128 rows cut along their columns (NJ = 2) have room for a fourth, and a launch of few such tiles is
  // bound by the loads a compute unit has in flight: calls of dense 4096 x 11008, 90 / 100 tokens 78.2 -> 73.6 / 81.2 -> 76.9 us, 128 tokens 85.8 -> 82.0.
  // Not below, where LDS reads and the barrier of a k-tile take longer than its loads: five stages gained 1 to 5 % with 48 and 64 tokens (4096 x
  // 8192 and x 4096) and lost 2 to 6 % with 8 and 24 (4864 x 1664 35.1 -> 37.4, 1024 x 1024 17.2 -> 17.9: the ring is full later).
  static constexpr bool DEEP = NJ == 2 && FA >= 3 && FA <= 4;
  static constexpr int NA = DEEP ? 4 : FA <= 5 ? 3 : 2;
  static constexpr int NB = DEEP || FA <= 2 ? 4 : FA <= 5 ? 3 : 2;
  static constexpr int A_STAGE = BM * 128;
  static constexpr int B_STAGE = BNW * 128;
  static constexpr int B_OFF = NA * A_STAGE;
  static constexpr int LDS = B_OFF + NB * B_STAGE;
  static constexpr int BL = NJ;                                    // direct-to-LDS loads of B per wave and k-tile
  static constexpr int R = NA > NB ? NA : NB;
  // fragments of a phase, fragments before it
  static constexpr int frags(int p) {
    return NP == 1 ? FA : NP == 2 ? (p == 0 ? (FA + 1) / 2 : FA / 2) : p == 0 ? 4 : p == 1 ? FA - 6 : 2;
  }
  static constexpr int frag0(int p) { return p == 0 ? 0 : frag0(p - 1) + frags(p - 1); }
  // A loads of a wave for a phase's region (32 rows per fragment, both groups): 8 rows each, for an odd number of fragments one
  // of 4 rows (half the lanes); loads before the phase's
  static constexpr int aloads(int p) { return (frags(p) + 1) / 2; }
  static constexpr int aload0(int p) { return p == 0 ? 0 : aload0(p - 1) + aloads(p - 1); }
  static constexpr int ALD = aload0(NP - 1) + aloads(NP - 1);
  static constexpr int phase_of(int i) { int p = 0; while (i >= aload0(p) + aloads(p)) ++p; return p; }
  static constexpr bool half(int i) { return frags(phase_of(i)) % 2 == 1 && i == aload0(phase_of(i)) + aloads(phase_of(i)) - 1; }

  // Loads of a wave that may still be in flight when the data of the phase after phase q of tile `it` must have landed, with
  // `rem` tiles after tile `it`: those issued later than the last load of that data.  The order of issue is the loop's.
  static constexpr int younger_at(int it, int q, int rem) {
    const int nk = it + 1 + rem;
    int pos = 0, last = 0;
    bool any = false;
    for (int step = -1; step < it * NP + q + 1; ++step) {
      const int t0 = step < 0 ? 0 : step / NP, q0 = step < 0 ? 0 : step % NP;
      const int n_t = step < 0 ? R : 1;  // the prologue issues tiles 0 .. R-1
      for (int t = 0; t < n_t; ++t)
        for (int p = 0; p < NP; ++p) {
          const int at = step < 0 ? (t < NA ? t : -1) : refill_a(t0, q0, p, nk), bt = p > 0 ? -1 : step < 0 ? (t < NB ? t : -1) : refill_b(t0, q0, nk);
          if (at >= 0 && at < nk) { pos += aloads(p); if (q < NP - 1 ? at == it && p == q + 1 : at == it + 1 && p == 0) { last = pos; any = true; } }
          if (bt >= 0 && bt < nk) { pos += BL; if (q == NP - 1 && bt == it + 1) { last = pos; any = true; } }
        }
    }
    return any ? pos - last : pos;
  }
  // tile whose region p of A (whose B) is issued in phase q of tile `it`, -1: none
  static constexpr int refill_a(int it, int q, int p, int nk) {
    if (p != (q == 0 ? NP - 1 : q - 1)) return -1;
    const int t = (q == 0 ? it - 1 : it) + NA;
    return (q == 0 && it == 0) || t >= nk ? -1 : t;
  }
  static constexpr int refill_b(int it, int q, int nk) {
    if (q != (NP == 1 ? 0 : 1)) return -1;
    const int t = (NP == 1 ? it - 1 : it) + NB;
    return (NP == 1 && it == 0) || t >= nk ? -1 : t;
  }
  static constexpr int younger(int q, int rem) {
    int n = 63;
    for (int it = 0; it < 2 * R + 2; ++it) { const int y = younger_at(it, q, rem); n = y < n ? y : n; }
    return n;
  }
  // the same for the first phase of tile 0 behind the prologue of a loop of nk tiles (a k-split of FC2 may have fewer than stages; a wait for all
  // of them there took dense 5120 x 1024, 120 tokens, from 57.7 to 58.7 us with the fourth stage)
  static constexpr int younger_start(int nk) {
    int n = ALD - aloads(0);
    for (int t = 1; t < nk && t < R; ++t) n += (t < NA ? ALD : 0) + (t < NB ? BL : 0);
    return n;
  }
  static_assert(LDS <= KERNEL_LDS, "ring does not fit");
};

// first LDS row of the rows that wave w's i-th A load of a k-tile fills
template <class P, int I> __device__ __forceinline__ int ring_a_row(int w) {
  constexpr int p = P::phase_of(I), f = P::frags(p);
  const int rr = P::half(I) ? f / 2 * 64 + w * 4 : (I - P::aload0(p)) * 64 + w * 8;  // row inside the phase's region of 2 x 16 f rows
  const int g = rr >= 16 * f ? 1 : 0;
  return g * 16 * P::FA + P::frag0(p) * 16 + rr - g * 16 * f;
}
template <int N, class F> __device__ __forceinline__ void unroll(F f) {
  if constexpr (N > 0) {
    unroll<N - 1>(f);
    f(std::integral_constant<int, N - 1>{});
  }
}

template <int R, class P, int Q> __device__ __forceinline__ void ring_wait(int rem) {
  if constexpr (R == 0) {
    wait_vmcnt<P::younger(Q, 0)>();
  } else {
    if (rem >= R) wait_vmcnt<P::younger(Q, R)>();
    else ring_wait<R - 1, P, Q>(rem);
  }
}

template <int N, class P> __device__ __forceinline__ void ring_wait_start(int nk) {
  if constexpr (N == 1) {
    wait_vmcnt<P::younger_start(1)>();
  } else {
    if (nk >= N) wait_vmcnt<P::younger_start(N)>();
    else ring_wait_start<N - 1, P>(nk);
  }
}

// acc[i][j] += the 16 x 16 tile (rows i*16.., B rows j*16..) of the wave over nk k-tiles, transposed: lane l holds row
// l%16 and the four consecutive B rows 4*(l/16) .. +3, i.e. output columns that are adjacent in memory.
//   issue_a(i, stage, kt): wave's i-th A load of tile kt into LDS at `stage` (rows ring_a_row);  issue_b(stage, kt): its 4 B
//   loads;  boff[ks]: byte offset of the lane's piece of B fragment 0 in k-step ks inside a B stage, BJ: bytes
//   between fragments.  (Fragment addresses are one lane offset per k-step and operand plus constants: the swizzle of
//   row r is that of r + 16.  Left to the compiler they were 16 registers.)
template <class P, int BJ, class IA, class IB>
__device__ __forceinline__ void gemm_pingpong(unsigned char* lds, int nk, int lane, int wr, f32x4 (&acc)[P::FA][P::NJ],
                                              IA issue_a, IB issue_b, const uint32_t (&boff)[2]) {
  constexpr int FP = P::frags(0);
  // With up to 64 rows a slot of matrix instructions is far shorter than one of loads and LDS reads, and the groups in turn
  // only add their latencies: there all waves read, pass one barrier per k-tile and multiply.  (What is read was waited for
  // before that barrier, and what is refilled after it was read before it.)  Dense layers of 13 to 61 tokens: 4352 x 7232
  // 62.3 -> 59.2 us, 3328 x 1472 41.4 -> 39.0, 2816 x 4928 47.3 -> 45.9; the 128-row body loses 2 to 12 % by it.
  constexpr bool PONG = P::FA > 2;
  bf16x8 fa[FP][2], fb[P::NJ][2];
  const uint32_t aoff[2] = {(uint32_t)swz(wr * 16 * P::FA + (lane & 15), lane >> 4), (uint32_t)swz(wr * 16 * P::FA + (lane & 15), 4 + (lane >> 4))};
  auto issue_region = [&](auto pc, int stage, int kt) {
    constexpr int p = decltype(pc)::value;
    unroll<P::aloads(p)>([&](auto i) { issue_a(std::integral_constant<int, P::aload0(p) + decltype(i)::value>{}, lds + stage * P::A_STAGE, kt); });
  };
  auto b_stage = [&](int stage) { return lds + P::B_OFF + stage * P::B_STAGE; };
  auto phase = [&](auto qc, int it, int sta, int stb) {
    constexpr int q = decltype(qc)::value;
    constexpr int nf = P::frags(q), f0 = P::frag0(q);
    const unsigned char *sa = lds + sta * P::A_STAGE, *sb = b_stage(stb);
    if constexpr (q == 0) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int j = 0; j < P::NJ; ++j) fb[j][ks] = as_bf16x8(*reinterpret_cast<const u32x4*>(sb + boff[ks] + j * BJ));
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < nf; ++i) fa[i][ks] = as_bf16x8(*reinterpret_cast<const u32x4*>(sa + aoff[ks] + (f0 + i) * 2048));
    // refill the regions that both groups have read: those of the previous phase
    if constexpr (q == 0) {
      if (it > 0 && it - 1 + P::NA < nk) issue_region(std::integral_constant<int, P::NP - 1>{}, sta == 0 ? P::NA - 1 : sta - 1, it - 1 + P::NA);
      if constexpr (P::NP == 1)
        if (it > 0 && it - 1 + P::NB < nk) issue_b(b_stage(stb == 0 ? P::NB - 1 : stb - 1), it - 1 + P::NB);
    } else {
      if (it + P::NA < nk) issue_region(std::integral_constant<int, q - 1>{}, sta, it + P::NA);
      if constexpr (q == 1)
        if (it + P::NB < nk) issue_b(b_stage(stb), it + P::NB);
    }
    ring_wait<P::R, P, q>(nk - 1 - it);
    wait_lgkmcnt0();
    __builtin_amdgcn_sched_barrier(0);
    block_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < nf; ++i)
#pragma unroll
        for (int jj = 0; jj < P::NJ; ++jj) {
          const int j = (i & 1) ? P::NJ - 1 - jj : jj;
          acc[f0 + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j][ks], fa[i][ks], acc[f0 + i][j], 0, 0, 0);
        }
    if constexpr (PONG) {
      __builtin_amdgcn_sched_barrier(0);
      block_barrier();
      __builtin_amdgcn_sched_barrier(0);
    }
  };
#pragma unroll
  for (int i = 0; i < P::FA; ++i)
#pragma unroll
    for (int j = 0; j < P::NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < P::R; ++t)
    if (t < nk)
      unroll<P::NP>([&](auto p) {
        if (t < P::NA) issue_region(p, t, t);
        if (p == 0 && t < P::NB) issue_b(b_stage(t), t);
      });
  ring_wait_start<P::R, P>(nk);  // the first region of A and B of tile 0
  block_barrier();
  __builtin_amdgcn_sched_barrier(0);
  if (PONG && wr == 1) block_barrier();
  __builtin_amdgcn_sched_barrier(0);
  int sta = 0, stb = 0;
  for (int it = 0; it < nk; ++it) {
    unroll<P::NP>([&](auto q) { phase(q, it, sta, stb); });
    sta = sta + 1 == P::NA ? 0 : sta + 1;
    stb = stb + 1 == P::NB ? 0 : stb + 1;
  }
  if (!PONG || wr == 0) block_barrier();  // the second group's last slot
}

// ---------------------------------------------------------------------------------------------
// The same loop for weights in the 4-bit storage form.  The codes of a B tile and their scales travel to LDS by direct loads
// like A, NQ tiles ahead, every wave its own 1/8 (lane: 16 bytes of codes, i.e. 32 weights of one row or column, and the
// aligned word that holds their scale).  A wave reads them back into registers and writes them as bf16((code - 8) * scale)
// into the B stage that both groups have just read, the stage of tile it + 2: the conversion is vector work in the slots of the
// matrix instructions, 2 between each two of them, so that the memory slots are those of the bf16 loop.  (Before, codes
// came in registers by inline loads and were converted in the memory slots; 777 tokens over 8 experts of 14336: 668 -> 605 us;
// dense 4096 x 28672, 32 / 128 / 192 / 256 / 1024 tokens: 164 / 215 / 246 / 264 / 695 -> 143 / 192 / 215 / 236 / 644, of that the
// vector work of the conversion about a tenth; with bf16 weights 243 / 569 for the last two.)
// Two phases (more than 128 rows): pieces 0 and 1 of tile it + 2 in the last slot of tile it, 2 and 3 in the first of it + 1; one
// phase: all four after the barrier.  A k-tile of 64 is one scale group of either projection.
// Layers that hold a scale of 2^117 or more (WeightView::q4) run it still; all others gemm_q4 below, which is 1.05 to 1.6 times as fast.
// ---------------------------------------------------------------------------------------------
template <int FAV> struct RingQ {
  static constexpr int FA = FAV;
  static constexpr int NJ = 4;
  static constexpr int BM = 32 * FA;
  static constexpr int NP = FA <= 4 ? 1 : 2;
  static constexpr int NA = FA <= 4 ? 3 : 2;                // LDS stages of A
  static constexpr int NB = 2;                              // of converted B
  static constexpr int NQ = 3;                              // of codes
  static constexpr int AHEAD = NQ + 2;                      // codes of tile it + AHEAD replace those of tile it + 2
  static constexpr int A_STAGE = BM * 128;
  static constexpr int Q_WAVE = 1024 + 256;                 // codes and scales of a wave
  static constexpr int Q_STAGE = 8 * Q_WAVE;
  static constexpr int B_OFF = NA * A_STAGE, Q_OFF = B_OFF + NB * B_BYTES;
  static constexpr int LDS = Q_OFF + NQ * Q_STAGE;
  static constexpr int R = AHEAD;
  static constexpr int frags(int p) { return NP == 1 ? FA : p == 0 ? (FA + 1) / 2 : FA / 2; }
  static constexpr int frag0(int p) { return p == 0 ? 0 : frag0(p - 1) + frags(p - 1); }
  static constexpr int aloads(int p) { return (frags(p) + 1) / 2; }
  static constexpr int aload0(int p) { return p == 0 ? 0 : aload0(p - 1) + aloads(p - 1); }
  static constexpr int ALD = aload0(NP - 1) + aloads(NP - 1);
  static constexpr int phase_of(int i) { int p = 0; while (i >= aload0(p) + aloads(p)) ++p; return p; }
  static constexpr bool half(int i) { return frags(phase_of(i)) % 2 == 1 && i == aload0(phase_of(i)) + aloads(phase_of(i)) - 1; }
  // as Ring::younger_at; needed after phase q: the A rows of the next phase, and the codes where that phase reads them.  The
  // codes' loads of a phase are issued after its wait.
  static constexpr int younger_at(int it, int q, int rem) {
    const int nk = it + 1 + rem, steps = it * NP + q;
    int pos = 0, last = 0;
    bool any = false;
    const int next_it = q < NP - 1 ? it : it + 1, next_q = q < NP - 1 ? q + 1 : 0;
    auto codes = [&](int t) { if (t < nk) { pos += 2; if (next_q == NP - 1 && t == next_it + 2) { last = pos; any = true; } } };
    auto a = [&](int t, int p) { if (t < nk) { pos += aloads(p); if (t == next_it && p == next_q) { last = pos; any = true; } } };
    for (int t = 0; t < NQ; ++t) codes(t);
    for (int t = 0; t < NA; ++t)
      for (int p = 0; p < NP; ++p) a(t, p);
    for (int t = NQ; t < AHEAD; ++t) codes(t);
    for (int s = 0; s <= steps; ++s) {
      const int t = s / NP, p = s % NP;
      if (p == 0) { if (t > 0) a(t - 1 + NA, NP - 1); }
      else a(t + NA, p - 1);
      if (p == NP - 1 && s < steps) codes(t + AHEAD);
    }
    return any ? pos - last : pos;
  }
  static constexpr int younger(int q, int rem) {
    int n = 63;
    for (int it = 0; it < 2 * R + 2; ++it) { const int y = younger_at(it, q, rem); n = y < n ? y : n; }
    return n;
  }
  static_assert(LDS <= KERNEL_LDS, "ring does not fit");
};

// 16-byte LDS store the compiler does not see as one: with a direct-to-LDS load in flight it would otherwise wait
// for ALL vector-memory operations (vmcnt(0)) before any LDS store it cannot prove disjoint from the load's
// target, which would drain the ring every iteration.  Disjointness is by construction here (the stage written is
// not the target of any load), and completion is covered by the loop's own lgkmcnt(0) before each barrier.
__device__ inline void lds_store_b128(unsigned char* p, const u32x4& v) {
  const uint32_t a = (uint32_t)(uintptr_t)SI_LPTR(p);
  asm volatile("ds_write_b128 %0, %1" ::"v"(a), "v"(v) : "memory");
}

// direct global -> LDS load of 4 bytes per lane
__device__ inline void load_lds4(const void* base, uint32_t off, unsigned char* l) {
  typedef const unsigned char __attribute__((address_space(1))) gchar;
  asm volatile("" : "+s"(base));
  __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)((gchar*)base + off), SI_LPTR(l), 4, 0, 0);
}

// The 8 codes of a word as (c - 8) * scale in fp32, exact: f[2i], f[2i + 1] of nibbles i, i + 4.  A nibble inserted into 0x6400 is
// the fp16 value 1024 + c at bit 0 and 1024 + 16 c at bit 4, which one mixed multiply-add turns into the product: 13 instructions
// and 4 for the rounding to bf16 (21 with c formed first, 617 against 605 us for 777 tokens over 8 experts of 14336; 23 by byte
// conversions).  1032 times a scale of 2^117 or more may overflow: WIDE forms c first, and c * scale - 8 scale is good to 2^125.
// A layer that holds such a scale takes kernels of its own (WeightView::q4: k_prefill_*_q4), whose results are the same.
template <bool WIDE> struct ScaledCodes {
  uint32_t lo = 0x000F000Fu, hi = 0x00F000F0u, magic = 0x64006400u;
  __device__ __forceinline__ void hide() { asm volatile("" : "+v"(lo), "+v"(hi), "+s"(magic)); }  // (one and-or instruction each)
  __device__ __forceinline__ void operator()(uint32_t w, float s, float (&f)[8]) const {
    const float s_hi = WIDE ? s : s * 0.0625f, c_lo = s * (WIDE ? -8.f : -1032.f), c_hi = s * (WIDE ? -8.f : -72.f);
    const uint32_t w8 = w >> 8;
    f16x2 a = __builtin_bit_cast(f16x2, (w & lo) | magic), b = __builtin_bit_cast(f16x2, (w & hi) | magic);
    f16x2 c = __builtin_bit_cast(f16x2, (w8 & lo) | magic), d = __builtin_bit_cast(f16x2, (w8 & hi) | magic);
    if constexpr (WIDE) {
      const f16x2 base = {(_Float16)1024.f, (_Float16)1024.f}, sixteenth = {(_Float16)0.0625f, (_Float16)0.0625f};
      a -= base;
      b = (b - base) * sixteenth;
      c -= base;
      d = (d - base) * sixteenth;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      f[h] = __builtin_fmaf((float)a[h], s, c_lo);
      f[2 + h] = __builtin_fmaf((float)b[h], s_hi, c_hi);
      f[4 + h] = __builtin_fmaf((float)c[h], s, c_lo);
      f[6 + h] = __builtin_fmaf((float)d[h], s_hi, c_hi);
    }
  }
};

//   issue_a as above;  issue_q(slot, kt): the two loads of the wave's codes and scales;  scale(word, kt): the lane's scale;
//   conv(stage, codes word, scale, i): convert and store piece i
template <class P, int BJ, class IA, class IQ, class SC, class CV>
__device__ __forceinline__ void gemm_pingpong_q4(unsigned char* lds, int nk, int w, int lane, int wr, f32x4 (&acc)[P::FA][4],
                                                 IA issue_a, IQ issue_q, SC scale, CV conv, const uint32_t (&boff)[2]) {
  constexpr int FP = P::frags(0);
  constexpr bool PONG = P::NP > 1;
  bf16x8 fa[FP][2], fb[4][2];
  const uint32_t aoff[2] = {(uint32_t)swz(wr * 16 * P::FA + (lane & 15), lane >> 4), (uint32_t)swz(wr * 16 * P::FA + (lane & 15), 4 + (lane >> 4))};
  auto b_stage = [&](int stage) { return lds + P::B_OFF + stage * B_BYTES; };
  auto q_slot = [&](int slot) { return lds + P::Q_OFF + slot * P::Q_STAGE + w * P::Q_WAVE; };
  auto issue_region = [&](auto pc, int stage, int kt) {
    constexpr int p = decltype(pc)::value;
    unroll<P::aloads(p)>([&](auto i) { issue_a(std::integral_constant<int, P::aload0(p) + decltype(i)::value>{}, lds + stage * P::A_STAGE, kt); });
  };
  u32x4 rq = {0u, 0u, 0u, 0u};
  float sc = 0.f;
  auto read_codes = [&](int slot, int kt) {
    const unsigned char* s = q_slot(slot);
    rq = *reinterpret_cast<const u32x4*>(s + lane * 16);
    sc = scale(*reinterpret_cast<const uint32_t*>(s + 1024 + lane * 4), kt);
  };
  // sq: slot of the codes of tile it + 2
  auto phase = [&](auto qc, int it, int sta, int stb, int sq) {
    constexpr int q = decltype(qc)::value;
    constexpr int nf = P::frags(q), f0 = P::frag0(q);
    const unsigned char *sa = lds + sta * P::A_STAGE, *sb = b_stage(stb);
    if constexpr (q == 0) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int j = 0; j < 4; ++j) fb[j][ks] = as_bf16x8(*reinterpret_cast<const u32x4*>(sb + boff[ks] + j * BJ));
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < nf; ++i) fa[i][ks] = as_bf16x8(*reinterpret_cast<const u32x4*>(sa + aoff[ks] + (f0 + i) * 2048));
    if constexpr (q == P::NP - 1) read_codes(sq, it + 2);
    if constexpr (q == 0) {
      if (it > 0 && it - 1 + P::NA < nk) issue_region(std::integral_constant<int, P::NP - 1>{}, sta == 0 ? P::NA - 1 : sta - 1, it - 1 + P::NA);
    } else {
      if (it + P::NA < nk) issue_region(std::integral_constant<int, q - 1>{}, sta, it + P::NA);
    }
    ring_wait<P::R, P, q>(nk - 1 - it);
    wait_lgkmcnt0();
    if constexpr (q == P::NP - 1)
      if (it + P::AHEAD < nk) issue_q(q_slot(sq), it + P::AHEAD);
    __builtin_amdgcn_sched_barrier(0);
    block_barrier();
    __builtin_amdgcn_sched_barrier(0);
    // (past the last tile stale codes are converted into a stage that nobody reads any more)
    if constexpr (P::NP == 1) {
#pragma unroll
      for (int i = 0; i < 4; ++i) conv(b_stage(stb), rq[i], sc, i);
    } else {
#pragma unroll
      for (int i = 0; i < 2; ++i) conv(b_stage(q == 0 ? stb ^ 1 : stb), rq[q == 0 ? i + 2 : i], sc, q == 0 ? i + 2 : i);
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < nf; ++i)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          const int j = (i & 1) ? 3 - jj : jj;
          acc[f0 + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j][ks], fa[i][ks], acc[f0 + i][j], 0, 0, 0);
        }
#pragma unroll
    for (int i = 0; i < nf * 8; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one matrix instruction,
      __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);  // two vector instructions
    }
    if constexpr (PONG) {
      __builtin_amdgcn_sched_barrier(0);
      block_barrier();
      __builtin_amdgcn_sched_barrier(0);
    }
  };
#pragma unroll
  for (int i = 0; i < P::FA; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < P::NQ; ++t)
    if (t < nk) issue_q(q_slot(t), t);
#pragma unroll
  for (int t = 0; t < P::NA; ++t)
    if (t < nk) unroll<P::NP>([&](auto p) { issue_region(p, t, t); });
  wait_vmcnt<0>();
  // B of tiles 0 and 1; with two phases the second half of tile 1 follows in the first slot
  read_codes(0, 0);
#pragma unroll
  for (int i = 0; i < 4; ++i) conv(b_stage(0), rq[i], sc, i);
  read_codes(1, 1);
#pragma unroll
  for (int i = 0; i < (P::NP == 1 ? 4 : 2); ++i) conv(b_stage(1), rq[i], sc, i);
  wait_lgkmcnt0();
#pragma unroll
  for (int t = P::NQ; t < P::AHEAD; ++t)
    if (t < nk) issue_q(q_slot(t - P::NQ), t);
  block_barrier();
  __builtin_amdgcn_sched_barrier(0);
  if (PONG && wr == 1) block_barrier();
  __builtin_amdgcn_sched_barrier(0);
  int sta = 0, stb = 0, sq = 2;
  for (int it = 0; it < nk; ++it) {
    unroll<P::NP>([&](auto q) { phase(q, it, sta, stb, sq); });
    sta = sta + 1 == P::NA ? 0 : sta + 1;
    stb ^= 1;
    sq = sq + 1 == P::NQ ? 0 : sq + 1;
  }
  if (PONG && wr == 0) block_barrier();  // the second group's last slot
  // No converted weights may still be on their way to LDS when a wave goes on: the next pass or tile may run a body of another
  // size, whose codes and rows lie where this one's stages of B were.  (A barrier of its own; the wait in front of the barrier of
  // every slot instead costs 1.4 %: 777 tokens over 8 experts of 14336, 603 us against 597.)
  wait_lgkmcnt0();
  block_barrier();
}

// ---------------------------------------------------------------------------------------------
// 4-bit weights, converted in the registers of the wave that multiplies them.  The 8 waves of a block own 32 B rows each and all
// rows of the tile (wave tile (32 FA) x 32), so that no converted weight is shared: the codes of a wave and their scales travel to LDS
// by direct loads, some k-tiles ahead, into slots that only this wave reads; a lane reads the two words of each of its two B
// fragments, and while tile `it` is multiplied they become its operand registers for tile it + 1 (two sets).  The order of the
// products and sums is that of the bf16 loop.  A is read from LDS by all eight waves (256 bytes a clock: a quarter to a half of the
// matrix cycles).  The two wave groups take turns as in gemm_pingpong.
// What bounded the loop before it (weights converted into a B stage in LDS): the slots of the loads, 18 LDS reads in the longer
// ones, and the address unit.  A direct load takes the CU's address unit 17 cycles where its lanes cover runs of 128 bytes, 32 with runs of 64 and 62 with
// runs of 32 bytes, also when only 4 bytes a lane are loaded (measured); the codes and scales of FC1, rows of 32 and 2 bytes a k-tile, took 1000
// cycles of 2000.  Hence blocks of four k-tiles for FC1, of which a row is 128 bytes and its scales are one load.
// What bounds it now: few rows: the instructions of a slot (one in 4 to 8 cycles and wave: 81 vector and 26 scalar ones a k-tile, 91 and 31 by the
// counters of 24 rows, which hold prologue and epilogue too: vector units busy 0.64, matrix cores 0.20, address unit 0.38; with
// the places in a block known at run time only, 80 scalar ones, 44 instead of 40 us below); many: the matrix cores, busy 0.61 to 0.66, two slots a
// phase of 450 matrix cycles with 47 vector instructions beside them and 80 cycles for the barriers.
// Measured, FC1 of a dense 4096 x 32768 layer (256 tiles), us before -> now: 24 rows 61.6 -> 39.8, 48 67.3 -> 47.7, 112 81.6 -> 64.6, 144 91.8
// -> 76.3, 208 107.5 -> 93.8, 240 113.1 -> 107.7; calls: 777 tokens over 8 experts of 14336 601 -> 536 (other cards 577 -> 508, 615 -> 545); 35 drawn 4-bit shapes 1.03 to 1.60.
// Tried: one barrier per k-tile without turns (24 rows 51, 112 76, 208 104); half of the conversion in the slots of the loads (57, 80, 100:
// it then waits for the LDS reads); five fragments of rows and more in one phase (208 rows 113).
// ---------------------------------------------------------------------------------------------
// KB: k-tiles of a block of codes (4 for FC1, whose rows then are read 128 bytes at a time; 1 for FC2)
template <int FAV, int KBV> struct RingQR {
  static constexpr int FA = FAV, RF = 2 * FAV;              // row fragments of a wave: all of the tile
  static constexpr int BM = 32 * FA;
  static constexpr int NP = FA <= 4 ? 1 : FA <= 7 ? 2 : 3;  // phases per k-tile (fewer: no registers left for the rows of one)
  static constexpr int KB = KBV;
  static constexpr int A_STAGE = BM * 128;
  static constexpr int Q_CODES = KB * 1024;                 // codes of a wave in a block, then their scales
  static constexpr int Q_WAVE = Q_CODES + (KB == 1 ? 256 : 512);
  static constexpr int Q_STAGE = 8 * Q_WAVE;
  // LDS stages of A, blocks of codes, parts of a block (1 KB) that are issued in one k-tile
  static constexpr int NA = KB == 1 ? (FA >= 8 ? 3 : FA >= 6 ? 4 : FA >= 4 ? 5 : FA == 3 ? 6 : 8)
                                    : (FA >= 8 ? 2 : FA >= 6 ? 3 : FA == 5 ? 4 : FA == 4 ? 3 : FA == 3 ? 4 : FA == 2 ? 6 : 8);
  static constexpr int NB_ROOM = (KERNEL_LDS - NA * A_STAGE) / Q_STAGE, NB_MAX = KB == 1 ? 8 : 3;
  static constexpr int NB = NB_ROOM < NB_MAX ? NB_ROOM : NB_MAX;
  static constexpr int PP = KB > 1 && NB == 2 ? 2 : 1;
  static constexpr int Q_OFF = NA * A_STAGE;
  static constexpr int LDS = Q_OFF + NB * Q_STAGE;
  static constexpr int R = NA > (NB - 1) * KB + 1 ? NA : (NB - 1) * KB + 1;
  static constexpr int frags(int p) { return RF / NP + (p < RF % NP ? 1 : 0); }
  static constexpr int frag0(int p) { return p == 0 ? 0 : frag0(p - 1) + frags(p - 1); }
  // direct-to-LDS loads of A per wave for a phase's rows, 8 rows each (where the waves are more than the rows need, the last rows are
  // loaded more than once)
  static constexpr int aloads(int p) { return (frags(p) + 3) / 4; }
  static constexpr int aload0(int p) { return p == 0 ? 0 : aload0(p - 1) + aloads(p - 1); }
  static constexpr int ALD = aload0(NP - 1) + aloads(NP - 1);
  static constexpr int phase_of(int i) { int p = 0; while (i >= aload0(p) + aloads(p)) ++p; return p; }
  // word j = 2 f + s of the codes (fragment f, k-step s) is converted in phase
  static constexpr int conv_phase(int j) { return j * NP / 4; }
  static constexpr int convs(int p) { int n = 0; for (int j = 0; j < 4; ++j) n += conv_phase(j) == p; return n; }
  // loads of a block that are issued in the k-tile in front of the u-th of another one: parts u PP .. + PP - 1, with the first the scales
  static constexpr int qloads(int u) { return (u * PP < KB ? PP : 0) + (u == 0 ? 1 : 0); }
  // Loads of a wave that may still be in flight when the rows of the phase after phase q of tile `it`, and after the last phase the
  // codes of tile it + 2, must have landed, with `rem` tiles after tile `it`: those issued after them.  The order of issue is the loop's.
  static constexpr int younger_at(int it, int q, int rem) {
    const int nk = it + 1 + rem;
    int pos = 0, last = 0;
    const int ni = q < NP - 1 ? it : it + 1, nq = q < NP - 1 ? q + 1 : 0;
    auto a = [&](int t, int p) { if (t < nk) { pos += aloads(p); if (t == ni && p == nq) last = pos; } };
    auto codes = [&](int b, int n) { if (b * KB < nk) { pos += n; if (n > 0 && q == NP - 1 && it + 2 < nk && b == (it + 2) / KB) last = pos; } };
    for (int t = 0; t < (NA > NB - 1 ? NA : NB - 1); ++t) {
      if (t < NB - 1) codes(t, KB + 1);
      if (t < NA) for (int p = 0; p < NP; ++p) a(t, p);
    }
    codes(NB - 1, qloads(0));
    for (int s = 0; s <= it * NP + q; ++s) {
      const int t = s / NP, p = s % NP;
      if (p > 0) a(t + NA, p - 1);
      else if (t > 0) a(t - 1 + NA, NP - 1);
      if (p == 0 && s < it * NP + q) codes((t + 1) / KB + NB - 1, qloads((t + 1) % KB));
    }
    return last ? pos - last : 63;
  }
  static constexpr int younger(int q, int rem) {
    int n = 63;
    for (int it = 0; it < 2 * R + 2 * KB; ++it) { const int y = younger_at(it, q, rem); n = y < n ? y : n; }
    return n;
  }
  // the same for the codes of tiles 0 and 1 and the rows of tile 0, which are waited for before the loop
  static constexpr int younger_first() {
    int pos = 0, last = 0;
    for (int t = 0; t < (NA > NB - 1 ? NA : NB - 1); ++t) {
      if (t < NB - 1) { pos += KB + 1; if (t <= 1 / KB) last = pos; }
      if (t < NA) { pos += ALD; if (t == 0) last = pos; }
    }
    return pos + qloads(0) - last;
  }
  static_assert(LDS <= KERNEL_LDS && NB >= (KB == 1 ? 3 : 2) && NA >= 2, "ring does not fit");
};
// first LDS row of the rows that wave w's i-th A load of a k-tile fills
template <class P, int I> __device__ __forceinline__ int qr_a_row(int w) {
  constexpr int p = P::phase_of(I), first = (I - P::aload0(p)) * 8, n = P::frags(p) * 2;
  return P::frag0(p) * 16 + 8 * (first + 8 <= n ? first + w : min(first + w, n - 1));
}

//   issue_a(i, stage, kt): wave's i-th A load of tile kt;  issue_q(slot, block, part): the load of a part of a block's codes, with part 0
//   that of its scales;  read(slot, u, f, words): the two words of codes of the lane's fragment f of the block's u-th tile, and
//   their scale as the result;  conv(word, scale): 8 codes -> operand registers
template <class P, class IA, class IQ, class RD, class CV>
__device__ __forceinline__ void gemm_q4(unsigned char* lds, int nk, int w, int lane, f32x4 (&acc)[P::RF][2], IA issue_a, IQ issue_q, RD read, CV conv) {
  const int wr = w >> 2;
  const uint32_t aoff[2] = {(uint32_t)swz(lane & 15, lane >> 4), (uint32_t)swz(lane & 15, 4 + (lane >> 4))};
  // (stages and slots are byte offsets)
  unsigned char* const q_lds = lds + P::Q_OFF + w * P::Q_WAVE;
  auto issue_rows = [&](auto pc, int stage, int kt) {
    constexpr int p = decltype(pc)::value;
    unroll<P::aloads(p)>([&](auto i) { issue_a(std::integral_constant<int, P::aload0(p) + decltype(i)::value>{}, lds + stage, kt); });
  };
  bf16x8 fa[P::frags(0)][2];
  u32x4 fb[2][2][2];  // [set][fragment][k-step]
  uint32_t wq[2][2];
  float sc[2];
  auto read_codes = [&](int slot, int u) {
#pragma unroll
    for (int f = 0; f < 2; ++f) sc[f] = read(q_lds + slot, u, f, wq[f]);
  };
  auto issue_parts = [&](int slot, int block, int u) {
#pragma unroll
    for (int i = 0; i < P::PP; ++i)
      if (P::PP * P::KB == 1 || u * P::PP < P::KB) issue_q(q_lds + slot, block, u * P::PP + i);
  };
  int sta = 0, stp = (P::NA - 1) * P::A_STAGE;  // stage of the rows of tile it, and of the tile before
  int b = 0, sq = 0, sp = (P::NB - 1) * P::Q_STAGE;  // the block that holds the codes of tile it + 1, its slot, that of the block before
  auto next_block = [&]() {
    ++b;
    sp = sq;
    sq = sq == (P::NB - 1) * P::Q_STAGE ? 0 : sq + P::Q_STAGE;
  };
  // steady: at least R more tiles follow;  u: the place of tile it + 1 in its block
  auto phase = [&](auto qc, auto setc, auto steady, int it, int u) {
    constexpr int q = decltype(qc)::value, set = decltype(setc)::value, nf = P::frags(q), f0 = P::frag0(q);
    constexpr bool ST = decltype(steady)::value;
    const unsigned char* sa = lds + sta;
    if constexpr (q == 0) read_codes(sq, u);  // of tile it + 1 (past the last tile stale ones, for operands that nobody uses)
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int i = 0; i < nf; ++i) fa[i][s] = as_bf16x8(*reinterpret_cast<const u32x4*>(sa + aoff[s] + (f0 + i) * 2048));
    // refill the rows that both groups have read: those of the previous phase
    if constexpr (q == 0) {
      if (ST ? it > 0 : it > 0 && it - 1 + P::NA < nk) issue_rows(std::integral_constant<int, P::NP - 1>{}, stp, it - 1 + P::NA);
    } else {
      if (ST || it + P::NA < nk) issue_rows(std::integral_constant<int, q - 1>{}, sta, it + P::NA);
    }
    if constexpr (ST) wait_vmcnt<P::younger(q, P::R)>();
    else ring_wait<P::R, P, q>(nk - 1 - it);
    wait_lgkmcnt0();
    if constexpr (q == 0)
      if (ST || (b + P::NB - 1) * P::KB < nk) issue_parts(sp, b + P::NB - 1, u);
    __builtin_amdgcn_sched_barrier(0);
    block_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (P::conv_phase(j) == q) fb[set ^ 1][j >> 1][j & 1] = conv(wq[j >> 1][j & 1], sc[j >> 1]);
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int i = 0; i < nf; ++i)
#pragma unroll
        for (int ff = 0; ff < 2; ++ff) {
          const int f = (i & 1) ? 1 - ff : ff;
          acc[f0 + i][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(fb[set][f][s]), fa[i][s], acc[f0 + i][f], 0, 0, 0);
        }
    // (kept here: what only the next tile uses would otherwise be formed in front of it)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (P::conv_phase(j) == q) asm volatile("" : "+v"(fb[set ^ 1][j >> 1][j & 1]));
    constexpr int nm = nf * 4, nv = (P::convs(q) * 20 + nm - 1) / nm;
#pragma unroll
    for (int i = 0; i < nm; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one matrix instruction,
      __builtin_amdgcn_sched_group_barrier(0x002, nv, 0);  // the vector instructions of its share
    }
    __builtin_amdgcn_sched_barrier(0);
    block_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int i = 0; i < P::RF; ++i)
#pragma unroll
    for (int f = 0; f < 2; ++f) acc[i][f] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < (P::NA > P::NB - 1 ? P::NA : P::NB - 1); ++t) {
    if (t < P::NB - 1 && t * P::KB < nk)
#pragma unroll
      for (int i = 0; i < P::KB; ++i) issue_q(q_lds + t * P::Q_STAGE, t, i);
    if (t < P::NA && t < nk) unroll<P::NP>([&](auto p) { issue_rows(p, t * P::A_STAGE, t); });
  }
  if ((P::NB - 1) * P::KB < nk) issue_parts((P::NB - 1) * P::Q_STAGE, P::NB - 1, 0);
  if (nk >= P::R) wait_vmcnt<P::younger_first()>();
  else wait_vmcnt<0>();
  read_codes(0, 0);
#pragma unroll
  for (int j = 0; j < 4; ++j) fb[0][j >> 1][j & 1] = conv(wq[j >> 1][j & 1], sc[j >> 1]);
  wait_lgkmcnt0();
  block_barrier();
  __builtin_amdgcn_sched_barrier(0);
  if (wr == 1) block_barrier();
  __builtin_amdgcn_sched_barrier(0);
  // (the places of the tiles in their blocks and the register sets of their operands are known in the unrolled loop)
  constexpr int U = P::KB == 1 ? 2 : P::KB;
  const std::integral_constant<int, 0> set0;
  auto next_stage = [&]() {
    stp = sta;
    sta = sta == (P::NA - 1) * P::A_STAGE ? 0 : sta + P::A_STAGE;
  };
  int it = 0;
  for (; it + U - 1 + P::R < nk; it += U)
    unroll<U>([&](auto kc) {
      constexpr int k = decltype(kc)::value, u = (k + 1) % P::KB;
      if (u == 0) next_block();
      unroll<P::NP>([&](auto q) { phase(q, std::integral_constant<int, k & 1>{}, std::true_type{}, it + k, u); });
      next_stage();
    });
  for (int u = 0; it < nk; ++it) {
    if (++u == P::KB) { u = 0; next_block(); }
    unroll<P::NP>([&](auto q) { phase(q, set0, std::false_type{}, it, u); });
    next_stage();
#pragma unroll
    for (int j = 0; j < 4; ++j) fb[0][j >> 1][j & 1] = fb[1][j >> 1][j & 1];
  }
  if (wr == 0) block_barrier();  // the second group's last slot
}

// Epilogue of FC1: SiLU(gate) * up of the wave's 32 hidden columns -> bf16 Hact.  The loader puts the hidden columns of a
// wave into LDS in an order (gu_col) that leaves 8 adjacent columns in a lane, for one 16-byte store per fragment row: with
// the plain order, 2-byte stores and a full division this epilogue was 1180 vector instructions per wave, 5 us of a tile.
// chunk: of the wave's columns; col: their first column inside the launch's range
template <int FA, int NJ>
__device__ __forceinline__ void gateup_store(const f32x4 (&acc)[FA][NJ], const TileInfo& ti, const WeightView& wv, int chunk, int col, int wr,
                                             int lane, uint16_t* __restrict__ hact, int ldh) {
  if (chunk >= wv.n_chunks) return;
  // (the lane index is made opaque here so that the output addresses are formed after the main loop: formed
  // ahead of it they are live through it, which the 320-row body has no registers for)
  int el = lane;
  asm volatile("" : "+v"(el));
  const int row0 = ti.row0 + wr * (16 * FA) + (el & 15);
  uint16_t* dst = hact + (size_t)row0 * ldh + (wv.col0 + col + (el >> 4) * 2 * NJ);
#pragma unroll
  for (int i = 0; i < FA; ++i) {
    typedef uint32_t out_t __attribute__((ext_vector_type(NJ)));
    out_t o;
#pragma unroll
    for (int j = 0; j < NJ / 2; ++j)
#pragma unroll
      for (int r = 0; r < 2; ++r)
        o[j * 2 + r] = pack_bf16(silu_f(acc[i][j][2 * r]) * acc[i][j + NJ / 2][2 * r], silu_f(acc[i][j][2 * r + 1]) * acc[i][j + NJ / 2][2 * r + 1]);
    if (row0 + i * 16 < ti.row_end) *reinterpret_cast<out_t*>(dst + (size_t)(i * 16) * ldh) = o;
  }
}
// hidden column (of the 32 of a wave) whose gate / up row sits at LDS row r of the wave's 32: fragment j = r / 16, row
// n = r % 16 of it holds column 8*(n/4) + 4*j + n%4
__device__ inline int gu_col(int r) { return ((r & 12) << 1) + ((r >> 4) << 2) + (r & 3); }

// Epilogue of FC2: the wave's 64 output columns, overwritten or accumulated, 16 bytes per lane
template <int FA, int NJ>
__device__ __forceinline__ void down_store(const f32x4 (&acc)[FA][NJ], const TileInfo& ti, int n0, int wr, int lane, int M,
                                           float* __restrict__ out, int accumulate) {
  int el = lane;  // opaque, as in gateup_store
  asm volatile("" : "+v"(el));
  const int row0 = ti.row0 + wr * (16 * FA) + (el & 15), m0 = n0 + (el >> 4) * 4;
  float* dst = out + (size_t)row0 * M + m0;
#pragma unroll
  for (int i = 0; i < FA; ++i) {
    if (row0 + i * 16 < ti.row_end) {
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        if (m0 + j * 16 < M) {
          f32x4* d = reinterpret_cast<f32x4*>(dst + (size_t)(i * 16) * M + j * 16);
          *d = accumulate ? *d + acc[i][j] : acc[i][j];
        }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// FC1 + SwiGLU.  Tile: BM rows x 128 hidden columns (two chunks).  B rows in LDS are ordered so
// that wave column wc owns hidden columns [32 wc, 32 wc + 32): LDS B row = wc*64 + f*32 + r with
// f = 0 the gate row and f = 1 the up row of column 32 wc + gu_col(r); SiLU(gate)*up is then formed in
// registers from the two accumulator tiles of a wave.
// ---------------------------------------------------------------------------------------------
template <class P, class Take>
__device__ __forceinline__ void gateup_body(const uint16_t* __restrict__ x, int M, const Plan& p, int tc, int half, const TileInfo& ti,
                                            const WeightView& wv, uint16_t* __restrict__ hact, int ldh, unsigned char* lds, Take take) {
  const int tid = thread_of_item(), lane = tid % WAVE, w = __builtin_amdgcn_readfirstlane(tid / WAVE);  // wave index, known to be uniform
  const int wr = w >> 2, wc = w & 3;
  const uint16_t* ebase = wv.base + (size_t)ti.se * wv.expert_stride;

  // loader: a wave instruction fills 8 LDS rows (1 KB); lane/8 is the row, lane%8 the slot inside the
  // 128-byte row, which holds logical piece slot ^ ((row >> 1) & 7)
  const int lrow = lane >> 3, lpp = lane & 7;
  uint32_t a_src[P::ALD];  // byte offsets from x (the host checks that x spans less than 2^31 elements)
  unroll<P::ALD>([&](auto i) {
    const int lr = ring_a_row<P, i>(w) + lrow;  // LDS row of the A tile
    int row = ti.row0 + lr;
    row = row < ti.row_end ? row : ti.row_end - 1;
    a_src[i] = ((uint32_t)(ti.row_t0 >= 0 ? row - ti.row_t0 : p.row_token[row]) * (uint32_t)M + ((lpp ^ ((lr >> 1) & 7)) * 8)) * 2;
  });
  // B: LDS row w*8*NJ + i*8 + lrow.  A whole tile: chunk 2*tc + w/4, f = w%2 (gate / up block), column-in-chunk
  // jc = ((w/2)%2)*32 + gu_col(i*8 + lrow); half a tile: chunk 2*tc + half, f = w%2, jc = (w/2)*16 + i*8 + lrow.
  // Blocks are [M/PW panels][64 j][PW m] (cc_worker.h).
  const int chunk = 2 * tc + (P::NJ == 4 ? wc >> 1 : half);
  const int chunk_rel = __builtin_amdgcn_readfirstlane(min(2 * tc + (P::NJ == 4 ? w >> 2 : half), wv.n_chunks - 1));
  const uint16_t* b_blk = ebase + (size_t)(wv.chunk0 + chunk_rel) * 3 * CHUNK_J * M + (size_t)(w & 1) * CHUNK_J * M;
  const int jc0 = P::NJ == 4 ? ((w >> 1) & 1) * 32 + gu_col(lrow) : (w >> 1) * 16 + lrow;
  const int PW = panel_width(M);
  const int lc0 = lpp ^ (lrow >> 1);  // B piece for even i; odd i uses lc0 ^ 4

  // uniform bases and 32-bit lane offsets: two vector registers for the B addresses instead of eight (a k-tile never
  // crosses a panel, PW being a multiple of 64)
  uint32_t b_lane[2] = {(uint32_t)(jc0 * PW + lc0 * 8) * 2u, (uint32_t)(jc0 * PW + (lc0 ^ 4) * 8) * 2u};
  auto issue_a = [&](auto i, unsigned char* stage, int kt) {
    if (!P::half(i) || lane < 32) load_lds16(x + kt * BK, a_src[i], stage + ring_a_row<P, i>(w) * 128);
  };
  auto issue_b = [&](unsigned char* stage, int kt) {
    unsigned char* sb = stage + w * (P::NJ * 1024);
    const int k0 = kt * BK;
    const uint16_t* bk = b_blk + (size_t)(k0 / PW) * CHUNK_J * PW + k0 % PW;
#pragma unroll
    for (int i = 0; i < P::NJ; ++i) load_lds16(bk + (P::NJ == 4 ? gu_col(i * 8) : i * 8) * PW, b_lane[i & 1], sb + i * 1024);
  };
  f32x4 acc[P::FA][P::NJ];
  const int br = wc * 16 * P::NJ + (lane & 15);
  const uint32_t boff[2] = {(uint32_t)swz(br, lane >> 4), (uint32_t)swz(br, 4 + (lane >> 4))};
  gemm_pingpong<P, 2048>(lds, M / BK, lane, wr, acc, issue_a, issue_b, boff);
  take();
  gateup_store<P::FA, P::NJ>(acc, ti, wv, chunk, tc * 128 + (P::NJ == 4 ? wc * 32 : half * 64 + wc * 16), wr, lane, hact, ldh);
}

// A block picks the body for the rows its tile really has (whole-block branch), so a 40-row tile costs a 64-row
// body and a 140-row tile a 160-row one.  The bodies above 256 rows (160 accumulator registers, 144 KB of LDS) exist for the last
// tile of an expert only.  Tiles of at most 192 rows that hold all rows of their expert are bound by HBM: they ran a loop
// of their own before (weights through registers, four k-tiles ahead), which the ping-pong loop overtook because an
// iteration of it is shorter, not because more bytes are in flight (Mixtral-8x7B-shaped prompt of 512 tokens, about
// 128 rows per expert: gate/up 398 -> 366 us, down 205 -> 165 us; 24 tokens, 6 rows per expert: equal).
#define SI_PICK_BODY(ti, CALL)                         \
  switch (((ti).row_end - (ti).row0 + 31) / 32) {      \
    case 1: CALL(1, 4); break;                         \
    case 2: CALL(2, 4); break;                         \
    case 3: CALL(3, 4); break;                         \
    case 4: CALL(4, 4); break;                         \
    case 5: CALL(5, 4); break;                         \
    case 6: CALL(6, 4); break;                         \
    case 7: CALL(7, 4); break;                         \
    case 8: CALL(8, 4); break;                         \
    case 9: CALL(9, 4); break;                         \
    default: CALL(10, 4); break;                       \
  }
// A tile of at most CUT_COLUMNS_ROWS rows is cut along its columns (such tiles are bound by the weights, which each half then
// reads half of), others along their rows.
constexpr int CUT_COLUMNS_ROWS = 160;
#define SI_PICK_HALF_BODY(ti, CALL)                    \
  switch (((ti).row_end - (ti).row0 + 31) / 32) {      \
    case 1: CALL(1, 2); break;                         \
    case 2: CALL(2, 2); break;                         \
    case 3: CALL(3, 2); break;                         \
    case 4: CALL(4, 2); break;                         \
    default: CALL(5, 2); break;                        \
  }
// The 4-bit bodies stop at 256 rows (they have no registers for more fragments of A): the rows a last tile holds beyond 256
// take a second pass of the same block.  When a body returns no wave still reads the LDS rings (its last barrier follows every
// fragment read; gemm_q4's last reads of codes are of slots of the wave itself and are not used) or has a store to them on its way
// (gemm_pingpong_q4 waits), so the next pass may refill them.
#define SI_PICK_BODY_2PASS(ti, CALL)                                  \
  for (const int row_end_all_ = (ti).row_end;;) {                     \
    (ti).row_end = min(row_end_all_, (ti).row0 + TILE_ROWS);          \
    const bool more_ = (ti).row_end < row_end_all_;                   \
    auto take_ = [&]() { if (!more_) take(); };                       \
    switch (((ti).row_end - (ti).row0 + 31) / 32) {                   \
      case 1: CALL(1); break;                                         \
      case 2: CALL(2); break;                                         \
      case 3: CALL(3); break;                                         \
      case 4: CALL(4); break;                                         \
      case 5: CALL(5); break;                                         \
      case 6: CALL(6); break;                                         \
      case 7: CALL(7); break;                                         \
      default: CALL(8); break;                                        \
    }                                                                 \
    if (!more_) break;                                                \
    (ti).row0 = (ti).row_end;                                         \
    (ti).row_end = row_end_all_;                                      \
  }

__global__ __launch_bounds__(THREADS, 1) void k_prefill_gateup(const uint16_t* __restrict__ x, int M, Plan p,
                                                               int expert_sel, int x2_only,
                                                               int n_ctiles, WeightView wv_r, WeightView wv_s,
                                                               uint16_t* __restrict__ hact_r, int ldh_r, long hact_s, int ldh_s) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int n_ctiles_s = (wv_s.n_chunks + 1) / 2;
  const TileQueues tq = tile_queues(p, expert_sel, x2_only, n_ctiles, n_ctiles_s, true);
  run_items(tq, p.queue, p.queue + N_XCD * QUEUE_STRIDE, lds, [&](int q, int item, auto take) {
    int tc, half, halves;
    TileInfo ti;
    item_tile(tq, p, expert_sel, x2_only, q, item, n_ctiles, tc, ti, half, halves);
    const WeightView wv = ti.sh ? wv_s : wv_r;
    const int ldh = ti.sh ? ldh_s : ldh_r;
    uint16_t* hact = hact_r + (ti.sh ? hact_s : 0);
    if (!storage_index(wv, ti.e, ti.se)) return take();
#define SI_CALL_GU(FAV, NJV) gateup_body<Ring<FAV, NJV>>(x, scalar_of_item(M), p, tc, half, ti, wv, hact, ldh, lds, take)
    if (halves == 2 && ti.row_end - ti.row0 <= CUT_COLUMNS_ROWS) {
      SI_PICK_HALF_BODY(ti, SI_CALL_GU)
    } else {
      if (halves == 2 && !half_rows(ti, half)) return take();
      SI_PICK_BODY(ti, SI_CALL_GU)
    }
#undef SI_CALL_GU
  });
}

// inner index of an FC2 tile -> output columns, k-split and its chunks
struct DownRange { int nt, split, c_begin, c_end; };
__device__ __forceinline__ DownRange down_range(int inner, int n_ntiles, int n_split, int n_chunks) {
  DownRange d;
  int rem;
  d.split = small_div(inner, n_ntiles, d.nt);
  d.c_begin = small_div(n_chunks * d.split, n_split, rem);
  d.c_end = small_div(n_chunks * (d.split + 1), n_split, rem);
  return d;
}

// ---------------------------------------------------------------------------------------------
// FC2.  Tile: BM rows x 256 output columns m; contraction over the hidden columns of this
// k-split's chunk range (one chunk = 64 per step).  B operand: the down block of a chunk is
// [8 groups][M][8 j], i.e. already "8 consecutive k per (group, m)"; it is kept in that order in
// LDS ([group][256 m] x 16 bytes), read conflict free by consecutive lanes.
// Output slab `split` of yp: rows x M fp32; overwritten or accumulated.
// ---------------------------------------------------------------------------------------------
template <class P, class Take>
__device__ __forceinline__ void down_body(const uint16_t* __restrict__ hact, int ldh, int M, const DownRange& dr, int half, const TileInfo& ti,
                                          const WeightView& wv, float* __restrict__ yp, size_t slab_stride, int accumulate,
                                          unsigned char* lds, Take take) {
  const int c_begin = dr.c_begin, c_end = dr.c_end;
  if (c_begin >= c_end && accumulate) return take();  // nothing to add
  const int tid = thread_of_item(), lane = tid % WAVE, w = __builtin_amdgcn_readfirstlane(tid / WAVE);  // wave index, known to be uniform
  const int wr = w >> 2, wc = w & 3;
  const int n0 = dr.nt * BN + (P::NJ == 4 ? 0 : half * P::BNW);
  const uint16_t* ebase = wv.base + (size_t)ti.se * wv.expert_stride;
  float* out = yp + (size_t)dr.split * slab_stride;

  const int lrow = lane >> 3, lpp = lane & 7;
  uint32_t a_src[P::ALD];  // byte offsets from hact (the host checks that it spans less than 2^31 elements)
  unroll<P::ALD>([&](auto i) {
    const int lr = ring_a_row<P, i>(w) + lrow;
    int row = ti.row0 + lr;
    row = row < ti.row_end ? row : ti.row_end - 1;
    a_src[i] = ((uint32_t)row * (uint32_t)ldh + wv.col0 + ((lpp ^ ((lr >> 1) & 7)) * 8)) * 2;
  });
  // B: wave w loads group q = w of the chunk's down block ([M/NW tiles][8 q][NW m][8 i]), NJ x 64 output columns
  const int NW = ntile_width(M);
  const int nw_shift = __builtin_ctz(NW);
  uint32_t b_off[P::NJ];  // bytes, inside one chunk's down block
#pragma unroll
  for (int i = 0; i < P::NJ; ++i) {
    const int n = min(n0 + i * 64 + lane, M - 1);
    b_off[i] = (((uint32_t)(n >> nw_shift) * 8 + w) * NW + (n & (NW - 1))) * 16;  // NW is a power of two
  }

  if (c_begin < c_end) {
    auto issue_a = [&](auto i, unsigned char* stage, int kt) {
      if (!P::half(i) || lane < 32) load_lds16(hact + (c_begin + kt) * CHUNK_J, a_src[i], stage + ring_a_row<P, i>(w) * 128);
    };
    auto issue_b = [&](unsigned char* stage, int kt) {
      unsigned char* sb = stage + w * (P::NJ * 1024);
      const uint16_t* dblk = ebase + (size_t)(wv.chunk0 + c_begin + kt) * 3 * CHUNK_J * M + (size_t)2 * CHUNK_J * M;
#pragma unroll
      for (int i = 0; i < P::NJ; ++i) load_lds16(dblk, b_off[i], sb + i * 1024);
    };
    f32x4 acc[P::FA][P::NJ];
    const uint32_t b0 = ((lane >> 4) * P::BNW + wc * 16 * P::NJ + (lane & 15)) * 16;
    const uint32_t boff[2] = {b0, b0 + 4 * P::BNW * 16};
    gemm_pingpong<P, 256>(lds, c_end - c_begin, lane, wr, acc, issue_a, issue_b, boff);
    take();
    down_store<P::FA, P::NJ>(acc, ti, n0 + wc * 16 * P::NJ, wr, lane, M, out, accumulate);
  } else {
    // an empty k-split of an overwriting launch still has to define its slab
    take();
    for (int i = tid; i < P::BM * P::BNW; i += THREADS) {
      const int row = ti.row0 + i / P::BNW, m = n0 + i % P::BNW;
      if (row < ti.row_end && m < M) out[(size_t)row * M + m] = 0.f;
    }
  }
}

__global__ __launch_bounds__(THREADS, 1) void k_prefill_down(const uint16_t* __restrict__ hact_r, int ldh_r, int M, Plan p,
                                                             int expert_sel, int x2_only,
                                                             int n_ntiles, int split_r, WeightView wv_r, WeightView wv_s,
                                                             int ldh_s, long hact_s, int split_s, float* __restrict__ yp,
                                                             size_t slab_stride, int accumulate) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int n_in_r = n_ntiles * split_r, n_in_s = wv_s.n_chunks ? n_ntiles * split_s : 0;
  // (ids in ranges also when every expert has a single row tile: one expert's Hact rows, the A operand, a few MB,
  // then stay in one L2; dealt one by one every XCD re-reads every expert's rows for each of its column tiles: 512 tokens over
  // 8 experts of 14336 columns 540 -> 552 us)
  const TileQueues tq = tile_queues(p, expert_sel, x2_only, n_in_r, n_in_s, false);
  run_items(tq, p.queue + N_XCD * QUEUE_STRIDE, p.queue, lds, [&](int q, int item, auto take) {
    int inner, half, halves;
    TileInfo ti;
    item_tile(tq, p, expert_sel, x2_only, q, item, n_in_r, inner, ti, half, halves);
    const WeightView wv = ti.sh ? wv_s : wv_r;
    const int ldh = ti.sh ? ldh_s : ldh_r, n_split = ti.sh ? split_s : split_r;
    const uint16_t* hact = hact_r + (ti.sh ? hact_s : 0);
    const DownRange dr = down_range(inner, n_ntiles, n_split, wv.n_chunks);
    if (!storage_index(wv, ti.e, ti.se)) return take();
#define SI_CALL_DN(FAV, NJV) down_body<Ring<FAV, NJV>>(hact, ldh, scalar_of_item(M), dr, half, ti, wv, yp, slab_stride, accumulate, lds, take)
    if (halves == 2 && ti.row_end - ti.row0 <= CUT_COLUMNS_ROWS) {
      SI_PICK_HALF_BODY(ti, SI_CALL_DN)
    } else {
      if (halves == 2 && !half_rows(ti, half)) return take();
      SI_PICK_BODY(ti, SI_CALL_DN)
    }
#undef SI_CALL_DN
  });
}

// ---------------------------------------------------------------------------------------------
// The same two GEMMs on weights in the 4-bit storage form (chunk layout in cc_worker.h), converted on the way
// into the B stage.  Tiles, LDS layouts, fragment reads, matrix instructions and epilogues are those above.
// ---------------------------------------------------------------------------------------------
template <class P, class Take>
__device__ __forceinline__ void gateup_body_q4(const uint16_t* __restrict__ x, int M, const Plan& p, int tc, const TileInfo& ti,
                                               const WeightView& wv, uint16_t* __restrict__ hact, int ldh, unsigned char* lds, Take take) {
  const int tid = thread_of_item(), lane = tid % WAVE, w = __builtin_amdgcn_readfirstlane(tid / WAVE);  // wave index, known to be uniform
  const int wr = w >> 2, wc = w & 3;
  const unsigned char* ebase = reinterpret_cast<const unsigned char*>(wv.base + (size_t)ti.se * wv.expert_stride);

  const int lrow = lane >> 3, lpp = lane & 7;
  uint32_t a_src[P::ALD];  // byte offsets from x
  unroll<P::ALD>([&](auto i) {
    const int lr = ring_a_row<P, i>(w) + lrow;
    int row = ti.row0 + lr;
    row = row < ti.row_end ? row : ti.row_end - 1;
    a_src[i] = ((uint32_t)(ti.row_t0 >= 0 ? row - ti.row_t0 : p.row_token[row]) * (uint32_t)M + ((lpp ^ ((lr >> 1) & 7)) * 8)) * 2;
  });
  auto issue_a = [&](auto i, unsigned char* stage, int kt) {
    if (!P::half(i) || lane < 32) load_lds16(x + kt * BK, a_src[i], stage + ring_a_row<P, i>(w) * 128);
  };
  // B: wave w fills LDS rows [32 w, 32 w + 32) = (chunk 2*tc + w/4, gate (w even) or up block, columns
  // ((w/2)%2)*32 + gu_col(row) of the chunk); lane = (row lane/2, k-half lane%2): the 32 weights of its half row are
  // 16 bytes of codes, i.e. the pieces 4*(lane%2) .. +3 of the LDS row
  const int chunk_rel = __builtin_amdgcn_readfirstlane(min(2 * tc + (w >> 2), wv.n_chunks - 1));
  const unsigned char* cb = ebase + (size_t)(wv.chunk0 + chunk_rel) * q4_chunk_u16(M) * 2;
  const unsigned char *codes = cb + q4_off_codes(w & 1, M), *scales = cb + q4_off_scales(w & 1, M);
  const int jc = ((w >> 1) & 1) * 32 + gu_col(lane >> 1), kh = lane & 1;
  uint32_t q_lane = (uint32_t)(jc * (M / 2) + kh * 16);
  const uint32_t z_row = (uint32_t)(jc * (M / 64));  // index of the row's first scale
  auto issue_q = [&](unsigned char* slot, int kt) {
    load_lds16(codes + kt * 32, q_lane, slot);
    load_lds4(scales, (z_row + kt) / 2 * 4, slot + 1024);
  };
  auto scale = [&](uint32_t word, int kt) { return __uint_as_float((z_row + kt) & 1 ? word & 0xffff0000u : word << 16); };
  const uint32_t brow = (uint32_t)(w * 32 + (lane >> 1)), b_dst = brow * 128 + (((kh * 4) ^ ((brow >> 1) & 7)) << 4);
  ScaledCodes<true> codes_of;
  codes_of.hide();
  // a word holds elements 8i .. 8i+7 of the half row: nibbles p and p + 4 are elements 2p, 2p + 1 (cc_worker.h)
  auto conv = [&](unsigned char* stage, uint32_t word, float sc, int i) {
    float f[8];
    codes_of(word, sc, f);
    lds_store_b128(stage + (b_dst ^ (i << 4)), u32x4{pack_bf16(f[0], f[1]), pack_bf16(f[2], f[3]), pack_bf16(f[4], f[5]), pack_bf16(f[6], f[7])});
  };
  f32x4 acc[P::FA][4];
  const uint32_t boff[2] = {(uint32_t)swz(wc * 64 + (lane & 15), lane >> 4), (uint32_t)swz(wc * 64 + (lane & 15), 4 + (lane >> 4))};
  gemm_pingpong_q4<P, 2048>(lds, M / BK, w, lane, wr, acc, issue_a, issue_q, scale, conv, boff);
  take();
  gateup_store<P::FA, 4>(acc, ti, wv, 2 * tc + (wc >> 1), tc * 128 + wc * 32, wr, lane, hact, ldh);
}

__global__ __launch_bounds__(THREADS, 1) void k_prefill_gateup_q4(const uint16_t* __restrict__ x, int M, Plan p,
                                                                  int expert_sel, int x2_only,
                                                                  int n_ctiles, WeightView wv_r, WeightView wv_s,
                                                                  uint16_t* __restrict__ hact_r, int ldh_r, long hact_s, int ldh_s) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int n_ctiles_s = (wv_s.n_chunks + 1) / 2;
  const TileQueues tq = tile_queues(p, expert_sel, x2_only, n_ctiles, n_ctiles_s, true);
  run_items(tq, p.queue, p.queue + N_XCD * QUEUE_STRIDE, lds, [&](int q, int item, auto take) {
    int tc, half, halves;
    TileInfo ti;
    item_tile(tq, p, expert_sel, x2_only, q, item, n_ctiles, tc, ti, half, halves);
    const WeightView wv = ti.sh ? wv_s : wv_r;
    const int ldh = ti.sh ? ldh_s : ldh_r;
    uint16_t* hact = hact_r + (ti.sh ? hact_s : 0);
    if (!storage_index(wv, ti.e, ti.se) || (halves == 2 && !half_rows(ti, half))) return take();
#define SI_CALL_GU(FAV) gateup_body_q4<RingQ<FAV>>(x, scalar_of_item(M), p, tc, ti, wv, hact, ldh, lds, take_)
    SI_PICK_BODY_2PASS(ti, SI_CALL_GU)
#undef SI_CALL_GU
  });
}

template <class P, class Take>
__device__ __forceinline__ void down_body_q4(const uint16_t* __restrict__ hact, int ldh, int M, const DownRange& dr, const TileInfo& ti,
                                             const WeightView& wv, float* __restrict__ yp, size_t slab_stride, int accumulate,
                                             unsigned char* lds, Take take) {
  const int c_begin = dr.c_begin, c_end = dr.c_end;
  if (c_begin >= c_end && accumulate) return take();
  const int tid = thread_of_item(), lane = tid % WAVE, w = __builtin_amdgcn_readfirstlane(tid / WAVE);  // wave index, known to be uniform
  const int wr = w >> 2, wc = w & 3;
  const int n0 = dr.nt * BN;
  const unsigned char* ebase = reinterpret_cast<const unsigned char*>(wv.base + (size_t)ti.se * wv.expert_stride);
  float* out = yp + (size_t)dr.split * slab_stride;

  const int lrow = lane >> 3, lpp = lane & 7;
  uint32_t a_src[P::ALD];  // byte offsets from hact
  unroll<P::ALD>([&](auto i) {
    const int lr = ring_a_row<P, i>(w) + lrow;
    int row = ti.row0 + lr;
    row = row < ti.row_end ? row : ti.row_end - 1;
    a_src[i] = ((uint32_t)row * (uint32_t)ldh + wv.col0 + ((lpp ^ ((lr >> 1) & 7)) * 8)) * 2;
  });
  auto issue_a = [&](auto i, unsigned char* stage, int kt) {
    if (!P::half(i) || lane < 32) load_lds16(hact + (c_begin + kt) * CHUNK_J, a_src[i], stage + ring_a_row<P, i>(w) * 128);
  };
  // B: thread = (output column n0 + (w%4)*64 + lane, j-half w/4): its 16 bytes of codes are the 32 hidden columns
  // of the half for that output column, i.e. the pieces 4*half .. +3 of the column in the [piece][column] B stage
  const int NW = ntile_width(M);
  const int half = w >> 2, col = (w & 3) * 64 + lane;
  const int n = min(n0 + col, M - 1);
  uint32_t q_lane = (uint32_t)(((n / NW) * 2 + half) * NW + (n & (NW - 1))) * 16;  // NW is a power of two
  const size_t cbytes = q4_chunk_u16(M) * 2;
  const unsigned char* cb0 = ebase + (size_t)(wv.chunk0 + c_begin) * cbytes;
  auto issue_q = [&](unsigned char* slot, int kt) {
    const unsigned char* cb = cb0 + (size_t)kt * cbytes;
    load_lds16(cb + q4_off_codes(2, M), q_lane, slot);
    load_lds4(cb + q4_off_scales(2, M), (uint32_t)n / 2 * 4, slot + 1024);
  };
  auto scale = [&](uint32_t word, int) { return __uint_as_float(n & 1 ? word & 0xffff0000u : word << 16); };
  ScaledCodes<true> codes_of;
  codes_of.hide();
  // a word holds hidden columns 8i .. 8i+7 of the half: nibbles p and p + 4 are elements (0, 2), (4, 6), (1, 3), (5, 7) (cc_worker.h)
  auto conv = [&](unsigned char* stage, uint32_t word, float sc, int i) {
    float f[8];
    codes_of(word, sc, f);
    lds_store_b128(stage + ((half * 4 + i) * BN + col) * 16, u32x4{pack_bf16(f[0], f[4]), pack_bf16(f[1], f[5]), pack_bf16(f[2], f[6]), pack_bf16(f[3], f[7])});
  };
  if (c_begin < c_end) {
    f32x4 acc[P::FA][4];
    const uint32_t b0 = ((lane >> 4) * BN + wc * 64 + (lane & 15)) * 16;
    const uint32_t boff[2] = {b0, b0 + 4 * BN * 16};
    gemm_pingpong_q4<P, 256>(lds, c_end - c_begin, w, lane, wr, acc, issue_a, issue_q, scale, conv, boff);
    take();
    down_store<P::FA, 4>(acc, ti, n0 + wc * 64, wr, lane, M, out, accumulate);
  } else {
    take();
    for (int i = tid; i < P::BM * BN; i += THREADS) {
      const int row = ti.row0 + i / BN, m = n0 + i % BN;
      if (row < ti.row_end && m < M) out[(size_t)row * M + m] = 0.f;
    }
  }
}

__global__ __launch_bounds__(THREADS, 1) void k_prefill_down_q4(const uint16_t* __restrict__ hact_r, int ldh_r, int M, Plan p,
                                                                int expert_sel, int x2_only,
                                                                int n_ntiles, int split_r, WeightView wv_r, WeightView wv_s,
                                                                int ldh_s, long hact_s, int split_s, float* __restrict__ yp,
                                                                size_t slab_stride, int accumulate) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int n_in_r = n_ntiles * split_r, n_in_s = wv_s.n_chunks ? n_ntiles * split_s : 0;
  const TileQueues tq = tile_queues(p, expert_sel, x2_only, n_in_r, n_in_s, false);
  run_items(tq, p.queue + N_XCD * QUEUE_STRIDE, p.queue, lds, [&](int q, int item, auto take) {
    int inner, half, halves;
    TileInfo ti;
    item_tile(tq, p, expert_sel, x2_only, q, item, n_in_r, inner, ti, half, halves);
    const WeightView wv = ti.sh ? wv_s : wv_r;
    const int ldh = ti.sh ? ldh_s : ldh_r, n_split = ti.sh ? split_s : split_r;
    const uint16_t* hact = hact_r + (ti.sh ? hact_s : 0);
    const DownRange dr = down_range(inner, n_ntiles, n_split, wv.n_chunks);
    if (!storage_index(wv, ti.e, ti.se) || (halves == 2 && !half_rows(ti, half))) return take();
#define SI_CALL_DN(FAV) down_body_q4<RingQ<FAV>>(hact, ldh, scalar_of_item(M), dr, ti, wv, yp, slab_stride, accumulate, lds, take_)
    SI_PICK_BODY_2PASS(ti, SI_CALL_DN)
#undef SI_CALL_DN
  });
}

// the bodies on gemm_q4 (above: on gemm_pingpong_q4, for layers with a scale of 2^117 or more)
template <class P, class Take>
__device__ __forceinline__ void gateup_body_qr(const uint16_t* __restrict__ x, int M, const Plan& p, int tc, const TileInfo& ti,
                                               const WeightView& wv, uint16_t* __restrict__ hact, int ldh, unsigned char* lds, Take take) {
  const int tid = thread_of_item(), lane = tid % WAVE, w = __builtin_amdgcn_readfirstlane(tid / WAVE);  // wave index, known to be uniform
  const unsigned char* ebase = reinterpret_cast<const unsigned char*>(wv.base + (size_t)ti.se * wv.expert_stride);

  const int lrow = lane >> 3, lpp = lane & 7;
  uint32_t a_src[P::ALD];  // byte offsets from x
  unroll<P::ALD>([&](auto i) {
    const int lr = qr_a_row<P, i>(w) + lrow;
    int row = ti.row0 + lr;
    row = row < ti.row_end ? row : ti.row_end - 1;
    a_src[i] = ((uint32_t)(ti.row_t0 >= 0 ? row - ti.row_t0 : p.row_token[row]) * (uint32_t)M + ((lpp ^ ((lr >> 1) & 7)) * 8)) * 2;
  });
  auto issue_a = [&](auto i, unsigned char* stage, int kt) {
    load_lds16(x + kt * BK, a_src[i], stage + qr_a_row<P, i>(w) * 128);
  };
  // B: wave w owns the hidden columns 16 (w % 4) .. + 15 of chunk 2 * tc + w / 4: rows 0 .. 15 of its 32 are their gate rows (fragment 0),
  // 16 .. 31 their up rows.  A part of a block is 128 bytes, four k-tiles, of 8 rows; the 16-byte piece c of row r sits at piece
  // c ^ ((r >> 1) & 7) of its 128 bytes in LDS.
  const int chunk = 2 * tc + (w >> 2), chunk_rel = __builtin_amdgcn_readfirstlane(min(chunk, wv.n_chunks - 1));
  const unsigned char* cb = ebase + (size_t)(wv.chunk0 + chunk_rel) * q4_chunk_u16(M) * 2;
  const int j0 = (w & 3) * 16, MG = M / 64;
  const unsigned char *codes = cb + q4_off_codes(0, M) + (size_t)j0 * (M / 2), *scales = cb + q4_off_scales(0, M);
  const uint32_t up_codes = (uint32_t)(q4_off_codes(1, M) - q4_off_codes(0, M)), up_scales = (uint32_t)(q4_off_scales(1, M) - q4_off_scales(0, M));
  // even parts hold rows 0 .. 7 of the 16 gate / up rows, odd ones 8 .. 15
  const uint32_t q_even = (uint32_t)(lrow * (M / 2) + ((lpp ^ (lrow >> 1)) * 16)), q_odd = (uint32_t)((8 + lrow) * (M / 2) + ((lpp ^ (4 + (lrow >> 1))) * 16));
  // scales of a block: 16 bytes of lane = row (0 .. 31), from the aligned word that holds the first
  const uint32_t z_row = (uint32_t)((j0 + (lane & 15)) * MG), z_lane = ((lane >> 4) & 1) * up_scales;
  auto issue_q = [&](unsigned char* slot, int block, int part) {
    uint32_t off = (part & 1) ? q_odd : q_even;
    load_lds16(codes + ((part & 2) ? up_codes : 0u) + block * 128, off, slot + part * 1024);
    if (part == 0 && lane < 32) {
      uint32_t z = z_lane + (z_row + block * 4) / 2 * 4;
      load_lds16(scales, z, slot + P::Q_CODES);
    }
  };
  const int n = lane & 15;
  const uint32_t q_rd = (uint32_t)(n * 128 + (((n >> 1) & 7) << 4) + (lane >> 4) * 4), s_rd = (uint32_t)(P::Q_CODES + n * 16 + ((((j0 + n) * MG) & 1) << 1));
  auto read = [&](const unsigned char* slot, int u, int f, uint32_t (&words)[2]) {
#pragma unroll
    for (int s = 0; s < 2; ++s) words[s] = *reinterpret_cast<const uint32_t*>(slot + (q_rd ^ (uint32_t)((2 * u + s) << 4)) + f * 2048);
    return __uint_as_float((uint32_t)*reinterpret_cast<const uint16_t*>(slot + s_rd + u * 2 + f * 256) << 16);
  };
  ScaledCodes<false> codes_of;
  codes_of.hide();
  auto conv = [&](uint32_t word, float sc) {
    float f[8];
    codes_of(word, sc, f);
    return u32x4{pack_bf16(f[0], f[1]), pack_bf16(f[2], f[3]), pack_bf16(f[4], f[5]), pack_bf16(f[6], f[7])};
  };
  f32x4 acc[P::RF][2];
  gemm_q4<P>(lds, M / BK, w, lane, acc, issue_a, issue_q, read, conv);
  take();
  gateup_store<P::RF, 2>(acc, ti, wv, chunk, tc * 128 + w * 16, 0, lane, hact, ldh);
}

template <class P, class Take>
__device__ __forceinline__ void down_body_qr(const uint16_t* __restrict__ hact, int ldh, int M, const DownRange& dr, const TileInfo& ti,
                                             const WeightView& wv, float* __restrict__ yp, size_t slab_stride, int accumulate,
                                             unsigned char* lds, Take take) {
  const int c_begin = dr.c_begin, c_end = dr.c_end;
  if (c_begin >= c_end && accumulate) return take();
  const int tid = thread_of_item(), lane = tid % WAVE, w = __builtin_amdgcn_readfirstlane(tid / WAVE);  // wave index, known to be uniform
  const int n0 = dr.nt * BN;
  const unsigned char* ebase = reinterpret_cast<const unsigned char*>(wv.base + (size_t)ti.se * wv.expert_stride);
  float* out = yp + (size_t)dr.split * slab_stride;

  const int lrow = lane >> 3, lpp = lane & 7;
  uint32_t a_src[P::ALD];  // byte offsets from hact
  unroll<P::ALD>([&](auto i) {
    const int lr = qr_a_row<P, i>(w) + lrow;
    int row = ti.row0 + lr;
    row = row < ti.row_end ? row : ti.row_end - 1;
    a_src[i] = ((uint32_t)row * (uint32_t)ldh + wv.col0 + ((lpp ^ ((lr >> 1) & 7)) * 8)) * 2;
  });
  auto issue_a = [&](auto i, unsigned char* stage, int kt) {
    load_lds16(hact + (c_begin + kt) * CHUNK_J, a_src[i], stage + qr_a_row<P, i>(w) * 128);
  };
  // B: wave w owns the output columns n0 + 32 w .. + 31.  A block is one chunk: 16 bytes, 32 hidden columns, of lane = (column lane % 32,
  // j-half lane / 32), and the words of the columns' scales
  const int NW = ntile_width(M);
  const int nl = min(n0 + w * 32 + (lane & 31), M - 1);
  uint32_t q_lane = (uint32_t)(((nl / NW) * 2 + (lane >> 5)) * NW + (nl & (NW - 1))) * 16;  // NW is a power of two
  const size_t cbytes = q4_chunk_u16(M) * 2;
  const unsigned char* cb0 = ebase + (size_t)(wv.chunk0 + c_begin) * cbytes;
  auto issue_q = [&](unsigned char* slot, int block, int) {
    const unsigned char* cb = cb0 + (size_t)block * cbytes;
    load_lds16(cb + q4_off_codes(2, M), q_lane, slot);
    load_lds4(cb + q4_off_scales(2, M), (uint32_t)nl / 2 * 4, slot + P::Q_CODES);
  };
  const uint32_t q_rd = (uint32_t)((lane & 15) * 16 + (lane >> 4) * 4), s_rd = (uint32_t)(P::Q_CODES + (lane & 15) * 4 + (lane & 1) * 2);
  auto read = [&](const unsigned char* slot, int, int f, uint32_t (&words)[2]) {
#pragma unroll
    for (int s = 0; s < 2; ++s) words[s] = *reinterpret_cast<const uint32_t*>(slot + q_rd + f * 256 + s * 512);
    return __uint_as_float((uint32_t)*reinterpret_cast<const uint16_t*>(slot + s_rd + f * 64) << 16);
  };
  ScaledCodes<false> codes_of;
  codes_of.hide();
  auto conv = [&](uint32_t word, float sc) {
    float f[8];
    codes_of(word, sc, f);
    return u32x4{pack_bf16(f[0], f[4]), pack_bf16(f[1], f[5]), pack_bf16(f[2], f[6]), pack_bf16(f[3], f[7])};
  };
  if (c_begin < c_end) {
    f32x4 acc[P::RF][2];
    gemm_q4<P>(lds, c_end - c_begin, w, lane, acc, issue_a, issue_q, read, conv);
    take();
    down_store<P::RF, 2>(acc, ti, n0 + w * 32, 0, lane, M, out, accumulate);
  } else {
    take();
    for (int i = tid; i < P::BM * BN; i += THREADS) {
      const int row = ti.row0 + i / BN, m = n0 + i % BN;
      if (row < ti.row_end && m < M) out[(size_t)row * M + m] = 0.f;
    }
  }
}

__global__ __launch_bounds__(THREADS, 1) void k_prefill_gateup_qr(const uint16_t* __restrict__ x, int M, Plan p,
                                                                  int expert_sel, int x2_only,
                                                                  int n_ctiles, WeightView wv_r, WeightView wv_s,
                                                                  uint16_t* __restrict__ hact_r, int ldh_r, long hact_s, int ldh_s) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int n_ctiles_s = (wv_s.n_chunks + 1) / 2;
  const TileQueues tq = tile_queues(p, expert_sel, x2_only, n_ctiles, n_ctiles_s, true);
  run_items(tq, p.queue, p.queue + N_XCD * QUEUE_STRIDE, lds, [&](int q, int item, auto take) {
    int tc, half, halves;
    TileInfo ti;
    item_tile(tq, p, expert_sel, x2_only, q, item, n_ctiles, tc, ti, half, halves);
    const WeightView wv = ti.sh ? wv_s : wv_r;
    const int ldh = ti.sh ? ldh_s : ldh_r;
    uint16_t* hact = hact_r + (ti.sh ? hact_s : 0);
    if (!storage_index(wv, ti.e, ti.se) || (halves == 2 && !half_rows(ti, half))) return take();
#define SI_CALL_GU(FAV) gateup_body_qr<RingQR<FAV, 4>>(x, scalar_of_item(M), p, tc, ti, wv, hact, ldh, lds, take_)
    SI_PICK_BODY_2PASS(ti, SI_CALL_GU)
#undef SI_CALL_GU
  });
}

__global__ __launch_bounds__(THREADS, 1) void k_prefill_down_qr(const uint16_t* __restrict__ hact_r, int ldh_r, int M, Plan p,
                                                                int expert_sel, int x2_only,
                                                                int n_ntiles, int split_r, WeightView wv_r, WeightView wv_s,
                                                                int ldh_s, long hact_s, int split_s, float* __restrict__ yp,
                                                                size_t slab_stride, int accumulate) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int n_in_r = n_ntiles * split_r, n_in_s = wv_s.n_chunks ? n_ntiles * split_s : 0;
  const TileQueues tq = tile_queues(p, expert_sel, x2_only, n_in_r, n_in_s, false);
  run_items(tq, p.queue + N_XCD * QUEUE_STRIDE, p.queue, lds, [&](int q, int item, auto take) {
    int inner, half, halves;
    TileInfo ti;
    item_tile(tq, p, expert_sel, x2_only, q, item, n_in_r, inner, ti, half, halves);
    const WeightView wv = ti.sh ? wv_s : wv_r;
    const int ldh = ti.sh ? ldh_s : ldh_r, n_split = ti.sh ? split_s : split_r;
    const uint16_t* hact = hact_r + (ti.sh ? hact_s : 0);
    const DownRange dr = down_range(inner, n_ntiles, n_split, wv.n_chunks);
    if (!storage_index(wv, ti.e, ti.se) || (halves == 2 && !half_rows(ti, half))) return take();
#define SI_CALL_DN(FAV) down_body_qr<RingQR<FAV, 1>>(hact, ldh, scalar_of_item(M), dr, ti, wv, yp, slab_stride, accumulate, lds, take_)
    SI_PICK_BODY_2PASS(ti, SI_CALL_DN)
#undef SI_CALL_DN
  });
}

constexpr int MERGE_TERMS = 4;
__global__ __launch_bounds__(256) void k_prefill_combine(const float* __restrict__ yp, size_t slab_stride, int n_split, int split_s,
                                                         const float* __restrict__ ycc, int T, int k, int M, int n_x1,
                                                         int has_shared, Plan p, float* __restrict__ y) {
  const int t = blockIdx.y;
  const int m4 = blockIdx.x * 256 + threadIdx.x;
  // (the launch before has cleared one queue and used the other)
  if (t == 0 && blockIdx.x == 0 && threadIdx.x < 2 * N_XCD) p.queue[threadIdx.x * QUEUE_STRIDE] = 0;
  if (m4 * 4 >= M) return;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  // MERGE_TERMS terms at a time: their row indices (scalar loads) and then their rows are in flight together, and are added in their
  // order.  One after the other, two trips to memory each, the merge of 2011 tokens, 8 + 1 terms of 3584 columns took 66 us, of
  // 1817 tokens, 4 terms of 5888 columns 45; now 55 and 33 (214 MB, 6.5 TB/s).
  for (int s0 = 0; s0 < k; s0 += MERGE_TERMS) {
    const float* row[MERGE_TERMS];
    float wgt[MERGE_TERMS];
    float4 v[MERGE_TERMS];
#pragma unroll
    for (int u = 0; u < MERGE_TERMS; ++u) {
      const int q = t * k + min(s0 + u, k - 1);
      row[u] = yp + (size_t)(p.dense_T ? q : table(p.inv, q)) * M;
      wgt[u] = p.dense_T ? 1.f : __int_as_float(table(reinterpret_cast<const int32_t*>(p.w), q));
    }
#pragma unroll
    for (int u = 0; u < MERGE_TERMS; ++u)
      if (s0 + u < k) v[u] = reinterpret_cast<const float4*>(row[u])[m4];
    for (int q = 1; q < n_split; ++q)
#pragma unroll
      for (int u = 0; u < MERGE_TERMS; ++u)
        if (s0 + u < k) {
          const float4 v2 = reinterpret_cast<const float4*>(row[u] + (size_t)q * slab_stride)[m4];
          v[u].x += v2.x; v[u].y += v2.y; v[u].z += v2.z; v[u].w += v2.w;
        }
#pragma unroll
    for (int u = 0; u < MERGE_TERMS; ++u)
      if (s0 + u < k) {
        acc.x = fmaf(wgt[u], v[u].x, acc.x); acc.y = fmaf(wgt[u], v[u].y, acc.y);
        acc.z = fmaf(wgt[u], v[u].z, acc.z); acc.w = fmaf(wgt[u], v[u].w, acc.w);
      }
  }
  if (has_shared) {
    const float* row = yp + (size_t)(T * k + t) * M;
    float4 v[MAX_KSPLIT];
#pragma unroll
    for (int q = 0; q < MAX_KSPLIT; ++q)
      if (q < split_s) v[q] = reinterpret_cast<const float4*>(row + (size_t)q * slab_stride)[m4];
#pragma unroll
    for (int q = 0; q < MAX_KSPLIT; ++q)
      if (q < split_s) { acc.x += v[q].x; acc.y += v[q].y; acc.z += v[q].z; acc.w += v[q].w; }
  }
  if (ycc && t < n_x1) {
    const float4 v = reinterpret_cast<const float4*>(ycc + (size_t)t * M)[m4];
    acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
  }
  reinterpret_cast<float4*>(y + (size_t)t * M)[m4] = acc;
}

// grid: (blocks over the n elements, slabs)
__global__ void k_fill_zero(float* __restrict__ p, size_t n, size_t slab_stride) {
  p += blockIdx.y * slab_stride;
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = 0.f;
}

}  // namespace

static hipError_t ensure_lds_attr() {
  static hipError_t st = [] {
    const void* kernels[] = {(const void*)k_prefill_gateup, (const void*)k_prefill_down, (const void*)k_prefill_gateup_qr,
                             (const void*)k_prefill_down_qr, (const void*)k_prefill_gateup_q4, (const void*)k_prefill_down_q4};
    for (const void* k : kernels) {
      hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, KERNEL_LDS + NEXT_LDS);
      if (e != hipSuccess) return e;
      // The main loops count their own vector-memory operations (wait_vmcnt<N> against Ring::younger): a
      // register spill would add scratch loads and stores to that count and let a barrier pass before a tile has
      // landed.  A build whose GEMM kernels use scratch memory is refused here instead of computing wrong results.
      hipFuncAttributes fa{};
      e = hipFuncGetAttributes(&fa, k);
      if (e != hipSuccess) return e;
      if (fa.localSizeBytes != 0) return hipErrorInvalidDeviceFunction;
    }
    return hipSuccess;
  }();
  return st;
}

hipError_t launch_prefill_gateup(const uint16_t* x, int M, const Plan& plan, int expert_sel, int x2_only,
                                 int n_row_tiles, const WeightView& wv, uint16_t* hact, int ldh, const SharedPart& sp,
                                 hipStream_t stream) {
  if (wv.n_chunks <= 0 || n_row_tiles <= 0) return hipSuccess;
  hipError_t e = ensure_lds_attr();
  if (e != hipSuccess) return e;
  const int n_ctiles = (wv.n_chunks + 1) / 2;
  if (wv.q4)
    hipLaunchKernelGGL(wv.q4 == Q4_WIDE ? k_prefill_gateup_q4 : k_prefill_gateup_qr, dim3(N_XCD * XCD_CU), dim3(THREADS), KERNEL_LDS + NEXT_LDS, stream, x, M, plan, expert_sel, x2_only,
                       n_ctiles, wv, sp.wv, hact, ldh, sp.hact, sp.ldh);
  else
    hipLaunchKernelGGL(k_prefill_gateup, dim3(N_XCD * XCD_CU), dim3(THREADS), KERNEL_LDS + NEXT_LDS, stream, x, M, plan, expert_sel, x2_only,
                       n_ctiles, wv, sp.wv, hact, ldh, sp.hact, sp.ldh);
  return hipGetLastError();
}

hipError_t launch_prefill_down(const uint16_t* hact, int ldh, int M, const Plan& plan, int expert_sel,
                               int x2_only, int n_row_tiles, const WeightView& wv, float* yp, size_t slab_stride,
                               int n_split, int accumulate, const SharedPart& sp, hipStream_t stream) {
  if (wv.n_chunks <= 0 || n_row_tiles <= 0) return hipSuccess;
  hipError_t e = ensure_lds_attr();
  if (e != hipSuccess) return e;
  const int n_ntiles = (M + BN - 1) / BN;
  if (wv.q4)
    hipLaunchKernelGGL(wv.q4 == Q4_WIDE ? k_prefill_down_q4 : k_prefill_down_qr, dim3(N_XCD * XCD_CU), dim3(THREADS), KERNEL_LDS + NEXT_LDS, stream, hact, ldh, M, plan, expert_sel,
                       x2_only, n_ntiles, n_split, wv, sp.wv, sp.ldh, sp.hact, sp.split, yp, slab_stride, accumulate);
  else
    hipLaunchKernelGGL(k_prefill_down, dim3(N_XCD * XCD_CU), dim3(THREADS), KERNEL_LDS + NEXT_LDS, stream, hact, ldh, M, plan, expert_sel,
                       x2_only, n_ntiles, n_split, wv, sp.wv, sp.ldh, sp.hact, sp.split, yp, slab_stride, accumulate);
  return hipGetLastError();
}

hipError_t launch_prefill_combine(const float* yp, size_t slab_stride, int n_split, int split_s, const float* ycc, int T, int k, int M,
                                  int n_x1, int has_shared, const Plan& plan, float* y, hipStream_t stream) {
  if (T <= 0) return hipSuccess;
  dim3 grid((M / 4 + 255) / 256, T);
  hipLaunchKernelGGL(k_prefill_combine, grid, dim3(256), 0, stream, yp, slab_stride, n_split, split_s, ycc, T, k, M, n_x1,
                     has_shared, plan, y);
  return hipGetLastError();
}

hipError_t launch_fill_zero(float* p, size_t n, int n_slabs, size_t slab_stride, hipStream_t stream) {
  if (n == 0 || n_slabs <= 0) return hipSuccess;
  int blocks = (int)std::min<size_t>((n + 255) / 256, 4096);
  hipLaunchKernelGGL(k_fill_zero, dim3(blocks, n_slabs), dim3(256), 0, stream, p, n, slab_stride);
  return hipGetLastError();
}

}  // namespace si
