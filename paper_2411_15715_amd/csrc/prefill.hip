// Prompt-phase grouped GEMMs on the bf16 matrix cores (v_mfma_f32_16x16x32_bf16), fp32 accumulate.
//   gateup : Hact[row][j] = SiLU(X_e . Wg_e[j]) * (X_e . Wu_e[j])   (FC1 + activation, Eq. 1)
//   down   : Yp[row][m] (+)= Hact[row][:] . Wd_e[:, m]              (FC2, one term of Eq. 2)
//   combine: y[t] = sum_s w[t][s] Yp[row(t,s)] (+ shared expert row) (+ Y^CC for X1 rows)
// Rows are the expert-sorted (token, slot) pairs of the token assignment; a row tile never
// crosses an expert.  The gather of x rows is fused into the A-operand load of the first GEMM.
//
// Both GEMMs: one 512-thread block (8 waves, 2 per SIMD) per BM x 256 output tile, BK = 64, a ring of LDS
// stages filled by direct global->LDS loads (global_load_lds_dwordx4, no VGPR staging), wave tile
// (BM/2) x 64.  A row tile holds up to 256 rows, the last one of an expert up to 320 (si_internal.h: n_row_tiles);
// the block runs the body instantiated for BM = 64, 128, 192, 256 or 320, the smallest that covers the rows the
// tile really has.  The main loop is a ping-pong of two wave groups on v_mfma_f32_16x16x32_bf16 (gemm_pingpong;
// gemm_pingpong_q4 converts 4-bit weights on their way into LDS).
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
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
#define SI_LPTR(p) ((void __attribute__((address_space(3)))*)(p))

constexpr int WAVE = 64;
constexpr int THREADS = 512;
constexpr int BN = 256;  // B rows per tile: 128 hidden columns (gate+up) or 256 output columns
constexpr int BK = 64;
constexpr int B_BYTES = BN * BK * 2;  // 32 KB
constexpr int KERNEL_LDS = 144 * 1024;  // the largest body

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

// Hardware block id -> logical tile id.
//  * XCD-aware remap: consecutive hardware block ids go round-robin over the 8 XCDs; give each XCD a
//    contiguous range of logical ids so that the row tiles that read the same weights share an L2.  The
//    ranges are cut from the number of ids that really have work (known on the device only), so that no
//    XCD is handed a range of empty ids (with ranges cut from the grid's upper bound the remap cost more than
//    it saved on small tiles: the last XCD idled while the others carried its share).
//    When no expert of the launch has more than one row tile nothing is shared through the L2 but the few rows
//    of x, and tiles of different experts differ in cost (a 192-row tile streams its weights a quarter slower than
//    a 128-row one): the ids are then dealt round-robin (`interleave`), every XCD gets the same mix, and the launch
//    takes the mean of the experts' times instead of the slowest XCD's.
//  * Tail split: N tiles on n_cu compute units run in ceil(N / n_cu) rounds; when the last round is at most
//    half full each of its tiles gets two blocks, which share its rows if it has more than 128 (LLaMA-shaped
//    gate/up GEMM: 896 tiles = 3.5 rounds; the last round then costs about half a round).
__device__ inline bool map_block(int b, int N, int n_cu, int interleave, int& L, int& half, int& halves) {
  int r = N % n_cu;
  if (2 * r > n_cu) r = 0;
  const int main_n = N - r;
  const int per = (main_n + 7) / 8;
  if (b < 8 * per) {
    L = interleave ? b : (b % 8) * per + b / 8;
    half = 0;
    halves = 1;
    return L < main_n;
  }
  const int bt = b - 8 * per;
  if (bt >= 2 * r) return false;
  L = main_n + (bt >> 1);
  half = bt & 1;
  halves = 2;
  return true;
}

// se: index of the expert inside the launch's weight storage; sh: the shared expert in a launch that covers it as well
struct TileInfo { int e, row0, row_end, se, sh; };

// Number of logical tile ids with work in this launch (row tiles x inner tiles); single: no expert of the launch
// has more than one row tile.
__device__ inline int launch_extent(const Plan& p, int expert_sel, int x2_only, int n_inner, int& single) {
  if (expert_sel >= 0) {
    const int start = p.off[expert_sel] + (x2_only ? p.count1[expert_sel] : 0);
    const int nrt = n_row_tiles(p.off[expert_sel + 1] - start);
    single = nrt <= 1;
    return nrt * n_inner;
  }
  single = (*p.tile_flags >> (x2_only ? 1 : 0)) & 1;
  return (x2_only ? *p.n_tiles_x2 : *p.n_tiles) * n_inner;  // row tiles of the routed experts
}

// logical id L -> (expert, inner index, row tile) with the row tile varying fastest inside an
// expert: L / n_inner indexes the row-tile table, which yields the expert.
__device__ inline bool decode_tile(const Plan& p, int expert_sel, int x2_only, int L, int n_inner, int& inner,
                                   TileInfo& ti) {
  int e, first, nrt, start, end;
  if (expert_sel >= 0) {
    e = expert_sel;
    start = p.off[e] + (x2_only ? p.count1[e] : 0);
    end = p.off[e + 1];
    nrt = n_row_tiles(end - start);
    if (L >= nrt * n_inner) return false;
    first = 0;
  } else {
    const int n_tiles = x2_only ? *p.n_tiles_x2 : *p.n_tiles;
    const int t = L / n_inner;
    if (t >= n_tiles) return false;
    e = x2_only ? p.tile_e_x2[t] : p.tile_e[t];
    if (e >= p.n_routed) return false;
    first = t - (x2_only ? p.tile_r_x2[t] : p.tile_r[t]);
    start = p.off[e] + (x2_only ? p.count1[e] : 0);
    end = p.off[e + 1];
    nrt = n_row_tiles(end - start);
  }
  const int Le = L - first * n_inner;
  inner = Le / nrt;
  const int r = Le % nrt;
  ti.e = e;
  ti.row0 = start + r * TILE_ROWS;
  ti.row_end = r == nrt - 1 ? end : ti.row0 + TILE_ROWS;
  return true;
}

// Launch over the routed experts and the shared one: every XCD gets a contiguous eighth of either kind's ids, the shared
// expert's first: its tiles are the longest of the down projection and alike, and the smaller ones of the routed experts
// even out the end (a split tail as in map_block is not needed).  2011 tokens, 64 experts of 2560 columns, top-8, a
// shared one of 20480: 1829 us with two launches, 1761 like this, 1790 with the routed tiles first, 1827 with the two
// kinds in turn (their operands then share the L2s).
__device__ inline bool joint_tile(const Plan& p, int expert_sel, int n_inner, int n_inner_s, int spread, int& inner, TileInfo& ti) {
  int single;
  const int n_r = launch_extent(p, expert_sel, 0, n_inner, single);
  const int n_s = n_row_tiles(p.off[p.n_routed + 1] - p.off[p.n_routed]) * n_inner_s;
  const int per_r = (n_r + 7) / 8, per_s = (n_s + 7) / 8;
  const int xcd = blockIdx.x % 8, i = blockIdx.x / 8;
  const bool sh = i < per_s;
  const int idx = sh ? i : i - per_s, per = sh ? per_s : per_r;
  if (idx >= per) return false;
  const int L = !sh && single && spread ? idx * 8 + xcd : xcd * per + idx;
  if (L >= (sh ? n_s : n_r)) return false;
  ti.sh = sh;
  return decode_tile(p, sh ? p.n_routed : expert_sel, 0, L, sh ? n_inner_s : n_inner, inner, ti);
}

// block id -> tile of this block (false: nothing to do)
// n_inner_s: inner tiles of the shared expert when the launch covers it along with the routed ones, else 0
// spread: deal single-tile launches round-robin over the XCDs (see map_block)
__device__ inline bool block_tile(const Plan& p, int expert_sel, int x2_only, int n_inner, int n_inner_s, int n_cu, int spread,
                                  int& inner, TileInfo& ti) {
  ti.sh = 0;
  if (n_inner_s) return joint_tile(p, expert_sel, n_inner, n_inner_s, spread, inner, ti);
  int L, half, halves, single;
  const int extent = launch_extent(p, expert_sel, x2_only, n_inner, single);
  if (!map_block(blockIdx.x, extent, n_cu, single && spread, L, half, halves)) return false;
  if (!decode_tile(p, expert_sel, x2_only, L, n_inner, inner, ti)) return false;
  if (halves == 2) {
    const int rows = ti.row_end - ti.row0;
    if (rows <= 128) return half == 0;  // too few rows to share: the first block takes them all
    const int hs = ((rows + 1) / 2 + 31) / 32 * 32;
    ti.row0 += half * hs;
    ti.row_end = min(ti.row_end, ti.row0 + hs);
    if (ti.row0 >= ti.row_end) return false;
  }
  return true;
}

// ---------------------------------------------------------------------------------------------
// Main loop of the bf16 tiles: ping-pong of two wave groups.
// 8 waves as 2 (rows) x 4 (B-row quarters of 64), wave tile (BM/2) x 64 in v_mfma_f32_16x16x32_bf16 tiles.  Waves w and
// w + 4 share a SIMD; the second row group runs one barrier behind the first, so that in every slot between two
// barriers one wave of each SIMD issues matrix instructions and nothing else while the other reads its next fragments
// from LDS, issues tile loads and waits.  A k-tile of 64 is cut into phases of up to 64 rows per group (2 loads per wave,
// 4 fragments, 32 matrix instructions of 16 cycles); B is read in the first phase and kept in registers.
// A region of a stage (the rows of one phase, with B in the first) is free once both groups have read it, i.e. one phase
// later, and is refilled then with tile it + NST: at BM = 256 a load has three phases = 3072 matrix cycles to land.
// What bounds it: the power limit.  Counters of a 1024 x 65536 x 8192 product: matrix cores busy 0.90 of the time at a
// shader clock of 1.68 GHz (the loop with one barrier per k-tile that it replaces: 0.65 at 1.84 GHz): 1461 TFLOP/s against
// 1181.  The 16 x 16 x 32 instruction is part of it: register-resident on random operands it sustains 2.06 PFLOP/s under
// the power limit where the 32 x 32 x 16 one sustains 1.81 (its accumulators cost twice the register traffic).  Four
// phases of 16 matrix instructions (64 x 32 quadrants) measured 1378, one wave per SIMD with 128 x 128 tiles 1064.
// ---------------------------------------------------------------------------------------------
template <int BM, int BL = 4> struct PingPong {  // BL: direct-to-LDS loads of B per wave and k-tile (0: B travels through registers)
  static constexpr int NST = BM >= 192 ? 2 : 3;     // LDS stages
  static constexpr int STAGE = BM * 128 + B_BYTES;  // bytes per stage
  static constexpr int LDS = NST * STAGE;           // 120, 144, 112, 128, 144 KB for BM = 64, 128, 192, 256, 320
  static constexpr int FA = BM / 32;                // A fragments (16 rows each) per wave
  static constexpr int ALD = BM / 64;               // A load instructions (8 rows each) per wave and k-tile
  static constexpr int NP = (ALD + 1) / 2;          // phases per k-tile
  static constexpr int LPW = ALD + BL;              // direct-to-LDS load instructions per wave and k-tile
  static constexpr int aloads(int p) { return ALD - 2 * p < 2 ? ALD - 2 * p : 2; }
  static constexpr int loads(int p) { return aloads(p) + (p == 0 ? BL : 0); }
  // loads of a wave that may still be in flight when the data of the phase after phase q of tile `it` must have landed:
  // those issued later than it, in the order (tile, phase region), when `rem` tiles follow tile `it`
  static constexpr int younger(int q, int rem) {
    int n = 0;
    if (q < NP - 1) {
      for (int p = q + 2; p < NP; ++p) n += loads(p);
      for (int t = 1; t < NST && t <= rem; ++t) n += LPW;
    } else {
      if (rem >= 1) for (int p = 1; p < NP; ++p) n += loads(p);
      for (int t = 2; t < NST && t <= rem; ++t) n += LPW;
    }
    if (rem >= NST) for (int p = 0; p < q; ++p) n += loads(p);
    return n;
  }
  static_assert(LDS <= KERNEL_LDS && (NST + 1) * LPW < 64, "ring does not fit");
};

// first LDS row of the 8 rows that wave w's i-th A load of a k-tile fills (region p = i / 2 of both row groups)
template <int BM> __device__ inline int pp_a_row(int w, int i) {
  using P = PingPong<BM>;
  const int p = i >> 1;
  if (P::ALD - 2 * p >= 2) {
    const int u = w * 2 + (i & 1);
    return (u >> 3) * (BM / 2) + p * 64 + (u & 7) * 8;
  }
  return (w >> 2) * (BM / 2) + p * 64 + (w & 3) * 8;
}

// P: PingPong; X: register loads of B that are younger than what is waited for as well
template <int R, class P, int Q, int X> __device__ __forceinline__ void pp_wait(int rem) {
  if constexpr (R == 0) {
    wait_vmcnt<P::younger(Q, 0) + X>();
  } else {
    if (rem >= R) wait_vmcnt<P::younger(Q, R) + X>();
    else pp_wait<R - 1, P, Q, X>(rem);
  }
}

// acc[i][j] += the 16 x 16 tile (rows i*16.., B rows j*16..) of the wave over nk k-tiles, transposed: lane l holds row
// l%16 and the four consecutive B rows 4*(l/16) .. +3, i.e. output columns that are adjacent in memory.
//   issue_a(i, stage, kt): wave's i-th A load of tile kt into LDS stage `stage` (rows pp_a_row);  issue_b(stage, kt): its 4 B
//   loads;  boff[ks]: byte offset of the lane's piece of B fragment 0 in k-step ks inside the B part of a stage, BJ: bytes
//   between fragments.  (Fragment addresses are one lane offset per k-step and operand plus constants: the swizzle of
//   row r is that of r + 16.  Left to the compiler they were 16 registers.)
template <int BM, int BJ, class IA, class IB>
__device__ __forceinline__ void gemm_pingpong(unsigned char* lds, int nk, int lane, int wr, f32x4 (&acc)[BM / 32][4],
                                              IA issue_a, IB issue_b, const uint32_t (&boff)[2]) {
  using P = PingPong<BM>;
  constexpr int FP = P::ALD >= 2 ? 4 : 2;  // fragments of a phase
  // With a 64-row body a slot of matrix instructions is far shorter than one of loads and LDS reads, and the groups in turn
  // only add their latencies: there all waves read, pass one barrier per k-tile and multiply.  (What is read was waited for
  // before that barrier, and what is refilled after it was read before it.)  Dense layers of 13 to 61 tokens: 4352 x 7232
  // 62.3 -> 59.2 us, 3328 x 1472 41.4 -> 39.0, 2816 x 4928 47.3 -> 45.9; the 128-row body loses 2 to 12 % by it.
  constexpr bool PONG = BM > 64;
  bf16x8 fa[FP][2], fb[4][2];
  const uint32_t aoff[2] = {(uint32_t)swz(wr * (BM / 2) + (lane & 15), lane >> 4), (uint32_t)swz(wr * (BM / 2) + (lane & 15), 4 + (lane >> 4))};
  auto issue = [&](auto pc, int stage, int kt) {
    constexpr int p = decltype(pc)::value;
#pragma unroll
    for (int i = 0; i < P::aloads(p); ++i) issue_a(2 * p + i, stage, kt);
    if constexpr (p == 0) issue_b(stage, kt);
  };
  auto next = [&](int st) { return st + 1 == P::NST ? 0 : st + 1; };
  auto phase = [&](auto qc, int it, int st) {
    constexpr int q = decltype(qc)::value;
    constexpr int nf = 2 * P::aloads(q);
    const unsigned char* sa = lds + st * P::STAGE;
    if constexpr (q == 0) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          fb[j][ks] = as_bf16x8(*reinterpret_cast<const u32x4*>(sa + boff[ks] + (BM * 128 + j * BJ)));
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < nf; ++i)
        fa[i][ks] = as_bf16x8(*reinterpret_cast<const u32x4*>(sa + aoff[ks] + (q * 64 + i * 16) * 128));
    // refill the region that both groups have read: that of the previous phase
    if constexpr (q == 0) {
      if (it > 0 && it - 1 + P::NST < nk) issue(std::integral_constant<int, P::NP - 1>{}, st == 0 ? P::NST - 1 : st - 1, it - 1 + P::NST);
    } else {
      if (it + P::NST < nk) issue(std::integral_constant<int, q - 1>{}, st, it + P::NST);
    }
    pp_wait<P::NST, P, q, 0>(nk - 1 - it);
    wait_lgkmcnt0();
    __builtin_amdgcn_sched_barrier(0);
    block_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < nf; ++i)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          const int j = (i & 1) ? 3 - jj : jj;
          acc[q * 4 + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j][ks], fa[i][ks], acc[q * 4 + i][j], 0, 0, 0);
        }
    if constexpr (PONG) {
      __builtin_amdgcn_sched_barrier(0);
      block_barrier();
      __builtin_amdgcn_sched_barrier(0);
    }
  };
#pragma unroll
  for (int i = 0; i < BM / 32; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  using C0 = std::integral_constant<int, 0>;
  using C1 = std::integral_constant<int, 1>;
  using C2 = std::integral_constant<int, 2>;
#pragma unroll
  for (int t = 0; t < P::NST; ++t)
    if (t < nk) {
      issue(C0{}, t, t);
      if constexpr (P::NP > 1) issue(C1{}, t, t);
      if constexpr (P::NP > 2) issue(C2{}, t, t);
    }
  if (nk >= P::NST) wait_vmcnt<P::NST * P::LPW - P::loads(0)>();  // the first region of tile 0
  else wait_vmcnt<0>();
  block_barrier();
  __builtin_amdgcn_sched_barrier(0);
  if (PONG && wr == 1) block_barrier();
  __builtin_amdgcn_sched_barrier(0);
  int st = 0;
  for (int it = 0; it < nk; ++it) {
    phase(C0{}, it, st);
    if constexpr (P::NP > 1) phase(C1{}, it, st);
    if constexpr (P::NP > 2) phase(C2{}, it, st);
    st = next(st);
  }
  if (!PONG || wr == 0) block_barrier();  // the second group's last slot
}

// register loads and the dependency tie used by the loops whose B operand travels through registers
__device__ inline void gload_b128(u32x4& q, const void* p) {
  asm volatile("global_load_dwordx4 %0, %1, off" : "=v"(q) : "v"(p) : "memory");
}
__device__ inline void gload_u16(uint32_t& z, const void* p) {
  asm volatile("global_load_ushort %0, %1, off" : "=v"(z) : "v"(p) : "memory");
}

struct Q4Regs { u32x4 q; uint32_t z; };  // codes and scale of one lane's share of a B tile
constexpr int Q4_GL = 2;                 // register loads of a Q4Regs

// 16-byte LDS store the compiler does not see as one: with a direct-to-LDS load in flight it would otherwise wait
// for ALL vector-memory operations (vmcnt(0)) before any LDS store it cannot prove disjoint from the load's
// target, which would drain the ring every iteration.  Disjointness is by construction here (the stage written is
// not the target of any load in flight), and completion is covered by the loop's own lgkmcnt(0) before each barrier.
__device__ inline void lds_store_b128(unsigned char* p, const u32x4& v) {
  const uint32_t a = (uint32_t)(uintptr_t)SI_LPTR(p);
  asm volatile("ds_write_b128 %0, %1" ::"v"(a), "v"(v) : "memory");
}

// Eight 4-bit codes (as two words of four byte-sized codes each: `lo` holds elements a0 a1 a2 a3 in its bytes
// 0..3 for the byte order given by the caller) -> bf16((code - 8) * scale), exact product, one rounding.
// s8 = -8 * scale.
__device__ inline uint32_t q4_pair(uint32_t bytes, int b0, int b1, float sc, float s8) {
  // (the compiler turns byte extraction + conversion into one v_cvt_f32_ubyteN)
  const float c0 = (float)((bytes >> (8 * b0)) & 0xffu), c1 = (float)((bytes >> (8 * b1)) & 0xffu);
  return pack_bf16(__builtin_fmaf(c0, sc, s8), __builtin_fmaf(c1, sc, s8));
}

// The same loop for weights in the 4-bit storage form.  The A operand arrives by direct global->LDS loads as above;
// the B operand cannot (it has to be turned into bf16 on the way), so every lane fetches 16 bytes of codes (32 weights)
// and their group scale into registers, and turns them into four 16-byte pieces of bf16((code - 8) * scale) that it
// writes into the B part of a stage.  A k-tile of 64 is one scale group of either projection.
// A wave converts B of tile it+1 in the memory slots of tile it, four pieces over its phases, while its partner on the
// SIMD issues matrix instructions; the registers that frees are refilled in the last phase with tile it+3 (two register
// sets, the loop unrolled by two, so that no fetched register is copied while its load is in flight).
// Order of a wave's vector-memory operations, which the wait counts rely on: per phase its A loads, and in the last phase
// of a tile, after them, the Q4_GL register loads (always issued, tile index clamped).  The register loads are inline
// assembly and their waits explicit: with direct-to-LDS loads in flight the compiler's own wait before the first use
// of a loaded register is vmcnt(0), which would drain the ring every iteration; bready ties the registers to the wait.
//   bload(kt, regs), bconv(stage, regs, i): fetch / convert-and-store piece i
template <int BM, int BJ, class IA, class BL, class BC>
__device__ __forceinline__ void gemm_pingpong_q4(unsigned char* lds, int nk, int lane, int wr, f32x4 (&acc)[BM / 32][4],
                                                 IA issue_a, BL bload, BC bconv, const uint32_t (&boff)[2]) {
  using P = PingPong<BM, 0>;
  constexpr int FP = P::ALD >= 2 ? 4 : 2;  // fragments of a phase
  // Bodies of up to 128 rows: one barrier per k-tile, as in gemm_pingpong; here the conversion makes the memory slot the
  // longer one up to 128 rows (12 experts of 3200 columns, d_model 5632, top-6, 62 tokens: 326 -> 268 us; dense
  // 5376 x 1472, 89 tokens: 118 -> 112; the 192- and 256-row bodies keep the two groups).
  constexpr bool PONG = BM > 128;
  bf16x8 fa[FP][2], fb[4][2];
  const uint32_t aoff[2] = {(uint32_t)swz(wr * (BM / 2) + (lane & 15), lane >> 4), (uint32_t)swz(wr * (BM / 2) + (lane & 15), 4 + (lane >> 4))};
  auto bready = [](Q4Regs& r) { asm volatile("" : "+v"(r.q), "+v"(r.z)::"memory"); };
  auto issue = [&](auto pc, int stage, int kt) {
    constexpr int p = decltype(pc)::value;
#pragma unroll
    for (int i = 0; i < P::aloads(p); ++i) issue_a(2 * p + i, stage, kt);
  };
  auto phase = [&](auto qc, int it, int st, Q4Regs& rg) {
    constexpr int q = decltype(qc)::value;
    constexpr int nf = 2 * P::aloads(q);
    constexpr int XB = Q4_GL * ((q + 1) % P::NP == P::NP - 1 ? P::NST - 1 : P::NST);  // register loads younger than the A region waited for
    constexpr int NB = P::ALD + P::aloads(P::NP - 1) + Q4_GL;           // operations younger than the codes of tile it+1
    const unsigned char* sa = lds + st * P::STAGE;
    const int nst = st + 1 == P::NST ? 0 : st + 1;
    if constexpr (q == 0) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          fb[j][ks] = as_bf16x8(*reinterpret_cast<const u32x4*>(sa + boff[ks] + (BM * 128 + j * BJ)));
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < nf; ++i)
        fa[i][ks] = as_bf16x8(*reinterpret_cast<const u32x4*>(sa + aoff[ks] + (q * 64 + i * 16) * 128));
    if constexpr (q == 0) {
      if (it > 0 && it - 1 + P::NST < nk) issue(std::integral_constant<int, P::NP - 1>{}, st == 0 ? P::NST - 1 : st - 1, it - 1 + P::NST);
      // (near the end, where A loads are no longer issued, the A part of the count is dropped)
      if (it - 1 + P::NST < nk) wait_vmcnt<NB>(); else wait_vmcnt<Q4_GL>();
      bready(rg);
    } else {
      if (it + P::NST < nk) issue(std::integral_constant<int, q - 1>{}, st, it + P::NST);
    }
#pragma unroll
    for (int i = 4 * q / P::NP; i < 4 * (q + 1) / P::NP; ++i) bconv(nst, rg, i);
    if constexpr (q == P::NP - 1) bload(min(it + 3, nk - 1), rg);
    pp_wait<P::NST, P, q, XB>(nk - 1 - it);
    wait_lgkmcnt0();
    __builtin_amdgcn_sched_barrier(0);
    block_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < nf; ++i)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          const int j = (i & 1) ? 3 - jj : jj;
          acc[q * 4 + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j][ks], fa[i][ks], acc[q * 4 + i][j], 0, 0, 0);
        }
    if constexpr (PONG) {
      __builtin_amdgcn_sched_barrier(0);
      block_barrier();
      __builtin_amdgcn_sched_barrier(0);
    }
  };
#pragma unroll
  for (int i = 0; i < BM / 32; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  using C0 = std::integral_constant<int, 0>;
  using C1 = std::integral_constant<int, 1>;
  Q4Regs ra, rb;
#pragma unroll
  for (int t = 0; t < P::NST; ++t)
    if (t < nk) {
      issue(C0{}, t, t);
      if constexpr (P::NP > 1) issue(C1{}, t, t);
    }
  Q4Regs r0;
  bload(0, r0);
  bload(min(1, nk - 1), ra);
  bload(min(2, nk - 1), rb);
  wait_vmcnt<0>();
  bready(r0);
  bready(ra);
  bready(rb);
#pragma unroll
  for (int i = 0; i < 4; ++i) bconv(0, r0, i);
  wait_lgkmcnt0();
  block_barrier();
  __builtin_amdgcn_sched_barrier(0);
  if (PONG && wr == 1) block_barrier();
  __builtin_amdgcn_sched_barrier(0);
  int st = 0;
  auto tile = [&](int it, Q4Regs& rg) {
    phase(C0{}, it, st, rg);
    if constexpr (P::NP > 1) phase(C1{}, it, st, rg);
    st = st + 1 == P::NST ? 0 : st + 1;
  };
  for (int it = 0; it < nk; it += 2) {
    tile(it, ra);
    if (it + 1 < nk) tile(it + 1, rb);
  }
  if (!PONG || wr == 0) block_barrier();  // the second group's last slot
  wait_vmcnt<0>();  // the clamped fetches past the last tile
  bready(ra);
  bready(rb);
}

// Epilogue of FC1: SiLU(gate) * up of the wave's 32 hidden columns -> bf16 Hact.  The loader puts the hidden columns of a
// wave into LDS in an order (gu_col) that leaves 8 adjacent columns in a lane, for one 16-byte store per fragment row: with
// the plain order, 2-byte stores and a full division this epilogue was 1180 vector instructions per wave, 5 us of a tile.
template <int BM>
__device__ __forceinline__ void gateup_store(const f32x4 (&acc)[BM / 32][4], const TileInfo& ti, const WeightView& wv, int tc, int wr,
                                             int wc, int lane, uint16_t* __restrict__ hact, int ldh) {
  using P = PingPong<BM>;
  if (2 * tc + (wc >> 1) >= wv.n_chunks) return;
  // (the lane index is made opaque here so that the output addresses are formed after the main loop: formed
  // ahead of it they are live through it, which the 320-row body has no registers for)
  int el = lane;
  asm volatile("" : "+v"(el));
  const int row0 = ti.row0 + wr * (BM / 2) + (el & 15);
  uint16_t* dst = hact + (size_t)row0 * ldh + (wv.col0 + tc * 128 + wc * 32 + (el >> 4) * 8);
#pragma unroll
  for (int i = 0; i < P::FA; ++i) {
    u32x4 o;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 2; ++r)
        o[j * 2 + r] = pack_bf16(silu_f(acc[i][j][2 * r]) * acc[i][j + 2][2 * r], silu_f(acc[i][j][2 * r + 1]) * acc[i][j + 2][2 * r + 1]);
    if (row0 + i * 16 < ti.row_end) *reinterpret_cast<u32x4*>(dst + (size_t)(i * 16) * ldh) = o;
  }
}
// hidden column (of the 32 of a wave) whose gate / up row sits at LDS row r of the wave's 32: fragment j = r / 16, row
// n = r % 16 of it holds column 8*(n/4) + 4*j + n%4
__device__ inline int gu_col(int r) { return ((r & 12) << 1) + ((r >> 4) << 2) + (r & 3); }

// Epilogue of FC2: the wave's 64 output columns, overwritten or accumulated, 16 bytes per lane
template <int BM>
__device__ __forceinline__ void down_store(const f32x4 (&acc)[BM / 32][4], const TileInfo& ti, int n0, int wr, int wc, int lane, int M,
                                           float* __restrict__ out, int accumulate) {
  using P = PingPong<BM>;
  int el = lane;  // opaque, as in gateup_store
  asm volatile("" : "+v"(el));
  const int row0 = ti.row0 + wr * (BM / 2) + (el & 15), m0 = n0 + wc * 64 + (el >> 4) * 4;
  float* dst = out + (size_t)row0 * M + m0;
#pragma unroll
  for (int i = 0; i < P::FA; ++i) {
    if (row0 + i * 16 < ti.row_end) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (m0 + j * 16 < M) {
          f32x4* d = reinterpret_cast<f32x4*>(dst + (size_t)(i * 16) * M + j * 16);
          *d = accumulate ? *d + acc[i][j] : acc[i][j];
        }
    }
  }
}

#define SI_BOFF_K8(col, pc) (((pc) * BN + (col)) * 16)

// ---------------------------------------------------------------------------------------------
// FC1 + SwiGLU.  Tile: BM rows x 128 hidden columns (two chunks).  B rows in LDS are ordered so
// that wave column wc owns hidden columns [32 wc, 32 wc + 32): LDS B row = wc*64 + f*32 + r with
// f = 0 the gate row and f = 1 the up row of column 32 wc + gu_col(r); SiLU(gate)*up is then formed in
// registers from the two accumulator tiles of a wave.
// ---------------------------------------------------------------------------------------------
template <int BM>
__device__ __forceinline__ void gateup_body(const uint16_t* __restrict__ x, int M, const Plan& p, int tc, const TileInfo& ti,
                                            const WeightView& wv, uint16_t* __restrict__ hact, int ldh,
                                            unsigned char* lds) {
  using P = PingPong<BM>;
  const int tid = threadIdx.x, lane = tid % WAVE, w = __builtin_amdgcn_readfirstlane(tid / WAVE);  // wave index, known to be uniform
  const int wr = w >> 2, wc = w & 3;
  const uint16_t* ebase = wv.base + (size_t)ti.se * wv.expert_stride;

  // loader: a wave instruction fills 8 LDS rows (1 KB); lane/8 is the row, lane%8 the slot inside the
  // 128-byte row, which holds logical piece slot ^ ((row >> 1) & 7)
  const int lrow = lane >> 3, lpp = lane & 7;
  uint32_t a_src[P::ALD];  // byte offsets from x (the host checks that x spans less than 2^31 elements)
#pragma unroll
  for (int i = 0; i < P::ALD; ++i) {
    const int lr = pp_a_row<BM>(w, i) + lrow;  // LDS row of the A tile
    int row = ti.row0 + lr;
    row = row < ti.row_end ? row : ti.row_end - 1;
    a_src[i] = ((uint32_t)p.row_token[row] * (uint32_t)M + ((lpp ^ ((lr >> 1) & 7)) * 8)) * 2;
  }
  // B: LDS row w*32 + i*8 + lrow  ->  chunk 2*tc + w/4, f = w%2 (gate / up block), column-in-chunk
  // jc = ((w/2)%2)*32 + gu_col(i*8 + lrow).  Blocks are [M/PW panels][64 j][PW m] (cc_worker.h).
  const int chunk_rel = min(2 * tc + (w >> 2), wv.n_chunks - 1);
  const uint16_t* b_blk = ebase + (size_t)(wv.chunk0 + chunk_rel) * 3 * CHUNK_J * M + (size_t)(w & 1) * CHUNK_J * M;
  const int jc0 = ((w >> 1) & 1) * 32 + gu_col(lrow);
  const int PW = panel_width(M);
  const int lc0 = lpp ^ (lrow >> 1);  // B piece for even i; odd i uses lc0 ^ 4

  // uniform bases and 32-bit lane offsets: two vector registers for the B addresses instead of eight (a k-tile never
  // crosses a panel, PW being a multiple of 64)
  uint32_t b_lane[2] = {(uint32_t)(jc0 * PW + lc0 * 8) * 2u, (uint32_t)(jc0 * PW + (lc0 ^ 4) * 8) * 2u};
  auto issue_a = [&](int i, int stage, int kt) {
    load_lds16(x + kt * BK, a_src[i], lds + stage * P::STAGE + pp_a_row<BM>(w, i) * 128);
  };
  auto issue_b = [&](int stage, int kt) {
    unsigned char* sb = lds + stage * P::STAGE + BM * 128 + w * 4096;
    const int k0 = kt * BK;
    const uint16_t* bk = b_blk + (size_t)(k0 / PW) * CHUNK_J * PW + k0 % PW;
#pragma unroll
    for (int i = 0; i < 4; ++i) load_lds16(bk + gu_col(i * 8) * PW, b_lane[i & 1], sb + i * 1024);
  };
  f32x4 acc[P::FA][4];
  const uint32_t boff[2] = {(uint32_t)swz(wc * 64 + (lane & 15), lane >> 4), (uint32_t)swz(wc * 64 + (lane & 15), 4 + (lane >> 4))};
  gemm_pingpong<BM, 2048>(lds, M / BK, lane, wr, acc, issue_a, issue_b, boff);
  gateup_store<BM>(acc, ti, wv, tc, wr, wc, lane, hact, ldh);
}

// A block picks the body for the rows its tile really has (whole-block branch), so a 40-row tile costs a 64-row
// body and a 140-row tile a 192-row one.  The 320-row body (160 accumulator registers, 144 KB of LDS) exists for the last
// tile of an expert only.  Tiles of at most 192 rows that hold all rows of their expert are bound by HBM: they ran a loop
// of their own before (weights through registers, four k-tiles ahead), which the ping-pong loop overtook because an
// iteration of it is shorter, not because more bytes are in flight (Mixtral-8x7B-shaped prompt of 512 tokens, about
// 128 rows per expert: gate/up 398 -> 366 us, down 205 -> 165 us; 24 tokens, 6 rows per expert: equal).
#define SI_PICK_BODY(ti, CALL)                  \
  {                                             \
    const int rows_ = (ti).row_end - (ti).row0; \
    if (rows_ > 256) CALL(320);                 \
    else if (rows_ > 192) CALL(256);            \
    else if (rows_ > 128) CALL(192);            \
    else if (rows_ > 64) CALL(128);             \
    else CALL(64);                              \
  }
// The 4-bit bodies stop at 256 rows (their B operand passes through registers, which leaves no room for a fifth
// A fragment): the rows a last tile holds beyond 256 take a second pass of the same block.  No wave still reads
// the LDS ring when a body returns (its last barrier follows every fragment read), so the next pass may refill it.
#define SI_PICK_BODY_2PASS(ti, CALL)                                  \
  for (const int row_end_all_ = (ti).row_end;;) {                     \
    (ti).row_end = min(row_end_all_, (ti).row0 + TILE_ROWS);          \
    const int rows_ = (ti).row_end - (ti).row0;                       \
    if (rows_ <= 64) CALL(64);                                        \
    else if (rows_ <= 128) CALL(128);                                 \
    else if (rows_ <= 192) CALL(192);                                 \
    else CALL(256);                                                   \
    if ((ti).row_end >= row_end_all_) break;                          \
    (ti).row0 = (ti).row_end;                                         \
  }

__global__ __launch_bounds__(THREADS, 1) void k_prefill_gateup(const uint16_t* __restrict__ x, int M, Plan p,
                                                               int expert_sel, int x2_only, int n_cu,
                                                               int n_ctiles, WeightView wv_r, WeightView wv_s,
                                                               uint16_t* __restrict__ hact, int ldh_r, long hact_s, int ldh_s) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  int tc;
  TileInfo ti;
  if (!block_tile(p, expert_sel, x2_only, n_ctiles, (wv_s.n_chunks + 1) / 2, n_cu, 1, tc, ti)) return;
  const WeightView wv = ti.sh ? wv_s : wv_r;
  const int ldh = ti.sh ? ldh_s : ldh_r;
  hact += ti.sh ? hact_s : 0;
  if (!storage_index(wv, ti.e, ti.se)) return;
#define SI_CALL_GU(BMV) gateup_body<BMV>(x, M, p, tc, ti, wv, hact, ldh, lds)
  SI_PICK_BODY(ti, SI_CALL_GU)
#undef SI_CALL_GU
}

// ---------------------------------------------------------------------------------------------
// FC2.  Tile: BM rows x 256 output columns m; contraction over the hidden columns of this
// k-split's chunk range (one chunk = 64 per step).  B operand: the down block of a chunk is
// [8 groups][M][8 j], i.e. already "8 consecutive k per (group, m)"; it is kept in that order in
// LDS ([group][256 m] x 16 bytes), read conflict free by consecutive lanes.
// Output slab `split` of yp: rows x M fp32; overwritten or accumulated.
// ---------------------------------------------------------------------------------------------
template <int BM>
__device__ __forceinline__ void down_body(const uint16_t* __restrict__ hact, int ldh, int M, int inner, const TileInfo& ti,
                                          int n_ntiles, int n_split, const WeightView& wv, float* __restrict__ yp,
                                          size_t slab_stride, int accumulate, unsigned char* lds) {
  using P = PingPong<BM>;
  const int nt = inner % n_ntiles, split = inner / n_ntiles;
  const int c_begin = (int)((long)wv.n_chunks * split / n_split), c_end = (int)((long)wv.n_chunks * (split + 1) / n_split);
  if (c_begin >= c_end && accumulate) return;  // nothing to add
  const int tid = threadIdx.x, lane = tid % WAVE, w = __builtin_amdgcn_readfirstlane(tid / WAVE);  // wave index, known to be uniform
  const int wr = w >> 2, wc = w & 3;
  const int n0 = nt * BN;
  const uint16_t* ebase = wv.base + (size_t)ti.se * wv.expert_stride;
  float* out = yp + (size_t)split * slab_stride;

  const int lrow = lane >> 3, lpp = lane & 7;
  uint32_t a_src[P::ALD];  // byte offsets from hact (the host checks that it spans less than 2^31 elements)
#pragma unroll
  for (int i = 0; i < P::ALD; ++i) {
    const int lr = pp_a_row<BM>(w, i) + lrow;
    int row = ti.row0 + lr;
    row = row < ti.row_end ? row : ti.row_end - 1;
    a_src[i] = ((uint32_t)row * (uint32_t)ldh + wv.col0 + ((lpp ^ ((lr >> 1) & 7)) * 8)) * 2;
  }
  // B: wave w loads group q = w of the chunk's down block ([M/NW tiles][8 q][NW m][8 i]), 4 x 64 output columns
  const int NW = ntile_width(M);
  const int nw_shift = __builtin_ctz(NW);
  uint32_t b_off[4];  // bytes, inside one chunk's down block
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int n = min(n0 + i * 64 + lane, M - 1);
    b_off[i] = (((uint32_t)(n >> nw_shift) * 8 + w) * NW + (n & (NW - 1))) * 16;  // NW is a power of two
  }

  if (c_begin < c_end) {
    auto issue_a = [&](int i, int stage, int kt) {
      load_lds16(hact + (c_begin + kt) * CHUNK_J, a_src[i], lds + stage * P::STAGE + pp_a_row<BM>(w, i) * 128);
    };
    auto issue_b = [&](int stage, int kt) {
      unsigned char* sb = lds + stage * P::STAGE + BM * 128 + w * 4096;
      const uint16_t* dblk = ebase + (size_t)(wv.chunk0 + c_begin + kt) * 3 * CHUNK_J * M + (size_t)2 * CHUNK_J * M;
#pragma unroll
      for (int i = 0; i < 4; ++i) load_lds16(dblk, b_off[i], sb + i * 1024);
    };
    f32x4 acc[P::FA][4];
    const uint32_t b0 = SI_BOFF_K8(wc * 64 + (lane & 15), lane >> 4);
    const uint32_t boff[2] = {b0, b0 + 4 * BN * 16};
    gemm_pingpong<BM, 256>(lds, c_end - c_begin, lane, wr, acc, issue_a, issue_b, boff);
    down_store<BM>(acc, ti, n0, wr, wc, lane, M, out, accumulate);
  } else {
    // an empty k-split of an overwriting launch still has to define its slab
    for (int i = tid; i < BM * BN; i += THREADS) {
      const int row = ti.row0 + i / BN, m = n0 + i % BN;
      if (row < ti.row_end && m < M) out[(size_t)row * M + m] = 0.f;
    }
  }
}

__global__ __launch_bounds__(THREADS, 1) void k_prefill_down(const uint16_t* __restrict__ hact, int ldh_r, int M, Plan p,
                                                             int expert_sel, int x2_only, int n_cu,
                                                             int n_ntiles, int split_r, WeightView wv_r, WeightView wv_s,
                                                             int ldh_s, long hact_s, int split_s, float* __restrict__ yp,
                                                             size_t slab_stride, int accumulate) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  int inner;
  TileInfo ti;
  // (XCD ranges also when every expert has a single row tile: one expert's Hact rows, the A operand, a few MB,
  // then stay in one L2; dealt round-robin every XCD re-reads every expert's rows for each of its column tiles,
  // which measured 3 % slower although the XCDs finish together)
  if (!block_tile(p, expert_sel, x2_only, n_ntiles * split_r, wv_s.n_chunks ? n_ntiles * split_s : 0, n_cu, 0, inner, ti)) return;
  const WeightView wv = ti.sh ? wv_s : wv_r;
  const int ldh = ti.sh ? ldh_s : ldh_r, n_split = ti.sh ? split_s : split_r;
  hact += ti.sh ? hact_s : 0;
  if (!storage_index(wv, ti.e, ti.se)) return;
#define SI_CALL_DN(BMV) down_body<BMV>(hact, ldh, M, inner, ti, n_ntiles, n_split, wv, yp, slab_stride, accumulate, lds)
  SI_PICK_BODY(ti, SI_CALL_DN)
#undef SI_CALL_DN
}

// ---------------------------------------------------------------------------------------------
// The same two GEMMs on weights in the 4-bit storage form (chunk layout in cc_worker.h), converted on the way
// into the B stage.  Tiles, LDS layouts, fragment reads, matrix instructions and epilogues are those above.
// ---------------------------------------------------------------------------------------------
template <int BM>
__device__ __forceinline__ void gateup_body_q4(const uint16_t* __restrict__ x, int M, const Plan& p, int tc, const TileInfo& ti,
                                               const WeightView& wv, uint16_t* __restrict__ hact, int ldh,
                                               unsigned char* lds) {
  using P = PingPong<BM, 0>;
  const int tid = threadIdx.x, lane = tid % WAVE, w = __builtin_amdgcn_readfirstlane(tid / WAVE);  // wave index, known to be uniform
  const int wr = w >> 2, wc = w & 3;
  const unsigned char* ebase = reinterpret_cast<const unsigned char*>(wv.base + (size_t)ti.se * wv.expert_stride);

  const int lrow = lane >> 3, lpp = lane & 7;
  uint32_t a_src[P::ALD];  // byte offsets from x
#pragma unroll
  for (int i = 0; i < P::ALD; ++i) {
    const int lr = pp_a_row<BM>(w, i) + lrow;
    int row = ti.row0 + lr;
    row = row < ti.row_end ? row : ti.row_end - 1;
    a_src[i] = ((uint32_t)p.row_token[row] * (uint32_t)M + ((lpp ^ ((lr >> 1) & 7)) * 8)) * 2;
  }
  auto issue_a = [&](int i, int stage, int kt) {
    load_lds16(x + kt * BK, a_src[i], lds + stage * P::STAGE + pp_a_row<BM>(w, i) * 128);
  };
  // B: wave w fills LDS rows [32 w, 32 w + 32) = (chunk 2*tc + w/4, gate (w even) or up block, columns
  // ((w/2)%2)*32 + gu_col(row) of the chunk); lane = (row lane/2, k-half lane%2): the 32 weights of its half row are
  // 16 bytes of codes, i.e. the pieces 4*(lane%2) .. +3 of the LDS row
  const int chunk_rel = min(2 * tc + (w >> 2), wv.n_chunks - 1);
  const unsigned char* cb = ebase + (size_t)(wv.chunk0 + chunk_rel) * q4_chunk_u16(M) * 2;
  const int jc = ((w >> 1) & 1) * 32 + gu_col(lane >> 1), kh = lane & 1;
  const unsigned char* qrow = cb + q4_off_codes(w & 1, M) + (size_t)jc * (M / 2) + kh * 16;
  const uint16_t* zrow = reinterpret_cast<const uint16_t*>(cb + q4_off_scales(w & 1, M)) + (size_t)jc * (M / 64);
  const int brow = w * 32 + (lane >> 1);
  const int bsw = (brow >> 1) & 7;
  auto bload = [&](int kt, Q4Regs& r) {
    gload_b128(r.q, qrow + (size_t)kt * 32);
    gload_u16(r.z, zrow + kt);
  };
  // word i of the lane's codes = elements 8i .. 8i+7 of its half row; even nibbles hold elements 0 4 1 5, odd
  // nibbles 2 6 3 7 (cc_worker.h)
  auto bconv = [&](int stage, const Q4Regs& r, int i) {
    const float sc = __uint_as_float(r.z << 16), s8 = -8.f * sc;
    const uint32_t wd = r.q[i], ev = wd & 0x0f0f0f0fu, od = (wd >> 4) & 0x0f0f0f0fu;
    u32x4 o;
    o.x = q4_pair(ev, 0, 2, sc, s8);
    o.y = q4_pair(od, 0, 2, sc, s8);
    o.z = q4_pair(ev, 1, 3, sc, s8);
    o.w = q4_pair(od, 1, 3, sc, s8);
    lds_store_b128(lds + stage * P::STAGE + BM * 128 + brow * 128 + (((kh * 4 + i) ^ bsw) << 4), o);
  };
  f32x4 acc[P::FA][4];
  const uint32_t boff[2] = {(uint32_t)swz(wc * 64 + (lane & 15), lane >> 4), (uint32_t)swz(wc * 64 + (lane & 15), 4 + (lane >> 4))};
  gemm_pingpong_q4<BM, 2048>(lds, M / BK, lane, wr, acc, issue_a, bload, bconv, boff);
  gateup_store<BM>(acc, ti, wv, tc, wr, wc, lane, hact, ldh);
}

__global__ __launch_bounds__(THREADS, 1) void k_prefill_gateup_q4(const uint16_t* __restrict__ x, int M, Plan p,
                                                                  int expert_sel, int x2_only, int n_cu,
                                                                  int n_ctiles, WeightView wv_r, WeightView wv_s,
                                                                  uint16_t* __restrict__ hact, int ldh_r, long hact_s, int ldh_s) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  int tc;
  TileInfo ti;
  if (!block_tile(p, expert_sel, x2_only, n_ctiles, (wv_s.n_chunks + 1) / 2, n_cu, 1, tc, ti)) return;
  const WeightView wv = ti.sh ? wv_s : wv_r;
  const int ldh = ti.sh ? ldh_s : ldh_r;
  hact += ti.sh ? hact_s : 0;
  if (!storage_index(wv, ti.e, ti.se)) return;
#define SI_CALL_GU(BMV) gateup_body_q4<BMV>(x, M, p, tc, ti, wv, hact, ldh, lds)
  SI_PICK_BODY_2PASS(ti, SI_CALL_GU);
#undef SI_CALL_GU
}

template <int BM>
__device__ __forceinline__ void down_body_q4(const uint16_t* __restrict__ hact, int ldh, int M, int inner, const TileInfo& ti,
                                             int n_ntiles, int n_split, const WeightView& wv, float* __restrict__ yp,
                                             size_t slab_stride, int accumulate, unsigned char* lds) {
  using P = PingPong<BM, 0>;
  const int nt = inner % n_ntiles, split = inner / n_ntiles;
  const int c_begin = (int)((long)wv.n_chunks * split / n_split), c_end = (int)((long)wv.n_chunks * (split + 1) / n_split);
  if (c_begin >= c_end && accumulate) return;
  const int tid = threadIdx.x, lane = tid % WAVE, w = __builtin_amdgcn_readfirstlane(tid / WAVE);  // wave index, known to be uniform
  const int wr = w >> 2, wc = w & 3;
  const int n0 = nt * BN;
  const unsigned char* ebase = reinterpret_cast<const unsigned char*>(wv.base + (size_t)ti.se * wv.expert_stride);
  float* out = yp + (size_t)split * slab_stride;

  const int lrow = lane >> 3, lpp = lane & 7;
  uint32_t a_src[P::ALD];  // byte offsets from hact
#pragma unroll
  for (int i = 0; i < P::ALD; ++i) {
    const int lr = pp_a_row<BM>(w, i) + lrow;
    int row = ti.row0 + lr;
    row = row < ti.row_end ? row : ti.row_end - 1;
    a_src[i] = ((uint32_t)row * (uint32_t)ldh + wv.col0 + ((lpp ^ ((lr >> 1) & 7)) * 8)) * 2;
  }
  auto issue_a = [&](int i, int stage, int kt) {
    load_lds16(hact + (c_begin + kt) * CHUNK_J, a_src[i], lds + stage * P::STAGE + pp_a_row<BM>(w, i) * 128);
  };
  // B: thread = (output column n0 + (w%4)*64 + lane, j-half w/4): its 16 bytes of codes are the 32 hidden columns
  // of the half for that output column, i.e. the pieces 4*half .. +3 of the column in the [piece][column] B stage
  const int NW = ntile_width(M);
  const int half = w >> 2, col = (w & 3) * 64 + lane;
  const int n = min(n0 + col, M - 1);
  const size_t qoff = q4_off_codes(2, M) + (((size_t)(n / NW) * 2 + half) * NW + (n % NW)) * 16;
  const size_t zoff = q4_off_scales(2, M) + (size_t)n * 2;
  const size_t cbytes = q4_chunk_u16(M) * 2;
  auto bload = [&](int kt, Q4Regs& r) {
    const unsigned char* cb = ebase + (size_t)(wv.chunk0 + c_begin + kt) * cbytes;
    gload_b128(r.q, cb + qoff);
    gload_u16(r.z, cb + zoff);
  };
  // word i = hidden columns 8i .. 8i+7 of the half; even nibbles hold elements 0 1 2 3, odd nibbles 4 5 6 7
  auto bconv = [&](int stage, const Q4Regs& r, int i) {
    const float sc = __uint_as_float(r.z << 16), s8 = -8.f * sc;
    const uint32_t wd = r.q[i], ev = wd & 0x0f0f0f0fu, od = (wd >> 4) & 0x0f0f0f0fu;
    u32x4 o;
    o.x = q4_pair(ev, 0, 1, sc, s8);
    o.y = q4_pair(ev, 2, 3, sc, s8);
    o.z = q4_pair(od, 0, 1, sc, s8);
    o.w = q4_pair(od, 2, 3, sc, s8);
    lds_store_b128(lds + stage * P::STAGE + BM * 128 + ((half * 4 + i) * BN + col) * 16, o);
  };
  if (c_begin < c_end) {
    f32x4 acc[P::FA][4];
    const uint32_t b0 = SI_BOFF_K8(wc * 64 + (lane & 15), lane >> 4);
    const uint32_t boff[2] = {b0, b0 + 4 * BN * 16};
    gemm_pingpong_q4<BM, 256>(lds, c_end - c_begin, lane, wr, acc, issue_a, bload, bconv, boff);
    down_store<BM>(acc, ti, n0, wr, wc, lane, M, out, accumulate);
  } else {
    for (int i = tid; i < BM * BN; i += THREADS) {
      const int row = ti.row0 + i / BN, m = n0 + i % BN;
      if (row < ti.row_end && m < M) out[(size_t)row * M + m] = 0.f;
    }
  }
}

__global__ __launch_bounds__(THREADS, 1) void k_prefill_down_q4(const uint16_t* __restrict__ hact, int ldh_r, int M, Plan p,
                                                                int expert_sel, int x2_only, int n_cu,
                                                                int n_ntiles, int split_r, WeightView wv_r, WeightView wv_s,
                                                                int ldh_s, long hact_s, int split_s, float* __restrict__ yp,
                                                                size_t slab_stride, int accumulate) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  int inner;
  TileInfo ti;
  if (!block_tile(p, expert_sel, x2_only, n_ntiles * split_r, wv_s.n_chunks ? n_ntiles * split_s : 0, n_cu, 0, inner, ti)) return;
  const WeightView wv = ti.sh ? wv_s : wv_r;
  const int ldh = ti.sh ? ldh_s : ldh_r, n_split = ti.sh ? split_s : split_r;
  hact += ti.sh ? hact_s : 0;
  if (!storage_index(wv, ti.e, ti.se)) return;
#define SI_CALL_DN(BMV) down_body_q4<BMV>(hact, ldh, M, inner, ti, n_ntiles, n_split, wv, yp, slab_stride, accumulate, lds)
  SI_PICK_BODY_2PASS(ti, SI_CALL_DN);
#undef SI_CALL_DN
}

__global__ __launch_bounds__(256) void k_prefill_combine(const float* __restrict__ yp, size_t slab_stride, int n_split, int split_s,
                                                         const float* __restrict__ ycc, int T, int k, int M, int n_x1,
                                                         int has_shared, Plan p, float* __restrict__ y) {
  const int t = blockIdx.y;
  const int m4 = blockIdx.x * 256 + threadIdx.x;
  if (m4 * 4 >= M) return;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int s = 0; s < k; ++s) {
    const float wgt = p.w[t * k + s];
    const float* row = yp + (size_t)p.inv[t * k + s] * M;
    float4 v = reinterpret_cast<const float4*>(row)[m4];
    for (int q = 1; q < n_split; ++q) {
      const float4 v2 = reinterpret_cast<const float4*>(row + (size_t)q * slab_stride)[m4];
      v.x += v2.x; v.y += v2.y; v.z += v2.z; v.w += v2.w;
    }
    acc.x = fmaf(wgt, v.x, acc.x); acc.y = fmaf(wgt, v.y, acc.y);
    acc.z = fmaf(wgt, v.z, acc.z); acc.w = fmaf(wgt, v.w, acc.w);
  }
  if (has_shared) {
    const float* row = yp + (size_t)(T * k + t) * M;
    for (int q = 0; q < split_s; ++q) {
      const float4 v = reinterpret_cast<const float4*>(row + (size_t)q * slab_stride)[m4];
      acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
    }
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

// compute units of the current device (a round of the tail split)
static int cu_count() {
  static int n = [] {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0)
      v = 256;
    return v;
  }();
  return n;
}

// grid of a launch over at most n_tiles logical ids: room for the XCD ranges (rounded up to 8) and for the
// second blocks of a split tail (at most half a round)
static int grid_blocks(int n_tiles) { return (n_tiles + 7) / 8 * 8 + 8 + cu_count() / 2 + 8; }

static hipError_t ensure_lds_attr() {
  static hipError_t st = [] {
    const void* kernels[] = {(const void*)k_prefill_gateup, (const void*)k_prefill_down, (const void*)k_prefill_gateup_q4,
                             (const void*)k_prefill_down_q4};
    for (const void* k : kernels) {
      hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, KERNEL_LDS);
      if (e != hipSuccess) return e;
      // The main loops count their own vector-memory operations (wait_vmcnt<N> against PingPong<>::younger): a
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
  const int total = grid_blocks(n_row_tiles * n_ctiles) + (sp.row_tiles * ((sp.wv.n_chunks + 1) / 2) + 7) / 8 * 8;
  if (wv.q4)
    hipLaunchKernelGGL(k_prefill_gateup_q4, dim3(total), dim3(THREADS), KERNEL_LDS, stream, x, M, plan, expert_sel, x2_only,
                       cu_count(), n_ctiles, wv, sp.wv, hact, ldh, sp.hact, sp.ldh);
  else
    hipLaunchKernelGGL(k_prefill_gateup, dim3(total), dim3(THREADS), KERNEL_LDS, stream, x, M, plan, expert_sel, x2_only,
                       cu_count(), n_ctiles, wv, sp.wv, hact, ldh, sp.hact, sp.ldh);
  return hipGetLastError();
}

hipError_t launch_prefill_down(const uint16_t* hact, int ldh, int M, const Plan& plan, int expert_sel,
                               int x2_only, int n_row_tiles, const WeightView& wv, float* yp, size_t slab_stride,
                               int n_split, int accumulate, const SharedPart& sp, hipStream_t stream) {
  if (wv.n_chunks <= 0 || n_row_tiles <= 0) return hipSuccess;
  hipError_t e = ensure_lds_attr();
  if (e != hipSuccess) return e;
  const int n_ntiles = (M + BN - 1) / BN;
  const int total = grid_blocks(n_row_tiles * n_ntiles * n_split) + (sp.wv.n_chunks ? (sp.row_tiles * n_ntiles * sp.split + 7) / 8 * 8 : 0);
  if (wv.q4)
    hipLaunchKernelGGL(k_prefill_down_q4, dim3(total), dim3(THREADS), KERNEL_LDS, stream, hact, ldh, M, plan, expert_sel,
                       x2_only, cu_count(), n_ntiles, n_split, wv, sp.wv, sp.ldh, sp.hact, sp.split, yp, slab_stride, accumulate);
  else
    hipLaunchKernelGGL(k_prefill_down, dim3(total), dim3(THREADS), KERNEL_LDS, stream, hact, ldh, M, plan, expert_sel,
                       x2_only, cu_count(), n_ntiles, n_split, wv, sp.wv, sp.ldh, sp.hact, sp.split, yp, slab_stride, accumulate);
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
