// Kernels for the 4-bit storage form of the weights (codes 0..15 standing for (code - 8) * scale, bf16 group
// scales; chunk layout in cc_worker.h).
//   k_decode_gateup_q4 / k_decode_down_q4 : the generation-phase GEMVs straight from the codes (exact products, fp32
//       sums; 4x fewer weight bytes than bf16, so the unpacking, about 1.5 vector instructions per weight, and not the
//       multiplication, which the matrix cores do, has to stay below the time the bytes take)
//   k_dequant_q4 : codes -> bf16 chunks (the layout the MFMA GEMMs read), piece by piece, for the prompt phase
#include "si_internal.h"
#include "decode_device.h"

#include <algorithm>

namespace si {
namespace {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
constexpr int WAVE = 64;
constexpr int QGU_THREADS = 512;
constexpr int QGU_JPB = 32;  // hidden columns per block
constexpr int QDN_THREADS = 256;

__device__ inline float bf16_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
// The generation-phase GEMVs on the matrix cores.  A 32-bit word of 8 codes becomes matrix operand data with one or two
// instructions per pair of codes, whatever the number of tokens: the rows of the other operand are the tokens (FC1) or
// the fp16 parts of fp32 activations (FC2).  FC1 inserts a nibble into 0x4300, the bf16 value 128 + c (3 shifts and 4 and-or
// per word), and per scale group forms acc = -136 sum(x) + sum x (128 + c), total += scale * acc, in fp32; FC2 sums
// h (c - 8) directly (SignedCodes).  The dot-product kernels these replaced (shift, insert and one dot instruction per pair
// and token) were bound by the vector units: LLaMA-shaped layer, 3 tokens, gate/up 107 us and down 77 us for 250 and
// 125 MB of codes; now 53 and 26.5 us.
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// the 8 codes of a word as bf16(128 + c): register i holds the nibbles i and i + 4.  mask / magic arrive in registers, so
// that and-then-or is one instruction.  (Not inline assembly: a matrix instruction may read a register that a vector
// instruction wrote only two wait states later, and the compiler inserts those for instructions it knows.)
__device__ __forceinline__ u32x4 expand_codes(uint32_t w, uint32_t mask, uint32_t magic) {
  u32x4 o;
#pragma unroll
  for (int i = 0; i < 4; ++i) o[i] = ((w >> (4 * i)) & mask) | magic;
  return o;
}

// FC2: a lane's 16-byte load holds 32 codes of a column, i.e. half a scale group: lanes of quarter q = lane/16 hold half q%2 of group q/2.
// Exchanging between the lane halves leaves words of one group in all four quarters, which one matrix instruction needs:
// g[0][i], g[1][i]: word pair i of group 0 / 1.  Quarter q then covers the contraction offset unit_k(q) + 8 i.
__device__ __forceinline__ void split_groups(const u32x4& w, uint32_t (&g)[2][2]) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const auto r = __builtin_amdgcn_permlane32_swap(w[i], w[i + 2], false, false);
    g[0][i] = r[0];
    g[1][i] = r[1];
  }
}
__device__ inline int unit_k(int q) { return ((q & 1) << 5) | ((q >> 1) << 4); }

// h[row][j] = SiLU(x . Wg[j]) * (x . Wu[j]).  A wave owns 4 hidden columns over the whole contraction: v_mfma_f32_4x4x4_16b
// multiplies 16 independent 4 x 4 x 4 blocks, and block b = lane / 4 takes the 32 codes of piece b (16 bytes) of a row, so
// that one load covers 256 contiguous bytes of 4 rows and a lane's codes lie in one scale group.  (With the 16 x 16 x 32
// instruction a load covers 64 bytes of 16 rows: the same loads without any arithmetic then took 57 us for 250 MB where
// 1 KB runs took 43.)  A lane ends up with 4 tokens of its column and piece, scaled and summed over the row in fp32;
// -136 sum(x) is the product of x with a constant operand.  LDS: x of up to 4 tokens.
// LLaMA-shaped layer, 3 tokens: 107 -> 55 us (250 MB of codes).
typedef short s16x4 __attribute__((ext_vector_type(4)));
constexpr int QU = 2;      // units (512 codes per row; 2 KB of gate and up codes per wave) in flight, refilled as they are consumed
                           // (3 and 4 units: 62 and 67 us instead of 55, the registers cost waves)
constexpr int QGU_TB = 4;  // tokens per pass over the weights
// LDS of a block: scales [2][32][M / 64], x [tb][2 M bytes], rows of both PADded (the 4 tokens of 4 pieces then cover all banks).  At
// M = 8192 and 4 tokens the padding would leave one block per compute unit (8192 x 28672: 70 us); without it there are two, and the
// 16-byte words of a 64-byte piece of x are kept in an order of the token's own, so that 4 tokens of 2 pieces cover all banks: 58.6 us.
// (Not for all: computing that order costs the smaller calls 0.5 us of 53.)
constexpr size_t QGU_LDS = 80 * 1024;
constexpr size_t gateup_lds(int tb, int M, bool pad) { return (size_t)2 * QGU_JPB * (M / 64 + 2 * pad) * 2 + (size_t)tb * (2 * M + 16 * pad); }
template <bool PAD>
__global__ __launch_bounds__(QGU_THREADS, 4) void k_decode_gateup_q4(const uint16_t* __restrict__ x, int M, Plan p,
                                                                     int expert_sel, int x2_only, WeightView wv_r, WeightView wv_s,
                                                                     int shared_y, float* __restrict__ h, int ldh, int tb) {
  extern __shared__ __attribute__((aligned(16))) unsigned char s_q[];
  int e, r0, r1, se;
  // the first shared_y rows of the grid are the blocks of the shared expert
  const int slot = (int)blockIdx.y - shared_y;
  const int bx = slot < 0 ? blockIdx.y * gridDim.x + blockIdx.x : blockIdx.x;
  const WeightView wv = slot < 0 ? wv_s : wv_r;
  if (!block_rows(p, expert_sel, x2_only, slot, e, r0, r1)) return;
  if (!storage_index(wv, e, se)) return;
  const int tid = threadIdx.x, lane = tid % WAVE, wid = __builtin_amdgcn_readfirstlane(tid / WAVE), j = lane & 3, pc = lane >> 2;
  constexpr int blocks_per_chunk = CHUNK_J / QGU_JPB;
  if (bx >= wv.n_chunks * blocks_per_chunk) return;
  const int chunk = wv.chunk0 + bx / blocks_per_chunk;
  const int jb = (bx % blocks_per_chunk) * QGU_JPB, jj0 = jb + wid * 4;
  const unsigned char* cb = reinterpret_cast<const unsigned char*>(wv.base + (size_t)se * wv.expert_stride + (size_t)chunk * q4_chunk_u16(M));
  const unsigned char* gq = cb + q4_off_codes(0, M) + (size_t)(jj0 + j) * (M / 2);
  const unsigned char* uq = cb + q4_off_codes(1, M) + (size_t)(jj0 + j) * (M / 2);
  const int n_pieces = M / 32, n_units = (n_pieces + 15) / 16;
  const int MG = M / 64, GS = MG + 2 * PAD, xstride = 2 * M + 16 * PAD;
  uint16_t* s_sc = reinterpret_cast<uint16_t*>(s_q);           // [2][32][GS]
  unsigned char* s_x = s_q + 2 * QGU_JPB * GS * 2;             // [tb][xstride]
  uint32_t mask = 0x000F000Fu, magic = 0x43004300u, m136 = 0xC308C308u;  // (m136: two bf16 values -136)
  asm volatile("" : "+v"(mask), "+s"(magic), "+v"(m136));  // kept out of the optimiser's sight (see expand_codes)
  const s16x4 neg136 = __builtin_bit_cast(s16x4, (u32x2{m136, m136}));

  u32x4 wg[QU], wu[QU];
  auto fetch1 = [&](int i, int u) {
    const int pp = min(u * 16 + pc, n_pieces - 1);  // (a piece past the row is fetched from its end and not used)
    wg[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(gq + (size_t)pp * 16));
    wu[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(uq + (size_t)pp * 16));
  };
  auto fetch = [&]() {
#pragma unroll
    for (int i = 0; i < QU; ++i) fetch1(i, i);
  };
  fetch();
  // the scales of the 32 rows are contiguous: 8 per load (32 * MG of them, so no load crosses the section).  Fetched by
  // each wave as it needs them, 16 bytes of a row at a time, they cost 7 us.
  for (int i = tid; i < 2 * 4 * MG; i += QGU_THREADS) {
    const int f = i >= 4 * MG, pos = (f ? i - 4 * MG : i) * 8;
    const u32x4 v = *reinterpret_cast<const u32x4*>(cb + q4_off_scales(f, M) + ((size_t)jb * MG + pos) * 2);
    int r = pos / MG, g = pos - r * MG;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      s_sc[(f * QGU_JPB + r) * GS + g] = (uint16_t)(v[k >> 1] >> (16 * (k & 1)));
      if (++g == MG) { g = 0; ++r; }
    }
  }
  const uint16_t* sc = s_sc + (wid * 4 + j) * GS;
  for (int rb = r0; rb < r1; rb += tb) {
    const int nt = min(tb, r1 - rb);
    if (rb != r0) {
      __syncthreads();
      fetch();
    }
    // x in batches of XB pieces of 16 bytes per thread, whose loads are in flight together
    constexpr int XB = 6;
    const int M8 = M / 8;
    for (int i0 = tid; i0 < nt * M8; i0 += XB * QGU_THREADS) {
      u32x4 v[XB];
#pragma unroll
      for (int b = 0; b < XB; ++b) {
        const int i = min(i0 + b * QGU_THREADS, nt * M8 - 1), t = i / M8;
        v[b] = reinterpret_cast<const u32x4*>(x + (size_t)token_of_row(p, rb + t) * M)[i - t * M8];
      }
#pragma unroll
      for (int b = 0; b < XB; ++b) {
        const int i = i0 + b * QGU_THREADS, t = i / M8, c = i - t * M8;
        if (i < nt * M8) *reinterpret_cast<u32x4*>(s_x + t * xstride + (PAD ? c : c ^ (t & 3)) * 16) = v[b];
      }
    }
    __syncthreads();
    // operand rows past the last token repeat it, their results are not read
    const int xt = min(j, nt - 1);
    const unsigned char* xrow = s_x + xt * xstride;
    f32x4 tg = {0.f, 0.f, 0.f, 0.f}, tu = tg;
    auto use = [&](int i, int u) {
      const int pp = min(u * 16 + pc, n_pieces - 1);
      const bool in = u * 16 + pc < n_pieces;
      const unsigned char* xp = xrow + pp * 64;
      f32x4 ag = {0.f, 0.f, 0.f, 0.f}, au = ag, as = ag;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const u32x4 xv = *reinterpret_cast<const u32x4*>(xp + (PAD ? w : w ^ xt) * 16);
        const u32x4 cg = expand_codes(wg[i][w], mask, magic), cu = expand_codes(wu[i][w], mask, magic);
#pragma unroll
        for (int f = 0; f < 2; ++f) {
          const s16x4 xa = __builtin_bit_cast(s16x4, (u32x2{xv[2 * f], xv[2 * f + 1]}));
          as = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(xa, neg136, as, 0, 0, 0);
          ag = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(xa, __builtin_bit_cast(s16x4, (u32x2{cg[2 * f], cg[2 * f + 1]})), ag, 0, 0, 0);
          au = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(xa, __builtin_bit_cast(s16x4, (u32x2{cu[2 * f], cu[2 * f + 1]})), au, 0, 0, 0);
        }
      }
      const float sg = in ? bf16_f32(sc[pp >> 1]) : 0.f, su = in ? bf16_f32(sc[QGU_JPB * GS + (pp >> 1)]) : 0.f;
#pragma unroll
      for (int r = 0; r < 4; ++r) { tg[r] = fmaf(sg, ag[r] + as[r], tg[r]); tu[r] = fmaf(su, au[r] + as[r], tu[r]); }
    };
    int u0 = 0;
    for (; u0 + QU < n_units; u0 += QU) {
#pragma unroll
      for (int i = 0; i < QU; ++i) {
        use(i, u0 + i);
        fetch1(i, u0 + QU + i);
      }
    }
#pragma unroll
    for (int i = 0; i < QU; ++i)
      if (u0 + i < n_units) use(i, u0 + i);
    // sum over the 16 pieces; then lanes 0..3 (gate; 32..35 up) and 16..19 hold the tokens 2g and 2g + 1 of columns 0..3
    float v[8] = {tg[0], tu[0], tg[1], tu[1], tg[2], tu[2], tg[3], tu[3]};
    wave_sums<8, 4>(v);
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const float u = __uint_as_float(__builtin_amdgcn_permlane32_swap(__float_as_uint(v[g]), __float_as_uint(v[g]), false, false)[1]);
      const int t = 2 * g + (lane >> 4);
      if ((lane & 15) < 4 && lane < 32 && t < nt) h[(size_t)(rb + t) * ldh + wv.col0 + (bx / blocks_per_chunk) * CHUNK_J + jj0 + j] = silu_f(v[g]) * u;
    }
  }
}

// The same for a launch over one expert whose rows are long (d_model > 6656), with the contraction split over the waves of a block: a wave
// keeps its 2 units of x (up to 4 tokens) and their -136 sum(x) in registers over all groups (4 columns) of the block, so that neither takes
// LDS or instructions per group; the partial sums of the waves meet in LDS at the end and are added in their order, which is the same for
// every launch.  The groups are dealt equally to two blocks per compute unit: k_decode_gateup_q4 with 28672 columns of d_model 8192 is 896
// blocks of 66 KB, 1.75 rounds, of which each stages 49 KB of x; with 1408 columns it is 44 blocks.
// Dense layers, call before -> now (us): 8192 x 28672, 3 tokens 81.0 -> 75.7 (gate/up 53.8 -> 46.2, 5.4 TB/s); 8192 x 14336, 4 tokens 48.9 -> 45.8; 8192 x
// 5632, 1 token 27.4 -> 24.8; 8192 x 1408, 4 tokens 25.2 -> 17.9; 7168 x 14336 equal, 7168 x 5632, 1 token 25.9 -> 23.8.  Shorter rows lose by it, as the
// waves' shares get uneven and x in LDS is small: 5120 x 14336, 4 tokens (10 units on 8 waves) 35.3 -> 38.2, 4096 x 14336 equal, 1024 x 5632
// 13.2 -> 14.7; so do launches over several experts (16 of 4864 x 3264, 8 tokens 45.2 -> 51.7: a block's share ends inside an expert and
// starts over with the next one's x and scales).
constexpr int QGS_WAVES = 8, QGS_THREADS = QGS_WAVES * WAVE, QGS_BLOCKS = 512;
constexpr int QGS_UNITS = 14;          // from so many units (of 16) up
constexpr int QGS_MAX_M = 8192;
constexpr size_t QGS_LDS = 78 * 1024;  // two blocks per compute unit
// (193 to 256 blocks of the other kernel are one good round of it, and but for the longest rows nothing is gained: 6720 x 7168, 4 tokens
// 27.3 -> 29.0, 7424 x 7168 30.0 -> 30.4, 8192 x 8192 33.5 -> 32.3; 192 blocks: 6720 x 6144, 1 / 4 tokens 25.4 -> 23.6 / 26.5 -> 26.3.
// The blocks are those of the whole expert, not of a launch over a part or a piece of one: the kernels sum a row in different orders, and
// a result must not depend on how a streamed part is cut.  Against a choice by the chunks of a launch, eleven calls of 6720 to 8192 x 6400 to 28672
// with 6 to 125 chunks streamed or on the host: 0.993 to 1.017, the worst 7168 x 6400, 6 chunks, 4 tokens 86.9 -> 87.5: they wait for their copies,
// 12 us a chunk, whichever kernel it is.)
constexpr bool gateup_split(int M, int e_chunks) {
  const int n_units = (M / 32 + 15) / 16, blocks = e_chunks * (CHUNK_J / QGU_JPB);
  return M <= QGS_MAX_M && n_units >= QGS_UNITS && (n_units == 2 * QGS_WAVES || blocks <= 192 || blocks > 256);
}
// LDS of a block per group: scales [2][4][M / 64 + 2], partial sums [waves][2][4 tokens][4]
constexpr size_t gateup_group_lds(int M) { return (size_t)16 * (M / 64 + 2) + 128 * QGS_WAVES; }
__global__ __launch_bounds__(QGS_THREADS, 4) void k_decode_gateup_q4_split(const uint16_t* __restrict__ x, int M, Plan p, int expert_sel,
                                                                           int x2_only, WeightView wv, int lds_groups,
                                                                           float* __restrict__ h, int ldh) {
  extern __shared__ __attribute__((aligned(16))) unsigned char s_q[];
  constexpr int GROUPS = CHUNK_J / 4;  // of a chunk
  constexpr int KU = 2;                // units of x of a wave
  const int tid = threadIdx.x, lane = tid % WAVE, w0 = __builtin_amdgcn_readfirstlane(tid / WAVE), j = lane & 3, pc = lane >> 2;
  int e, r0, r1, se;
  if (!block_rows(p, expert_sel, x2_only, 0, e, r0, r1)) return;
  if (!storage_index(wv, e, se)) return;
  const unsigned char* cb0 = reinterpret_cast<const unsigned char*>(wv.base + (size_t)se * wv.expert_stride + (size_t)wv.chunk0 * q4_chunk_u16(M));
  const size_t cbytes = q4_chunk_u16(M) * 2;
  const int n_pieces = M / 32, n_units = (n_pieces + 15) / 16;
  const int MG = M / 64, GS = MG + 2;
  uint16_t* s_sc = reinterpret_cast<uint16_t*>(s_q);                           // [2][lds_groups * 4][GS]
  float* s_p = reinterpret_cast<float*>(s_q + (size_t)16 * lds_groups * GS);  // [waves][lds_groups][2][4 tokens][4]
  uint32_t mask = 0x000F000Fu, magic = 0x43004300u, m136 = 0xC308C308u;  // (m136: two bf16 values -136)
  asm volatile("" : "+v"(mask), "+s"(magic), "+v"(m136));  // kept out of the optimiser's sight (see expand_codes)
  const s16x4 neg136 = __builtin_bit_cast(s16x4, (u32x2{m136, m136}));

  // an equal share of the groups for every block, in stretches that LDS holds
  const long long ng = wv.n_chunks * GROUPS;
  const int hi = (int)(ng * (blockIdx.x + 1) / gridDim.x);
  for (int g0 = (int)(ng * blockIdx.x / gridDim.x), n_g; g0 < hi; g0 += n_g) {
    n_g = min(hi - g0, lds_groups);
    // the lane's pieces of the wave's units w0 and w0 + 8
    uint32_t off[KU], sidx[KU];  // bytes from the group's first gate code; its scale (past the row: a zero beside the row's scales)
    const int n_mine = (n_units - w0 + QGS_WAVES - 1) / QGS_WAVES;
#pragma unroll
    for (int i = 0; i < KU; ++i) {
      const int q = (w0 + QGS_WAVES * i) * 16 + pc;
      off[i] = (uint32_t)(j * (M / 2) + min(q, n_pieces - 1) * 16);  // (a piece past the row is fetched from its end and not used)
      sidx[i] = q < n_pieces ? q >> 1 : MG;
    }
    const uint32_t up = (uint32_t)(q4_off_codes(1, M) - q4_off_codes(0, M));
    u32x4 wg[KU], wu[KU];
    auto fetch = [&](int i, int gl) {  // unit i of group gl of the stretch
      const int g = g0 + gl;
      const unsigned char* base = cb0 + (size_t)(g / GROUPS) * cbytes + q4_off_codes(0, M) + (size_t)(g % GROUPS) * (2 * M);
      wg[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(base + off[i]));
      wu[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(base + up + off[i]));
    };
    auto fetch_first = [&]() {
#pragma unroll
      for (int i = 0; i < KU; ++i)
        if (i < n_mine) fetch(i, 0);
    };
    fetch_first();
    __syncthreads();  // (the stretch before is done with LDS)
    // the scales of a group's 4 rows are contiguous: 4 per load (4 * MG of them)
    for (int i = tid; i < 2 * n_g * MG; i += QGS_THREADS) {
      const int f = i >= n_g * MG, k = f ? i - n_g * MG : i, gl = k / MG, pos = (k - gl * MG) * 4, g = g0 + gl;
      const u32x2 v = *reinterpret_cast<const u32x2*>(cb0 + (size_t)(g / GROUPS) * cbytes + q4_off_scales(f, M) + ((size_t)(g % GROUPS) * 4 * MG + pos) * 2);
      int r = pos / MG, c = pos - r * MG;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        s_sc[((f * lds_groups + gl) * 4 + r) * GS + c] = (uint16_t)(v[q >> 1] >> (16 * (q & 1)));
        if (++c == MG) { c = 0; ++r; }
      }
    }
    for (int i = tid; i < 8 * n_g; i += QGS_THREADS) s_sc[((i & 1) * lds_groups * 4 + (i >> 1)) * GS + MG] = 0;
    for (int rb = r0; rb < r1; rb += QGU_TB) {
      const int nt = min(QGU_TB, r1 - rb);
      // operand rows past the last token repeat it, their results are not read
      const uint16_t* xrow = x + (size_t)token_of_row(p, rb + min(j, nt - 1)) * M;
      if (rb != r0) fetch_first();
      u32x4 xv[KU][4];
      f32x4 as[KU];
#pragma unroll
      for (int i = 0; i < KU; ++i) {
#pragma unroll
        for (int w = 0; w < 4; ++w) xv[i][w] = reinterpret_cast<const u32x4*>(xrow + (off[i] - j * (M / 2)) * 2)[w];
        as[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
          for (int f = 0; f < 2; ++f)
            as[i] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(s16x4, (u32x2{xv[i][w][2 * f], xv[i][w][2 * f + 1]})), neg136, as[i], 0, 0, 0);
      }
      __syncthreads();  // the scales are in LDS, and the sums of the rows before have been taken from it
      for (int gl = 0; gl < n_g; ++gl) {
        const uint16_t* sc = s_sc + (gl * 4 + j) * GS;
        f32x4 tg = {0.f, 0.f, 0.f, 0.f}, tu = tg;
#pragma unroll
        for (int i = 0; i < KU; ++i)
          if (i < n_mine) {
            f32x4 ag = {0.f, 0.f, 0.f, 0.f}, au = ag;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
              const u32x4 cg = expand_codes(wg[i][w], mask, magic), cu = expand_codes(wu[i][w], mask, magic);
#pragma unroll
              for (int f = 0; f < 2; ++f) {
                const s16x4 xa = __builtin_bit_cast(s16x4, (u32x2{xv[i][w][2 * f], xv[i][w][2 * f + 1]}));
                ag = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(xa, __builtin_bit_cast(s16x4, (u32x2{cg[2 * f], cg[2 * f + 1]})), ag, 0, 0, 0);
                au = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(xa, __builtin_bit_cast(s16x4, (u32x2{cu[2 * f], cu[2 * f + 1]})), au, 0, 0, 0);
              }
            }
            if (gl + 1 < n_g) fetch(i, gl + 1);
            const float sg = bf16_f32(sc[sidx[i]]), su = bf16_f32(sc[lds_groups * 4 * GS + sidx[i]]);
#pragma unroll
            for (int r = 0; r < 4; ++r) { tg[r] = fmaf(sg, ag[r] + as[i][r], tg[r]); tu[r] = fmaf(su, au[r] + as[i][r], tu[r]); }
          }
        // sum over the 16 pieces; then lanes 0..3 (gate; 32..35 up) and 16..19 hold the tokens 2g and 2g + 1 of columns 0..3
        float v[8] = {tg[0], tu[0], tg[1], tu[1], tg[2], tu[2], tg[3], tu[3]};
        wave_sums<8, 4>(v);
        if ((lane & 15) < 4) {
          float* d = s_p + ((w0 * lds_groups + gl) * 2 + (lane >> 5)) * 16 + ((lane >> 4) & 1) * 4 + j;
#pragma unroll
          for (int g = 0; g < 2; ++g) d[8 * g] = v[g];
        }
      }
      __syncthreads();
      for (int i = tid; i < n_g * 4 * nt; i += QGS_THREADS) {
        const int c = i & 3, t = (i >> 2) % nt, gl = (i >> 2) / nt, g = g0 + gl;
        float vg = 0.f, vu = 0.f;
#pragma unroll
        for (int w = 0; w < QGS_WAVES; ++w) {
          const float* s = s_p + (w * lds_groups + gl) * 32 + t * 4 + c;
          vg += s[0];
          vu += s[16];
        }
        h[(size_t)(rb + t) * ldh + wv.col0 + g * 4 + c] = silu_f(vg) * vu;
      }
    }
  }
}

// 8 codes as the fp16 values c - 8 (exact), in the order of expand_codes.  A nibble inserted into 0x6400 is 1024 + c at bit 0
// and 1024 + 16 c at bit 4, which a packed addition and a packed multiply-add turn into c - 8.
struct SignedCodes {
  uint32_t lo = 0x000F000Fu, hi = 0x00F000F0u, magic = 0x64006400u, m1032 = 0xE408E408u, r16 = 0x2C002C00u, m72 = 0xD480D480u;
  __device__ __forceinline__ void hide() { asm volatile("" : "+v"(lo), "+v"(hi), "+s"(magic), "+v"(m1032), "+s"(r16), "+v"(m72)); }
  __device__ __forceinline__ f16x8 operator()(uint32_t w) const {
    const uint32_t w8 = w >> 8;
    const f16x2 a = __builtin_bit_cast(f16x2, (w & lo) | magic) + __builtin_bit_cast(f16x2, m1032);
    const f16x2 b = __builtin_elementwise_fma(__builtin_bit_cast(f16x2, (w & hi) | magic), __builtin_bit_cast(f16x2, r16), __builtin_bit_cast(f16x2, m72));
    const f16x2 c = __builtin_bit_cast(f16x2, (w8 & lo) | magic) + __builtin_bit_cast(f16x2, m1032);
    const f16x2 d = __builtin_elementwise_fma(__builtin_bit_cast(f16x2, (w8 & hi) | magic), __builtin_bit_cast(f16x2, r16), __builtin_bit_cast(f16x2, m72));
    return __builtin_shufflevector(__builtin_shufflevector(a, b, 0, 1, 2, 3), __builtin_shufflevector(c, d, 0, 1, 2, 3), 0, 1, 2, 3, 4, 5, 6, 7);
  }
};

// part[slot][row][m] = sum over the chunks of the slot of scale_c[m] * sum_j h_j (code[j][m] - 8).  Block: 128 output
// columns (32 per wave) of one slot; a load covers 256 contiguous bytes of two halves of two chunks.
// The fp32 activations of a chunk are scaled by a power of two that brings the largest to [2^14, 2^15) and split into three
// fp16 parts (11 bits each; what a part of an element 2^15 times smaller than that still drops is below 2^-39 of the
// largest), which are three operand rows: rows 4t .. 4t+2 belong to token t, so a lane ends up with the parts of one token.
// The products h (c - 8) are exact and at most 8 |h|, and a weight of 0 adds nothing.  LLaMA-shaped layer, 3 tokens: 26.5 us
// (125 MB of codes, 4.7 TB/s; four pairs of chunks in flight instead of two cost waves).  bf16 parts against 128 + c and
// -136 sum(h) took 24.4 us, but their sums carried 136 |h| until the offset cancelled: 10 to 20 times the rounding error,
// against 64 bits 2.5e-6 instead of 1.5e-6 of a whole call.
constexpr int QDN_COLS = 128, QDN_TB = 4;
__global__ __launch_bounds__(QDN_THREADS) void k_decode_down_q4(const float* __restrict__ h, int ldh, int M, Plan p,
                                                                int expert_sel, int x2_only, WeightView wv_r, WeightView wv_s,
                                                                int shared_z, int cps_s, int slot0, int chunks_per_slot,
                                                                float* __restrict__ part, size_t slot_stride, int tb) {
  extern __shared__ __attribute__((aligned(16))) unsigned char s_h[];
  int e, r0, r1, se;
  // the first shared_z layers of the grid are the j-slots of the shared expert
  const int slot = (int)blockIdx.z - shared_z;
  if (!block_rows(p, expert_sel, x2_only, slot, e, r0, r1)) return;
  const WeightView wv = slot < 0 ? wv_s : wv_r;
  if (slot < 0) chunks_per_slot = cps_s;
  const int s = slot < 0 ? blockIdx.z * gridDim.y + blockIdx.y : blockIdx.y;
  const int c_begin = s * chunks_per_slot;
  const int n_c = min(chunks_per_slot, wv.n_chunks - c_begin);
  if (n_c <= 0) return;
  if (!storage_index(wv, e, se)) return;
  const int tid = threadIdx.x, lane = tid % WAVE, wid = __builtin_amdgcn_readfirstlane(tid / WAVE), q = lane >> 4;
  const int NW = ntile_width(M);
  const size_t cbytes = q4_chunk_u16(M) * 2;
  const unsigned char* base = reinterpret_cast<const unsigned char*>(wv.base + (size_t)se * wv.expert_stride) + (size_t)(wv.chunk0 + c_begin) * cbytes;
  float* out = part + (size_t)(slot0 + s) * slot_stride;
  int m[2];
  size_t qo[2], zo[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    m[i] = blockIdx.x * QDN_COLS + wid * 32 + i * 16 + (lane & 15);
    const int mm = min(m[i], M - 1);
    qo[i] = q4_off_codes(2, M) + (((size_t)(mm / NW) * 2 + (q & 1)) * NW + mm % NW) * 16;
    zo[i] = q4_off_scales(2, M) + (size_t)mm * 2;
  }
  const int n_j = n_c * CHUNK_J, hstride = 2 * n_j + 16;
  float* s_inv = reinterpret_cast<float*>(s_h + (size_t)tb * 3 * hstride);  // [n_c][tb]: 1 / scale of the chunk's activations
  SignedCodes signed_codes;
  signed_codes.hide();

  constexpr int DU = 2;  // pairs of chunks fetched ahead
  u32x4 wd[DU][2];
  uint32_t zd[DU][2];
  auto fetch = [&](int c0) {
#pragma unroll
    for (int d = 0; d < DU; ++d)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const unsigned char* cb = base + (size_t)min(c0 + 2 * d + (q >> 1), n_c - 1) * cbytes;
        wd[d][i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(cb + qo[i]));
        zd[d][i] = *reinterpret_cast<const uint16_t*>(cb + zo[i]);
      }
  };
  fetch(0);
  for (int rb = r0; rb < r1; rb += tb) {
    const int nt = min(tb, r1 - rb);
    if (rb != r0) {
      __syncthreads();
      fetch(0);
    }
    // eight activations per thread, stored in the order in which a word delivers its codes: 0 2 4 6 1 3 5 7
    for (int i = tid; i < nt * (n_j / 8); i += QDN_THREADS) {
      const int t = i / (n_j / 8), c8 = i % (n_j / 8);
      const f32x4* src = reinterpret_cast<const f32x4*>(h + (size_t)(rb + t) * ldh + wv.col0 + c_begin * CHUNK_J + c8 * 8);
      const f32x4 lo = src[0], hi = src[1];
      float v[8] = {lo[0], lo[2], hi[0], hi[2], lo[1], lo[3], hi[1], hi[3]};
      float top = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) top = fmaxf(top, fabsf(v[e]));
#pragma unroll
      for (int d = 1; d < 8; d <<= 1) top = fmaxf(top, __shfl_xor(top, d, WAVE));  // (the 8 threads of a chunk are adjacent lanes)
      // biased exponent; from 15 up the scale and its reciprocal are normal numbers
      const uint32_t ex = max(__float_as_uint(top) >> 23, 15u);
      const float up = __uint_as_float((268u - ex) << 23);
      f16x2 o[3][4];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float rest = v[e] * up;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          const _Float16 pv = (_Float16)rest;
          rest -= (float)pv;
          o[a][e >> 1][e & 1] = pv;
        }
      }
#pragma unroll
      for (int a = 0; a < 3; ++a) *reinterpret_cast<u32x4*>(s_h + (t * 3 + a) * hstride + c8 * 16) = __builtin_bit_cast(u32x4, o[a]);
      if ((c8 & 7) == 0) s_inv[(size_t)(c8 >> 3) * tb + t] = __uint_as_float((ex - 14u) << 23);
    }
    __syncthreads();
    const unsigned char* hrow = s_h + (min((lane & 15) >> 2, nt - 1) * 3 + min(lane & 3, 2)) * hstride + unit_k(q) * 2;
    const float* irow = s_inv + min(q, nt - 1);
    float tot[2] = {0.f, 0.f};
    for (int c0 = 0; c0 < n_c; c0 += 2 * DU) {
      u32x4 cd[DU][2];
      uint32_t cz[DU][2];
#pragma unroll
      for (int d = 0; d < DU; ++d)
#pragma unroll
        for (int i = 0; i < 2; ++i) { cd[d][i] = wd[d][i]; cz[d][i] = zd[d][i]; }
      if (c0 + 2 * DU < n_c) fetch(c0 + 2 * DU);
#pragma unroll
      for (int d = 0; d < DU; ++d) {
        uint32_t g[2][2][2];
        float sc[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          split_groups(cd[d][i], g[i]);
          const auto z = __builtin_amdgcn_permlane32_swap(cz[d][i], cz[d][i], false, false);
          sc[0][i] = __uint_as_float(z[0] << 16);
          sc[1][i] = __uint_as_float(z[1] << 16);
        }
#pragma unroll
        for (int gi = 0; gi < 2; ++gi) {
          const int c = c0 + 2 * d + gi;
          if (c < n_c) {
            const float inv = irow[(size_t)c * tb];
            f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int k = 0; k < 2; ++k) {
              const f16x8 hv = __builtin_bit_cast(f16x8, *reinterpret_cast<const u32x4*>(hrow + c * 128 + k * 16));
#pragma unroll
              for (int i = 0; i < 2; ++i)
                acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hv, signed_codes(g[i][gi][k]), acc[i], 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) tot[i] = fmaf(sc[gi][i], (acc[i][0] + (acc[i][1] + acc[i][2])) * inv, tot[i]);
          }
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
      if (q < nt && m[i] < M) out[(size_t)(rb + q) * M + m[i]] = tot[i];
  }
}

__device__ inline uint32_t pack_bf16x2(float a, float b) {
  uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
  ua += 0x7fffu + ((ua >> 16) & 1u);  // round to nearest even
  ub += 0x7fffu + ((ub >> 16) & 1u);
  return (ua >> 16) | (ub & 0xffff0000u);
}

// 4-bit chunks [c0, c0+n) of the selected experts -> bf16 chunks 0..n of `dst` (expert e at dst + e*dst_estride),
// value = bf16((code - 8) * scale).  One thread per 32-bit word of codes (8 weights -> one 16-byte store).
// grid: (n * 24, experts): 8 blocks of work per gate block, 8 per up block, 8 per down block of a chunk.
__global__ __launch_bounds__(256) void k_dequant_q4(const uint16_t* __restrict__ src, size_t src_estride,
                                                    const int32_t* __restrict__ e_map, int c0, int M, Plan p,
                                                    int expert_sel, int x2_only, uint16_t* __restrict__ dst,
                                                    size_t dst_estride) {
  int e, de;
  if (expert_sel >= 0) {
    e = expert_sel;
    de = 0;
  } else {
    e = blockIdx.y;
    de = e;
    if (e >= p.n_routed) return;
  }
  if (row_end(p, e) - row_begin(p, e, x2_only) <= 0) return;  // no rows: nobody reads these weights
  const int se = e_map ? e_map[e] : e;
  if (se < 0) return;
  const int c = blockIdx.x / 24, sec = (blockIdx.x % 24) / 8, oct = blockIdx.x % 8;
  const unsigned char* cb = reinterpret_cast<const unsigned char*>(src + (size_t)se * src_estride + (size_t)(c0 + c) * q4_chunk_u16(M));
  uint16_t* ob = dst + (size_t)de * dst_estride + (size_t)c * 3 * CHUNK_J * M + (size_t)sec * CHUNK_J * M;
  const uint32_t* q = reinterpret_cast<const uint32_t*>(cb + q4_off_codes(sec, M));
  const uint16_t* z = reinterpret_cast<const uint16_t*>(cb + q4_off_scales(sec, M));
  float v[8];
  if (sec < 2) {
    // rows oct*8 .. oct*8+7 of the gate / up block; destination [M/PW panels][64 j][PW m]
    const int PW = panel_width(M), M8 = M / 8;
    for (int i = threadIdx.x; i < 8 * M8; i += 256) {
      const int j = oct * 8 + i / M8, m0 = (i % M8) * 8;
      const uint32_t w = q[(size_t)j * M8 + m0 / 8];
      const float sc = bf16_f32(z[(size_t)j * (M / 64) + m0 / 64]);
#pragma unroll
      for (int el = 0; el < 8; ++el) v[el] = (float)((int)((w >> (4 * q4_fc1_nibble(el))) & 15u) - 8) * sc;
      const uint4 o = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
      *reinterpret_cast<uint4*>(ob + gu_off(j, m0, PW)) = o;
    }
  } else {
    // j = oct*8 .. oct*8+7 of the down block for every column m; destination [M/NW][8 q][NW m][8 i]
    const int NW = ntile_width(M);
    for (int m = threadIdx.x; m < M; m += 256) {
      const uint32_t w = q[q4_fc2_word(oct * 8, m, NW)];
      const float sc = bf16_f32(z[m]);
#pragma unroll
      for (int el = 0; el < 8; ++el) v[el] = (float)((int)((w >> (4 * q4_fc2_nibble(el))) & 15u) - 8) * sc;
      const uint4 o = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
      *reinterpret_cast<uint4*>(ob + dn_off(oct * 8, m, NW)) = o;
    }
  }
}

size_t down_lds(int tb, int cps) { return (size_t)tb * 3 * (2 * cps * CHUNK_J + 16) + (size_t)cps * tb * 4; }
constexpr size_t Q4_LDS = 81 * 1024;  // two blocks per compute unit

hipError_t ensure_q4_lds() {
  static hipError_t st = [] {
    const void* kernels[] = {(const void*)k_decode_gateup_q4<true>, (const void*)k_decode_gateup_q4<false>, (const void*)k_decode_gateup_q4_split, (const void*)k_decode_down_q4};
    for (const void* k : kernels) {
      const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)Q4_LDS);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }();
  return st;
}

}  // namespace

hipError_t launch_decode_gateup_q4(const uint16_t* x, int M, const Plan& plan, int tb_hint, int expert_sel, int x2_only,
                                   int max_touched, const WeightView& wv, int e_chunks, const WeightView& ws, float* h, int ldh, hipStream_t stream) {
  if (wv.n_chunks <= 0) return hipSuccess;
  if (hipError_t e = ensure_q4_lds(); e != hipSuccess) return e;
  if (expert_sel >= 0 && ws.n_chunks == 0 && gateup_split(M, e_chunks)) {
    const int ng = wv.n_chunks * (CHUNK_J / 4), blocks = std::min(QGS_BLOCKS, ng);
    const int groups = std::min((ng + blocks - 1) / blocks, (int)(QGS_LDS / gateup_group_lds(M)));
    hipLaunchKernelGGL(k_decode_gateup_q4_split, dim3(blocks), dim3(QGS_THREADS), groups * gateup_group_lds(M), stream, x, M, plan, expert_sel, x2_only, wv,
                       groups, h, ldh);
    return hipGetLastError();
  }
  const int shared_y = (ws.n_chunks + wv.n_chunks - 1) / wv.n_chunks;
  dim3 grid(wv.n_chunks * (CHUNK_J / QGU_JPB), shared_y + (expert_sel >= 0 ? 1 : max_touched));
  const int tb = std::max(1, std::min(tb_hint, QGU_TB));
  const bool pad = gateup_lds(tb, M, true) <= QGU_LDS;
  hipLaunchKernelGGL(pad ? k_decode_gateup_q4<true> : k_decode_gateup_q4<false>, grid, dim3(QGU_THREADS), gateup_lds(tb, M, pad), stream, x, M, plan, expert_sel, x2_only, wv, ws, shared_y, h, ldh, tb);
  return hipGetLastError();
}

hipError_t launch_decode_down_q4(const float* h, int ldh, int M, const Plan& plan, int tb_hint, int expert_sel, int x2_only,
                                 int max_touched, const WeightView& wv, const WeightView& ws, int cps_s, int slot0,
                                 int chunks_per_slot, float* part, size_t slot_stride, hipStream_t stream) {
  if (wv.n_chunks <= 0) return hipSuccess;
  if (hipError_t e = ensure_q4_lds(); e != hipSuccess) return e;
  const int n_slots = (wv.n_chunks + chunks_per_slot - 1) / chunks_per_slot;
  const int slots_s = ws.n_chunks > 0 ? (ws.n_chunks + cps_s - 1) / cps_s : 0, shared_z = (slots_s + n_slots - 1) / n_slots;
  const int cps_max = std::max(chunks_per_slot, slots_s ? cps_s : 0);
  dim3 grid((M + QDN_COLS - 1) / QDN_COLS, n_slots, shared_z + (expert_sel >= 0 ? 1 : max_touched));
  int tb = std::max(1, std::min(tb_hint, QDN_TB));
  while (tb > 1 && down_lds(tb, cps_max) > Q4_LDS) --tb;
  hipLaunchKernelGGL(k_decode_down_q4, grid, dim3(QDN_THREADS), down_lds(tb, cps_max), stream, h, ldh, M, plan, expert_sel, x2_only, wv, ws, shared_z, cps_s, slot0, chunks_per_slot, part, slot_stride, tb);
  return hipGetLastError();
}

hipError_t launch_dequant_q4(const WeightView& wv, int M, const Plan& plan, int expert_sel, int x2_only, int n_experts,
                             uint16_t* dst, size_t dst_estride, hipStream_t stream) {
  if (wv.n_chunks <= 0) return hipSuccess;
  dim3 grid(wv.n_chunks * 24, expert_sel >= 0 ? 1 : n_experts);
  hipLaunchKernelGGL(k_dequant_q4, grid, dim3(256), 0, stream, wv.base, wv.expert_stride, wv.e_map, wv.chunk0, M, plan,
                     expert_sel, x2_only, dst, dst_estride);
  return hipGetLastError();
}

}  // namespace si
