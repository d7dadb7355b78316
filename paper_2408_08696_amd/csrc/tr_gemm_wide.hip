// Projection GEMM whose waves share both operands in LDS: y[n, O] = a[n, K] * w[O, K]^T with n up to WIDE_MAX_ROWS rows at
// once.  All projections of prompt ingestion above TR_MAX_NODES rows, and a tree step's matrices of many out-tiles (rows8_plan).
//
// A workgroup of eight waves owns NW consecutive out-tiles and RB row tiles (16 x 16 tiles = 256 x 256 outputs in the
// largest shape); its waves form a WR x WC grid over that block, so that a tile loaded once serves WC or WR of them.
// Both operands travel memory -> LDS without passing through registers (global_load_lds, 16 bytes a lane: a fragment
// tile is one contiguous KiB on both sides) into a ring of D k-steps, D - 1 of them under way while one is multiplied.
// A wave reads the operands of k-step s + 1 between the MFMAs of k-step s and meets the others once per k-step; the
// MFMAs that follow the barrier have their operands in registers already.  A wave ends with the sums over its k range
// for its outputs, and the epilogue runs from registers: no cross-wave reduction, but for the form of two groups of waves
// (KG = 2), whose sums meet in LDS once.  Projections with few out-tiles (o and
// down) are split over k so that the launch still fills the chip; the residual kernel adds the partial sums.  Row
// blocks of one out-tile group have linear ids congruent modulo 8, land on one XCD and share its weights in that L2.
//
// What bounds it.  A compute unit takes tiles in at 47-52 GB/s when part of them comes from memory, against 100-107
// when all are in L2 and whatever the share of the chip that is busy (96 to 256 workgroups alike): its load path
// holds about 48 KB and returns in order, so every tile waits as long as a weight tile does.  The time of a k-step is
// therefore its tiles over that rate, and the shapes with the most MFMAs per tile win wherever they fill the chip:
// us per k-step (tile pairs per workgroup) 0.28-0.31 (64), 0.40-0.42 (96), 0.43-0.45 (128), 0.57-0.59 (192), 0.66-0.74
// (256, 1.4 PFLOP/s in full rounds, the matrix pipe 73 % busy).  LDS reads are conflict-free and take a quarter of
// that unit's time.  Measured without effect: weight tiles at other strides or in another k order per workgroup, wave
// priorities; slower: touching lines ahead of the loads to bring them into L2 (the touches go through the same path).
// 512 rows, us per launch, this kernel / one that took weights through registers and activations straight to the
// operands (8 x 1 wave grid): 7B gate/up 79 / 94, Q/K/V 60 / 61, o + down 80 / 103, 70B gate/up 392 / 489, o + down 276 /
// 360, Q/K/V 108 / 97.
//
// Same packed weight layout, fragment-ordered activations and epilogues (plain store, RoPE + cache append,
// SwiGLU, residual update) as the decode kernel.
#include <type_traits>
#include <utility>

#include "tr_kernels.h"

namespace tr {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

__device__ inline f32x16 mfma32w(const u32x4 &a, const u32x4 &b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

constexpr int WIDE_WAVES = 8;

// Weight tiles carry the streaming hint: few workgroups read them and the activations keep their place in L2 (7B, 511
// rows: o and down 84.2 -> 79.7 us, Q/K/V 63.3 -> 61.6; nothing at 70B width with eight row blocks).
__device__ inline void w_tile_to_lds(uint32_t lds_off, uint32_t voff, uint64_t gbase) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds_off), "v"(voff), "s"(gbase)
               : "memory");
}
// tile_to_lds for lanes 0 .. 31 alone: half a tile.  (Called with all lanes active.)
__device__ inline void half_tile_to_lds(uint32_t lds_off, uint32_t voff, uint64_t gbase) {
  asm volatile("s_mov_b32 m0, %0\n\ts_mov_b64 exec, 0xffffffff\n\tglobal_load_lds_dwordx4 %1, %2 nt\n\ts_mov_b64 exec, -1"
               ::"s"(lds_off), "v"(voff), "s"(gbase) : "memory");
}
// Words (a0, a1) hold features 4 hb .. + 3 and (b0, b1) 8 + 4 hb .. + 3 of a row's sixteen in lane 32 hb + row; the result holds
// features 8 hb .. + 7.
__device__ inline uint4 eight_features(uint32_t a0, uint32_t a1, uint32_t b0, uint32_t b1) {
  const auto s0 = __builtin_amdgcn_permlane32_swap(a0, b0, false, false); // lanes 32 .. 63 of the first with 0 .. 31 of the second
  const auto s1 = __builtin_amdgcn_permlane32_swap(a1, b1, false, false);
  return uint4{s0[0], s1[0], s0[1], s1[1]};
}
template <typename F, int... J>
__device__ inline void for_each_step(F f, std::integer_sequence<int, J...>) {
  (f(std::integral_constant<int, J>{}), ...);
}

// RP2 x NP2: pairs of row tiles x pairs of out-tiles per wave; WR x WC: the workgroup's wave grid (WR * WC = 8).
// KG = 2: two such groups of waves take even and odd k-tiles (both in each step of the ring, T tiles each) and the first adds the
// other's sums at the end; WR * WC * KG = 8.
// SwiGLU: an out-tile pair is (gate tile, up tile) of the same 16 features.
// What the first tiles need leads the arguments and comes in scalar registers with the wave (w1: up, or the second of Q/K/V).
template <int MODE, bool SCALED, int RP2, int NP2, int WR, int WC, int D, int CHAIN, int KG>
__global__ __launch_bounds__(WIDE_WAVES * 64) void k_gemm_wide(const bf16_t *a_frag, const bf16_t *w0, const bf16_t *w1,
                                                              int32_t KT, int32_t row_tiles, int32_t groups, int32_t splits,
                                                              int32_t part_q, int32_t part_rem, GemmArgs g) {
  constexpr bool ROPE = MODE == GEMM_ROPE; // GEMM_STORE with the fused Q/K/V epilogue
  constexpr int RB = 2 * RP2 * WR, NW = 2 * NP2 * WC; // row tiles and out-tiles of the workgroup
  constexpr int T = RB + NW;                          // tiles per k-step
  constexpr int TS = KG * T;                          // tiles per step of the ring
  constexpr int C = (TS + WIDE_WAVES - 1) / WIDE_WAVES;     // tile loads of a wave per step
  constexpr bool HALVES = TS % WIDE_WAVES != 0;             // the last of them is half a tile
  static_assert(TS % WIDE_WAVES == 0 || TS % WIDE_WAVES == WIDE_WAVES / 2, "whole and half tiles only");
  static_assert(WR * WC * KG == WIDE_WAVES && D * TS <= 160 && D >= 3, "the ring is the compute unit's LDS at most");
  extern __shared__ u32x4 ring[]; // [D][TS][64]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6); // in a scalar register: what depends on it alone is uniform
  const int kg = wave / (WR * WC), wr = wave / WC % WR, wc = wave % WC;
  // linear id -> (k-split, out-tile group, row block): ids that differ by 8 share an XCD, so the row blocks of
  // a group are 8 apart; groups are numbered (id % 8) + 8 * (id / (8 * row_blocks))
  const int row_blocks = (row_tiles + RB - 1) / RB;
  const int per_split = ((groups + 7) / 8) * 8 * row_blocks;
  const int split = blockIdx.x / per_split, id = blockIdx.x - split * per_split;
  const int bx = (id & 7) + 8 * (id / (8 * row_blocks));
  const int rb = (id >> 3) % row_blocks;
  if (bx >= groups) return; // uniform over the workgroup (group count not a multiple of 8)
  const int per_k = (KT + splits - 1) / splits;
  const int k0 = split * per_k, k1 = k0 + per_k < KT ? k0 + per_k : KT;
  const int nk = (k1 - k0) / KG; // >= 1: the launch leaves no split empty; KG = 2: an even number of k-tiles
  const int tile0 = bx * part_q + (bx < part_rem ? bx : part_rem);
  const int n_valid = part_q + (bx < part_rem ? 1 : 0);

  // The tiles of a k-step this wave loads: tile j = wave + 8 i, the first RB of them row tiles, then out-tiles (with
  // T = 8 c + 4 the last four are loaded by two waves each, half by half: every wave then has the same number of loads
  // to wait for).  Row tiles past the last and unused out-tile slots load a neighbour again; nothing of theirs is stored.
  uint64_t src[C];
  uint32_t dst[C], step[C];
  bool of_rows[C]; // KG = 2 mixes both kinds in a load (all without the streaming hint: 7B gate/up of 128 rows 44 -> 47 us)
#pragma unroll
  for (int i = 0; i < C; ++i) {
    const bool half = HALVES && i == C - 1;
    const int slot = WIDE_WAVES * i + (half ? wave >> 1 : wave), k = KG > 1 ? slot / T : 0, j = slot - k * T;
    of_rows[i] = j < RB;
    if (j < RB) {
      int rt = rb * RB + j;
      rt = rt < row_tiles ? rt : row_tiles - 1;
      src[i] = reinterpret_cast<uint64_t>(a_frag) + ((uint64_t)(k0 + k) * row_tiles + rt) * 1024;
      step[i] = (uint32_t)row_tiles * KG * 1024;
    } else {
      const int u = j - RB;
      const int uu = MODE == GEMM_SWIGLU ? u >> 1 : u;
      int t = tile0 + (uu < n_valid ? uu : 0);
      const bf16_t *mat = MODE == GEMM_SWIGLU && (u & 1) ? w1 : w0;
      if constexpr (ROPE || MODE == GEMM_PARTS) {
        if (t >= g.seg[0].out_tiles + g.seg[1].out_tiles) {
          t -= g.seg[0].out_tiles + g.seg[1].out_tiles;
          mat = g.seg[2].w;
        } else if (t >= g.seg[0].out_tiles) {
          t -= g.seg[0].out_tiles;
          mat = w1;
        }
      }
      src[i] = reinterpret_cast<uint64_t>(mat) + ((uint64_t)t * KT + k0 + k) * 1024;
      step[i] = KG * 1024;
    }
    dst[i] = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)ring + slot * 1024;
    if (half) {
      src[i] += (wave & 1) * 512;
      dst[i] += (wave & 1) * 512;
    }
  }
  const uint32_t voff = lane * 16;
  auto load = [&](int i, uint32_t slot_off) { // the i-th load of the next k-step, into the ring slot at this offset
    if (HALVES && i == C - 1) half_tile_to_lds(dst[i] + slot_off, voff, src[i]);
    else if (KG > 1 ? of_rows[i] : i * WIDE_WAVES < RB) tile_to_lds(dst[i] + slot_off, voff, src[i]);
    else w_tile_to_lds(dst[i] + slot_off, voff, src[i]);
    src[i] += step[i];
  };

  // MFMA shape: v_mfma_f32_32x32x16_bf16 (same rate per flop as the 16x16x32 form, half as many instructions).  Its
  // operands are rebuilt from the 16x32 fragment tiles by addressing alone: for k-half h of a k-step, lane l supplies
  // 8 k-values 16 h + 8 (l / 32) .. + 7 of item l % 32, i.e. lane slot (l % 16) + 16 (2 h + l / 32) of the first
  // (l % 32 < 16) or second tile of a pair.  The 32 x 32 result leaves lane l with row l % 32 of the row pair and, in
  // elements 4q .. 4q + 3, features 8 q + 4 (l / 32) .. + 3 of the 32 the out-tile pair spans.
  const int half_sel = (lane >> 4) & 1, hb = lane >> 5;
  const int frag = half_sel * 64 + (lane & 15) + 16 * hb; // in 16-byte units; + 32 for the second k-half
  const char *abase = reinterpret_cast<const char *>(ring + (kg * T + wr * (2 * RP2)) * 64 + frag);
  const char *wbase = reinterpret_cast<const char *>(ring + (kg * T + RB + wc * (2 * NP2)) * 64 + frag);

  f32x16 acc[NP2][RP2];
#pragma unroll
  for (int u = 0; u < NP2; ++u)
#pragma unroll
    for (int j = 0; j < RP2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[u][j][e] = 0.f;
  u32x4 wf[2][NP2][2], af[2][RP2][2]; // operands of the current and the next k-step
  // CHAIN > 0: sums of CHAIN k-steps, added up here.  A chain over all of k loses more to rounding than the decode kernel.
  f32x16 total[CHAIN > 0 ? NP2 : 1][CHAIN > 0 ? RP2 : 1];
  int chained = 0;
  if constexpr (CHAIN > 0) {
#pragma unroll
    for (int u = 0; u < NP2; ++u)
#pragma unroll
      for (int j = 0; j < RP2; ++j) total[u][j] = acc[u][j];
  }
  auto end_chain = [&](int steps) {
    if constexpr (CHAIN > 0) {
      chained += steps;
      if (chained < CHAIN) return;
      chained = 0;
#pragma unroll
      for (int u = 0; u < NP2; ++u)
#pragma unroll
        for (int j = 0; j < RP2; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            total[u][j][e] += acc[u][j][e];
            acc[u][j][e] = 0.f;
          }
    }
  };

  constexpr int READS = 2 * (NP2 + RP2), MFMAS = 2 * NP2 * RP2;
  constexpr int RPM = (READS + MFMAS - 2) / (MFMAS - 1); // operand reads behind an MFMA (1 where they fit, 2 cost 1 %)
  auto read_frag = [&](int set, int i, uint32_t at) { // i-th of the READS operand reads of the k-step in ring slot `at`
    const int h = i / (NP2 + RP2), r = i % (NP2 + RP2);
    if (r < RP2) af[set][r][h] = *reinterpret_cast<const u32x4 *>(abase + at + (2 * r * 64 + 32 * h) * 16);
    else wf[set][r - RP2][h] = *reinterpret_cast<const u32x4 *>(wbase + at + (2 * (r - RP2) * 64 + 32 * h) * 16);
  };
  // One k-step s in ring slot `slot` (a byte offset): its operands (set SET) were read during s - 1; the tiles of s + 1
  // must have landed for every wave, and its own slot, which every wave has read, takes k-step s + D.  Of the
  // min(s + D, nk) k-steps requested so far, those past s + 1 may stay under way.  STEADY: s + D < nk.
  constexpr uint32_t SLOT = TS * 1024;
  uint32_t slot = 0;
  auto k_step = [&](auto set_c, auto steady_c, int s) {
    constexpr int SET = decltype(set_c)::value;
    constexpr bool STEADY = decltype(steady_c)::value;
    if constexpr (STEADY) {
      wait_tiles<(D - 2) * C>();
    } else {
      const int under_way = nk - 2 - s;
      if (under_way >= D - 2) wait_tiles<(D - 2) * C>();
      else
        for_each_step([&](auto j) {
          constexpr int J = decltype(j)::value;
          if (under_way == J) wait_tiles<J * C>();
        }, std::make_integer_sequence<int, D - 2>{});
    }
    meet_waves();
    const uint32_t next = slot + SLOT < D * SLOT ? slot + SLOT : 0;
#pragma unroll
    for (int i = 0; i < MFMAS; ++i) {
      const int h = i / (NP2 * RP2), p = (i / RP2) % NP2, j = i % RP2;
      acc[p][j] = mfma32w(wf[SET][p][h], af[SET][j][h], acc[p][j]);
#pragma unroll
      for (int r = 0; r < READS; ++r)
        if (r / RPM == i) read_frag(SET ^ 1, r, next);
      __builtin_amdgcn_sched_barrier(0); // keep this order: left alone, the scheduler bunches the reads
#pragma unroll
      for (int c = 0; c < C; ++c)
        if (i == 1 + c * ((MFMAS - 2) / C) && (STEADY || s + D < nk)) load(c, slot);
    }
    slot = next;
  };

#pragma unroll
  for (int s = 0; s < D; ++s)
    if (s < nk) {
#pragma unroll
      for (int c = 0; c < C; ++c) load(c, s * SLOT);
    }
  if (nk >= D) wait_tiles<(D - 1) * C>();
  else wait_tiles<0>();
  meet_waves();
#pragma unroll
  for (int r = 0; r < READS; ++r) read_frag(0, r, 0);
  constexpr std::integral_constant<int, 0> set0{};
  constexpr std::integral_constant<int, 1> set1{};
  int s = 0;
  if (nk & 1) { // one k-step ahead of the pairs
    if (nk - 2 >= D - 2) wait_tiles<(D - 2) * C>();
    else wait_tiles<0>();
    meet_waves();
#pragma unroll
    for (int i = 0; i < MFMAS; ++i) {
      const int h = i / (NP2 * RP2), p = (i / RP2) % NP2, j = i % RP2;
      acc[p][j] = mfma32w(wf[0][p][h], af[0][j][h], acc[p][j]);
    }
    if (D < nk) {
#pragma unroll
      for (int c = 0; c < C; ++c) load(c, 0);
    }
#pragma unroll
    for (int r = 0; r < READS; ++r) read_frag(0, r, SLOT);
    slot = SLOT;
    s = 1;
  }
  for (; s + 2 <= nk - D; s += 2) {
    k_step(set0, std::true_type{}, s);
    k_step(set1, std::true_type{}, s + 1);
    end_chain(2);
  }
  // The last tiles are under way: what the epilogue needs of its rows comes behind them.
  const int pos0 = ROPE ? *g.rope.d_len : 0;
  float ssq[SCALED ? RP2 : 1][4];
  if (SCALED) {
#pragma unroll
    for (int j = 0; j < RP2; ++j) {
      const int row = 16 * (rb * RB + wr * 2 * RP2 + 2 * j) + (lane & 31);
      const float *at = g.row_ssq + (size_t)(row < g.n ? row : g.n - 1) * g.n_ssq;
      if (CHAIN > 0 || g.n_ssq <= 8) {
#pragma unroll
        for (int c = 0; c < 4; ++c) ssq[j][c] = at[hb + 2 * c < g.n_ssq ? hb + 2 * c : 0];
      } else { // a multiple of 4, of which the row's two lanes take alternate fours
        float4 sum = float4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
        for (int c = 4 * hb; c < g.n_ssq; c += 8) {
          const float4 q = *reinterpret_cast<const float4 *>(at + c);
          sum.x += q.x; sum.y += q.y; sum.z += q.z; sum.w += q.w;
        }
        ssq[j][0] = sum.x; ssq[j][1] = sum.y; ssq[j][2] = sum.z; ssq[j][3] = sum.w;
      }
    }
    asm volatile("" ::: "memory"); // here and not where they are used
  }
  for (; s < nk; s += 2) {
    k_step(set0, std::false_type{}, s);
    k_step(set1, std::false_type{}, s + 1);
    end_chain(2);
  }
  if constexpr (CHAIN > 0) {
#pragma unroll
    for (int u = 0; u < NP2; ++u)
#pragma unroll
      for (int j = 0; j < RP2; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[u][j][e] += total[u][j][e];
  }
  if constexpr (KG > 1) {
    static_assert(KG == 2 && WR * WC * NP2 * RP2 * 4 <= D * TS, "the second group's sums fit the ring");
    f32x4 *xa = reinterpret_cast<f32x4 *>(ring) + (size_t)(wave % (WR * WC)) * (NP2 * RP2 * 4 * 64) + lane;
    wait_tiles<0>();
    __syncthreads(); // everyone has read the last k-step
    if (kg == 1) {
#pragma unroll
      for (int i = 0; i < NP2 * RP2 * 4; ++i) {
        const f32x16 &a = acc[i / (4 * RP2)][i / 4 % RP2];
        xa[i * 64] = f32x4{a[4 * (i & 3)], a[4 * (i & 3) + 1], a[4 * (i & 3) + 2], a[4 * (i & 3) + 3]};
      }
    }
    __syncthreads();
    if (kg == 1) return;
#pragma unroll
    for (int i = 0; i < NP2 * RP2 * 4; ++i) {
      const f32x4 o = xa[i * 64];
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i / (4 * RP2)][i / 4 % RP2][4 * (i & 3) + e] += o[e];
    }
  }
  const int rt0 = rb * RB + wr * 2 * RP2;
  if (rt0 >= row_tiles) return;

  // Epilogue from registers, bound by its vector instructions and stores.  us of a workgroup's time, with the RMS partial sums, the
  // rotary factors and the committed length asked for one after another where they were used, an integer division per four
  // features, rounding to bf16 by integer arithmetic and 8-byte stores / now: 7B, 511 rows: gate/up 4.8 / 2.2 of 77, Q/K/V 7.7 / 4.9
  // of 57; 70B, 2048 rows, a round: gate/up 7.2 / 2.9 of 190, Q/K/V 20.7 / 11.5 of 165.  (Gate/up's second figure is with a
  // reciprocal for SwiGLU's division; the division adds 0.2 % to a prompt of 511 tokens at 7B width, 0.5 % to 4095 at 70B width.)
#pragma unroll
  for (int j = 0; j < RP2; ++j) {
    const int row = 16 * (rt0 + 2 * j) + (lane & 31);
    const int rt = row >> 4, r = row & 15;
    f32x2 rope_c[ROPE ? NP2 * 4 : 1], rope_s[ROPE ? NP2 * 4 : 1];
    if constexpr (ROPE) { // head_dim is 128 (tiled cache): eight out-tiles a head
      const float *cs = g.rope.rope + (size_t)(row < g.n ? row : g.n - 1) * 128;
#pragma unroll
      for (int i = 0; i < NP2 * 4; ++i) {
        const int t = tile0 + 2 * (wc * NP2 + (i >> 2)) + ((i & 3) >> 1);
        const float *at = cs + (t & 7) * 8 + 4 * (i & 1) + 2 * hb;
        rope_c[i] = *reinterpret_cast<const f32x2 *>(at);
        rope_s[i] = *reinterpret_cast<const f32x2 *>(at + 64);
      }
      __builtin_amdgcn_sched_barrier(0); // all of them on their way before the first store
    }
    if (rt >= row_tiles) continue;
    // x += the sums, the next projection's operand and this wave's sums of squares.  Bound by memory: where a launch is one round, all
    // workgroups read and write x at once.  us at 2048 rows, plain store + residual kernel / this: 70B o 199 + 55 / 219, down 676 + 55 / 697;
    // prompts of 1023 and 2047 tokens at 7B width (16 layers) 6706 / 6533 and 12290 / 11970, 2047 at 13B width (8) 9092 / 8925, 4095 at
    // 70B (4) 17720 / 17580.  Streaming hints on x lose 1 to 5 %, on the operand 0.
    if constexpr (MODE == GEMM_RESID) {
      const bool on = row < g.n;
      float *const xr = g.resid.x + (size_t)(on ? row : g.n - 1) * g.ldy + (tile0 + 2 * wc * NP2) * 16 + 4 * hb;
      const bf16_t *const gr = g.resid.gain + (tile0 + 2 * wc * NP2) * 16 + 4 * hb;
      float4 x[NP2 * 4];
      uint2 gain[NP2 * 4];
#pragma unroll
      for (int i = 0; i < NP2 * 4; ++i) { // out-tiles that the workgroup does not have read its first one again
        const int at = 2 * wc * NP2 + (i >> 1) < n_valid ? 8 * i : -(2 * wc * NP2) * 16;
        x[i] = *reinterpret_cast<const float4 *>(xr + at);
        gain[i] = *reinterpret_cast<const uint2 *>(gr + at);
      }
      __builtin_amdgcn_sched_barrier(0); // all of them on their way before the first store
      float ss = 0.f;
#pragma unroll
      for (int u2 = 0; u2 < 2 * NP2; ++u2) {
        if (2 * wc * NP2 + u2 >= n_valid) continue;
        const int t = tile0 + 2 * wc * NP2 + u2;
        uint32_t w[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int q = 2 * u2 + i;
          const f32x16 &a = acc[u2 >> 1][j];
          const int e = 4 * (q & 3);
          const f32x4 v = f32x4{x[q].x + a[e], x[q].y + a[e + 1], x[q].z + a[e + 2], x[q].w + a[e + 3]};
          if (on) *reinterpret_cast<float4 *>(xr + 8 * q) = float4{v[0], v[1], v[2], v[3]};
          ss += (v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]);
          w[i][0] = bf16_pair(v[0] * __uint_as_float(gain[q].x << 16), v[1] * __uint_as_float(gain[q].x & 0xFFFF0000u));
          w[i][1] = bf16_pair(v[2] * __uint_as_float(gain[q].y << 16), v[3] * __uint_as_float(gain[q].y & 0xFFFF0000u));
        }
        uint4 e = eight_features(w[0][0], w[0][1], w[1][0], w[1][1]);
        if (!on) e = uint4{0u, 0u, 0u, 0u};
        const size_t fslot = ((size_t)(t >> 1) * row_tiles + rt) * 64 + r + 16 * (2 * (t & 1) + hb);
        reinterpret_cast<uint4 *>(g.resid.xg_frag)[fslot] = e;
      }
      ss += __shfl_xor(ss, 32);
      if (on && hb == 0) {
        float *const at = g.resid.ssq + (size_t)row * g.resid.ld_ssq;
        at[bx * WC + wc] = ss;
        if (bx == groups - 1 && wc == WC - 1)
          for (int c = groups * WC; c < g.resid.ld_ssq; ++c) at[c] = 0.f; // sums of no wave
      }
      continue;
    }
    float sc_row = 1.0f;
    if (SCALED) { // per-row RMS scale; the row's two lanes hold alternate partial sums
      float ss = 0.f;
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (hb + 2 * c < g.n_ssq) ss += ssq[j][c];
      ss += __shfl_xor(ss, 32);
      sc_row = 1.0f / sqrtf(ss / (float)g.norm_dim + g.eps);
    }
    // A lane's accumulator elements are features 8 q + 4 hb .. + 3 of an out-tile for q = 0, 1.  In 16 bits the two lanes of a row
    // exchange halves, so that each has eight neighbouring features and stores them at once.
#pragma unroll
    for (int p2 = 0; p2 < NP2; ++p2) {
      const f32x16 &a = acc[p2][j];
#pragma unroll
      for (int half = 0; half < (MODE == GEMM_SWIGLU ? 1 : 2); ++half) { // out-tile u; SWIGLU: gate elements 0 .. 7, up 8 .. 15
        const int u = MODE == GEMM_SWIGLU ? wc * NP2 + p2 : 2 * (wc * NP2 + p2) + half;
        if (u >= n_valid) continue;
        const int t = tile0 + u;
        if constexpr (MODE == GEMM_STORE || MODE == GEMM_PARTS) {
          if (row >= g.n) continue;
#pragma unroll
          for (int q = 2 * half; q < 2 * half + 2; ++q) {
            const f32x4 v = f32x4{a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]} * sc_row;
            *reinterpret_cast<float4 *>(g.y + (size_t)split * g.split_stride + (size_t)row * g.ldy + t * 16 + 8 * (q & 1) + 4 * hb) =
                float4{v[0], v[1], v[2], v[3]};
          }
        } else if constexpr (ROPE) {
          // fused Q/K/V epilogue, as in the decode kernel, into a tiled cache: neighbouring features are rotation pairs
          const GemmRope &rp = g.rope;
          const int head = t >> 3, pos = pos0 + row;
          uint32_t w[2][2];
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const int q = 2 * half + i;
            const f32x4 v = f32x4{a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]} * sc_row;
            if (head < rp.H + rp.Hkv) {
              const f32x2 c = rope_c[p2 * 4 + q], sn = rope_s[p2 * 4 + q];
              w[i][0] = bf16_pair(v[0] * c[0] - v[1] * sn[0], v[1] * c[0] + v[0] * sn[0]);
              w[i][1] = bf16_pair(v[2] * c[1] - v[3] * sn[1], v[3] * c[1] + v[2] * sn[1]);
            } else {
              w[i][0] = bf16_pair(v[0], v[1]);
              w[i][1] = bf16_pair(v[2], v[3]);
            }
          }
          const uint4 e = eight_features(w[0][0], w[0][1], w[1][0], w[1][1]);
          const int dd = (t & 7) * 16 + 8 * hb;
          if (row >= g.n) continue;
          if (head < rp.H + rp.Hkv) {
            bf16_t *dst;
            if (head < rp.H) dst = rp.q + ((size_t)row * rp.H + head) * 128 + dd;
            else dst = rp.k_layer + (size_t)(head - rp.H) * rp.cap * 128 + kv_k_index(pos, dd);
            *reinterpret_cast<uint4 *>(dst) = e;
          } else {
            bf16_t *dst = rp.v_layer + (size_t)(head - rp.H - rp.Hkv) * 128 * rp.cap + kv_v_index(pos, dd);
            const uint32_t ew[4] = {e.x, e.y, e.z, e.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) { // features of an out-tile sit in neighbouring lane slots
              dst[16 * i] = (bf16_t)ew[i];
              dst[16 * i + 8] = (bf16_t)(ew[i] >> 16);
            }
          }
        } else {
          // h[row, ..] = bf16(silu(gate) * up) in fragment order over all row tiles; rows past n are zeros
          uint32_t w[4];
#pragma unroll
          for (int i = 0; i < 4; ++i)
            w[i] = bf16_pair(silu(a[2 * i] * sc_row) * (a[8 + 2 * i] * sc_row), silu(a[2 * i + 1] * sc_row) * (a[9 + 2 * i] * sc_row));
          const uint4 e = eight_features(w[0], w[1], w[2], w[3]);
          const bool live = row < g.n;
          const u32x4 hv = live ? u32x4{e.x, e.y, e.z, e.w} : u32x4{0u, 0u, 0u, 0u};
          const size_t fslot = ((size_t)(t >> 1) * row_tiles + rt) * 64 + r + 16 * (2 * (t & 1) + hb);
          __builtin_nontemporal_store(hv, reinterpret_cast<u32x4 *>(g.h_frag) + fslot);
        }
      }
    }
  }
}

bool gemm_wide_supported(int32_t n, int32_t K, int32_t O) {
  return n >= 1 && n <= WIDE_MAX_ROWS && K % 32 == 0 && K >= 64 && O % 32 == 0;
}

template <int MODE, bool SCALED, int RP2, int NP2, int WR, int WC, int D, int CHAIN, int KG = 1>
static hipError_t launch_ks(const GemmArgs &g, int row_tiles, unsigned grid, hipStream_t st, KernelTimer tm) {
  constexpr auto kernel = &k_gemm_wide<MODE, SCALED, RP2, NP2, WR, WC, D, CHAIN, KG>;
  constexpr int smem = D * KG * (2 * RP2 * WR + 2 * NP2 * WC) * 1024;
  static bool once = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                         smem) == hipSuccess;
  if (!once) return hipErrorInvalidValue;
  return launch(kernel, dim3(grid), dim3(WIDE_WAVES * 64), smem, st, tm, g.a_frag, g.seg[0].w,
                MODE == GEMM_SWIGLU ? g.w2 : g.seg[1].w, g.K / 32, row_tiles, g.groups, g.splits, g.part_q, g.part_rem, g);
}
template <int RP2, int NP2, int WR, int WC, int D>
static hipError_t launch_shape(GemmArgs &g, int row_tiles, unsigned grid, hipStream_t st, KernelTimer tm) {
  if (g.mode == GEMM_SWIGLU) return launch_ks<GEMM_SWIGLU, true, RP2, NP2, WR, WC, D, 0>(g, row_tiles, grid, st, tm);
  if (g.resid.x != nullptr) {
    g.resid.ld_ssq = (g.groups * WC + 3) & ~3;
    return launch_ks<GEMM_RESID, false, RP2, NP2, WR, WC, D, 0>(g, row_tiles, grid, st, tm);
  }
  if (g.rope.q != nullptr) return launch_ks<GEMM_ROPE, true, RP2, NP2, WR, WC, D, 0>(g, row_tiles, grid, st, tm);
  return launch_ks<GEMM_STORE, false, RP2, NP2, WR, WC, D, 0>(g, row_tiles, grid, st, tm);
}

// The workgroup shapes: row tiles x out-tiles, and the measured us of one k-step when every compute unit has a
// workgroup (see the header).  The smallest leaves room for two workgroups on a compute unit.
struct WideShape {
  int rb, nw;
  double step_us;
};
static constexpr WideShape WIDE_SHAPES[5] = {{8, 8, 0.27}, {8, 12, 0.42}, {16, 8, 0.45}, {16, 12, 0.585}, {16, 16, 0.70}};

struct WidePlan {
  int shape, splits;
};
static int wide_groups(int total, int nw, int unit) { return (total + nw / unit - 1) / (nw / unit); }

// The workgroup shape and the K-splits of n rows; total out-tiles, of which `unit` tiles of the weights each.
static WidePlan wide_choose(int n, int K, int total, int unit, int max_splits) {
  const int row_tiles = (n + 15) / 16;
  // Cost in us: rounds of 256 workgroups, each its k-steps plus 8 for ramp and epilogue, plus what a partial sum costs
  // to write (4.6 TB/s) and to read back in the residual kernel (2.9 TB/s).
  const int KT = K / 32;
  WidePlan plan{0, 1};
  double best = 1e30;
  for (int v = 0; v < 5; ++v) {
    const int row_blocks = (row_tiles + WIDE_SHAPES[v].rb - 1) / WIDE_SHAPES[v].rb;
    // A single row block with fewer tiles than the shape has loads a neighbour in their place, which costs next to nothing:
    // 161 rows, 8192 -> 8192, 8 x 8 tiles in two shares 60.8 us, 16 x 8 in four 49.8; 145 rows, 13824 -> 5120, 65.5 / 59.6.
    const int row_here = row_tiles < WIDE_SHAPES[v].rb ? row_tiles : WIDE_SHAPES[v].rb;
    const double step_us = WIDE_SHAPES[v].step_us * (row_here + WIDE_SHAPES[v].nw) / (WIDE_SHAPES[v].rb + WIDE_SHAPES[v].nw);
    for (int sp = 1; sp <= max_splits; ++sp) {
      const int per_k = (KT + sp - 1) / sp;
      if (sp > 1 && (per_k < 16 || (sp - 1) * per_k >= KT)) continue; // no empty share, none that is all ramp
      const int rounds = (wide_groups(total, WIDE_SHAPES[v].nw, unit) * row_blocks * sp + 255) / 256;
      double cost = rounds * (per_k * step_us + 8.0);
      if (sp > 1) cost += sp * (64.0 * n * total) * (1 / 4.6e6 + 1 / 2.9e6);
      if (cost < best) {
        best = cost;
        plan = WidePlan{v, sp};
      }
    }
  }
  return plan;
}
WideProjection wide_plan(int32_t n, int32_t K, int32_t out_tiles) {
  const WidePlan p = wide_choose(n, K, out_tiles, 1, wide_max_splits(n));
  const WideShape &s = WIDE_SHAPES[p.shape];
  return WideProjection{s.rb, s.nw, wide_groups(out_tiles, s.nw, 1), p.splits};
}

// Fills the plan and the tile assignment and launches.  g.n is the total row count
// (<= WIDE_MAX_ROWS); a_frag / h_frag use ceil(n / 16) row tiles; SwiGLU and Q/K/V come with the RMS scale of partial
// sums per row (at most 8, or a multiple of 4 on 16 bytes), a plain store without.  max_splits > 1 (plain store only): y[s] = y + s *
// split_stride receives the partial sum of k-range s, and *out_splits how many the launch used.  With GemmResid it is the sums of
// squares per row that *out_splits receives.
hipError_t launch_gemm_wide(const GemmArgs &args, int32_t max_splits, int32_t *out_splits, hipStream_t st, KernelTimer tm) {
  GemmArgs g = args;
  if (g.n < 1 || g.n > WIDE_MAX_ROWS || g.K % 32 != 0 || g.K < 64) return hipErrorInvalidValue;
  if (g.row_ssq != nullptr && g.n_ssq > 8 && (g.n_ssq % 4 != 0 || !starts_on_16(g.row_ssq))) return hipErrorInvalidValue;
  if (g.n_seg != (g.rope.q != nullptr ? 3 : 1)) return hipErrorInvalidValue; // only Q/K/V walks several matrices
  int32_t total = 0;
  for (int i = 0; i < g.n_seg; ++i) total += g.seg[i].out_tiles;
  if (total < 1 || (g.mode != GEMM_STORE && g.mode != GEMM_SWIGLU)) return hipErrorInvalidValue;
  if ((g.mode == GEMM_SWIGLU || g.rope.q != nullptr) != (g.row_ssq != nullptr)) return hipErrorInvalidValue;
  if (g.rope.q != nullptr && (!g.rope.tiled || g.rope.hd != 128 || g.mode != GEMM_STORE)) return hipErrorInvalidValue;
  const bool may_split = g.row_ssq == nullptr && g.resid.x == nullptr && max_splits > 1;
  const int row_tiles = (g.n + 15) / 16;
  const int unit = g.mode == GEMM_SWIGLU ? 2 : 1; // a gate/up pair occupies two of the NW tiles
  const WidePlan plan = wide_choose(g.n, g.K, total, unit, may_split ? max_splits : 1);
  const int shape = plan.shape;
  const int nw = WIDE_SHAPES[shape].nw, row_blocks = (row_tiles + WIDE_SHAPES[shape].rb - 1) / WIDE_SHAPES[shape].rb;
  g.total_tiles = total;
  g.tiles_per_wg = nw / unit;
  g.groups = wide_groups(total, nw, unit);
  g.part_q = total / g.groups;
  g.part_rem = total % g.groups;
  g.splits = plan.splits;
  if (out_splits != nullptr) *out_splits = g.splits;
  const unsigned grid = (unsigned)(((g.groups + 7) / 8) * 8 * row_blocks * g.splits);
  hipError_t e;
  switch (shape) {
  case 0: e = launch_shape<1, 2, 4, 2, 5>(g, row_tiles, grid, st, tm); break;
  case 1: e = launch_shape<1, 3, 4, 2, 7>(g, row_tiles, grid, st, tm); break;
  case 2: e = launch_shape<2, 2, 4, 2, 6>(g, row_tiles, grid, st, tm); break;
  case 3: e = launch_shape<2, 3, 4, 2, 5>(g, row_tiles, grid, st, tm); break;
  default: e = launch_shape<2, 4, 4, 2, 5>(g, row_tiles, grid, st, tm); break;
  }
  if (out_splits != nullptr && g.resid.x != nullptr) *out_splits = g.resid.ld_ssq;
  return e;
}

// Tree steps (n <= 128) of matrices with many out-tiles: one block of eight row tiles x 8 or 16 out-tiles per workgroup.
// Every workgroup loads the activations of its k range, so what the compute units pull is (out-tiles + row tiles) per out-tile;
// the decode kernel, whose waves each hold all accumulators of the workgroup, ends at 6 or 8 out-tiles (6 from 81 rows on),
// this one shares them out over its waves.  It needs the chip full of workgroups, since each pulls no faster for being
// alone: 200 workgroups per round of 256 at least.  All figures are of one launch behind 128 MiB of other traffic, new activations and
// weights that no cache holds, as in a step (launched back to back this kernel looks 3 to 8 % better: the 7B LM head, 80 rows, is
// 49.7 / 47.2 so, 49.5 / 51.8 here and 50.0 / 52.0 in a step).  us, decode kernel / this, 48 / 80 / 96 / 128 rows:
//   70B gate/up, 224 x 16 out-tiles   159 / 148   161 / 143   198 / 148   227 / 151
//   70B LM head, 501 x 16             384 / 346   390 / 340   462 / 333   506 / 342
//   70B down, 64 x 8 in four shares    77 /  79    82 /  84    99 /  86   118 /  95
//   13B gate/up, 216 x 8               52 /  48    54 /  51    68 /  55    78 /  58
//   13B LM head, 250 x 8               58 /  54    58 /  57    76 /  60    89 /  64
//   7B LM head, 250 x 8                49 /  53    50 /  52    63 /  50    73 /  53
// Which rows, from this kernel's time over the decode kernel's at K = 4096, 5120, 6656 and 8192, plain and gate/up:
//   16 out-tiles, one round   1-16 rows 0.83-1.18; 17-32 rows: 200 to 230 groups, K >= 5120 0.82-0.95, the others 0.69-1.07;
//                             33-48 0.70-1.00; 49-64 0.76-1.01; 80 0.73-0.98; 96 and more 0.57-0.84
//     two rounds and more     17-32 0.93-1.10; 33-48: K >= 5120 0.86-1.00, K = 4096 0.93-1.04; 49-64 0.87-1.02; 80 0.83-0.97;
//                             96 and more 0.68-0.87
//   8 out-tiles, whole k      1-32 0.87-1.22; 33-48: K >= 5120 0.84-0.98, K = 4096 0.84-1.14; 49-64 0.95-1.11 (the decode kernel's own
//                             form of eight out-tiles is for four and five row tiles); 80: 200 to 230 groups 0.92-0.99, more
//                             0.93-1.05; 96 and more 0.70-0.94
//   6, gate/up alone          80 1.02-1.08; 96 1.00-1.03; 112 0.93-0.99; 128 0.94-0.99
// 6 out-tiles are for the matrices that have no 200 workgroups of 8 (7B gate/up, 172), by two groups of waves on even and odd k-tiles (a
// wave's 2 x 2 tiles of 8 x 6 leave four waves idle): 112, 128 rows 42.6 / 40.6, 44.6 / 42.7 us.
// Shares of k (o and down, in four, 50 to 64 groups) from 128 k-steps on: 17-48 rows 0.92-1.11, 49-64 0.96-1.10, 80 0.98-1.02; 96 0.86-0.91;
// 112 and more 0.79-0.87.  A wave of the decode kernel has an eighth of a share in one chain, so with shorter ones its sums are the better
// (relative error against float64, decode kernel / this, 80 rows: 4096 -> 6656 0.99e-7 / 1.28e-7, 6656 -> 6656 1.20e-7 / 1.30e-7, 16384 -> 6656
// 1.85e-7 / 1.37e-7), and with 64 groups this kernel is slower there (6656 -> 8192 at 96 rows 25.7 / 28.5 us).
// Matrices with K below 4096 were not measured and stay.
bool rows8_plan(int32_t n, int32_t K, int32_t total_tiles, bool swiglu, int32_t max_splits, Rows8Plan *plan) {
  if (n < 1 || n > NP || K < 4096 || K % 32 != 0) return false;
  const int unit = swiglu ? 2 : 1, NT = (n + 15) / 16, KT = K / 32;
  auto fills = [](int wgs) { return wgs >= (wgs + 255) / 256 * 200; };
  const int g16 = (total_tiles + 16 / unit - 1) / (16 / unit), g8 = (total_tiles + 8 / unit - 1) / (8 / unit);
  if (max_splits == 1 && fills(g16) && (NT >= 4 || (NT == 3 && (g16 <= 256 || K >= 5120)) || (NT == 2 && g16 <= 230 && K >= 5120))) {
    *plan = Rows8Plan{16, g16, 1};
    return true;
  }
  for (int sp = max_splits; sp >= 1; --sp) {
    const int per_k = (KT + sp - 1) / sp;
    if ((sp - 1) * per_k >= KT || !fills(g8 * sp)) continue;
    const bool faster = sp > 1 ? per_k >= 128 && NT >= 6
                               : NT >= 6 || (NT == 5 && g8 <= 230) || (NT == 3 && g8 <= 256 && K >= 5120);
    if (!faster) continue;
    *plan = Rows8Plan{8, g8, sp};
    return true;
  }
  const int g6 = (total_tiles + 2) / 3;
  if (swiglu && NT >= 7 && KT % 2 == 0 && fills(g6)) {
    *plan = Rows8Plan{6, g6, 1};
    return true;
  }
  return false;
}

// Q/K/V: 8 out-tiles and as many shares of k as fill one round.  Whole, every workgroup of the decode kernel has 3 or 4 out-tiles and all
// of the activations to load; in shares they load a half or a third of that, and the launch that adds the shares (6.4 us at 80 rows of
// 70B width) is less than they save from where the activations are many.  us of the launches at 70B width, 80 rows: 48.5 / 35.5 + 6.4.  A
// step on the same buffers, whole / in shares:
//   three shares   K = 8192 (3 layers) 33 rows 1288 / 1276, 48 1320 / 1311, 64 1350 / 1342, 80 1384 / 1363, 128 1480 / 1443;
//                  7168 (5) 81 rows 1462 / 1426, 96 1482 / 1450, 128 1655 / 1614
//   four           8192 (3) 33 rows 848 / 836, 64 906 / 897, 96 1031 / 1006; 5120 (8) 81 rows 1356 / 1326, 128 1545 / 1526; 6144 (6) 96 rows 1285 / 1276
//   two            5120 (20) 81 rows 3294 / 3337, 96 3388 / 3418, 97 3801 / 3766, (8) 128 rows 1685 / 1653; 7168 (4) 81 rows 1323 / 1301; 8192 (3)
//                  33 rows 1060 / 1074, 64 1109 / 1123, 80 1164 / 1164, 81 1212 / 1195
// Three and four shares of K < 8192 and fewer rows were not measured and stay whole.  At 7B width two shares of 96 groups do not
// fill the chip.  Chains of 16 k-steps, where a wave of the decode kernel has 20 at K = 5120 and 32 at 8192.
bool qkv_split_plan(int32_t n, int32_t K, int32_t total_tiles, Rows8Plan *plan) {
  const int NT = (n + 15) / 16, g8 = (total_tiles + 7) / 8;
  if (n > NP || K < 5120 || K % 32 != 0) return false;
  for (int sp = 2; sp <= GEMM_MAX_SPLITS; ++sp)
    if (g8 * sp >= 200 && g8 * sp <= 256) {
      if (NT < (sp == 2 ? (K < 7168 ? 7 : 6) : (K < 8192 ? 6 : 3))) return false;
      *plan = Rows8Plan{8, g8, sp};
      return true;
    }
  return false;
}

hipError_t launch_gemm_rows8(const GemmArgs &args, const Rows8Plan &plan, hipStream_t st, KernelTimer tm) {
  GemmArgs g = args;
  g.total_tiles = 0;
  for (int i = 0; i < g.n_seg; ++i) g.total_tiles += g.seg[i].out_tiles;
  g.tiles_per_wg = plan.out_tiles / (g.mode == GEMM_SWIGLU ? 2 : 1);
  g.groups = plan.groups;
  g.part_q = g.total_tiles / g.groups;
  g.part_rem = g.total_tiles % g.groups;
  g.splits = plan.splits;
  const int row_tiles = (g.n + 15) / 16;
  const unsigned grid = (unsigned)(((g.groups + 7) / 8) * 8 * g.splits);
  const bool swiglu = g.mode == GEMM_SWIGLU, scaled = g.row_ssq != nullptr;
  if (g.n < 1 || g.n > NP || (scaled ? g.n_ssq > 8 || g.splits != 1 : swiglu)) return hipErrorInvalidValue;
  if (g.n_seg != 1 && g.n_seg != 3) return hipErrorInvalidValue;
  // Chains of 16 k-steps: as long as a wave's in the decode kernel at K = 4096 in eight waves, or in shares of 128, and shorter than
  // all others there.  Its MFMA adds 32 products, these 16 twice, and the errors are the same: relative to float64 1.31e-7 with both for
  // 4096 -> 32064, 96 and 128 rows; where the decode kernel has four waves (80 rows) 1.81e-7 / 1.32e-7.
  if (g.n_seg == 3) { // partial sums of Q/K/V
    if (swiglu || scaled || plan.out_tiles != 8) return hipErrorInvalidValue;
    return launch_ks<GEMM_PARTS, false, 1, 2, 4, 2, 5, 16>(g, row_tiles, grid, st, tm);
  }
  if (plan.out_tiles == 6 && swiglu) return launch_ks<GEMM_SWIGLU, true, 1, 3, 4, 1, 5, 16, 2>(g, row_tiles, grid, st, tm);
  if (plan.out_tiles == 8 && swiglu) return launch_ks<GEMM_SWIGLU, true, 1, 2, 4, 2, 5, 16>(g, row_tiles, grid, st, tm);
  if (plan.out_tiles == 8 && scaled) return launch_ks<GEMM_STORE, true, 1, 2, 4, 2, 5, 16>(g, row_tiles, grid, st, tm);
  if (plan.out_tiles == 8) return launch_ks<GEMM_STORE, false, 1, 2, 4, 2, 5, 16>(g, row_tiles, grid, st, tm);
  if (plan.out_tiles == 16 && swiglu) return launch_ks<GEMM_SWIGLU, true, 2, 2, 2, 4, 6, 16>(g, row_tiles, grid, st, tm);
  if (plan.out_tiles == 16 && scaled) return launch_ks<GEMM_STORE, true, 2, 2, 2, 4, 6, 16>(g, row_tiles, grid, st, tm);
  return hipErrorInvalidValue;
}

} // namespace tr
