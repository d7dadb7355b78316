// Tree attention on the matrix cores (Section 2.2 "Tree Attention"): head_dim 128, bf16 Q/K/V, float32
// softmax statistics and accumulators.  HBM-bound: every K/V byte of the head is read once per call.
//
// A workgroup owns HPW query heads that share one K/V head (HPW = 2 under grouped-query attention with an
// even group, else 1) and every nsplit-th 32-key tile; its waves own one (head, tile of 16 tree nodes)
// each, so no cross-wave reduction is needed.  K and V tiles are staged through LDS (double buffered,
// one barrier per tile) and shared by the waves, so two heads of a group read their K/V once instead of
// twice.  The grid is (K/V head, head group, split): workgroups that read the same K/V head have linear
// ids congruent modulo the number of K/V heads and, with 8 of those and round-robin dispatch, land on one
// XCD, whose L2 then serves the remaining re-reads.
//
// Everything is computed transposed so that no value ever changes lanes between the two contractions:
//   S^T[key][node] = K[key][:] . Q[node][:]      A = K tile (16 keys x 32 d), B = Q^T; lane l receives
//                                                keys 4*(l/16) .. +3 of node l%16
//   O^T[d][node]  += V^T[d][key] * P^T[key][node] A = V^T tile (16 d x 32 keys), B = P^T built in place from
//                                                the lane's own 8 probabilities (two 16-key S^T tiles)
// The KV cache is kept in exactly these operand orders (TR_KV_TILED, see kv_k_index / kv_v_index), so a
// tile is one contiguous 8 KiB block in memory and an LDS read of 16 bytes per lane is an MFMA operand.
//
// Mask: key position p is visible to node i when p < L (committed prefix), or L <= p < L + N and bit
// p - L of the node's ancestor mask is set.  Invisible keys get probability exactly 0.
// With more than one split, split s owns tiles s, s + nsplit, ...; each writes (max, sum, normalised O in
// half precision) per node and k_attn_merge combines them in split order.  K/V are read with streaming
// loads: they are used once per call and would otherwise push the activations out of L2 (the direct loads of
// k_attn_ring do without: steps of the 13B and 70B shapes were the same with the hint, within 1 % of noise).
#include <type_traits>

#include "tr_kernels.h"

namespace tr {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) _Float16 f16x4;

__device__ inline f32x4 mfma16a(const u32x4 &a, const u32x4 &b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

constexpr int ATT_TILE_BYTES = 16384; // 32 keys: K 8 KiB + V 8 KiB
constexpr float NEG_BIG = -1e30f;

// End of a wave of the split forms, (head, tile of 16 nodes) over one key share: the result itself if there is only one share.
// `lds` has 4 KiB per wave for it once every wave is done with the K/V tiles.
__device__ inline void finish_share(const f32x4 (&acc)[8], float m, float lsum, void *lds_all, int wave, int lane, int wt, int h,
                                    int split, int nsplit, int32_t H, int32_t n, float *__restrict__ part_ml,
                                    float *__restrict__ part_acc, bf16_t *__restrict__ out, int32_t out_row_tiles) {
  const int r = lane & 15, g = lane >> 4, node = wt * 16 + r;
  if (nsplit == 1) {
    if (node >= n) return;
    const float inv = 1.0f / lsum;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) {
      const int d = 16 * dt + 4 * g;
      ushort4 o;
      o.x = f32_to_bf16(acc[dt][0] * inv); o.y = f32_to_bf16(acc[dt][1] * inv);
      o.z = f32_to_bf16(acc[dt][2] * inv); o.w = f32_to_bf16(acc[dt][3] * inv);
      const size_t idx = out_row_tiles > 0 ? act_frag_index(node, h * 128 + d, out_row_tiles)
                                           : ((size_t)node * H + h) * 128 + d;
      store_stream(out + idx, o);
    }
    return;
  }
  // a split's partial result is its own normalised output (a convex combination of V rows, so it fits
  // half precision with 2^-11 relative error, below the bf16 rounding of the merged output) plus (m, l).
  // The wave's 16 x 128 block is turned through LDS so that a node's 256 bytes leave as whole lines.
  const size_t prow = ((size_t)split * H + h) * NP + wt * 16;
  if (g == 0 && node < n) {
    part_ml[(prow + r) * 2] = m;
    part_ml[(prow + r) * 2 + 1] = lsum;
  }
  const float inv = lsum > 0.f ? 1.0f / lsum : 0.f;
  __syncthreads(); // every wave is done with the last K/V tile
  // row r keeps its 16-byte chunk c at slot c ^ r, so the 16 rows of one store hit distinct banks
  char *blk = reinterpret_cast<char *>(lds_all) + wave * 4096;
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) {
    // clamped to the half-precision range: a value-cache entry beyond +-65504 saturates instead of
    // turning into an infinity that the merge would spread over the row
    f32x4 o = acc[dt] * inv;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = fminf(fmaxf(o[e], -65504.0f), 65504.0f);
    *reinterpret_cast<f16x4 *>(blk + r * 256 + (((2 * dt + (g >> 1)) ^ r) << 4) + 8 * (g & 1)) =
        __builtin_convertvector(o, f16x4);
  }
  // the wave reads back only what it wrote itself; its LDS operations complete in order
  asm volatile("" ::: "memory");
  u32x4 *pa = reinterpret_cast<u32x4 *>(part_acc);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int c = i * 64 + lane, rr = c >> 4, cc = c & 15;
    const u32x4 v = *reinterpret_cast<const u32x4 *>(blk + rr * 256 + ((cc ^ rr) << 4));
    if (wt * 16 + rr < n) pa[(prow + rr) * 16 + cc] = v; // plain store: the merge pass finds these in L2
  }
}

template <int NT, int HPW>
__global__ __launch_bounds__(NT * HPW * 64) void k_attn_mfma(const bf16_t *__restrict__ q, const bf16_t *__restrict__ Kl,
                                                       const bf16_t *__restrict__ Vl, int32_t H, int32_t Hkv,
                                                       int32_t cap, int32_t n, const uint64_t *__restrict__ anc,
                                                       const int32_t *__restrict__ d_len, int32_t nsplit,
                                                       float *__restrict__ part_ml, float *__restrict__ part_acc,
                                                       bf16_t *__restrict__ out, int32_t out_row_tiles) {
  constexpr int THREADS = NT * HPW * 64;
  constexpr int SLOTS = ATT_TILE_BYTES / 16;                 // 16-byte slots per tile
  constexpr int PER_THREAD = (SLOTS + THREADS - 1) / THREADS;
  // two tile buffers; reused at the end for one 4 KiB block per wave
  constexpr int LDS_SLOTS = 2 * SLOTS > NT * HPW * 256 ? 2 * SLOTS : NT * HPW * 256;
  __shared__ u32x4 lds_all[LDS_SLOTS];
  u32x4 (*lds)[SLOTS] = reinterpret_cast<u32x4 (*)[SLOTS]>(lds_all);

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int r = lane & 15, g = lane >> 4;
  const int wt = wave % NT;                                  // node tile of this wave
  // grid (K/V head, head group inside it, split): linear ids of one K/V head differ by multiples of Hkv
  const int hk = blockIdx.x, split = blockIdx.z;
  const int h = hk * (H / Hkv) + blockIdx.y * HPW + wave / NT;
  // split s owns tiles s, s + nsplit, s + 2 nsplit, ...: its first tile does not depend on the committed
  // length, so that fetch is issued before the length has arrived, and the masked tiles at the end of
  // the sequence spread over the splits

  const int node = wt * 16 + r;
  const int node_c = node < n ? node : n - 1;
  // Q^T operand: lane (node r, group g) holds Q[node][32c + 8g .. +7] for d-step c
  u32x4 qf[4];
  {
    const u32x4 *qp = reinterpret_cast<const u32x4 *>(q + ((size_t)node_c * H + h) * 128 + 8 * g);
#pragma unroll
    for (int c = 0; c < 4; ++c) qf[c] = qp[c * 4];
  }
  const uint64_t a0 = anc[2 * node_c], a1 = anc[2 * node_c + 1];

  const u32x4 *Kh = reinterpret_cast<const u32x4 *>(Kl + (size_t)hk * cap * 128);
  const u32x4 *Vh = reinterpret_cast<const u32x4 *>(Vl + (size_t)hk * cap * 128);

  f32x4 acc[8];
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) acc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  // running sum l of the (bf16-rounded) probabilities, kept as the product of an all-ones A tile with
  // P^T: every row of that product is the column sum, so each lane ends with l of its own node
  f32x4 accl = f32x4{0.f, 0.f, 0.f, 0.f};
  const u32x4 ones = u32x4{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
  float m = NEG_BIG;
  const float sc = 0.08838834764831845f * 1.4426950408889634f; // 1/sqrt(128) * log2(e)

  // K/V tiles travel global -> registers -> LDS with one tile of loads in flight.  More were measured and
  // are no faster: the per-tile chain of dependent steps (stage, barrier, score contraction, softmax, value
  // contraction) is the limit, 0.7 to 0.9 us of it.  Longer shares go through k_attn_ring for that.
  u32x4 stage[PER_THREAD];
  auto fetch = [&](int tile) {
    // K tile: 512 slots at Kh + tile*512; V tile: 512 slots at Vh + tile*512
#pragma unroll
    for (int i = 0; i < PER_THREAD; ++i) {
      const int s = tid + i * THREADS;
      if (s < SLOTS)
        stage[i] = __builtin_nontemporal_load(s < 512 ? Kh + (size_t)tile * 512 + s : Vh + (size_t)tile * 512 + (s - 512));
    }
  };
  auto publish = [&](int buf) {
#pragma unroll
    for (int i = 0; i < PER_THREAD; ++i) {
      const int s = tid + i * THREADS;
      if (s < SLOTS) lds[buf][s] = stage[i];
    }
  };

  // The loop is bound by the vector ALU work per score, not by the K/V stream, so that work is kept
  // minimal: tiles that lie wholly in the committed prefix skip the mask, the scale is folded into the
  // exponent with one fma, the accumulators are rescaled only when some lane's maximum moved, and the
  // bf16 rounding of the probabilities is the hardware's packed conversion.
  if ((split + 1) * 32 <= cap) fetch(split); // inside the cache allocation even if beyond the sequence
  const int L = *d_len;
  const int total = L + n;
  const int n_tiles = (total + 31) >> 5;
  int buf = 0;
  for (int t = split; t < n_tiles; t += nsplit, buf ^= 1) {
    publish(buf);
    __syncthreads();
    if (t + nsplit < n_tiles) fetch(t + nsplit);
    const u32x4 *kt = lds[buf];
    const u32x4 *vt = lds[buf] + 512;

    f32x4 s0 = f32x4{0.f, 0.f, 0.f, 0.f}, s1 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      s0 = mfma16a(kt[c * 64 + lane], qf[c], s0);
      s1 = mfma16a(kt[(4 + c) * 64 + lane], qf[c], s1);
    }
    const bool in_prefix = t * 32 + 32 <= L; // uniform: every key of the tile is visible to every node
    float pr[8];
    if (in_prefix) {
      float mx = fmaxf(fmaxf(fmaxf(s0[0], s0[1]), fmaxf(s0[2], s0[3])), fmaxf(fmaxf(s1[0], s1[1]), fmaxf(s1[2], s1[3])));
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float m_new = fmaxf(m, mx * sc);
      if (__any(m_new > m)) {
        const float corr = __builtin_amdgcn_exp2f(m - m_new);
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) {
          acc[dt][0] *= corr; acc[dt][1] *= corr; acc[dt][2] *= corr; acc[dt][3] *= corr;
        }
        accl[0] *= corr; accl[1] *= corr; accl[2] *= corr; accl[3] *= corr;
        m = m_new;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        pr[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s0[e], sc, -m));
        pr[4 + e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s1[e], sc, -m));
      }
    } else {
      float x[8];
      bool vis[8];
      const int pbase = t * 32 + 4 * g;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int p = pbase + (e >> 2) * 16 + (e & 3);
        bool v = p < L;
        if (!v && p < total) {
          const int j = p - L;
          v = j < 64 ? ((a0 >> j) & 1ull) : ((a1 >> (j - 64)) & 1ull);
        }
        vis[e] = v;
        const float sv = (e < 4 ? s0[e & 3] : s1[e & 3]) * sc;
        x[e] = v ? sv : NEG_BIG;
      }
      float mx = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float m_new = fmaxf(m, mx);
      if (__any(m_new > m)) {
        const float corr = __builtin_amdgcn_exp2f(m - m_new);
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) {
          acc[dt][0] *= corr; acc[dt][1] *= corr; acc[dt][2] *= corr; acc[dt][3] *= corr;
        }
        accl[0] *= corr; accl[1] *= corr; accl[2] *= corr; accl[3] *= corr;
        m = m_new;
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) pr[e] = vis[e] ? __builtin_amdgcn_exp2f(x[e] - m) : 0.f;
    }
    // P^T operand: the lane's own 8 probabilities, rounded to bf16 (round to nearest even)
    u32x4 pf;
#pragma unroll
    for (int e = 0; e < 8; e += 2)
      pf[e >> 1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{pr[e], pr[e + 1]}, bf16x2));
    accl = mfma16a(ones, pf, accl);
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) acc[dt] = mfma16a(vt[dt * 64 + lane], pf, acc[dt]);
  }
  finish_share(acc, m, accl[0], lds_all, wave, lane, wt, h, split, nsplit, H, n, part_ml, part_acc, out, out_row_tiles);
}

// ---------------------------------------------------------------------------------------------
// The split form for longer shares.  Same mapping, shares and arithmetic per score as k_attn_mfma, but tiles go memory -> LDS by
// direct loads, 64 keys (32 KiB) a step in a ring of two, the first of them asked for before the committed length is known;
// the waves meet once per 64 keys, and the operands of a contraction are read from LDS together.  The running maximum moves
// after every 32 keys as there, and the errors are the same (moved once per 64 keys they are 0.2 to 1 % larger, the time 1 to 5 %
// shorter).
// Queries and ancestor masks come the same way, in front of the tiles, through what is the second step's place: a plain load
// behind them would wait for every tile.
// What bounds it: the stream of K and V on long sequences (32 heads, 80 nodes, 16000 positions: 264 MB in 58 us, 4.5 TB/s); below
// about 2000 positions launch, a trip to memory (1.8 us), 1 to 1.5 us per 64 keys and write-back.  us without the merge, k_attn_mfma /
// this, 80 nodes: 32 heads on 32 19.8 / 18.9 at 4013 positions, 34.2 / 31.8 at 8192, 60.8 / 58.0 at 16000; 40 on 40 16.6 / 16.2 at 2221,
// 25.1 / 24.0 at 4096; 64 on 8 25.3 / 24.3 at 4096, 73.2 / 67.6 at 16000; 48 nodes, 32 on 32 21.1 / 18.4 at 4045.
// A ring of four steps, all asked for at once, takes 1.2 us more: the burst holds up its own first tiles.
// ---------------------------------------------------------------------------------------------
constexpr int RING_STEPS = 2;
constexpr int RING_STEP_BYTES = 2 * ATT_TILE_BYTES; // 64 keys
constexpr int RING_WAVE_BYTES = 5 * 1024;           // a wave's queries (16 x 128) and ancestor masks at the start
constexpr int ring_lds_bytes(int waves) {
  const int steps = RING_STEPS * RING_STEP_BYTES, start = (RING_STEPS - 1) * RING_STEP_BYTES + waves * RING_WAVE_BYTES;
  return steps > start ? steps : start;
}

template <int NT, int HPW>
__global__ __launch_bounds__(NT * HPW * 64) void k_attn_ring(const bf16_t *__restrict__ q, const bf16_t *__restrict__ Kl,
                                                            const bf16_t *__restrict__ Vl, int32_t H, int32_t Hkv,
                                                            int32_t cap, int32_t n, const uint64_t *__restrict__ anc,
                                                            const int32_t *__restrict__ d_len, int32_t bound_tiles,
                                                            int32_t nsplit, float *__restrict__ part_ml,
                                                            float *__restrict__ part_acc, bf16_t *__restrict__ out,
                                                            int32_t out_row_tiles) {
  constexpr int W = NT * HPW, D = RING_STEPS;
  constexpr int B = 32 / W, REM = 32 % W; // tile loads (1 KiB) of a wave per step; the first REM waves take one more
  extern __shared__ u32x4 ring[];         // [D][tile 0: K 8 | V 8, tile 1: K 8 | V 8][64]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, g = lane >> 4;
  const int wt = wave % NT;
  const int hk = blockIdx.x, split = blockIdx.z;
  const int h = hk * (H / Hkv) + blockIdx.y * HPW + wave / NT;
  const int node = wt * 16 + r, node_c = node < n ? node : n - 1;
  const uint32_t ring0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)ring;

  // queries and masks: Q^T operand of lane (node r, group g) is Q[node][32 c + 8 g .. + 7] for d-step c
  constexpr int OWN = (D - 1) * RING_STEP_BYTES;
  {
    const uint32_t own = ring0 + OWN + wave * RING_WAVE_BYTES;
    const uint32_t qoff = ((uint32_t)(node_c * H + h) * 128 + 8 * g) * 2;
#pragma unroll
    for (int c = 0; c < 4; ++c) tile_to_lds(own + c * 1024, qoff + c * 64, reinterpret_cast<uint64_t>(q));
    tile_to_lds(own + 4096, node_c * 16, reinterpret_cast<uint64_t>(anc));
  }
  const uint64_t kbase = reinterpret_cast<uint64_t>(Kl + (size_t)hk * cap * 128);
  const uint64_t vbase = reinterpret_cast<uint64_t>(Vl + (size_t)hk * cap * 128);
  const uint32_t voff = lane * 16;
  // step s of this share: tiles split + 2 s nsplit and nsplit further; a tile past `last` loads `last` again
  auto load_step = [&](int s, int last) {
    const uint32_t at = ring0 + (s % D) * RING_STEP_BYTES;
    const int t0 = split + 2 * s * nsplit, t1 = t0 + nsplit;
    const int c0 = t0 < last ? t0 : last, c1 = t1 < last ? t1 : last;
#pragma unroll 8 // one wave alone has 32: their addresses at once would spill
    for (int i = 0; i < B + (REM > 0 ? 1 : 0); ++i) {
      const int j = wave + W * i;
      if (i < B || wave < REM)
        tile_to_lds(at + j * 1024, voff, ((j & 8) ? vbase : kbase) + ((uint64_t)(j < 16 ? c0 : c1) * 8 + (j & 7)) * 1024);
    }
  };
  // at most `steps` (0 or 1) steps of this wave's loads still under way
  auto wait_steps = [&](int steps) {
    static_assert(D == 2, "one step ahead");
    if (steps <= 0) wait_tiles<0>();
    else if (REM > 0 && wave < REM) wait_tiles<B + 1>();
    else wait_tiles<B>();
  };
  auto steps_of = [&](int tiles) { return tiles > split ? (tiles - split + 2 * nsplit - 1) / (2 * nsplit) : 0; };

  // the host's bound of the sequence says what to ask for before the length is known
  const int cap_tiles = cap >> 5;
  const int early = bound_tiles < cap_tiles ? bound_tiles : cap_tiles;
  int issued = steps_of(early);
  issued = issued < D - 1 ? issued : D - 1;
  for (int s = 0; s < issued; ++s) load_step(s, early - 1);
  const int L = *d_len;

  wait_steps(issued); // the queries and masks are this wave's own
  u32x4 qf[4];
  uint64_t a0, a1;
  {
    const u32x4 *own = ring + (OWN + wave * RING_WAVE_BYTES) / 16;
#pragma unroll
    for (int c = 0; c < 4; ++c) qf[c] = own[c * 64 + lane];
    const u32x4 am = own[256 + lane];
    a0 = (uint64_t)am[0] | ((uint64_t)am[1] << 32);
    a1 = (uint64_t)am[2] | ((uint64_t)am[3] << 32);
  }
  const int total = L + n, n_tiles = (total + 31) >> 5;
  const int steps = steps_of(n_tiles);
  if (n_tiles > early) { // a sequence beyond the bound: what was clamped to it is asked for again
    wait_tiles<0>();
    issued = 0;
  }

  f32x4 acc[8];
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) acc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 accl = f32x4{0.f, 0.f, 0.f, 0.f}; // row sums of the rounded probabilities, as in k_attn_mfma
  const u32x4 ones = u32x4{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
  float m = NEG_BIG;
  const float sc = 0.08838834764831845f * 1.4426950408889634f; // 1/sqrt(128) * log2(e)

  auto multiply = [&](auto tiles_c, const u32x4 *kv, int t0) {
    constexpr int TILES = decltype(tiles_c)::value;
    // all of a contraction's LDS reads first: left alone, the compiler puts each in front of its product and waits for it
    u32x4 op[TILES][8];
#pragma unroll
    for (int k = 0; k < TILES; ++k)
#pragma unroll
      for (int c = 0; c < 8; ++c) op[k][c] = kv[k * 1024 + c * 64 + lane];
    __builtin_amdgcn_sched_barrier(0);
    f32x4 sv[2 * TILES];
#pragma unroll
    for (int i = 0; i < 2 * TILES; ++i) sv[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int i = 0; i < 2 * TILES; ++i) sv[i] = mfma16a(op[i >> 1][(i & 1) * 4 + c], qf[c], sv[i]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < TILES; ++k)
#pragma unroll
      for (int c = 0; c < 8; ++c) op[k][c] = kv[k * 1024 + (8 + c) * 64 + lane]; // the values, behind the softmax
    __builtin_amdgcn_sched_barrier(0);
    if ((t0 + (TILES - 1) * nsplit) * 32 + 32 > L) { // uniform: some keys are tree nodes, or past the last
#pragma unroll
      for (int i = 0; i < 2 * TILES; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int j = (t0 + (i >> 1) * nsplit) * 32 + (i & 1) * 16 + 4 * g + e - L;
          const int bit = (int)((j < 64 ? a0 : a1) >> (j & 63)) & 1; // no branch: 32 of them would cost more than the tile
          sv[i][e] = ((int)(j < 0) | ((int)(j < n) & bit)) != 0 ? sv[i][e] : -INFINITY;
        }
    }
    float mx[TILES];
#pragma unroll
    for (int k = 0; k < TILES; ++k) {
      mx[k] = sv[2 * k][0];
#pragma unroll
      for (int i = 2 * k; i < 2 * k + 2; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) mx[k] = fmaxf(mx[k], sv[i][e]);
      mx[k] = fmaxf(mx[k], __shfl_xor(mx[k], 16));
      mx[k] = fmaxf(mx[k], __shfl_xor(mx[k], 32));
    }
    // tile by tile, as in k_attn_mfma: each new maximum's probability is exactly 1 and has no rounding (with one maximum for
    // both tiles the result is 0.2 to 1 % further from float64)
#pragma unroll
    for (int k = 0; k < TILES; ++k) {
      const float m_new = fmaxf(m, mx[k] * sc);
      if (__any(m_new > m)) {
        const float corr = __builtin_amdgcn_exp2f(m - m_new);
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) {
          acc[dt][0] *= corr; acc[dt][1] *= corr; acc[dt][2] *= corr; acc[dt][3] *= corr;
        }
        accl[0] *= corr; accl[1] *= corr; accl[2] *= corr; accl[3] *= corr;
        m = m_new;
      }
      // m is finite, so an invisible key's probability is exactly 0, also in a row that has seen no key yet
      u32x4 pf;
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        const f32x4 &s4 = sv[2 * k + (e >> 2)];
        const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s4[e & 3], sc, -m));
        const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s4[(e & 3) + 1], sc, -m));
        pf[e >> 1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{p0, p1}, bf16x2));
      }
      accl = mfma16a(ones, pf, accl);
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) acc[dt] = mfma16a(op[k][dt], pf, acc[dt]);
    }
  };

  for (int s = 0; s < steps; ++s) { // uniform over the workgroup
    if (issued <= s) { // nothing was asked for ahead (only behind a sequence beyond the bound)
      load_step(s, n_tiles - 1);
      issued = s + 1;
    }
    wait_steps(issued - s - 1);
    meet_waves(); // this step's tiles are there, and every wave has read the previous step's and its queries
    while (issued < steps && issued < s + D) {
      load_step(issued, n_tiles - 1);
      ++issued;
    }
    const int t0 = split + 2 * s * nsplit;
    const u32x4 *kv = ring + (s % D) * (RING_STEP_BYTES / 16);
    if constexpr (W <= 8) { // the registers of three waves on a SIMD do not hold the operands of two tiles
      if (t0 + nsplit < n_tiles) multiply(std::integral_constant<int, 2>{}, kv, t0);
      else multiply(std::integral_constant<int, 1>{}, kv, t0);
    } else {
      multiply(std::integral_constant<int, 1>{}, kv, t0);
      if (t0 + nsplit < n_tiles) multiply(std::integral_constant<int, 1>{}, kv + 1024, t0 + nsplit);
    }
  }
  wait_tiles<0>(); // loads beyond a sequence shorter than the bound have landed
  finish_share(acc, m, accl[0], ring, wave, lane, wt, h, split, nsplit, H, n, part_ml, part_acc, out, out_row_tiles);
}

// ---------------------------------------------------------------------------------------------
// One-launch form for short sequences: a workgroup owns one (query head, tile of 16 nodes) and its eight
// waves split the keys (wave w takes the 32-key tiles w, w+8, ...), each reading its K/V tiles from memory
// straight into matrix-core operand registers (the cache layout is that order; nothing is shared between the
// waves, so nothing is staged).  The waves' (max, sum, accumulator) meet in LDS and wave w finishes features
// 16w .. 16w+15 of all 16 nodes, so no partial result ever leaves the compute unit and no merge launch
// follows.  The node tiles of a head read the same K/V: their workgroups are numbered so that round-robin
// placement puts them on one XCD, whose L2 serves the repeats.  Every compute unit then pulls the whole
// sequence of its head, (L + N) * 512 bytes, which is why this form is only chosen for short sequences.
// ---------------------------------------------------------------------------------------------
constexpr int ATT1_WAVES = 8;
constexpr size_t ATT1_LDS_BYTES = (size_t)ATT1_WAVES * 8 * 64 * 16 + (size_t)ATT1_WAVES * 16 * 2 * 4;
template <int DUMMY>
__global__ __launch_bounds__(ATT1_WAVES * 64) void k_attn_tile(const bf16_t *__restrict__ q, const bf16_t *__restrict__ Kl,
                                                             const bf16_t *__restrict__ Vl, int32_t H, int32_t Hkv,
                                                             int32_t cap, int32_t n, const uint64_t *__restrict__ anc,
                                                             const int32_t *__restrict__ d_len, bf16_t *__restrict__ out,
                                                             int32_t out_row_tiles) {
  extern __shared__ f32x4 att1_lds[]; // ATT1_LDS_BYTES
  f32x4 (*s_acc)[8][64] = reinterpret_cast<f32x4 (*)[8][64]>(att1_lds);                         // [waves][8][64], 64 KiB
  float (*s_ml)[16][2] = reinterpret_cast<float (*)[16][2]>(att1_lds + ATT1_WAVES * 8 * 64);    // [waves][16][2]
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int r = lane & 15, g = lane >> 4;
  // linear id -> (head, node tile): ids that differ by 8 share a head's XCD; x = id % 8 picks the head inside
  // a block of 8 heads, y = id / 8 runs over (node tile, head block)
  const int id = blockIdx.x, x8 = id & 7, y = id >> 3;
  const int NT = (n + 15) / 16, wt = y % NT, h = (y / NT) * 8 + x8;
  if (h >= H) return; // uniform over the workgroup (H not a multiple of 8)
  const int hk = h / (H / Hkv);

  const int node = wt * 16 + r;
  const int node_c = node < n ? node : n - 1;
  u32x4 qf[4];
  {
    const u32x4 *qp = reinterpret_cast<const u32x4 *>(q + ((size_t)node_c * H + h) * 128 + 8 * g);
#pragma unroll
    for (int c = 0; c < 4; ++c) qf[c] = qp[c * 4];
  }
  const uint64_t a0 = anc[2 * node_c], a1 = anc[2 * node_c + 1];
  const u32x4 *Kh = reinterpret_cast<const u32x4 *>(Kl + (size_t)hk * cap * 128) + lane;
  const u32x4 *Vh = reinterpret_cast<const u32x4 *>(Vl + (size_t)hk * cap * 128) + lane;

  f32x4 acc[8];
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) acc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 accl = f32x4{0.f, 0.f, 0.f, 0.f};
  const u32x4 ones = u32x4{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
  float m = NEG_BIG;
  const float sc = 0.08838834764831845f * 1.4426950408889634f; // 1/sqrt(128) * log2(e)

  u32x4 kq[2][8], vq[2][8]; // two tiles of operands in registers: the one in use and the next
  auto fetch = [&](int buf, int tile) {
#pragma unroll
    for (int c = 0; c < 8; ++c) kq[buf][c] = __builtin_nontemporal_load(Kh + (size_t)tile * 512 + c * 64);
#pragma unroll
    for (int c = 0; c < 8; ++c) vq[buf][c] = __builtin_nontemporal_load(Vh + (size_t)tile * 512 + c * 64);
  };
  if ((wave + 1) * 32 <= cap) fetch(0, wave); // inside the allocation even if beyond the sequence
  const int L = *d_len;
  const int total = L + n;
  const int n_tiles = (total + 31) >> 5;
  int i = 0;
  for (int t = wave; t < n_tiles; t += ATT1_WAVES, ++i) {
    const bool has_next = t + ATT1_WAVES < n_tiles;
    // the buffers alternate by compile-time index: two copies of the body
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if ((i & 1) != b) continue;
      if (has_next) fetch(b ^ 1, t + ATT1_WAVES);
      f32x4 s0 = f32x4{0.f, 0.f, 0.f, 0.f}, s1 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        s0 = mfma16a(kq[b][c], qf[c], s0);
        s1 = mfma16a(kq[b][4 + c], qf[c], s1);
      }
      float xs[8];
      bool vis[8];
      const bool in_prefix = t * 32 + 32 <= L; // uniform: every key of the tile is visible to every node
      const int pbase = t * 32 + 4 * g;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int p = pbase + (e >> 2) * 16 + (e & 3);
        bool v = in_prefix || p < L;
        if (!v && p < total) {
          const int j = p - L;
          v = j < 64 ? ((a0 >> j) & 1ull) : ((a1 >> (j - 64)) & 1ull);
        }
        vis[e] = v;
        const float sv = (e < 4 ? s0[e & 3] : s1[e & 3]) * sc;
        xs[e] = v ? sv : NEG_BIG;
      }
      float mx = fmaxf(fmaxf(fmaxf(xs[0], xs[1]), fmaxf(xs[2], xs[3])), fmaxf(fmaxf(xs[4], xs[5]), fmaxf(xs[6], xs[7])));
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float m_new = fmaxf(m, mx);
      if (__any(m_new > m)) {
        const float corr = __builtin_amdgcn_exp2f(m - m_new);
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) {
          acc[dt][0] *= corr; acc[dt][1] *= corr; acc[dt][2] *= corr; acc[dt][3] *= corr;
        }
        accl[0] *= corr; accl[1] *= corr; accl[2] *= corr; accl[3] *= corr;
        m = m_new;
      }
      float pr[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) pr[e] = vis[e] ? __builtin_amdgcn_exp2f(xs[e] - m) : 0.f;
      u32x4 pf;
#pragma unroll
      for (int e = 0; e < 8; e += 2)
        pf[e >> 1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{pr[e], pr[e + 1]}, bf16x2));
      accl = mfma16a(ones, pf, accl);
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) acc[dt] = mfma16a(vq[b][dt], pf, acc[dt]);
    }
  }

  // meet in LDS: every wave leaves its accumulators (unnormalised), its running maximum and its sum
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) s_acc[wave][dt][lane] = acc[dt];
  if (g == 0) {
    s_ml[wave][r][0] = m;
    s_ml[wave][r][1] = accl[0];
  }
  __syncthreads();
  // wave w finishes features 16w .. 16w+15: out = sum_v acc_v 2^(m_v - M) / sum_v l_v 2^(m_v - M) in wave order
  float M = NEG_BIG;
#pragma unroll
  for (int v = 0; v < ATT1_WAVES; ++v)
    if (s_ml[v][r][1] > 0.f) M = fmaxf(M, s_ml[v][r][0]);
  float den = 0.f;
  f32x4 num = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int v = 0; v < ATT1_WAVES; ++v) {
    const float lv = s_ml[v][r][1];
    if (lv > 0.f) {
      const float w = __builtin_amdgcn_exp2f(s_ml[v][r][0] - M);
      den += w * lv;
      num += s_acc[v][wave][lane] * w;
    }
  }
  if (node >= n) return;
  const float inv = 1.0f / den;
  const int d = 16 * wave + 4 * g;
  ushort4 o;
  o.x = f32_to_bf16(num[0] * inv); o.y = f32_to_bf16(num[1] * inv);
  o.z = f32_to_bf16(num[2] * inv); o.w = f32_to_bf16(num[3] * inv);
  const size_t idx = out_row_tiles > 0 ? act_frag_index(node, h * 128 + d, out_row_tiles) : ((size_t)node * H + h) * 128 + d;
  store_stream(out + idx, o);
}

// out[node, h, :] = sum_s w_s o_s / sum_s w_s with w_s = l_s 2^(m_s - max m), o_s the split's normalised
// output; splits without visible keys (l_s == 0) contribute nothing.  Block (8 nodes, head), 32 threads x
// 4 features per node; all loads of a thread are issued before any arithmetic.
template <int MOST>
__global__ __launch_bounds__(256) void k_attn_merge(const float *__restrict__ part_ml, const float *__restrict__ part_acc,
                                                    int32_t part_rows, int32_t H, int32_t n, int32_t nsplit,
                                                    bf16_t *__restrict__ out,
                                                    int32_t out_row_tiles) {
  const int node = blockIdx.x * 8 + (threadIdx.x >> 5), h = blockIdx.y, d = (threadIdx.x & 31) * 4;
  if (node >= n) return;
  float2 ml[MOST];
  f16x4 av[MOST];
#pragma unroll
  for (int s = 0; s < MOST; ++s) {
    if (s < nsplit) {
      const size_t row = ((size_t)s * H + h) * part_rows + node;
      ml[s] = *reinterpret_cast<const float2 *>(part_ml + row * 2);
      av[s] = reinterpret_cast<const f16x4 *>(part_acc)[row * 32 + (d >> 2)];
    }
  }
  float M = NEG_BIG;
#pragma unroll
  for (int s = 0; s < MOST; ++s)
    if (s < nsplit && ml[s].y > 0.f) M = fmaxf(M, ml[s].x);
  float den = 0.f;
  float4 num = float4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < MOST; ++s) {
    if (s < nsplit && ml[s].y > 0.f) {
      const float w = exp2f(ml[s].x - M) * ml[s].y;
      den += w;
      num.x += w * (float)av[s][0]; num.y += w * (float)av[s][1];
      num.z += w * (float)av[s][2]; num.w += w * (float)av[s][3];
    }
  }
  const float inv = 1.0f / den;
  ushort4 o;
  o.x = f32_to_bf16(num.x * inv); o.y = f32_to_bf16(num.y * inv);
  o.z = f32_to_bf16(num.z * inv); o.w = f32_to_bf16(num.w * inv);
  const size_t idx = out_row_tiles > 0 ? act_frag_index(node, h * 128 + d, out_row_tiles)
                                       : ((size_t)node * H + h) * 128 + d;
  store_stream(out + idx, o);
}

// part_rows: rows reserved per (split, head)
hipError_t launch_attn_merge(const float *part_ml, const float *part_acc, int32_t part_rows, int32_t H, int32_t n, int32_t nsplit,
                             bf16_t *out, int32_t out_row_tiles, KernelTimer tm, hipStream_t st) {
  const dim3 grid((n + 7) / 8, H);
  if (nsplit > ATTN_MAX_SPLITS)
    return launch(k_attn_merge<2 * ATTN_MAX_SPLITS>, grid, dim3(256), 0, st, tm, part_ml, part_acc, part_rows, H, n, nsplit, out, out_row_tiles);
  if (nsplit <= ATTN_MAX_SPLITS / 2)
    return launch(k_attn_merge<ATTN_MAX_SPLITS / 2>, grid, dim3(256), 0, st, tm, part_ml, part_acc, part_rows, H, n, nsplit, out, out_row_tiles);
  return launch(k_attn_merge<ATTN_MAX_SPLITS>, grid, dim3(256), 0, st, tm, part_ml, part_acc, part_rows, H, n, nsplit, out, out_row_tiles);
}

int attn_heads_per_wg(int32_t H, int32_t Hkv, int32_t n) {
  const int G = H / Hkv, NT = (n + 15) / 16;
  return (G % 2 == 0 && NT * 2 <= 12) ? 2 : 1; // up to 12 waves keep 3 per SIMD and the registers they need
}

// As many key-axis splits as keep the launch within one workgroup per CU (a second workgroup on a CU
// shares that CU's memory rate and doubles the critical path), at least two 32-key tiles per split.
int attn_choose_splits(int32_t head_groups, int32_t len_bound) {
  const int tiles = (len_bound + 31) / 32;
  int s = 256 / (head_groups > 0 ? head_groups : 1);
  if (s > tiles / 2) s = tiles / 2;
  if (s > ATTN_MAX_SPLITS) s = ATTN_MAX_SPLITS;
  return s < 1 ? 1 : s;
}

// 32-key tiles a workgroup takes one after another.  us a layer that whole steps are longer with k_attn_ring than with k_attn_mfma (runs of
// a side within 0.7 us): 80 nodes, 32 heads on 32 +0.4 at 12 tiles, 0.0 at 13, -0.6 at 16, -2.1 at 20, -3.1 at 32, -7.2 at 63; 40 on 40 +1.4
// at 12, -1.2 at 17, -2.2 at 21, -7.6 at 43, -17 at 84; 64 on 8 -0.9 at 17, -1.6 at 24, -3.7 at 63; 48 nodes, 32 on 32 -1.8 at 16, -2.9 at 20, 64
// on 8 -3.3 at 17; 96 nodes, 32 on 32 +0.8 at 16, -0.5 at 20, -1.4 at 32, 40 on 40 -1.3 at 21, 64 on 8 -1.5 at 16; 112 nodes, 32 on 32 +1.8 at 16,
// +0.1 at 20, -0.5 at 32, 40 on 40 -0.7 at 22; 128 nodes, 32 on 32 +1.2 at 16, +1.0 at 21, +0.5 at 32, -1.3 at 63, 40 on 40 -0.2 at 17, -2.9 at 27,
// -4.2 at 43.  (Kernel times alone put the lines at 12 and 14; launched back to back, with the queries in L2, it gains from 7 on.)
bool attn_long_shares(int32_t node_tiles, int32_t hpw, int32_t len_bound, int32_t nsplit) {
  const int chain = ((len_bound + 31) / 32 + nsplit - 1) / nsplit;
  return chain >= (hpw > 1 || node_tiles <= 5 ? 16 : node_tiles <= 7 ? 24 : 40);
}

template <int NT, int HPW>
static hipError_t launch_attn_k(const bf16_t *q, const bf16_t *Kl, const bf16_t *Vl, int32_t H, int32_t Hkv, int32_t cap,
                                int32_t n, const uint64_t *anc, const int32_t *d_len, int32_t len_bound, int32_t nsplit,
                                float *part_ml, float *part_acc, bf16_t *out, int32_t out_row_tiles, KernelTimer tm,
                                hipStream_t st) {
  const dim3 grid(Hkv, H / Hkv / HPW, nsplit), block(NT * HPW * 64);
  if (attn_long_shares(NT, HPW, len_bound, nsplit) && starts_on_16(q) && starts_on_16(Kl) && starts_on_16(Vl) && starts_on_16(anc)) {
    constexpr int smem = ring_lds_bytes(NT * HPW);
    static bool once = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_attn_ring<NT, HPW>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, smem) == hipSuccess;
    if (!once) return hipErrorInvalidValue;
    return launch(k_attn_ring<NT, HPW>, grid, block, smem, st, tm, q, Kl, Vl, H, Hkv, cap, n, anc, d_len,
                  (len_bound + 31) / 32, nsplit, part_ml, part_acc, out, out_row_tiles);
  }
  return launch(k_attn_mfma<NT, HPW>, grid, block, 0, st, tm, q, Kl, Vl, H, Hkv, cap, n, anc, d_len, nsplit, part_ml, part_acc,
                out, out_row_tiles);
}

template <int NT>
static hipError_t launch_attn_nt(int hpw, const bf16_t *q, const bf16_t *Kl, const bf16_t *Vl, int32_t H, int32_t Hkv,
                                 int32_t cap, int32_t n, const uint64_t *anc, const int32_t *d_len, int32_t len_bound,
                                 int32_t nsplit, float *part_ml, float *part_acc, bf16_t *out, int32_t out_row_tiles,
                                 KernelTimer tm, hipStream_t st) {
  if constexpr (NT <= 6) {
    if (hpw == 2)
      return launch_attn_k<NT, 2>(q, Kl, Vl, H, Hkv, cap, n, anc, d_len, len_bound, nsplit, part_ml, part_acc, out, out_row_tiles, tm, st);
  }
  if (hpw != 1) return hipErrorInvalidValue;
  return launch_attn_k<NT, 1>(q, Kl, Vl, H, Hkv, cap, n, anc, d_len, len_bound, nsplit, part_ml, part_acc, out, out_row_tiles, tm, st);
}

// The one-launch form pays when a compute unit can pull its head's whole sequence in less time than the
// split form spends on its second launch: up to about this many positions (prefix + nodes), and only when few
// query heads share a K/V head (each of them re-reads it).  Measured at 32 heads, 80 nodes (us per layer, one
// launch / split + merge): 7.8 / 11.0 at 256 positions, 10.3 / 12.5 at 512, 12.5 / 13.3 at 768, 14.5 / 14.2
// at 1024, 22.2 / 17.9 at 2048.
constexpr int ATT1_MAX_LEN = 832;
bool attn_one_launch(int32_t H, int32_t Hkv, int32_t len_bound) { return len_bound <= ATT1_MAX_LEN && H / Hkv <= 2; }

hipError_t launch_attn_mfma(const bf16_t *q, const bf16_t *Kl, const bf16_t *Vl, int32_t H, int32_t Hkv, int32_t cap,
                            int32_t n, const uint64_t *anc, const int32_t *d_len, int32_t len_bound, float *part_ml,
                            float *part_acc, bf16_t *out, int32_t out_row_tiles, Profiler *prof, hipStream_t st) {
  if (Hkv < 1 || H % Hkv != 0) return hipErrorInvalidValue;
  if (attn_rows_better(H, Hkv, n, len_bound) && starts_on_16(Kl) && starts_on_16(Vl))
    return launch_attn_rows(q, Kl, Vl, H, Hkv, cap, n, anc, d_len, len_bound, part_ml, part_acc, out, out_row_tiles, prof, st);
  const KernelTimer tm = prof_next(prof, PC_ATTN);
  if (attn_one_launch(H, Hkv, len_bound)) {
    const int NT = (n + 15) / 16;
    static bool once = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_attn_tile<0>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)ATT1_LDS_BYTES) == hipSuccess;
    if (!once) return hipErrorInvalidValue;
    return launch(k_attn_tile<0>, dim3(((H + 7) / 8) * 8 * NT), dim3(ATT1_WAVES * 64), ATT1_LDS_BYTES, st, tm, q, Kl, Vl,
                  H, Hkv, cap, n, anc, d_len, out, out_row_tiles);
  }
  const int hpw = attn_heads_per_wg(H, Hkv, n);
  const int nsplit = attn_choose_splits(H / hpw, len_bound);
  hipError_t e = hipErrorInvalidValue;
  switch ((n + 15) / 16) {
  case 1: e = launch_attn_nt<1>(hpw, q, Kl, Vl, H, Hkv, cap, n, anc, d_len, len_bound, nsplit, part_ml, part_acc, out, out_row_tiles, tm, st); break;
  case 2: e = launch_attn_nt<2>(hpw, q, Kl, Vl, H, Hkv, cap, n, anc, d_len, len_bound, nsplit, part_ml, part_acc, out, out_row_tiles, tm, st); break;
  case 3: e = launch_attn_nt<3>(hpw, q, Kl, Vl, H, Hkv, cap, n, anc, d_len, len_bound, nsplit, part_ml, part_acc, out, out_row_tiles, tm, st); break;
  case 4: e = launch_attn_nt<4>(hpw, q, Kl, Vl, H, Hkv, cap, n, anc, d_len, len_bound, nsplit, part_ml, part_acc, out, out_row_tiles, tm, st); break;
  case 5: e = launch_attn_nt<5>(hpw, q, Kl, Vl, H, Hkv, cap, n, anc, d_len, len_bound, nsplit, part_ml, part_acc, out, out_row_tiles, tm, st); break;
  case 6: e = launch_attn_nt<6>(hpw, q, Kl, Vl, H, Hkv, cap, n, anc, d_len, len_bound, nsplit, part_ml, part_acc, out, out_row_tiles, tm, st); break;
  case 7: e = launch_attn_nt<7>(hpw, q, Kl, Vl, H, Hkv, cap, n, anc, d_len, len_bound, nsplit, part_ml, part_acc, out, out_row_tiles, tm, st); break;
  case 8: e = launch_attn_nt<8>(hpw, q, Kl, Vl, H, Hkv, cap, n, anc, d_len, len_bound, nsplit, part_ml, part_acc, out, out_row_tiles, tm, st); break;
  }
  if (e != hipSuccess || nsplit == 1) return e;
  return launch_attn_merge(part_ml, part_acc, NP, H, n, nsplit, out, out_row_tiles, prof_next(prof, PC_ATTN_MERGE), st);
}

} // namespace tr
