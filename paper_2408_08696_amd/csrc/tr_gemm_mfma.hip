// Weight-streaming skinny GEMM on the matrix cores: y[n, O] = a[n, K] * w[O, K]^T with n <= 128 rows
// (the tree nodes), bf16 operands, float32 accumulation.  Every weight byte is read from HBM exactly
// once per call; the kernel is bound by that stream, the MFMA work (2*n flop per weight element) only
// has to keep up.
//
// Operand layouts.  v_mfma_f32_16x16x32_bf16 computes D[16 x 16] += A[16 x 32] * B[32 x 16] where lane l
// supplies A[l%16][8*(l/16) .. +7] and B[8*(l/16) .. +7][l%16] as one 16-byte register group, and receives
// D[4*(l/16) .. +3][l%16].  Both operands are therefore stored in memory in "fragment order": a tile of
// 16 rows x 32 k is 1 KiB, lane l's 16 bytes at offset 16*l, so that one wave-wide 16-byte load is one
// fully contiguous KiB and lands directly in MFMA operand registers.
//   weights (packed once by k_pack_weight):   tile (ot, kt) at ((ot * K/32 + kt) * 1 KiB)
//   activations (written so by their producers): tile (kt, nt) at ((kt * NT + nt) * 1 KiB), NT = ceil(n/16)
// With A = weight tile and B = activation tile, lane l ends with outputs o0 + 4*(l/16) .. +3 of row
// 16*nt + l%16.
//
// Mapping.  One workgroup owns up to NW consecutive out-tiles (16*NW output features; the tiles are dealt
// evenly over the workgroups) and one of `splits` K-ranges; its GW = 8 wavefronts (4 in the NW = 8
// variant) take interleaved k-tiles of that range, keep PF k-steps of loads in flight in registers, and
// reduce through LDS at the end, each wave ending up with (and storing) its share of the output tiles.
// splits > 1 writes one partial result per split (summed in a fixed order by the consumer), so results
// are run-to-run deterministic.
//
// Why NW is large.  Every workgroup reads the whole activation block of its K-range from L2 (16*NT rows),
// so L2 carries (1 + 16*NT / (16*NW)) bytes per weight byte; measured L2->CU throughput on MI355X is only
// about twice the HBM rate, so the kernel stays HBM-bound only while NW >= NT.  gemm_choose picks
// (NW, workgroups, splits) from a cost model of exactly this trade, close to one workgroup per compute
// unit with NW as large as the register file allows.
//
// Epilogues: plain float32 store (per K-split), gate/up pairs through SwiGLU into the next GEMM's operand
// order, for the fused Q/K/V projection RoPE plus the query and KV-cache writes (GemmRope), or for o and down of few rows the update of
// the residual stream (GemmResid).
#include "tr_kernels.h"

namespace tr {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr int GEMM_WAVES = 8;
// k-steps of loads in flight per wave, bounded by the register file: accumulators take 4*NW*NT VGPRs,
// every stage 4*(NW+NT); 256 VGPRs per wave at two waves per SIMD, about 208 of them usable here
__host__ __device__ constexpr int gemm_pf(int nw, int nt, int waves) {
  // four waves per workgroup leave one wave per SIMD and 512 registers per wave: the accumulators then
  // sit in the upper half of the unified register file and four stages of 4*(8+5) fit the lower half
  const int pf = waves <= 4 ? 4 : (208 - 4 * nw * nt) / (4 * (nw + nt));
  return pf < 1 ? 1 : (pf > 4 ? 4 : pf);
}

__device__ inline f32x4 mfma16(const u32x4 &a, const u32x4 &b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// ---------------------------------------------------------------------------------------------
// one-time repack of a row-major [O, K] bf16 matrix into fragment order
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_pack_weight(const bf16_t *__restrict__ src, int32_t O, int32_t K,
                                                     int32_t rope_hd, uint4 *__restrict__ dst) {
  const int KT = K / 32;
  const size_t slot = (size_t)blockIdx.x * 256 + threadIdx.x; // one 16-byte lane slot
  const size_t total = (size_t)(O / 16) * KT * 64;
  if (slot >= total) return;
  const int lane = (int)(slot & 63);
  const size_t tile = slot >> 6;
  const int kt = (int)(tile % KT);
  const int ot = (int)(tile / KT);
  int row = ot * 16 + (lane & 15);
  if (rope_hd > 0) { // packed row h*hd + 2j + b <- source row h*hd + j + b*hd/2
    const int i = row % rope_hd;
    row = row - i + (i >> 1) + (i & 1) * (rope_hd / 2);
  }
  const int k = kt * 32 + 8 * (lane >> 4);
  dst[slot] = *reinterpret_cast<const uint4 *>(src + (size_t)row * K + k);
}

hipError_t launch_pack_weight(const bf16_t *src, bf16_t *dst, int32_t O, int32_t K, int32_t rope_hd, hipStream_t st) {
  const size_t total = (size_t)(O / 16) * (K / 32) * 64;
  return launch(k_pack_weight, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, KernelTimer{}, src, O, K, rope_hd,
                reinterpret_cast<uint4 *>(dst));
}

// ---------------------------------------------------------------------------------------------
// the GEMM
// ---------------------------------------------------------------------------------------------
// LDS the tail needs: the GW partials of the tiles of one reduce-scatter pass, plus the per-row scales when
// the epilogue applies an RMS scale.  One pass if all tiles fit the 160 KB of a CU, else two (the first
// covers the units of waves 0 .. GW/2-1).
// The sums of squares a row comes with lie in the place of its scale.
constexpr size_t gemm_scale_lds_bytes(int nt, bool scaled) { return scaled ? (size_t)nt * 16 * gemm_most_ssq(nt) * sizeof(float) : 0; }
// Tail units a wave owns: an even share, or with GEMM_RESID a row tile's.
constexpr int gemm_units_per_wave(int p, int nt, int mode, int gw) { return mode == GEMM_RESID ? p : (p * nt + gw - 1) / gw; }
constexpr bool gemm_tail_one_pass(int p, int nt, int mode, int gw, bool scaled) {
  return (size_t)p * nt * (mode == GEMM_SWIGLU ? 2 : 1) * gw * 1024 + gemm_scale_lds_bytes(nt, scaled) <= 160 * 1024;
}
constexpr size_t gemm_tail_red_bytes(int p, int nt, int mode, int gw, bool scaled) {
  const int u = p * nt, upw = gemm_units_per_wave(p, nt, mode, gw);
  const int own0 = gemm_tail_one_pass(p, nt, mode, gw, scaled) ? gw : gw / 2;
  const int units0 = own0 * upw < u ? own0 * upw : u;
  return (size_t)units0 * (mode == GEMM_SWIGLU ? 2 : 1) * gw * 1024;
}

// keeps a uniform kernel argument in scalar registers across the main loop; left alone the compiler reads it again behind
// the reduction, a scalar memory round trip in the tail
template <typename T>
__device__ inline T hold(T v) {
  asm volatile("" : "+s"(v));
  return v;
}
template <typename T>
__device__ inline T *hold(T *p) {
  auto g = (__attribute__((address_space(1))) T *)p;
  asm volatile("" : "+s"(g));
  return (T *)g;
}

// What the first weight tiles need leads the arguments: 14 words, which come in scalar registers with the wave.  w1: the second
// matrix of Q/K/V or gate/up, w2: the third of Q/K/V.
template <int NT, int NW, int MODE, int GW, bool SCALED>
__global__ __launch_bounds__(GW * 64) void k_gemm_mfma(const bf16_t *w0, const bf16_t *w1, const bf16_t *a_frag, const bf16_t *w2,
                                                       int32_t KT, int32_t part_q, int32_t part_rem, int32_t split_kt, int32_t end0,
                                                       int32_t end1, GemmArgs g) {
  // GEMM_ROPE is GEMM_STORE with the fused Q/K/V epilogue: its rotary factors and the committed length are asked for behind
  // the first weight tiles, so that the tail has no load left (it took three dependent round trips there)
  // SWIGLU: NW = 2P; weight tiles 0..P-1 come from the gate matrix, P..2P-1 from the up matrix
  constexpr int P = MODE == GEMM_SWIGLU ? NW / 2 : NW; // distinct out-tiles per workgroup
  constexpr int PF = gemm_pf(NW, NT, GW);
  extern __shared__ float red[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6); // in a scalar register: the k-loop's branches are uniform

  // out-tiles owned by this workgroup: the T tiles are dealt to the G workgroups in contiguous ranges of
  // T/G tiles, the first T%G of them one longer (the host picks G >= T/P, so no range exceeds P).  Tiles
  // are numbered across the concatenated segments (weight matrices) and each looks up its own segment,
  // so a workgroup may straddle two matrices.
  // All arguments are needed at once and come in one batch of scalar loads.  A loop over the matrices per tile, the scale's
  // loads and the rotary factors in front of the first weight tile took 0.9 to 1.9 us to get there, this takes 0.3 to 0.5:
  // step of the 7B shape with 1 / 128 nodes 3003 / 4949 -> 2955 / 4849 us (runs of one side differ by 0.8 / 0.4 %); with 80 nodes
  // and the step of the 13B shape the difference is within that of the runs.
  const int bx = blockIdx.x;
  const int tile0 = bx * part_q + (bx < part_rem ? bx : part_rem);
  const int n_valid = part_q + (bx < part_rem ? 1 : 0);
  typedef __attribute__((address_space(1))) const u32x4 *global_tiles; // said outright: the masks below hide it
  global_tiles wbase[NW];
#pragma unroll
  for (int u = 0; u < P; ++u) {
    const int t = tile0 + (u < n_valid ? u : 0); // unused slots re-read the first tile (a cache hit), never stored
    const bf16_t *w = w0;
    int at = t;
    if (MODE == GEMM_ROPE) { // bit masks, no branch or loop over the matrices: their loads came one after another
      const int64_t in1 = -(int64_t)(t >= end0 && t < end1), in2 = -(int64_t)(t >= end1);
      const uint64_t b0 = (uint64_t)w0, b1 = (uint64_t)w1, b2 = (uint64_t)w2;
      w = reinterpret_cast<const bf16_t *>(b0 ^ ((b0 ^ b1) & in1) ^ ((b0 ^ b2) & in2));
      at = t - (end0 & (int)in1) - (end1 & (int)in2);
    }
    wbase[u] = (global_tiles)reinterpret_cast<const u32x4 *>(w) + (size_t)at * KT * 64 + lane;
    if (MODE == GEMM_SWIGLU) wbase[P + u] = (global_tiles)reinterpret_cast<const u32x4 *>(w1) + (size_t)at * KT * 64 + lane;
  }
  const u32x4 *abase = reinterpret_cast<const u32x4 *>(a_frag) + lane;

  // this workgroup's K-range and this wave's k-tiles in it: kt = kt0 + wave + 8*i
  const int split = blockIdx.y;
  const int n_rows = hold(g.n);
  float *const y = MODE == GEMM_STORE ? hold(g.y + (size_t)split * g.split_stride) : nullptr;
  const int ldy = MODE == GEMM_STORE ? hold(g.ldy) : 0;
  bf16_t *const h_frag = MODE == GEMM_SWIGLU ? hold(g.h_frag) : nullptr;
  const int kt0 = split * split_kt;
  const int kt1 = kt0 + split_kt < KT ? kt0 + split_kt : KT;
  const int first = kt0 + wave;
  const int nsteps = first < kt1 ? (kt1 - first + GW - 1) / GW : 0;

  f32x4 acc[NW][NT];
#pragma unroll
  for (int u = 0; u < NW; ++u)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[u][t] = f32x4{0.f, 0.f, 0.f, 0.f};

  u32x4 wq[PF][NW], aq[PF][NT];
  auto issue = [&](int stage, int step) {
    const size_t kt = (size_t)(first + step * GW);
#pragma unroll
    for (int u = 0; u < NW; ++u) wq[stage][u] = __builtin_nontemporal_load(wbase[u] + kt * 64);
#pragma unroll
    for (int t = 0; t < NT; ++t) aq[stage][t] = abase[(kt * NT + t) * 64];
  };
  constexpr int TPU = MODE == GEMM_SWIGLU ? 2 : 1;
  constexpr int U = P * NT;
  constexpr int UPW = gemm_units_per_wave(P, NT, MODE, GW);
  const int r = lane & 15, gq = lane >> 4;
  // What only the epilogue needs is asked for behind the first weight tiles.  Sums of squares go straight to LDS: wave w
  // fetches those of row tiles w, w + GW, .. and turns them into scales itself.
  float *const ssq_lds = red + gemm_tail_red_bytes(P, NT, MODE, GW, SCALED) / sizeof(float); // [NT][16][n_ssq], SCALED only
  GemmResid rs{};
  GemmRope rp{};
  int L = 0;
  f32x2 rope_c[MODE == GEMM_ROPE ? UPW : 1], rope_s[MODE == GEMM_ROPE ? UPW : 1];
  auto issue_epilogue = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    if (SCALED) {
      for (int t = wave; t < NT; t += GW) {
        const int words = (n_rows - 16 * t < 16 ? n_rows - 16 * t : 16) * g.n_ssq;
        for (int i = 0; i < words; i += 256)
          if (i + lane * 4 < words)
            tile_to_lds((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)(ssq_lds + t * 16 * g.n_ssq + i),
                        lane * 16, reinterpret_cast<uint64_t>(g.row_ssq + t * 16 * g.n_ssq + i));
      }
    }
    if (MODE == GEMM_RESID) {
      rs.x = hold(g.resid.x); rs.gain = hold(g.resid.gain); rs.xg_frag = hold(g.resid.xg_frag); rs.ssq = hold(g.resid.ssq);
      rs.ld_ssq = hold(g.resid.ld_ssq);
    }
    if (MODE == GEMM_ROPE) {
      rp.q = hold(g.rope.q); rp.k_layer = hold(g.rope.k_layer); rp.v_layer = hold(g.rope.v_layer);
      rp.H = hold(g.rope.H); rp.Hkv = hold(g.rope.Hkv); rp.hd = hold(g.rope.hd); rp.cap = hold(g.rope.cap);
      rp.tiled = hold(g.rope.tiled);
      L = *g.rope.d_len;
#pragma unroll
      for (int i = 0; i < UPW; ++i) {
        const int id = wave * UPW + i, u = id / NT, row = 16 * (id - u * NT) + r;
        const int o = (tile0 + u) * 16 + 4 * gq, head = o / rp.hd, dd = o - head * rp.hd;
        const bool on = id < U && u < n_valid && row < n_rows && head < rp.H + rp.Hkv;
        const float *cs = g.rope.rope + (on ? (size_t)row * rp.hd + (dd >> 1) : 0);
        rope_c[i] = *reinterpret_cast<const f32x2 *>(cs);
        rope_s[i] = *reinterpret_cast<const f32x2 *>(cs + rp.hd / 2);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  auto multiply = [&](int j) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int u = 0; u < NW; ++u) acc[u][t] = mfma16(wq[j][u], aq[j][t], acc[u][t]);
  };
  // The steady part has no condition in it, so that the compiler's wait for a stage leaves the younger ones under way;
  // with a test per step it waits for every load once in PF steps (80 rows: 7B gate/up 36.6 -> 36.3 us, Q/K/V with the
  // loads out of its tail 26.3 -> 25.9, o and down 34.2 -> 33.7).  One row tile keeps the tests: 70B gate/up takes 173 us
  // without them against 155.
  int base = 0;
  if (NT > 1 && nsteps >= 2 * PF) {
#pragma unroll
    for (int j = 0; j < PF; ++j) issue(j, j);
    issue_epilogue();
    do {
#pragma unroll
      for (int j = 0; j < PF; ++j) {
        multiply(j);
        __builtin_amdgcn_sched_barrier(0); // keep this order: the scheduler would gather the loads behind several stages
        issue(j, base + j + PF);
        __builtin_amdgcn_sched_barrier(0);
      }
      base += PF;
    } while (base + 2 * PF <= nsteps);
  } else {
#pragma unroll
    for (int j = 0; j < PF; ++j)
      if (j < nsteps) issue(j, j);
    issue_epilogue();
  }
  for (; base < nsteps; base += PF) {
#pragma unroll
    for (int j = 0; j < PF; ++j) {
      if (base + j < nsteps) {
        multiply(j);
        if (base + j + PF < nsteps) issue(j, base + j + PF);
      }
    }
  }

  // Cross-wave reduction as a reduce-scatter through LDS, then a distributed epilogue.  The NW*NT
  // accumulator tiles form U units of TPU tiles (one tile; for SWIGLU a gate tile and its up tile); wave w
  // owns units w*UPW .. w*UPW+UPW-1.  Every wave publishes its partial of each tile and the owner adds the
  // GW partials in wave order (a fixed order: results are run-to-run identical).  When the GW partials of
  // all tiles fit LDS this is one pass; otherwise two, the first for the units of waves 0 .. GW/2-1.
  // Every wave then scales, activates and stores its own few tiles, instead of one wave storing them all.
  constexpr int OWN0 = gemm_tail_one_pass(P, NT, MODE, GW, SCALED) ? GW : GW / 2; // waves 0 .. OWN0-1 own pass 0
  static_assert(MODE != GEMM_RESID || (OWN0 == GW && NT <= GW), "a wave has whole row tiles of one pass");
  float4 *red4 = reinterpret_cast<float4 *>(red); // [unit slot * TPU + k][GW][64]
  if (SCALED) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    for (int t = wave; t < NT; t += GW) {
      float *const at = ssq_lds + t * 16 * g.n_ssq;
      float ss = 0.f;
      const int n4 = g.n_ssq / 4, turn = n4 >= 16 ? r : 0; // rows start apart: theirs are a multiple of all banks apart
#pragma unroll 8
      for (int i = gq; i < n4; i += 4) {
        const int c = i + turn < n4 ? i + turn : i + turn - n4;
        const float4 q = *reinterpret_cast<const float4 *>(at + r * g.n_ssq + 4 * c);
        ss += (q.x + q.y) + (q.z + q.w);
      }
      ss += __shfl_xor(ss, 16);
      ss += __shfl_xor(ss, 32);
      if (lane < 16) at[lane] = 1.0f / sqrtf(ss / (float)g.norm_dim + g.eps); // in the place of its row tile's sums
    }
  }
  f32x4 x_old[MODE == GEMM_RESID ? UPW : 1];
  uint2 gains[MODE == GEMM_RESID ? UPW : 1];
  if (MODE == GEMM_RESID) { // on their way while the waves' sums meet
#pragma unroll
    for (int i = 0; i < UPW; ++i) {
      const int row = 16 * wave + r, o = (tile0 + i) * 16 + 4 * gq;
      x_old[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      gains[i] = uint2{0u, 0u};
      if (wave < NT && i < n_valid && row < n_rows) {
        const float4 xv = *reinterpret_cast<const float4 *>(rs.x + (size_t)row * g.ldy + o);
        x_old[i] = f32x4{xv.x, xv.y, xv.z, xv.w};
        gains[i] = *reinterpret_cast<const uint2 *>(rs.gain + o);
      }
    }
  }
  f32x4 fin[UPW][TPU];
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    if (pass == 1 && OWN0 * UPW >= U) break; // every unit was owned by a pass-0 wave
#pragma unroll
    for (int u = 0; u < P; ++u)
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int id = MODE == GEMM_RESID ? t * P + u : u * NT + t;
        if ((id / UPW >= OWN0) != (pass == 1)) continue;
        const int slot = (id - pass * OWN0 * UPW) * TPU;
        red4[((size_t)slot * GW + wave) * 64 + lane] = float4{acc[u][t][0], acc[u][t][1], acc[u][t][2], acc[u][t][3]};
        if (MODE == GEMM_SWIGLU)
          red4[((size_t)(slot + 1) * GW + wave) * 64 + lane] =
              float4{acc[P + u][t][0], acc[P + u][t][1], acc[P + u][t][2], acc[P + u][t][3]};
      }
    __syncthreads();
    if ((wave >= OWN0) == (pass == 1)) {
#pragma unroll
      for (int i = 0; i < UPW; ++i) {
        const int id = wave * UPW + i;
#pragma unroll
        for (int k = 0; k < TPU; ++k) {
          f32x4 sum = f32x4{0.f, 0.f, 0.f, 0.f};
          if (id < U) {
            const float4 *src = red4 + ((size_t)((id - pass * OWN0 * UPW) * TPU + k) * GW) * 64 + lane;
#pragma unroll
            for (int w = 0; w < GW; ++w) {
              const float4 o = src[w * 64];
              sum[0] += o.x; sum[1] += o.y; sum[2] += o.z; sum[3] += o.w;
            }
          }
          fin[i][k] = sum;
        }
      }
    }
    if (pass == 0 && OWN0 * UPW < U) __syncthreads(); // pass 1 reuses the buffer
  }

  if constexpr (MODE == GEMM_RESID) { // this wave's row tile and all out-tiles of the workgroup
    const int row = 16 * wave + r;
    float ss = 0.f;
#pragma unroll
    for (int u = 0; u < P; ++u) {
      if (wave >= NT || u >= n_valid) continue;
      const int o = (tile0 + u) * 16 + 4 * gq;
      const f32x4 v = x_old[u] + fin[u][0];
      u32x2s xg = u32x2s{0u, 0u};
      if (row < n_rows) {
        *reinterpret_cast<float4 *>(rs.x + (size_t)row * g.ldy + o) = float4{v[0], v[1], v[2], v[3]};
        xg = u32x2s{bf16_pair(v[0] * __uint_as_float(gains[u].x << 16), v[1] * __uint_as_float(gains[u].x & 0xFFFF0000u)),
                    bf16_pair(v[2] * __uint_as_float(gains[u].y << 16), v[3] * __uint_as_float(gains[u].y & 0xFFFF0000u))};
        ss += (v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]);
      }
      const size_t slot = ((size_t)(o >> 5) * NT + wave) * 64 + r + 16 * ((o & 31) >> 3);
      *reinterpret_cast<u32x2s *>(rs.xg_frag + slot * 8 + (o & 7)) = xg;
    }
    ss += __shfl_xor(ss, 16);
    ss += __shfl_xor(ss, 32);
    if (wave < NT && row < n_rows) {
      if (gq == 0) rs.ssq[(size_t)row * rs.ld_ssq + bx] = ss;
      if (bx == 0 && gq < rs.ld_ssq - g.groups) rs.ssq[(size_t)row * rs.ld_ssq + g.groups + gq] = 0.f; // sums of no group
    }
    return;
  }

#pragma unroll
  for (int i = 0; i < UPW; ++i) {
    const int id = wave * UPW + i;
    if (id >= U) continue;
    const int u = id / NT, t = id - u * NT;
    if (u >= n_valid) continue;
    const int row = 16 * t + r;
    const float sc_row = SCALED ? ssq_lds[t * 16 * g.n_ssq + r] : 1.0f;
    const int o = (tile0 + u) * 16 + 4 * gq;
    if (MODE != GEMM_SWIGLU) {
      if (row >= n_rows) continue;
      const f32x4 v = f32x4{fin[i][0][0] * sc_row, fin[i][0][1] * sc_row, fin[i][0][2] * sc_row, fin[i][0][3] * sc_row};
      if (MODE == GEMM_STORE) {
        *reinterpret_cast<float4 *>(y + (size_t)row * ldy + o) = float4{v[0], v[1], v[2], v[3]};
      } else {
        // fused Q/K/V epilogue: features o .. o+3 of the concatenated [q | k | v] outputs, in the
        // interleaved order of the packed wq / wk rows: (o, o+1) and (o+2, o+3) are rotation pairs
        const int hd = rp.hd, head = o / hd, dd = o - head * hd;
        const int pos = L + row;
        float a0 = v[0], b0 = v[1], a1 = v[2], b1 = v[3];
        if (head < rp.H + rp.Hkv) {
          const float c0 = rope_c[i][0], c1 = rope_c[i][1], s0 = rope_s[i][0], s1 = rope_s[i][1];
          a0 = v[0] * c0 - v[1] * s0; b0 = v[1] * c0 + v[0] * s0;
          a1 = v[2] * c1 - v[3] * s1; b1 = v[3] * c1 + v[2] * s1;
        }
        const bf16_t e0 = f32_to_bf16(a0), e1 = f32_to_bf16(b0), e2 = f32_to_bf16(a1), e3 = f32_to_bf16(b1);
        if (head < rp.H + rp.Hkv) {
          bf16_t *dst;
          if (head < rp.H) dst = rp.q + ((size_t)row * rp.H + head) * hd + dd;
          else if (rp.tiled) dst = rp.k_layer + (size_t)(head - rp.H) * rp.cap * hd + kv_k_index(pos, dd);
          else dst = rp.k_layer + ((size_t)(head - rp.H) * rp.cap + pos) * hd + dd;
          *reinterpret_cast<ushort4 *>(dst) = ushort4{e0, e1, e2, e3};
        } else {
          bf16_t *dst = rp.v_layer + (size_t)(head - rp.H - rp.Hkv) * hd * rp.cap;
          if (rp.tiled) {
            dst[kv_v_index(pos, dd)] = e0; dst[kv_v_index(pos, dd + 1)] = e1;
            dst[kv_v_index(pos, dd + 2)] = e2; dst[kv_v_index(pos, dd + 3)] = e3;
          } else {
            dst[(size_t)dd * rp.cap + pos] = e0; dst[(size_t)(dd + 1) * rp.cap + pos] = e1;
            dst[(size_t)(dd + 2) * rp.cap + pos] = e2; dst[(size_t)(dd + 3) * rp.cap + pos] = e3;
          }
        }
      }
    } else {
      // h[row, o .. o+3] = bf16(silu(gate) * up), written in fragment order over (k = o, NT row tiles);
      // rows past n are written as zeros so the consumer's operand tiles are fully defined
      const bool live = row < n_rows;
      const f32x4 gt = f32x4{fin[i][0][0] * sc_row, fin[i][0][1] * sc_row, fin[i][0][2] * sc_row, fin[i][0][3] * sc_row};
      const f32x4 up = f32x4{fin[i][TPU - 1][0] * sc_row, fin[i][TPU - 1][1] * sc_row, fin[i][TPU - 1][2] * sc_row, fin[i][TPU - 1][3] * sc_row};
      const u32x2s hv = u32x2s{live ? bf16_pair(silu(gt[0]) * up[0], silu(gt[1]) * up[1]) : 0u,
                               live ? bf16_pair(silu(gt[2]) * up[2], silu(gt[3]) * up[3]) : 0u};
      const size_t slot = ((size_t)(o >> 5) * NT + t) * 64 + r + 16 * ((o & 31) >> 3);
      __builtin_nontemporal_store(hv, reinterpret_cast<u32x2s *>(h_frag + slot * 8 + (o & 7)));
    }
  }
}

bool gemm_mfma_supported(int32_t n, int32_t K, int32_t O) {
  return n >= 1 && n <= TR_MAX_NODES && K % 32 == 0 && O % 32 == 0;
}

// Kernel variants: (P out-tiles per workgroup, waves).  Accumulators take 4*P*NT registers (twice that
// for SWIGLU pairs), so the larger ones exist only for few row tiles; 8 weight tiles need the four-wave
// form, whose accumulators live in the upper half of the unified register file.
static bool variant_ok(int NT, int p, bool swiglu) {
  const int wt = swiglu ? 2 * p : p;
  if (wt == 8) return NT == 4 || NT == 5;
  if (wt == 6) return true; // eight waves up to 5 row tiles, the four-wave form beyond
  if (wt == 5) return !swiglu && NT <= 5;
  if (swiglu) return wt == 2 || wt == 4;
  return wt >= 1 && wt <= 4;
}

// Pick (P, workgroups per K-split, K-splits).  About max(ceil(T/P), min(T, 256/S)) workgroups share the T
// out-tiles evenly.  The estimate is the slowest workgroup's time in each round of 256 workgroups: the
// KiB it pulls through L2 (its weight tiles once, the activation block of its K-range once) at the
// per-CU rate, or the round's weight stream at the HBM rate if that is slower, plus a fixed cost per
// round and what the consumer pays to re-read K-split partial sums.  Rates in KiB/us, fitted to
// measurements on MI355X.
void gemm_choose(int32_t n, int32_t K, int32_t total_tiles, bool swiglu, int32_t max_splits, bool feeds_x, int32_t *out_p,
                 int32_t *out_groups, int32_t *out_splits) {
  const int NT = (n + 15) / 16, KT = K / 32;
  const double wmul = swiglu ? 2.0 : 1.0;
  static const int cand[] = {1, 2, 3, 4, 5, 6, 8};
  double best = 1e30;
  int bp = swiglu ? 1 : 1, bg = total_tiles, bs = 1;
  for (int ci = 0; ci < 7; ++ci) {
    const int p = cand[ci];
    if (!variant_ok(NT, p, swiglu)) continue;
    for (int s = 1; s <= max_splits; s *= 2) {
      if (KT / s < GEMM_WAVES) break;
      int groups = 256 / s < total_tiles ? 256 / s : total_tiles;
      if (groups * p < total_tiles) groups = (total_tiles + p - 1) / p;
      const int tpw = (total_tiles + groups - 1) / groups;
      groups = (total_tiles + tpw - 1) / tpw; // fewest workgroups with the same largest share
      const int rounds = (groups * s + 255) / 256;
      const double kts = (double)((KT + s - 1) / s);
      const double l2_kib = kts * (tpw * wmul + NT);
      const double hbm_kib = kts * tpw * wmul * (groups * s < 256 ? groups * s : 256);
      double t = l2_kib / 48.0;
      if (hbm_kib / 6000.0 > t) t = hbm_kib / 6000.0;
      t = rounds * (t + 3.0) + 3.0;
      if (s > 1) t += 2.0 * (s - 1) * NT * total_tiles / 8000.0 + 0.5; // extra KiB of partials written and re-read
      // What a whole projection that updates the residual stream saves against another plan and k_add_frag.  us a step, the plan without / with it:
      //   two out-tiles a workgroup (6432 .. 7744 outputs, o of 17 to 32 rows): six layers of 6656, 17, 20, 32 nodes 1334 / 1379, 1346 / 1384, 1359 / 1366
      //   one, up to 16 rows: 12 layers of 3328, 3456, 3712, 16 nodes 912 / 907, 910 / 892, 1023 / 958; but with 2.5 us instead of 1.5 3200 too, 862 / 867 with one
      //     node, and down from 18944 features to 3584 (10 layers), 1 and 15 nodes 1087 / 1092, 1106 / 1117
      //   one, 17 to 32 rows (o): 10 layers of 4096, 17, 24, 32 nodes 1221 / 1199, 1196 / 1178, 1234 / 1213; 12 of 3840 1095 / 1079, 1104 / 1082, 1110 / 1080; but
      //     fewer workgroups, or waves with unequal numbers of k-steps: 3328 958 / 967, 963 / 975, 973 / 986, 3968 1150 / 1158, 1157 / 1167, 1163 / 1176
      if (feeds_x && tpw == 1 && gemm_updates_residual(n, groups, s)) t -= NT == 1 ? 1.5 : (groups >= 240 && KT % GEMM_WAVES == 0 ? 2.5 : 0.0);
      if (t < best) {
        best = t;
        bp = p;
        bg = groups;
        bs = s;
      }
    }
  }
  *out_p = bp;
  *out_groups = bg;
  *out_splits = bs;
}

template <int NT, int P, int MODE, int GW, bool SCALED>
static hipError_t launch_ks(const GemmArgs &g, hipStream_t st, KernelTimer tm) {
  constexpr int NW = MODE == GEMM_SWIGLU ? 2 * P : P;
  const size_t smem = gemm_tail_red_bytes(P, NT, MODE, GW, SCALED) + (SCALED ? (size_t)NT * 16 * g.n_ssq * sizeof(float) : 0);
  if (smem > 65536) {
    static bool once = [] {
      return hipFuncSetAttribute(reinterpret_cast<const void *>(&k_gemm_mfma<NT, NW, MODE, GW, SCALED>),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) == hipSuccess;
    }();
    if (!once) return hipErrorInvalidValue;
  }
  const int32_t end0 = g.seg[0].out_tiles, split_kt = (g.K / 32 + g.splits - 1) / g.splits;
  return launch(k_gemm_mfma<NT, NW, MODE, GW, SCALED>, dim3(g.groups, g.splits), dim3(GW * 64), smem, st, tm, g.seg[0].w,
                MODE == GEMM_SWIGLU ? g.w2 : g.seg[1].w, g.a_frag, g.seg[2].w, g.K / 32, g.part_q, g.part_rem, split_kt, end0,
                end0 + g.seg[1].out_tiles, g);
}
// the epilogue's RMS scale is a compile-time property: without it the tail needs no scale hand-out and
// the whole of LDS can hold partial tiles
template <int NT, int P, int MODE, int GW = GEMM_WAVES>
static hipError_t launch_k(const GemmArgs &g, hipStream_t st, KernelTimer tm) {
  if (MODE == GEMM_STORE && g.rope.q != nullptr) { // the fused Q/K/V projection: complete sums of a normalised input
    if (g.row_ssq == nullptr || g.splits != 1 || g.n_seg != 3) return hipErrorInvalidValue;
    return launch_ks<NT, P, GEMM_ROPE, GW, true>(g, st, tm);
  }
  if (g.n_seg != 1) return hipErrorInvalidValue;
  if (g.resid.x != nullptr) {
    if constexpr (MODE == GEMM_STORE && NT <= GEMM_RESID_ROW_TILES) {
      if (g.row_ssq == nullptr && g.splits == 1) return launch_ks<NT, P, GEMM_RESID, GW, false>(g, st, tm);
    }
    return hipErrorInvalidValue;
  }
  if (g.row_ssq != nullptr) return launch_ks<NT, P, MODE, GW, true>(g, st, tm);
  return launch_ks<NT, P, MODE, GW, false>(g, st, tm);
}

template <int NT>
static hipError_t launch_nt(const GemmArgs &g, hipStream_t st, KernelTimer tm) {
  const int p = g.tiles_per_wg;
  const bool swiglu = g.mode == GEMM_SWIGLU;
  if (!variant_ok(NT, p, swiglu) || g.groups < 1 || g.groups > g.total_tiles ||
      (int64_t)g.groups * p < g.total_tiles)
    return hipErrorInvalidValue;
  if (swiglu) {
    if constexpr (NT == 4 || NT == 5) {
      if (p == 4) return launch_k<NT, 4, GEMM_SWIGLU, 4>(g, st, tm);
    }
    if constexpr (NT <= 5) {
      if (p == 3) return launch_k<NT, 3, GEMM_SWIGLU>(g, st, tm);
    } else {
      if (p == 3) return launch_k<NT, 3, GEMM_SWIGLU, 4>(g, st, tm);
    }
    if (p == 2) return launch_k<NT, 2, GEMM_SWIGLU>(g, st, tm);
    if (p == 1) return launch_k<NT, 1, GEMM_SWIGLU>(g, st, tm);
    return hipErrorInvalidValue;
  }
  if constexpr (NT == 4 || NT == 5) {
    if (p == 8) return launch_k<NT, 8, GEMM_STORE, 4>(g, st, tm);
  }
  if constexpr (NT <= 5) {
    if (p == 6) return launch_k<NT, 6, GEMM_STORE>(g, st, tm);
  } else {
    if (p == 6) return launch_k<NT, 6, GEMM_STORE, 4>(g, st, tm);
  }
  if constexpr (NT <= 5) {
    if (p == 5) return launch_k<NT, 5, GEMM_STORE>(g, st, tm);
  }
  switch (p) {
  case 1: return launch_k<NT, 1, GEMM_STORE>(g, st, tm);
  case 2: return launch_k<NT, 2, GEMM_STORE>(g, st, tm);
  case 3: return launch_k<NT, 3, GEMM_STORE>(g, st, tm);
  case 4: return launch_k<NT, 4, GEMM_STORE>(g, st, tm);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_gemm_mfma(const GemmArgs &args, hipStream_t st, KernelTimer tm) {
  if (args.groups < 1 || args.total_tiles < 1) return hipErrorInvalidValue;
  GemmArgs g = args;
  g.part_q = g.total_tiles / g.groups;
  g.part_rem = g.total_tiles % g.groups;
  if (g.row_ssq != nullptr && (g.n_ssq > gemm_most_ssq((g.n + 15) / 16) || g.n_ssq % 4 != 0 || !starts_on_16(g.row_ssq)))
    return hipErrorInvalidValue;
  switch ((g.n + 15) / 16) {
  case 1: return launch_nt<1>(g, st, tm);
  case 2: return launch_nt<2>(g, st, tm);
  case 3: return launch_nt<3>(g, st, tm);
  case 4: return launch_nt<4>(g, st, tm);
  case 5: return launch_nt<5>(g, st, tm);
  case 6: return launch_nt<6>(g, st, tm);
  case 7: return launch_nt<7>(g, st, tm);
  case 8: return launch_nt<8>(g, st, tm);
  }
  return hipErrorInvalidValue;
}

} // namespace tr
