// Causal attention of a prompt-ingestion pass: row r (cache position L + r) sees the positions 0 .. L + r.  head_dim 128,
// bf16 Q/K/V, float32 softmax statistics and accumulators, the cache in the tiled layout (kv_k_index / kv_v_index).
//
// One launch covers all rows and heads.  A workgroup owns 128 rows of HPW query heads that share a K/V head, a wave 32
// rows of one of them and every KS-th block of 64 keys; K and V pass through LDS KS * 64 keys at a time, loaded straight
// from memory (every 1 KiB tile is contiguous on both sides) into one of two buffers while the other is in use: one
// barrier per step.  What bounds it is the chain of a step (scores, maximum, exponentials, values: about 2700 clocks, the
// matrix pipe a third of them), so the shapes keep two waves on every SIMD: two heads of a group (which also share the
// tiles), or, when the launch has at most one workgroup per compute unit, two waves that split the keys of the same
// rows and meet in LDS at the end.
// Measured: per layer of 70B width, passes of 2048 rows behind 0 and 2048 positions, 153 us on average; 274 with 16
// rows per wave on the 16x16x32 form in the same passes; 8 launches of the decode kernel and its merge per 512 rows
// took 843 us per layer for the same 4095 rows, now 306.  7B width, 511 rows: 15.5 us against 27.4
// (19.5 with one wave per 32 rows).
//
// Everything is
// computed transposed on v_mfma_f32_32x32x16_bf16, so that no value changes lanes between the two contractions:
//   S^T[32 keys][32 rows] = K . Q^T: lane l ends with keys 8 q + 4 (l / 32) .. + 3 (q = 0 .. 3) of row l % 32
//   O^T[d][row] += V^T . P^T: of a 32-key tile, contraction half h takes the keys whose V elements sit in lane slots
//                  16 (2 h + l / 32) ..: positions 8 h + 4 (l / 32) .. + 3 and 16 more, i.e. the lane's own q = h, h + 2
// and an operand is rebuilt from the cache's 16 x 32 tiles by addressing alone, as in the projection kernel.
#include "tr_kernels.h"

namespace tr {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

__device__ inline f32x16 mfma32c(const u32x4 &a, const u32x4 &b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

constexpr int CAUSAL_ROWS = 128; // rows of a workgroup
constexpr int CAUSAL_KEYS = 64;  // keys per step: 16 KiB of K, 16 KiB of V

template <int HPW, int KS>
__global__ __launch_bounds__(HPW * KS * 256) void k_attn_causal(const bf16_t *__restrict__ q, const bf16_t *__restrict__ Kl,
                                                           const bf16_t *__restrict__ Vl, int32_t H, int32_t Hkv, int32_t cap,
                                                           int32_t n, const int32_t *__restrict__ d_len,
                                                           bf16_t *__restrict__ out, int32_t out_row_tiles) {
  constexpr int WAVES = HPW * KS * 4, LOADS = KS * 32 / WAVES;
  extern __shared__ u32x4 buf[]; // [2][KS][K 16 tiles | V 16 tiles][64]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half_sel = (lane >> 4) & 1, hb = lane >> 5;
  const int hk = blockIdx.x, h = hk * (H / Hkv) + blockIdx.y * HPW + wave / 4 % HPW;
  const int ks = wave / 4 / HPW;
  // the row blocks with the longest prefix come first: what is left for the launch's end is short
  const int block0 = (gridDim.z - 1 - blockIdx.z) * CAUSAL_ROWS;
  const int wrow0 = block0 + (wave & 3) * 32, row = wrow0 + (lane & 31);
  const int last_row = block0 + CAUSAL_ROWS < n ? block0 + CAUSAL_ROWS - 1 : n - 1;

  // Q^T operand: contraction step c, half s: Q[row][32 c + 16 s + 8 hb .. + 7]; rows past n repeat the last one
  u32x4 qf[4][2];
  {
    const u32x4 *qp = reinterpret_cast<const u32x4 *>(q + ((size_t)(row < n ? row : n - 1) * H + h) * 128 + 8 * hb);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      qf[c][0] = qp[c * 4];
      qf[c][1] = qp[c * 4 + 2];
    }
  }
  const int L = *d_len;
  const int n_tiles = (L + last_row) / 32 + 1, n_steps = (n_tiles + 2 * KS - 1) / (2 * KS); // 32-key tiles and steps this block needs

  // tile j of a step: of each 32, 0 .. 15 are K (8 per 32-key tile), 16 .. 31 V.  The end of the last step may lie past
  // the sequence: it loads the last tile again, and its keys are masked by their nominal position.
  const uint64_t kbase = reinterpret_cast<uint64_t>(Kl + (size_t)hk * cap * 128);
  const uint64_t vbase = reinterpret_cast<uint64_t>(Vl + (size_t)hk * cap * 128);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)buf;
  const uint32_t voff = lane * 16;
  auto load_step = [&](int step, int b) {
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int j = wave + WAVES * i;
      int t = 2 * (step * KS + (j >> 5)) + ((j >> 3) & 1);
      t = t < n_tiles ? t : n_tiles - 1;
      tile_to_lds(lds0 + b * (KS * 32768) + j * 1024, voff, ((j & 31) < 16 ? kbase : vbase) + ((uint64_t)t * 8 + (j & 7)) * 1024);
    }
  };

  f32x16 acc[4];
#pragma unroll
  for (int d = 0; d < 4; ++d)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[d][e] = 0.f;
  float m = -1e30f, l = 0.f; // running maximum of the row (base 2), this lane's share of its sum
  const float sc = 0.08838834764831845f * 1.4426950408889634f; // 1/sqrt(128) * log2(e)
  const int frag = half_sel * 64 + (lane & 15) + 16 * hb;      // a pair of neighbouring tiles; + 32 for the second half
  const int kfrag = half_sel * 256 + (lane & 15) + 16 * hb;    // K: the pair is 4 tiles apart
  const bf16x2 ones = __builtin_bit_cast(bf16x2, 0x3F803F80u);

  load_step(0, 0);
  for (int step = 0; step < n_steps; ++step) {
    const int b = step & 1;
    wait_tiles<0>();
    meet_waves(); // this step's tiles are there for everyone, and everyone has read the other buffer
    if (step + 1 < n_steps) load_step(step + 1, b ^ 1);
    const int key0 = (step * KS + ks) * CAUSAL_KEYS;
    if (key0 > L + wrow0 + 31) continue; // uniform over the wave: all its rows lie before these keys
    const u32x4 *kt = buf + (b * KS + ks) * 2048, *vt = kt + 1024;

    f32x16 s[2];
#pragma unroll
    for (int e = 0; e < 16; ++e) s[0][e] = s[1][e] = 0.f;
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int hh = 0; hh < 2; ++hh)
#pragma unroll
        for (int u = 0; u < 2; ++u) s[u] = mfma32c(kt[u * 512 + c * 64 + kfrag + 32 * hh], qf[c][hh], s[u]);
    if (key0 + CAUSAL_KEYS - 1 > L + wrow0) { // some row of the wave does not see all of these keys
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (key0 + 32 * u + 8 * (e >> 2) + 4 * hb + (e & 3) > L + row) s[u][e] = -INFINITY;
    }
    float mx = s[0][0];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[u][e]);
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float m_new = fmaxf(m, mx * sc);
    if (__any(m_new > m)) {
      const float corr = __builtin_amdgcn_exp2f(m - m_new);
#pragma unroll
      for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[d][e] *= corr;
      l *= corr;
      m = m_new;
    }
    // m is finite, so a masked key's probability is exactly 0, also in a row that has seen no key of this wave's yet
    u32x4 pf[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int e = 0; e < 16; e += 2) {
        const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[u][e], sc, -m));
        const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[u][e + 1], sc, -m));
        const bf16x2 p = __builtin_convertvector(f32x2{p0, p1}, bf16x2);
        l = __builtin_amdgcn_fdot2_f32_bf16(p, ones, l, false); // the sum of the rounded probabilities
        pf[u][(e >> 2) & 1][(e >> 3) * 2 + ((e & 3) >> 1)] = __builtin_bit_cast(uint32_t, p);
      }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int hh = 0; hh < 2; ++hh)
#pragma unroll
        for (int d = 0; d < 4; ++d) acc[d] = mfma32c(vt[u * 512 + d * 128 + frag + 32 * hh], pf[u][hh], acc[d]);
  }
  l += __shfl_xor(l, 32);
  if constexpr (KS == 2) { // the second wave of a pair leaves (accumulator, maximum, sum) in LDS, the first combines
    f32x4 *xa = reinterpret_cast<f32x4 *>(buf) + (wave & 3) * (16 * 64) + lane;
    float2 *xm = reinterpret_cast<float2 *>(buf + 4 * 16 * 64) + (wave & 3) * 64 + lane;
    wait_tiles<0>();
    meet_waves(); // everyone has read the last buffers
    if (ks == 1) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        xa[i * 64] = f32x4{acc[i >> 2][4 * (i & 3)], acc[i >> 2][4 * (i & 3) + 1], acc[i >> 2][4 * (i & 3) + 2], acc[i >> 2][4 * (i & 3) + 3]};
      *xm = float2{m, l};
    }
    __syncthreads();
    if (ks == 1) return;
    const float2 o = *xm;
    const float top = fmaxf(m, o.x), w0 = __builtin_amdgcn_exp2f(m - top), w1 = __builtin_amdgcn_exp2f(o.x - top);
    l = l * w0 + o.y * w1;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const f32x4 v = xa[i * 64];
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i >> 2][4 * (i & 3) + e] = acc[i >> 2][4 * (i & 3) + e] * w0 + v[e] * w1;
    }
  }
  if (row >= n) return;
  const float inv = 1.0f / l;
#pragma unroll
  for (int d = 0; d < 4; ++d)
#pragma unroll
    for (int e = 0; e < 16; e += 4) {
      ushort4 o;
      o.x = f32_to_bf16(acc[d][e] * inv); o.y = f32_to_bf16(acc[d][e + 1] * inv);
      o.z = f32_to_bf16(acc[d][e + 2] * inv); o.w = f32_to_bf16(acc[d][e + 3] * inv);
      store_stream(out + act_frag_index(row, h * 128 + 32 * d + 2 * e + 4 * hb, out_row_tiles), o);
    }
}

template <int HPW, int KS>
static hipError_t launch_shape(const bf16_t *q, const bf16_t *Kl, const bf16_t *Vl, int32_t H, int32_t Hkv, int32_t cap,
                               int32_t n, const int32_t *d_len, bf16_t *out, int32_t out_row_tiles, hipStream_t st) {
  static bool once = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_attn_causal<HPW, KS>),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, KS * 65536) == hipSuccess;
  if (!once) return hipErrorInvalidValue;
  return launch(k_attn_causal<HPW, KS>, dim3(Hkv, H / Hkv / HPW, (n + CAUSAL_ROWS - 1) / CAUSAL_ROWS), dim3(HPW * KS * 256),
                KS * 65536, st, KernelTimer{}, q, Kl, Vl, H, Hkv, cap, n, d_len, out, out_row_tiles);
}

hipError_t launch_attn_causal(const bf16_t *q, const bf16_t *Kl, const bf16_t *Vl, int32_t H, int32_t Hkv, int32_t cap,
                              int32_t n, const int32_t *d_len, bf16_t *out, int32_t out_row_tiles, hipStream_t st) {
  if (Hkv < 1 || H % Hkv != 0 || n < 1) return hipErrorInvalidValue;
  const int blocks = (n + CAUSAL_ROWS - 1) / CAUSAL_ROWS;
  if (H * blocks <= 256) return launch_shape<1, 2>(q, Kl, Vl, H, Hkv, cap, n, d_len, out, out_row_tiles, st);
  if (H / Hkv % 2 == 0) return launch_shape<2, 1>(q, Kl, Vl, H, Hkv, cap, n, d_len, out, out_row_tiles, st);
  return launch_shape<1, 1>(q, Kl, Vl, H, Hkv, cap, n, d_len, out, out_row_tiles, st);
}

} // namespace tr
