// Tree attention for few query rows per K/V head (up to 64 nodes and 128 pairs of node and query head): every K/V byte is read once.
//
// The queries that share a K/V head are the rows of one operand, row = node * group + head of the group, so that a group's
// heads share each K/V tile in a workgroup's LDS instead of re-reading it from L2 one workgroup after another.  A workgroup
// owns one K/V head and one of nsplit shares of the keys; its waves form a grid of RW tiles of 32 rows x KS key groups.  A
// key group takes a 32-key tile per step (16 KiB, loaded straight from memory into a ring of D slots, D - 1 under way) and
// its RW waves multiply it (v_mfma_f32_32x32x16_bf16, operands and lanes as in tr_attn_causal.hip); with one row tile a
// wave's ring is its own and the loop has no barrier.  At the end the key groups meet in LDS, and the workgroup writes the
// result (one share) or (maximum, sum, normalised output in half precision) for k_attn_merge.
#include "tr_kernels.h"

namespace tr {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(4))) _Float16 f16x4;

__device__ inline f32x16 mfma32r(const u32x4 &a, const u32x4 &b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

constexpr int ROWS_NODES = NP / 2; // most nodes: half as many as the partial buffers are made for, in twice the shares

constexpr size_t rows_lds_bytes(int rw, int ks, int d) { // the rings; at the end the accumulators and (maximum, sum)
  const size_t ring = (size_t)ks * d * 16384, meet = (size_t)ks * rw * 32 * (512 + 8);
  return ring > meet ? ring : meet;
}

template <int RW, int KS, int D>
__global__ __launch_bounds__(RW * KS * 64) void k_attn_rows(const bf16_t *__restrict__ q, const bf16_t *__restrict__ Kl,
                                                            const bf16_t *__restrict__ Vl, int32_t H, int32_t Hkv,
                                                            int32_t cap, int32_t n, const uint64_t *__restrict__ anc,
                                                            const int32_t *__restrict__ d_len, int32_t nsplit,
                                                            float *__restrict__ part_ml, float *__restrict__ part_acc,
                                                            bf16_t *__restrict__ out, int32_t out_row_tiles) {
  constexpr int LOADS = (16 + RW - 1) / RW; // tile loads of a wave per step
  extern __shared__ u32x4 lds[];            // [KS][D][K 8 tiles | V 8 tiles][64]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rw = wave % RW, ks = wave / RW;
  const int half_sel = (lane >> 4) & 1, hb = lane >> 5;
  const int hk = blockIdx.x, split = blockIdx.y, G = H / Hkv, R = n * G;
  const int row = rw * 32 + (lane & 31), rc = row < R ? row : R - 1;
  const int node = rc / G, h = hk * G + (rc - node * G);

  const uint64_t kbase = reinterpret_cast<uint64_t>(Kl + (size_t)hk * cap * 128);
  const uint64_t vbase = reinterpret_cast<uint64_t>(Vl + (size_t)hk * cap * 128);
  const uint32_t ring0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)lds + ks * (D * 16384);
  const uint32_t voff = lane * 16;
  auto tile_of = [&](int step) { return (step * nsplit + split) * KS + ks; };
  auto load_step = [&](int slot, int t) { // 32-key tile t into ring slot `slot`
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      int j = rw + RW * i;
      j = j < 16 ? j : 15; // three waves: two of the 18 loads repeat the last tile
      tile_to_lds(ring0 + slot * 16384 + j * 1024, voff, (j < 8 ? kbase : vbase) + ((uint64_t)t * 8 + (j & 7)) * 1024);
    }
  };
  // the first tiles are asked for before the committed length is known: inside the cache even if beyond the sequence
  const int cap_tiles = cap / 32;
#pragma unroll
  for (int s = 0; s < D - 1; ++s) {
    const int t = tile_of(s);
    load_step(s, t < cap_tiles ? t : cap_tiles - 1);
  }
  // Q^T operand: contraction step c, half s: Q[row][32 c + 16 s + 8 hb .. + 7]; rows past the last repeat it
  u32x4 qf[4][2];
  {
    const u32x4 *qp = reinterpret_cast<const u32x4 *>(q + ((size_t)node * H + h) * 128 + 8 * hb);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      qf[c][0] = qp[c * 4];
      qf[c][1] = qp[c * 4 + 2];
    }
  }
  const uint64_t a0 = anc[2 * node], a1 = anc[2 * node + 1];
  const int L = *d_len, total = L + n, n_tiles = (total + 31) >> 5;

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

  int slot = 0;
  for (int step = 0; (step * nsplit + split) * KS < n_tiles; ++step) { // uniform over the workgroup
    wait_tiles<(D - 2) * LOADS>();
    if (RW > 1) meet_waves(); // this step's tiles are there for the group, and it has read the slot that is refilled next
    {
      int t = tile_of(step + D - 1);
      t = t < n_tiles ? t : n_tiles - 1; // past the end: again the last one, so that the counts under way stay constant
      load_step(slot == 0 ? D - 1 : slot - 1, t);
    }
    const u32x4 *kt = lds + (ks * D + slot) * 1024, *vt = kt + 512;
    slot = slot + 1 < D ? slot + 1 : 0;
    const int key0 = tile_of(step) * 32;
    if (key0 >= total) continue; // uniform over the wave

    f32x16 s, s2; // two chains of four products
#pragma unroll
    for (int e = 0; e < 16; ++e) s[e] = s2[e] = 0.f;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      s = mfma32r(kt[c * 64 + kfrag], qf[c][0], s);
      s2 = mfma32r(kt[c * 64 + kfrag + 32], qf[c][1], s2);
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) s[e] += s2[e];
    if (key0 + 32 > L) { // some keys are tree nodes, or past the last
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int p = key0 + 8 * (e >> 2) + 4 * hb + (e & 3), j = p - L;
        const bool vis = j < 0 || (j < n && (((j < 64 ? a0 >> j : a1 >> (j - 64)) & 1ull) != 0));
        s[e] = vis ? s[e] : -INFINITY;
      }
    }
    float mx = s[0];
#pragma unroll
    for (int e = 1; e < 16; ++e) mx = fmaxf(mx, s[e]);
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
    // m is finite, so an invisible key's probability is exactly 0, also in a row that has seen no key of this wave's yet
    u32x4 pf[2];
#pragma unroll
    for (int e = 0; e < 16; e += 2) {
      const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], sc, -m));
      const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e + 1], sc, -m));
      const bf16x2 p = __builtin_convertvector(f32x2{p0, p1}, bf16x2);
      l = __builtin_amdgcn_fdot2_f32_bf16(p, ones, l, false); // the sum of the rounded probabilities
      pf[(e >> 2) & 1][(e >> 3) * 2 + ((e & 3) >> 1)] = __builtin_bit_cast(uint32_t, p);
    }
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
      for (int d = 0; d < 4; ++d) acc[d] = mfma32r(vt[d * 128 + frag + 32 * hh], pf[hh], acc[d]);
  }
  l += __shfl_xor(l, 32);

  // the key groups meet: accumulators as rows of 32 chunks of 4 features, chunk c of a row in place c ^ (row % 32) so that
  // the 32 rows a wave stores at once hit distinct banks
  wait_tiles<0>(); // the repeated loads past the end have landed
  __syncthreads(); // and everyone has read the last tiles
  f32x4 *xa = reinterpret_cast<f32x4 *>(lds);                        // [KS][RW * 32][32]
  float2 *xm = reinterpret_cast<float2 *>(xa + KS * RW * 32 * 32);   // [KS][RW * 32]
#pragma unroll
  for (int d = 0; d < 4; ++d)
#pragma unroll
    for (int qd = 0; qd < 4; ++qd)
      xa[(ks * RW * 32 + row) * 32 + ((8 * d + 2 * qd + hb) ^ (row & 31))] =
          f32x4{acc[d][4 * qd], acc[d][4 * qd + 1], acc[d][4 * qd + 2], acc[d][4 * qd + 3]};
  if (hb == 0) xm[ks * RW * 32 + row] = float2{m, l};
  __syncthreads();
  for (int i = tid; i < R * 32; i += RW * KS * 64) {
    const int r = i >> 5, c = i & 31;
    float top = -1e30f, den = 0.f;
#pragma unroll
    for (int k = 0; k < KS; ++k) top = fmaxf(top, xm[k * RW * 32 + r].x);
    f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      const float2 ml = xm[k * RW * 32 + r];
      const float w = __builtin_amdgcn_exp2f(ml.x - top);
      den += ml.y * w;
      v += xa[(k * RW * 32 + r) * 32 + (c ^ (r & 31))] * w;
    }
    v *= nsplit == 1 || den > 0.f ? 1.0f / den : 0.f; // a share may have seen no key of the row, the whole sequence not
    const int nd = r / G, hh = hk * G + (r - nd * G);
    if (nsplit == 1) {
      const ushort4 o = ushort4{f32_to_bf16(v[0]), f32_to_bf16(v[1]), f32_to_bf16(v[2]), f32_to_bf16(v[3])};
      const size_t idx = out_row_tiles > 0 ? act_frag_index(nd, hh * 128 + 4 * c, out_row_tiles) : ((size_t)nd * H + hh) * 128 + 4 * c;
      store_stream(out + idx, o);
    } else {
      const size_t prow = ((size_t)split * H + hh) * ROWS_NODES + nd;
      if (c == 0) *reinterpret_cast<float2 *>(part_ml + prow * 2) = float2{top, den};
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = fminf(fmaxf(v[e], -65504.0f), 65504.0f); // saturate, as in k_attn_mfma
      reinterpret_cast<f16x4 *>(part_acc)[prow * 32 + c] = __builtin_convertvector(v, f16x4);
    }
  }
}

template <int RW, int KS, int D>
static hipError_t launch_grid(const bf16_t *q, const bf16_t *Kl, const bf16_t *Vl, int32_t H, int32_t Hkv, int32_t cap,
                              int32_t n, const uint64_t *anc, const int32_t *d_len, int32_t nsplit, float *part_ml,
                              float *part_acc, bf16_t *out, int32_t out_row_tiles, hipStream_t st, KernelTimer tm) {
  constexpr int smem = (int)rows_lds_bytes(RW, KS, D);
  static bool once = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_attn_rows<RW, KS, D>),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, smem) == hipSuccess;
  if (!once) return hipErrorInvalidValue;
  return launch(k_attn_rows<RW, KS, D>, dim3(Hkv, nsplit), dim3(RW * KS * 64), smem, st, tm, q, Kl, Vl, H, Hkv, cap, n, anc,
                d_len, nsplit, part_ml, part_acc, out, out_row_tiles);
}

static int key_groups(int rows) { return rows <= 64 ? 4 : 2; }

// Where this form is the faster one.  Measured: 25 head layouts (8 to 128 heads, groups of 1 to 32), 1 to 128 rows per K/V
// head, 20 to 16000 positions, 4040 points; the rule leaves one of them more than 1.5 % slower than the split form (1.8).
//   One share (up to 768 positions, where the split form has not taken over as one launch): a step costs 1.3 us and 32
//   rows 2 us more than 8, against the split form's merge launch.  64 heads on 8, 1 / 4 nodes, split form / this: 4.4 /
//   5.2 and 4.5 / 6.8 at 20 positions, 7.3 / 5.4 and 7.5 / 7.0 at 100, 9.3 / 10.9 and 9.4 / 12.6 at 600.
//   Several shares: both end with the merge, so what counts is the split form's chain, the 32-key tiles a workgroup of it
//   takes one after another (1.0 us each, 1.25 if one wave stages them), against this form's 2 us for every 32 rows.  64
//   on 8: 1 node 10.3 / 9.0 at 840 positions and 69 / 22 at 16000, 4 nodes 10.4 / 10.5 at 840 (4 tiles) and 11.5 / 10.9 at
//   1100 (5), 8 nodes 12.7 / 13.0 at 1420 (6) and 14.8 / 13.9 at 2000 (8), 16 nodes 20.6 / 20.7 at 3090 (13) and 23.6 /
//   20.6 at 4000 (16); 32 on 8: 8 nodes 10.6 / 11.7 at 1500 (3) and 16.6 / 16.2 at 4100 (9).
//   Without sharing heads (group 1) more nodes only pay where K and V come at the memory's rate: 32 on 32, 1 node 11.0 /
//   9.6 at 840, 32 nodes 11.7 / 13.1 at 1000 and 20.0 / 18.7 at 3000 (12); 64 nodes on 16 heads are slower up to 12000.
//   Groups of two share little either way: 32 on 16, 1 node 1.06 times as fast at 3100, 0.94 to 1.0 below.
bool attn_rows_better(int32_t H, int32_t Hkv, int32_t n, int32_t len_bound) {
  const int G = H / Hkv, rows = n * G;
  if (n > ROWS_NODES || rows > 128 || attn_one_launch(H, Hkv, len_bound)) return false;
  const int hpw = attn_heads_per_wg(H, Hkv, n), splits = attn_choose_splits(H / hpw, len_bound);
  const int chain = ((len_bound + 31) / 32 + splits - 1) / splits;
  const bool one_wave = hpw * ((n + 15) / 16) == 1;
  if (len_bound <= 768) {
    if (rows <= 8) return len_bound > 32 && len_bound <= (one_wave ? 416 : 256);
    return rows <= 32 && len_bound > 96 && len_bound <= (rows <= 16 || one_wave ? 256 : 224);
  }
  if (G == 2 && (rows > 32 || len_bound < 3072)) return false;
  if (rows <= 8) return true;
  if (rows <= 16) return chain >= (one_wave || G >= 8 ? 3 : 4);
  if (rows <= 32) return chain >= (one_wave ? 3 : G >= 8 ? 5 : G >= 3 ? 6 : 11);
  if (rows <= 64) return G >= 8 ? chain >= 7 : G >= 3 ? len_bound >= 5120 : len_bound >= 7168 && chain >= 24;
  return G >= 8 ? chain >= (rows <= 96 ? 12 : 14) : G >= 3 && len_bound >= 8192;
}

// Key shares: one, without a merge launch (4.8 us), up to six steps; else all compute units, at least a step each.
int attn_rows_splits(int32_t H, int32_t Hkv, int32_t n, int32_t len_bound) {
  const int steps = ((len_bound + 31) / 32 + key_groups(n * (H / Hkv)) - 1) / key_groups(n * (H / Hkv));
  if (steps <= 6) return 1;
  int s = 256 / Hkv;
  if (s > 2 * ATTN_MAX_SPLITS) s = 2 * ATTN_MAX_SPLITS; // what the partial buffers hold with ROWS_NODES nodes each
  if (s > steps) s = steps;
  return s < 1 ? 1 : s;
}

hipError_t launch_attn_rows(const bf16_t *q, const bf16_t *Kl, const bf16_t *Vl, int32_t H, int32_t Hkv, int32_t cap,
                            int32_t n, const uint64_t *anc, const int32_t *d_len, int32_t len_bound, float *part_ml,
                            float *part_acc, bf16_t *out, int32_t out_row_tiles, Profiler *prof, hipStream_t st) {
  if (Hkv < 1 || H % Hkv != 0 || n < 1 || n > ROWS_NODES || n * (H / Hkv) > 128) return hipErrorInvalidValue;
  const int rows = n * (H / Hkv), nsplit = attn_rows_splits(H, Hkv, n, len_bound);
  const KernelTimer tm = prof_next(prof, PC_ATTN);
  hipError_t e;
  if (rows <= 32)
    e = launch_grid<1, 4, 2>(q, Kl, Vl, H, Hkv, cap, n, anc, d_len, nsplit, part_ml, part_acc, out, out_row_tiles, st, tm);
  else if (rows <= 64)
    e = launch_grid<2, 4, 2>(q, Kl, Vl, H, Hkv, cap, n, anc, d_len, nsplit, part_ml, part_acc, out, out_row_tiles, st, tm);
  else if (rows <= 96)
    e = launch_grid<3, 2, 4>(q, Kl, Vl, H, Hkv, cap, n, anc, d_len, nsplit, part_ml, part_acc, out, out_row_tiles, st, tm);
  else
    e = launch_grid<4, 2, 4>(q, Kl, Vl, H, Hkv, cap, n, anc, d_len, nsplit, part_ml, part_acc, out, out_row_tiles, st, tm);
  if (e != hipSuccess || nsplit == 1) return e;
  return launch_attn_merge(part_ml, part_acc, ROWS_NODES, H, n, nsplit, out, out_row_tiles, prof_next(prof, PC_ATTN_MERGE), st);
}

} // namespace tr
