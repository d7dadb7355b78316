// Verification forward: one pass of a Llama-style decoder over the N tree nodes (Section 2.2).
// This file holds the orchestration, the embedding and residual / norm kernels and the shape-generic
// attention (any head_dim, f32 or bf16 storage, plain ALU arithmetic).  Models in the packed layout go
// through the projections in tr_gemm_mfma.hip / tr_gemm_wide.hip, all others through tr_rows.hip; a tiled
// cache through the attention in tr_attn_*.hip.
//
// Arithmetic contract of the bf16 path (both generic and packed): the residual stream, the
// softmax statistics, all accumulators and the logits are float32; operands of every contraction
// (normalised activations, rotated Q/K, V, attention output, SwiGLU output) are rounded to bf16.
// The RMS scale is applied after the contraction (it is a per-row scalar), i.e. the rounded operand
// is x * gain instead of x * gain * scale, in float32 models too.
#include "tr_internal.h"
#include "tr_kernels.h"

namespace tr {

typedef __attribute__((ext_vector_type(4))) float f32x4q;

static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

static bool packed_supported(const tr_model &m);

Workspace plan_workspace(const tr_model &m, int rows) {
  Workspace w;
  const bool generic = !packed_supported(m);
  const size_t esz = dtype_size(m.dtype);
  const size_t hq = (size_t)m.n_heads * m.head_dim;
  const size_t R = generic ? NP : rows; // rows of the activation buffers
  const size_t packed = generic ? 0 : 1; // what only the packed path uses
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += align256(bytes); return o; };
  w.x = take(R * m.d_model * 4);
  w.xn = take(packed * R * m.d_model * esz);
  w.q = take(R * hq * esz);
  w.attn = take(R * hq * esz);
  w.h = take(R * m.d_ffn * esz);
  w.rope = take(R * m.head_dim * 4);
  w.logits = take((size_t)NP * m.vocab * 4);
  w.part_ml = take((size_t)ATTN_MAX_SPLITS * NP * m.n_heads * 2 * 4);
  w.part_acc = take((size_t)ATTN_MAX_SPLITS * NP * m.n_heads * m.head_dim * 4);
  w.ypart = take(packed * WIDE_PART_ROWS * m.d_model * 4);
  static_assert(WIDE_PART_ROWS >= GEMM_MAX_SPLITS * NP && WIDE_PART_ROWS >= NPW_MOST, "ypart serves steps and passes");
  w.ssq = take(packed * R * ((m.d_model + 1023) / 1024) * 4);
  w.total = off;
  return w;
}

// ---------------------------------------------------------------------------------------------
// Rotary table of one row: cos/sin of pos * f_i with f_i = theta^(-2i/hd), evaluated in double so that long positions
// keep float32 accuracy.
// ---------------------------------------------------------------------------------------------
__device__ inline void rope_row(int pos, int32_t hd, float theta, float *__restrict__ rope_n) {
  const int half = hd / 2;
  for (int i = threadIdx.x; i < half; i += blockDim.x) {
    const double f = pow((double)theta, -2.0 * (double)i / (double)hd);
    double sn, cs;
    sincos((double)pos * f, &sn, &cs);
    rope_n[i] = (float)cs;
    rope_n[half + i] = (float)sn;
  }
}

// ---------------------------------------------------------------------------------------------
// Embedding gather + rotary table.  Row n: x[n,:] = E[tok[n],:]; cos/sin of position L + depth[n].
// depth == nullptr: row n sits n positions after L (a run of consecutive prompt tokens).
// Block (n, 0) writes row n of the table, block (n, 1 + c) columns 1024 c .. of x: the table's double-precision chain
// (2 us) and the copy run side by side.
// ---------------------------------------------------------------------------------------------
constexpr int EMBED_CHUNK = 1024;
template <typename T>
__global__ __launch_bounds__(256) void k_embed_rope(const T *__restrict__ E, int32_t V, int32_t d,
                                                    const int32_t *__restrict__ tok, const int32_t *__restrict__ depth,
                                                    const int32_t *__restrict__ d_len, int32_t hd, float theta,
                                                    float *__restrict__ x, float *__restrict__ rope) {
  const int n = blockIdx.x;
  if (blockIdx.y == 0) {
    rope_row(*d_len + (depth != nullptr ? depth[n] : n), hd, theta, rope + (size_t)n * hd);
    return;
  }
  int t = tok[n];
  t = t < 0 ? 0 : (t >= V ? V - 1 : t);
  const int j = (blockIdx.y - 1) * EMBED_CHUNK + threadIdx.x * 4; // d is a multiple of 4
  if (j >= d) return;
  T v[4];
  __builtin_memcpy(v, E + (size_t)t * d + j, 4 * sizeof(T));
  *reinterpret_cast<float4 *>(x + (size_t)n * d + j) =
      float4{to_f32<T>(v[0]), to_f32<T>(v[1]), to_f32<T>(v[2]), to_f32<T>(v[3])};
}

// ---------------------------------------------------------------------------------------------
// Generic tree attention (Section 2.2 "Tree Attention"), plain cache layout: block (node n, head h).  Keys are the
// committed positions 0..L-1 and the tree nodes j whose bit is set in anc[n] (cache position L+j);
// everything else is skipped exactly.  Online softmax over chunks of 256 keys: a thread scores one key (its row of K
// in 16-byte loads), then the value contraction splits the chunk's keys over 256 / hd groups of hd threads (one
// feature each, V is position-contiguous) that meet in LDS once at the end.  With one group, hd of the 256 threads
// walked all keys one by one and the launch took 15.5 us on the tiny model's 100 to 150 positions.
// ---------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void k_attn_generic(const T *__restrict__ q, const T *__restrict__ Kl,
                                                      const T *__restrict__ Vl, int32_t H, int32_t Hkv, int32_t hd,
                                                      int32_t cap, int32_t n_nodes, const uint64_t *__restrict__ anc,
                                                      const int32_t *__restrict__ d_len, T *__restrict__ out,
                                                      int32_t out_row_tiles) {
  constexpr int E = 16 / (int)sizeof(T);
  __shared__ float sq[256];
  __shared__ __align__(16) float sp[256];
  __shared__ float red[4], red2[4];
  const int n = blockIdx.x, h = blockIdx.y, tid = threadIdx.x;
  const int hk = h / (H / Hkv);
  const int L = *d_len;
  const uint64_t a0 = anc[2 * n], a1 = anc[2 * n + 1];
  const T *Kh = Kl + (size_t)hk * cap * hd;
  const T *Vh = Vl + (size_t)hk * hd * cap;
  if (tid < hd) sq[tid] = to_f32<T>(q[((size_t)n * H + h) * hd + tid]);
  __syncthreads();
  const float scale = 1.0f / sqrtf((float)hd);
  const int groups = 256 / hd, grp = tid / hd, dd = tid - grp * hd; // threads past groups * hd hold no feature
  const int span = ((256 + groups - 1) / groups + 3) & ~3;          // keys of a chunk per group
  float m = -1e30f, l = 0.f, acc = 0.f; // acc: feature dd, keys of this thread's group
  const int total = L + n_nodes;
  for (int base = 0; base < total; base += 256) {
    const int j = base + tid;
    bool vis = j < L;
    if (!vis && j < total) {
      const int t = j - L;
      vis = t < 64 ? ((a0 >> t) & 1) : ((a1 >> (t - 64)) & 1);
    }
    float s = -1e30f;
    if (vis) {
      const T *kr = Kh + (size_t)j * hd;
      float dot = 0.f;
      int e = 0;
      for (; e + E <= hd; e += E) {
        T kv[E];
        __builtin_memcpy(kv, kr + e, 16);
#pragma unroll
        for (int i = 0; i < E; ++i) dot += sq[e + i] * to_f32<T>(kv[i]);
      }
      for (; e < hd; ++e) dot += sq[e] * to_f32<T>(kr[e]);
      s = dot * scale;
    }
    float cm = s;
    for (int off = 32; off > 0; off >>= 1) cm = fmaxf(cm, __shfl_xor(cm, off));
    if ((tid & 63) == 0) red[tid >> 6] = cm;
    __syncthreads();
    cm = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    const float m_new = fmaxf(m, cm);
    const float p = vis ? expf(s - m_new) : 0.f;
    sp[tid] = p;
    float ps = p;
    for (int off = 32; off > 0; off >>= 1) ps += __shfl_xor(ps, off);
    if ((tid & 63) == 0) red2[tid >> 6] = ps;
    __syncthreads();
    const float corr = expf(m - m_new);
    l = l * corr + ((red2[0] + red2[1]) + (red2[2] + red2[3]));
    m = m_new;
    acc *= corr;
    if (grp < groups) {
      const T *vr = Vh + (size_t)dd * cap + base;
      const int cnt = total - base < 256 ? total - base : 256;
      int e = grp * span;
      const int e1 = e + span < cnt ? e + span : cnt;
      // a key without weight adds nothing, whatever its value: another branch of the tree may hold no finite one
      auto seen = [](float pe, T v) { return pe != 0.f ? to_f32<T>(v) : 0.f; };
      for (; e + 4 <= e1; e += 4) {
        T vv[4];
        __builtin_memcpy(vv, vr + e, 4 * sizeof(T));
        const float4 pe = *reinterpret_cast<const float4 *>(sp + e);
        acc += pe.x * seen(pe.x, vv[0]) + pe.y * seen(pe.y, vv[1]) + pe.z * seen(pe.z, vv[2]) + pe.w * seen(pe.w, vv[3]);
      }
      for (; e < e1; ++e) acc += sp[e] * seen(sp[e], vr[e]);
    }
    __syncthreads();
  }
  sp[tid] = acc;
  __syncthreads();
  if (tid < hd) {
    float o = sp[tid];
    for (int i = 1; i < groups; ++i) o += sp[i * hd + tid];
    // row-major [n, H*hd], or fragment order for the o-projection when out_row_tiles > 0
    const size_t idx = out_row_tiles > 0 ? act_frag_index(n, h * hd + tid, out_row_tiles)
                                         : ((size_t)n * H + h) * hd + tid;
    out[idx] = from_f32<T>(o / l);
  }
}

// ---------------------------------------------------------------------------------------------
// orchestration
// ---------------------------------------------------------------------------------------------
#define TR_TRY(expr)                   \
  do {                                 \
    hipError_t e__ = (expr);           \
    if (e__ != hipSuccess) return e__; \
  } while (0)

template <typename T>
static hipError_t attention_dispatch(const tr_kv &kv, int32_t layer, int32_t H, const TreeDev &tree, int32_t n,
                                     const T *q, T *out, int32_t out_row_tiles, float *part_ml, float *part_acc,
                                     Profiler *prof, hipStream_t st) {
  const size_t lsz = (size_t)kv.n_kv_heads * kv.capacity * kv.head_dim;
  const T *Kl = (const T *)kv.k + (size_t)layer * lsz;
  const T *Vl = (const T *)kv.v + (size_t)layer * lsz;
  if (kv.layout == TR_KV_TILED) {
    return launch_attn_mfma((const bf16_t *)q, (const bf16_t *)Kl, (const bf16_t *)Vl, H, kv.n_kv_heads, kv.capacity,
                            n, tree.anc, kv.d_len, kv.len_bound + n, part_ml, part_acc, (bf16_t *)out, out_row_tiles,
                            prof, st);
  }
  return launch(k_attn_generic<T>, dim3(n, H), dim3(256), 0, st, prof_next(prof, PC_ATTN), q, Kl, Vl, H, kv.n_kv_heads,
                kv.head_dim, kv.capacity, n, tree.anc, kv.d_len, out, out_row_tiles);
}

// ---------------------------------------------------------------------------------------------
// generic forward: row-major weights, any shape, f32 or bf16 storage
// ---------------------------------------------------------------------------------------------
template <typename T>
static hipError_t forward_generic(const tr_model &m, const tr_kv &kv, const TreeDev &tree, int32_t n,
                                  const int32_t *tok, float *logits_out, unsigned char *ws, Profiler *prof,
                                  hipStream_t st) {
  const Workspace w = plan_workspace(m);
  const int d = m.d_model, H = m.n_heads, Hkv = m.n_kv_heads, hd = m.head_dim, F = m.d_ffn;
  const int hq = H * hd;
  float *x = (float *)(ws + w.x);
  T *q = (T *)(ws + w.q);
  T *attn = (T *)(ws + w.attn);
  T *hbuf = (T *)(ws + w.h);
  float *rope = (float *)(ws + w.rope);
  const size_t lsz = (size_t)Hkv * kv.capacity * hd;
  auto normed = [&](const void *gain, int epilogue) { // norm(x) as the input
    RowsArgs p{};
    p.a = x; p.gain = gain; p.eps = m.rms_eps; p.n = n; p.K = d; p.epilogue = epilogue;
    return p;
  };
  auto residual = [&](const void *a, int K, const void *wt) { // x += a * wt^T
    RowsArgs p{};
    p.a = a; p.w[0] = wt; p.n = n; p.K = K; p.O = d; p.epilogue = ROWS_ADD; p.y = x; p.ldy = d;
    return p;
  };

  TR_TRY(launch(k_embed_rope<T>, dim3(n, 1 + (d + EMBED_CHUNK - 1) / EMBED_CHUNK), dim3(256), 0, st,
                prof_next(prof, PC_EMBED), (const T *)m.embed, m.vocab, d, tok, tree.depth, kv.d_len, hd, m.rope_theta, x,
                rope));
  for (int l = 0; l < m.n_layers; ++l) {
    const tr_layer &lw = m.layers[l];
    RowsArgs p = normed(lw.attn_norm, ROWS_ROPE);
    p.w[0] = lw.wq; p.w[1] = lw.wk; p.w[2] = lw.wv; p.O = (H + 2 * Hkv) * hd;
    p.q = q; p.k_layer = (T *)kv.k + (size_t)l * lsz; p.v_layer = (T *)kv.v + (size_t)l * lsz;
    p.rope = rope; p.d_len = kv.d_len; p.H = H; p.Hkv = Hkv; p.hd = hd; p.cap = kv.capacity; p.tiled = kv.layout;
    TR_TRY(launch_rows(p, m.dtype, st, prof_next(prof, PC_QKV)));
    if (l == m.n_layers - 1 && logits_out == nullptr) break; // ingestion only needs the cache: nothing reads the last layer's output
    TR_TRY(attention_dispatch<T>(kv, l, H, tree, n, q, attn, 0, (float *)(ws + w.part_ml), (float *)(ws + w.part_acc),
                                 prof, st));
    TR_TRY(launch_rows(residual(attn, hq, lw.wo), m.dtype, st, prof_next(prof, PC_OPROJ)));
    p = normed(lw.ffn_norm, ROWS_SWIGLU);
    p.w[0] = lw.w_gate; p.w[1] = lw.w_up; p.O = F; p.h = hbuf;
    TR_TRY(launch_rows(p, m.dtype, st, prof_next(prof, PC_GATEUP)));
    TR_TRY(launch_rows(residual(hbuf, F, lw.w_down), m.dtype, st, prof_next(prof, PC_DOWN)));
  }
  if (logits_out != nullptr) {
    RowsArgs p = normed(m.final_norm, ROWS_STORE);
    p.w[0] = m.lm_head; p.O = m.vocab; p.y = logits_out; p.ldy = m.vocab;
    TR_TRY(launch_rows(p, m.dtype, st, prof_next(prof, PC_LMHEAD)));
  }
  return hipSuccess;
}

// ---------------------------------------------------------------------------------------------
// packed bf16 forward: MFMA GEMMs on packed weights, activations handed from kernel to kernel in
// fragment order, projection outputs that feed the residual stream kept as per-split partial sums
// which the next normalisation kernel folds into x in a fixed order, or added to it by the projection itself.
// ---------------------------------------------------------------------------------------------
// Residual update and normalisation input, block (row, chunk of 1024 columns), 128 threads x 8 columns:
//   x[row, c] += sum_s part[s][row, c]        (in split order)
//   xg_frag    = bf16(x * g)                   fragment order; rows n..16*row_tiles-1 are zeros
//   ssq[row, chunk] = sum over the chunk of x^2
// The RMS scale 1/sqrt(mean(x^2) + eps) is a per-row scalar, so the GEMM that consumes xg_frag applies
// it to its output rows (gemm row_ssq arguments) instead of this kernel needing a whole-row reduction.
// k_embed_frag is the same for the first layer, where x comes from the embedding table, and writes the rotary table
// beside it (blocks of chunk n_chunks).
constexpr int NORM_CHUNK = 1024;
static_assert(NORM_CHUNK == 128 * 8, "one block iteration covers 128 threads x 8 columns");
constexpr int NORM_MAX_PARTS = 4;
static_assert(NORM_MAX_PARTS >= GEMM_MAX_SPLITS && NORM_MAX_PARTS >= WIDE_MAX_SPLITS, "all partial sums are read at once");

// Both are one memory round trip long and nothing else counts: every load, the gain's too, is issued before the first
// use, and the stores come after the last wait (a wait for a load also waits for the stores before it).
__device__ inline void norm_operand(const float (&v)[8], bool live, const uint4 &gv, int row, int j, int32_t d, int32_t row_tiles,
                                    bf16_t *__restrict__ xg_frag, float *__restrict__ ssq, int32_t ld_ssq, int chunk, bool row_on) {
  __shared__ float red[2];
  float ss = 0.f;
  uint4 pk = uint4{0u, 0u, 0u, 0u};
  if (live) {
    const uint32_t gw[4] = {gv.x, gv.y, gv.z, gv.w};
    uint32_t o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float g0 = bf16_to_f32((bf16_t)(gw[e] & 0xFFFFu)), g1 = bf16_to_f32((bf16_t)(gw[e] >> 16));
      o[e] = (uint32_t)f32_to_bf16(v[2 * e] * g0) | ((uint32_t)f32_to_bf16(v[2 * e + 1] * g1) << 16);
      ss += v[2 * e] * v[2 * e] + v[2 * e + 1] * v[2 * e + 1];
    }
    pk = uint4{o[0], o[1], o[2], o[3]};
  }
  // Written through in steps of four row tiles and more, from 2560 columns on and up to 1 MiB: the stores then reach memory before the
  // launch ends, which costs small operands more than the lines left dirty.  us a step, plain / through, on the same buffers: 7B
  // width, 80 nodes (640 KiB) 3714 / 3641, 13B (20 layers, 800 KiB) 3170 / 3115, 10 layers of 7B width, 64, 96, 128 nodes 1152 / 1115, 1377 / 1365,
  // 1542 / 1538, 12 layers of 2560, 3072, 3200, 80 nodes 934 / 918, 1016 / 1013, 1199 / 1163, but two of 512 (80 KiB) 81.9 / 83.3, 16 of 1024 650 / 658, of
  // 2048 1019 / 1020, and 15 nodes at 1024, 2560, 3072 523 / 526, 658 / 663, 756 / 761, 33 and 48 at 4096 1069 / 1072, 1082 / 1087.  70B (6 layers, 80 nodes, 1.3 MiB)
  // 2411 / 2419; prompts: 511 tokens at 7B width (16 layers) 3913 / 3986, 300 tokens of the two layers of 512 92.1 / 96.2.  7B, 80 nodes, without the streaming
  // hint 3685, with that alone 3727; with the rows of a line on one XCD 3726 plain, 3668 through.  No gain in the partial sums, x, the
  // queries or SwiGLU's output.
  const size_t at = act_frag_index(row, j, row_tiles);
  if (j < d) {
    if (row_tiles >= 4 && row_tiles <= NP / 16 && d >= 2560 && row_tiles * 16 * d <= (1 << 20) / 2) store_through(xg_frag, (uint32_t)at * 2, pk);
    else *reinterpret_cast<uint4 *>(xg_frag + at) = pk;
  }
  for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  if (threadIdx.x == 0 && row_on) {
    float *at = ssq + (size_t)row * ld_ssq;
    at[chunk] = red[0] + red[1];
    if (chunk == (d - 1) / NORM_CHUNK)
      for (int c = chunk + 1; c < ld_ssq; ++c) at[c] = 0.f; // sums of no chunk
  }
}

// From this many row tiles on the eight rows that share the operand's 128-byte lines are on one XCD, whose L2 writes a line back once.  us of
// a prompt on the same buffers, other order / this: 497 tokens at 2048 (12 layers) 1344 / 1327, 4096 (8) 1848 / 1829, 5120 (6) 1854 / 1829, 6144 (5) 1725 / 1705,
// 8192 (3) 1738 / 1724; 700 tokens 1637 / 1626, 2779 / 2763, 2589 / 2569, 2510 / 2487, 2440 / 2416; 1000 tokens 1966 / 1950, 3125 / 3121, 3387 / 3349, 2970 / 2939,
// 3096 / 3085.  300 tokens 4096 1716 / 1731, 5120 1677 / 1699, 400 4096 1855 / 1868.  From 28 row tiles on (440 to 480 tokens, 0.5 to 1.5 %) it would be the
// faster order too; that has not been compared in whole rounds of widths and the line stays.
constexpr int ADD_LINE_TILES = 32;

template <int PARTS>
__global__ __launch_bounds__(128) void k_add_frag(float *__restrict__ x, const float *__restrict__ part,
                                                  size_t part_stride, const bf16_t *__restrict__ g, int32_t n, int32_t d,
                                                  int32_t row_tiles, bf16_t *__restrict__ xg_frag,
                                                  float *__restrict__ ssq, int32_t ld_ssq) {
  int row = blockIdx.x, chunk = blockIdx.y;
  if (row_tiles >= ADD_LINE_TILES) { // block id -> (eight rows, chunk) on XCD id % 8, row of the eight
    const int groups = row_tiles * 2, n_chunks = (d + NORM_CHUNK - 1) / NORM_CHUNK, eighth = blockIdx.x >> 3;
    const int at = (eighth >> 3) * 8 + (blockIdx.x & 7);
    if (at >= groups * n_chunks) return;
    chunk = at / groups;
    row = (at - chunk * groups) * 8 + (eighth & 7);
  }
  const int j = chunk * NORM_CHUNK + threadIdx.x * 8;
  const bool live = row < n && j < d;
  float v[8];
  uint4 gv;
  if (live) {
    float *xr = x + (size_t)row * d + j;
    const float *pr = part + (size_t)row * d + j;
    float4 a = *reinterpret_cast<const float4 *>(xr), b = *reinterpret_cast<const float4 *>(xr + 4);
    gv = *reinterpret_cast<const uint4 *>(g + j);
    float4 pa[PARTS], pb[PARTS];
#pragma unroll
    for (int s = 0; s < PARTS; ++s) {
      pa[s] = *reinterpret_cast<const float4 *>(pr + (size_t)s * part_stride);
      pb[s] = *reinterpret_cast<const float4 *>(pr + (size_t)s * part_stride + 4);
    }
    __builtin_amdgcn_sched_barrier(0); // all of them on their way before the first sum
#pragma unroll
    for (int s = 0; s < PARTS; ++s) {
      a.x += pa[s].x; a.y += pa[s].y; a.z += pa[s].z; a.w += pa[s].w;
      b.x += pb[s].x; b.y += pb[s].y; b.z += pb[s].z; b.w += pb[s].w;
    }
    *reinterpret_cast<float4 *>(xr) = a;
    *reinterpret_cast<float4 *>(xr + 4) = b;
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  }
  norm_operand(v, live, gv, row, j, d, row_tiles, xg_frag, ssq, ld_ssq, chunk, row < n);
}

// n_part 1 .. NORM_MAX_PARTS partial sums
static hipError_t launch_add_frag(int n_part, int chunks, float *x, const float *part, size_t part_stride, const bf16_t *g,
                                  int32_t n, int32_t d, int32_t row_tiles, bf16_t *xg_frag, float *ssq, int32_t ld_ssq,
                                  KernelTimer tm, hipStream_t st) {
  const dim3 block(128);
  const dim3 grid = row_tiles >= ADD_LINE_TILES ? dim3((row_tiles * 2 * chunks + 7) / 8 * 64) : dim3(row_tiles * 16, chunks);
  switch (n_part) {
  case 1: return launch(k_add_frag<1>, grid, block, 0, st, tm, x, part, part_stride, g, n, d, row_tiles, xg_frag, ssq, ld_ssq);
  case 2: return launch(k_add_frag<2>, grid, block, 0, st, tm, x, part, part_stride, g, n, d, row_tiles, xg_frag, ssq, ld_ssq);
  case 3: return launch(k_add_frag<3>, grid, block, 0, st, tm, x, part, part_stride, g, n, d, row_tiles, xg_frag, ssq, ld_ssq);
  case 4: return launch(k_add_frag<4>, grid, block, 0, st, tm, x, part, part_stride, g, n, d, row_tiles, xg_frag, ssq, ld_ssq);
  }
  return hipErrorInvalidValue;
}

__global__ __launch_bounds__(128) void k_embed_frag(const bf16_t *__restrict__ E, int32_t V, const int32_t *__restrict__ tok,
                                                    const int32_t *__restrict__ depth, const int32_t *__restrict__ d_len,
                                                    int32_t hd, float theta, float *__restrict__ x,
                                                    float *__restrict__ rope, const bf16_t *__restrict__ g, int32_t n,
                                                    int32_t d, int32_t row_tiles, bf16_t *__restrict__ xg_frag,
                                                    float *__restrict__ ssq, int32_t ld_ssq) {
  const int row = blockIdx.x, chunk = blockIdx.y, n_chunks = (d + NORM_CHUNK - 1) / NORM_CHUNK;
  if (chunk == n_chunks) {
    if (row < n) rope_row(*d_len + (depth != nullptr ? depth[row] : row), hd, theta, rope + (size_t)row * hd);
    return;
  }
  const int j = chunk * NORM_CHUNK + threadIdx.x * 8;
  const bool live = row < n && j < d;
  float v[8];
  uint4 gv;
  if (live) {
    gv = *reinterpret_cast<const uint4 *>(g + j);
    int t = tok[row];
    t = t < 0 ? 0 : (t >= V ? V - 1 : t);
    bf16_t e[8];
    __builtin_memcpy(e, E + (size_t)t * d + j, 16);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = bf16_to_f32(e[i]);
    float *xr = x + (size_t)row * d + j;
    *reinterpret_cast<float4 *>(xr) = float4{v[0], v[1], v[2], v[3]};
    *reinterpret_cast<float4 *>(xr + 4) = float4{v[4], v[5], v[6], v[7]};
  }
  norm_operand(v, live, gv, row, j, d, row_tiles, xg_frag, ssq, ld_ssq, chunk, row < n);
}

// Q/K/V from partial sums: what the projection's own epilogue does where it is not split over k.  One memory round trip.  A block has 32
// features and all rows, so that the cache lines of keys and values are its own; a thread four features of every 32nd row.  (64
// features a block, half as many blocks: 7.2 us instead of 6.4 at 80 rows of 70B width.)
template <int ROWS>
__global__ __launch_bounds__(256) void k_qkv_finish(const float *__restrict__ part, const float *__restrict__ ssq,
                                                    const float *__restrict__ rope, const int32_t *__restrict__ d_len,
                                                    int32_t n, int32_t O, int32_t n_part, int32_t n_ssq, int32_t H, int32_t norm_dim,
                                                    float eps, int32_t Hkv, int32_t cap, bf16_t *__restrict__ q,
                                                    bf16_t *__restrict__ k_layer, bf16_t *__restrict__ v_layer) {
  const int o = blockIdx.x * 32 + (threadIdx.x & 7) * 4, row0 = threadIdx.x >> 3;
  const int head = o >> 7, dd = o & 127;
  const bool rotated = head < H + Hkv;
  f32x4q p[ROWS][GEMM_MAX_SPLITS];
  f32x4q sq[ROWS][2];
  float2 c[ROWS], s[ROWS];
  const int L = *d_len;
#pragma unroll
  for (int i = 0; i < ROWS; ++i) {
    const int row = row0 + 32 * i, r = row < n ? row : n - 1;
#pragma unroll
    for (int j = 0; j < GEMM_MAX_SPLITS; ++j)
      p[i][j] = *reinterpret_cast<const f32x4q *>(part + ((size_t)(j < n_part ? j : 0) * n + r) * O + o);
#pragma unroll
    for (int j = 0; j < 2; ++j) sq[i][j] = *reinterpret_cast<const f32x4q *>(ssq + (size_t)r * n_ssq + (4 * j < n_ssq ? 4 * j : 0));
    c[i] = *reinterpret_cast<const float2 *>(rope + (size_t)r * 128 + (dd >> 1));
    s[i] = *reinterpret_cast<const float2 *>(rope + (size_t)r * 128 + 64 + (dd >> 1));
  }
  __builtin_amdgcn_sched_barrier(0); // all of them on their way before the first sum
#pragma unroll
  for (int i = 0; i < ROWS; ++i) {
    const int row = row0 + 32 * i, pos = L + row;
    if (row >= n) continue;
    f32x4q v = p[i][0];
#pragma unroll
    for (int j = 1; j < GEMM_MAX_SPLITS; ++j)
      if (j < n_part) v += p[i][j];
    float ss = (sq[i][0][0] + sq[i][0][1]) + (sq[i][0][2] + sq[i][0][3]);
    if (n_ssq > 4) ss += (sq[i][1][0] + sq[i][1][1]) + (sq[i][1][2] + sq[i][1][3]);
    v *= 1.0f / sqrtf(ss / (float)norm_dim + eps);
    if (rotated) {
      const uint2 w = uint2{bf16_pair(v[0] * c[i].x - v[1] * s[i].x, v[1] * c[i].x + v[0] * s[i].x),
                            bf16_pair(v[2] * c[i].y - v[3] * s[i].y, v[3] * c[i].y + v[2] * s[i].y)};
      bf16_t *dst = head < H ? q + ((size_t)row * H + head) * 128 + dd
                             : k_layer + (size_t)(head - H) * cap * 128 + kv_k_index(pos, dd);
      *reinterpret_cast<uint2 *>(dst) = w;
    } else {
      const uint32_t w[2] = {bf16_pair(v[0], v[1]), bf16_pair(v[2], v[3])};
      bf16_t *dst = v_layer + (size_t)(head - H - Hkv) * 128 * cap;
#pragma unroll
      for (int e = 0; e < 4; ++e) dst[kv_v_index(pos, dd + e)] = (bf16_t)(w[e >> 1] >> (16 * (e & 1)));
    }
  }
}

// row-major bf16 [n, K] -> fragment order (standalone linear op only)
__global__ __launch_bounds__(256) void k_rows_to_frag(const bf16_t *__restrict__ a, int32_t n, int32_t K,
                                                      int32_t row_tiles, bf16_t *__restrict__ frag) {
  const int row = blockIdx.x;
  for (int j = threadIdx.x * 8; j < K; j += 2048) {
    uint4 v = uint4{0u, 0u, 0u, 0u};
    if (row < n) v = *reinterpret_cast<const uint4 *>(a + (size_t)row * K + j);
    *reinterpret_cast<uint4 *>(frag + act_frag_index(row, j, row_tiles)) = v;
  }
}

__global__ __launch_bounds__(256) void k_sum_parts(const float *__restrict__ part, int32_t n_part, size_t part_stride,
                                                   size_t count, float *__restrict__ y) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= count) return;
  float v = part[i];
  for (int s = 1; s < n_part; ++s) v += part[(size_t)s * part_stride + i];
  y[i] = v;
}

static bool packed_supported(const tr_model &m) {
  const int hq = m.n_heads * m.head_dim, hk = m.n_kv_heads * m.head_dim;
  return m.dtype == TR_BF16 && m.layout == TR_PACKED && m.d_model % 32 == 0 && m.d_model <= 8 * NORM_CHUNK && m.d_ffn % 32 == 0 && hq % 32 == 0 &&
         hk % 32 == 0 && m.vocab % 32 == 0;
}

static bool operands_on_16(const GemmArgs &g) { // what goes straight into LDS
  bool on = starts_on_16(g.a_frag) && starts_on_16(g.w2);
  for (int i = 0; i < g.n_seg; ++i) on = on && starts_on_16(g.seg[i].w);
  return on;
}
static bool project_rows8(const GemmArgs &g, int32_t max_splits, Rows8Plan *plan) {
  int32_t total = 0;
  for (int i = 0; i < g.n_seg; ++i) total += g.seg[i].out_tiles;
  const bool swiglu = g.mode == GEMM_SWIGLU, scaled = g.row_ssq != nullptr;
  return operands_on_16(g) && g.rope.q == nullptr && (scaled ? g.n_ssq <= 8 : !swiglu) && rows8_plan(g.n, g.K, total, swiglu, swiglu || scaled ? 1 : max_splits, plan);
}
// One projection of a tree step by the faster of its two kernels; fills g.splits.  (tr_plan_step_projection says which.)
static hipError_t project(GemmArgs &g, int32_t max_splits, KernelTimer tm, hipStream_t st) {
  Rows8Plan plan;
  if (project_rows8(g, max_splits, &plan)) {
    g.splits = plan.splits;
    return launch_gemm_rows8(g, plan, st, tm);
  }
  gemm_plan(g, max_splits, max_splits > 1); // o and down alone may be split
  return launch_gemm_mfma(g, st, tm);
}

// Q/K/V in shares of k, whose sums lie in ypart behind a step's other partial sums and the sums of squares.
bool step_qkv_plan(int32_t n, int32_t d, int32_t H, int32_t Hkv, int32_t hd, int32_t layout, Rows8Plan *plan) {
  const int O = (H + 2 * Hkv) * hd;
  return hd == 128 && layout == TR_KV_TILED && qkv_split_plan(n, d, O / 16, plan) &&
         (size_t)plan->splits * n * O + 8192 + 4 <= (size_t)(WIDE_PART_ROWS - GEMM_MAX_SPLITS * NP) * d;
}

static hipError_t forward_packed(const tr_model &m, const tr_kv &kv, const TreeDev &tree, int32_t n, const int32_t *tok,
                                 float *logits_out, unsigned char *ws, Profiler *prof, hipStream_t st) {
  typedef bf16_t T;
  const Workspace w = plan_workspace(m);
  const int d = m.d_model, H = m.n_heads, Hkv = m.n_kv_heads, hd = m.head_dim, F = m.d_ffn;
  const int hq = H * hd, hk = Hkv * hd;
  const int NT = (n + 15) / 16;
  float *x = (float *)(ws + w.x);
  T *xn = (T *)(ws + w.xn);
  T *q = (T *)(ws + w.q);
  T *attn = (T *)(ws + w.attn);
  T *hbuf = (T *)(ws + w.h);
  float *rope = (float *)(ws + w.rope);
  float *ypart = (float *)(ws + w.ypart);
  const size_t ystride = (size_t)NP * d;
  const size_t lsz = (size_t)Hkv * kv.capacity * hd;
  const int nch = (d + NORM_CHUNK - 1) / NORM_CHUNK;
  // The sums of squares sit behind a step's partial sums, where ypart has room for many times as much, on 16 bytes whatever the
  // workspace starts on.
  float *ssq = (float *)(((uintptr_t)(ypart + GEMM_MAX_SPLITS * ystride) + 15) & ~(uintptr_t)15);
  static_assert((size_t)(WIDE_PART_ROWS - GEMM_MAX_SPLITS * NP) * 32 >= (size_t)NP * 64 + 4, "d >= 32 columns hold 32 rows of 256 sums");

  int n_ssq = (nch + 3) & ~3; // sums of squares a row has at the moment
  TR_TRY(launch(k_embed_frag, dim3(NT * 16, nch + 1), dim3(128), 0, st,
                prof_next(prof, PC_EMBED), (const T *)m.embed, m.vocab, tok, tree.depth, kv.d_len, hd, m.rope_theta, x, rope,
                (const T *)m.layers[0].attn_norm, n, d, NT, xn, ssq, n_ssq));
  // x += a * wt^T and the operand of the projection behind it: in one launch where that is faster (gemm_updates_residual) and `next`,
  // whose sums of squares these become, is the decode kernel's
  auto residual = [&](const T *a, int K, const void *wt, const void *gain, GemmArgs &next, ProfCat cat) {
    GemmArgs g{};
    g.a_frag = a; g.n = n; g.K = K;
    g.seg[0] = GemmSeg{(const T *)wt, d / 16};
    g.n_seg = 1; g.y = ypart; g.ldy = d; g.split_stride = ystride; g.mode = GEMM_STORE;
    n_ssq = (nch + 3) & ~3;
    next.row_ssq = ssq; next.n_ssq = n_ssq; next.norm_dim = d; next.eps = m.rms_eps;
    Rows8Plan r8;
    if (!project_rows8(g, GEMM_MAX_SPLITS, &r8) && !project_rows8(next, 1, &r8)) {
      gemm_plan(g, GEMM_MAX_SPLITS, true);
      if (gemm_updates_residual(n, g.groups, g.splits)) {
        next.n_ssq = n_ssq = (g.groups + 3) & ~3;
        g.resid = GemmResid{x, (const T *)gain, xn, ssq, n_ssq};
        return launch_gemm_mfma(g, st, prof_next(prof, cat));
      }
    }
    TR_TRY(project(g, GEMM_MAX_SPLITS, prof_next(prof, cat), st));
    return launch_add_frag(g.splits, nch, x, ypart, ystride, (const T *)gain, n, d, NT, xn, ssq, n_ssq, prof_next(prof, PC_NORM), st);
  };
  for (int l = 0; l < m.n_layers; ++l) {
    const tr_layer &lw = m.layers[l];
    {
      GemmArgs g{};
      g.a_frag = xn; g.n = n; g.K = d;
      g.seg[0] = GemmSeg{(const T *)lw.wq, hq / 16};
      g.seg[1] = GemmSeg{(const T *)lw.wk, hk / 16};
      g.seg[2] = GemmSeg{(const T *)lw.wv, hk / 16};
      g.n_seg = 3; g.mode = GEMM_STORE;
      g.row_ssq = ssq; g.n_ssq = n_ssq; g.norm_dim = d; g.eps = m.rms_eps;
      // RoPE and the query / cache writes happen in the projection's epilogue (one K-split: the epilogue
      // needs complete sums); wq and wk are packed with interleaved rows for that
      g.rope = GemmRope{q, (T *)kv.k + (size_t)l * lsz, (T *)kv.v + (size_t)l * lsz, rope, kv.d_len,
                        H, Hkv, hd, kv.capacity, kv.layout};
      const int O = hq + 2 * hk;
      Rows8Plan plan;
      if (n_ssq <= 8 && operands_on_16(g) && step_qkv_plan(n, d, H, Hkv, hd, kv.layout, &plan)) {
        const GemmRope rp = g.rope;
        float *const parts = ssq + 8192; // behind the sums of squares
        g.rope = GemmRope{};
        g.row_ssq = nullptr;
        g.y = parts; g.ldy = O; g.split_stride = (size_t)n * O;
        TR_TRY(launch_gemm_rows8(g, plan, st, prof_next(prof, PC_QKV)));
        auto finish = [&](auto kernel) {
          return launch(kernel, dim3(O / 32), dim3(256), 0, st, prof_next(prof, PC_QKV), parts, ssq, rope, kv.d_len, n, O, plan.splits,
                        n_ssq, H, d, m.rms_eps, Hkv, kv.capacity, q, rp.k_layer, rp.v_layer);
        };
        TR_TRY(n <= 64 ? finish(k_qkv_finish<2>) : n <= 96 ? finish(k_qkv_finish<3>) : finish(k_qkv_finish<4>));
      } else {
        TR_TRY(project(g, 1, prof_next(prof, PC_QKV), st));
      }
    }
    if (l == m.n_layers - 1 && logits_out == nullptr) break; // as in forward_wide
    TR_TRY(attention_dispatch<T>(kv, l, H, tree, n, q, attn, NT, (float *)(ws + w.part_ml), (float *)(ws + w.part_acc),
                                 prof, st));
    GemmArgs up{};
    up.a_frag = xn; up.n = n; up.K = d;
    up.seg[0] = GemmSeg{(const T *)lw.w_gate, F / 16};
    up.n_seg = 1; up.w2 = (const T *)lw.w_up; up.h_frag = hbuf; up.mode = GEMM_SWIGLU;
    TR_TRY(residual(attn, hq, lw.wo, lw.ffn_norm, up, PC_OPROJ));
    TR_TRY(project(up, 1, prof_next(prof, PC_GATEUP), st));
    GemmArgs next{}; // the LM head, or nothing for Q/K/V: of the up to two row tiles that count here the decode kernel takes it always
    if (l == m.n_layers - 1) {
      next.a_frag = xn; next.n = n; next.K = d;
      next.seg[0] = GemmSeg{(const T *)m.lm_head, m.vocab / 16};
      next.n_seg = 1; next.y = logits_out; next.ldy = m.vocab; next.mode = GEMM_STORE;
    }
    TR_TRY(residual(hbuf, F, lw.w_down, l + 1 < m.n_layers ? m.layers[l + 1].attn_norm : m.final_norm, next, PC_DOWN));
    if (l == m.n_layers - 1) TR_TRY(project(next, 1, prof_next(prof, PC_LMHEAD), st));
  }
  return hipSuccess;
}

// ---------------------------------------------------------------------------------------------
// Prompt ingestion on the packed path: up to `most` rows per pass (what the workspace was sized for).  The projections
// (tr_gemm_wide.hip) and the attention (tr_attn_causal.hip; the Q/K/V projection has cached the keys and values of the
// whole pass by then) take all rows in one launch each.  Same arithmetic per row as forward_packed with one K-split.
// ---------------------------------------------------------------------------------------------
static hipError_t forward_wide(const tr_model &m, const tr_kv &kv, int32_t n, int32_t most, const int32_t *tok,
                               unsigned char *ws, hipStream_t st) {
  typedef bf16_t T;
  const Workspace w = plan_workspace(m, most);
  const int d = m.d_model, H = m.n_heads, Hkv = m.n_kv_heads, hd = m.head_dim, F = m.d_ffn;
  const int hq = H * hd, hk = Hkv * hd;
  const int RT = (n + 15) / 16;
  float *x = (float *)(ws + w.x);
  T *xn = (T *)(ws + w.xn);
  T *q = (T *)(ws + w.q);
  T *attn = (T *)(ws + w.attn);
  T *hbuf = (T *)(ws + w.h);
  float *rope = (float *)(ws + w.rope);
  float *ypart = (float *)(ws + w.ypart);
  const size_t lsz = (size_t)Hkv * kv.capacity * hd;
  float *ssq = (float *)(ws + w.ssq);
  const int nch = (d + NORM_CHUNK - 1) / NORM_CHUNK;
  const KernelTimer no_timer{};
  const size_t ystride = (size_t)RT * 16 * d; // the fewer rows a pass has, the more partial sums fit ypart
  const int max_splits = wide_max_splits(n);

  TR_TRY(launch(k_embed_frag, dim3(RT * 16, nch + 1), dim3(128), 0, st, no_timer, (const T *)m.embed, m.vocab, tok,
                (const int32_t *)nullptr, kv.d_len, hd, m.rope_theta, x, rope, (const T *)m.layers[0].attn_norm, n, d, RT,
                xn, ssq, nch));
  // Without partial sums of either o or down, ypart holds the sums of squares they leave (a row of x is as long as its sums at least).
  const bool fused = wide_plan(n, hq, d / 16).splits == 1 && wide_plan(n, F, d / 16).splits == 1;
  float *const fused_ssq = (float *)(((uintptr_t)ypart + 15) & ~(uintptr_t)15);
  int n_ssq = nch;
  auto residual = [&](const T *a, int K, const void *wt, const void *gain) { // x += a * wt^T and the next operand
    GemmArgs g{};
    g.a_frag = a; g.n = n; g.K = K;
    g.seg[0] = GemmSeg{(const T *)wt, d / 16};
    g.n_seg = 1; g.y = ypart; g.ldy = d; g.split_stride = ystride; g.mode = GEMM_STORE;
    if (fused) {
      ssq = fused_ssq;
      g.resid = GemmResid{x, (const T *)gain, xn, ssq, 0};
      return launch_gemm_wide(g, 1, &n_ssq, st);
    }
    int pending = 0;
    TR_TRY(launch_gemm_wide(g, max_splits, &pending, st));
    return launch_add_frag(pending, nch, x, ypart, ystride, (const T *)gain, n, d, RT, xn, ssq, nch, no_timer, st);
  };
  for (int l = 0; l < m.n_layers; ++l) {
    const tr_layer &lw = m.layers[l];
    {
      GemmArgs g{};
      g.a_frag = xn; g.n = n; g.K = d;
      g.seg[0] = GemmSeg{(const T *)lw.wq, hq / 16};
      g.seg[1] = GemmSeg{(const T *)lw.wk, hk / 16};
      g.seg[2] = GemmSeg{(const T *)lw.wv, hk / 16};
      g.n_seg = 3; g.mode = GEMM_STORE;
      g.row_ssq = ssq; g.n_ssq = n_ssq; g.norm_dim = d; g.eps = m.rms_eps;
      g.rope = GemmRope{q, (T *)kv.k + (size_t)l * lsz, (T *)kv.v + (size_t)l * lsz, rope, kv.d_len,
                        H, Hkv, hd, kv.capacity, kv.layout};
      TR_TRY(launch_gemm_wide(g, 1, nullptr, st));
    }
    if (l == m.n_layers - 1) break; // ingestion only needs the cache: nothing reads the last layer's output
    TR_TRY(launch_attn_causal(q, (const T *)kv.k + (size_t)l * lsz, (const T *)kv.v + (size_t)l * lsz, H, Hkv, kv.capacity, n,
                              kv.d_len, attn, RT, st));
    TR_TRY(residual(attn, hq, lw.wo, lw.ffn_norm));
    {
      GemmArgs g{};
      g.a_frag = xn; g.n = n; g.K = d;
      g.seg[0] = GemmSeg{(const T *)lw.w_gate, F / 16};
      g.n_seg = 1; g.w2 = (const T *)lw.w_up; g.h_frag = hbuf; g.mode = GEMM_SWIGLU;
      g.row_ssq = ssq; g.n_ssq = n_ssq; g.norm_dim = d; g.eps = m.rms_eps;
      TR_TRY(launch_gemm_wide(g, 1, nullptr, st));
    }
    TR_TRY(residual(hbuf, F, lw.w_down, m.layers[l + 1].attn_norm));
  }
  return hipSuccess;
}

static bool wide_supported(const tr_model &m, const tr_kv &kv, const void *ws) {
  if (!packed_supported(m) || kv.layout != TR_KV_TILED || kv.dtype != TR_BF16 || m.head_dim != 128 || m.d_model < 64 ||
      m.d_ffn < 64)
    return false;
  bool on = starts_on_16(ws) && starts_on_16(kv.k) && starts_on_16(kv.v); // what its kernels load straight into LDS
  for (int l = 0; l < m.n_layers; ++l) {
    const tr_layer &w = m.layers[l];
    for (const void *p : {w.wq, w.wk, w.wv, w.wo, w.w_gate, w.w_up, w.w_down}) on = on && starts_on_16(p);
  }
  return on;
}

int32_t prefill_rows(const tr_model &m, const tr_kv &kv, const void *ws, size_t ws_bytes) {
  if (!wide_supported(m, kv, ws)) return NP;
  return ws_bytes >= plan_workspace(m, NPW_MOST).total ? NPW_MOST : NPW;
}

hipError_t run_prefill_pass(const tr_model &m, const tr_kv &kv, const TreeDev &chain, int32_t n, int32_t most,
                            const int32_t *d_tokens, void *ws, hipStream_t st) {
  if (n > most) return hipErrorInvalidValue;
  if (n > NP) return forward_wide(m, kv, n, most, d_tokens, (unsigned char *)ws, st);
  return run_forward(m, kv, chain, n, d_tokens, nullptr, ws, nullptr, st);
}

hipError_t run_forward(const tr_model &m, const tr_kv &kv, const TreeDev &tree, int32_t n, const int32_t *d_tokens,
                       float *write_logits, void *ws, Profiler *prof, hipStream_t st) {
  if (packed_supported(m)) return forward_packed(m, kv, tree, n, d_tokens, write_logits, (unsigned char *)ws, prof, st);
  if (m.dtype == TR_BF16)
    return forward_generic<bf16_t>(m, kv, tree, n, d_tokens, write_logits, (unsigned char *)ws, prof, st);
  return forward_generic<float>(m, kv, tree, n, d_tokens, write_logits, (unsigned char *)ws, prof, st);
}

bool model_layout_ok(const tr_model &m) { return m.layout == TR_ROW_MAJOR || packed_supported(m); }

hipError_t run_tree_attention(const tr_kv &kv, int32_t layer, int32_t H, const TreeDev &tree, const void *d_q,
                              void *d_out, void *ws, hipStream_t st) {
  // standalone op: the split partials sit at the start of the caller's workspace
  float *ml = (float *)ws;
  float *acc = ws ? (float *)((unsigned char *)ws + align256((size_t)ATTN_MAX_SPLITS * NP * H * 2 * 4)) : nullptr;
  if (kv.dtype == TR_BF16)
    return attention_dispatch<bf16_t>(kv, layer, H, tree, tree.n_nodes, (const bf16_t *)d_q, (bf16_t *)d_out, 0, ml,
                                      acc, nullptr, st);
  return attention_dispatch<float>(kv, layer, H, tree, tree.n_nodes, (const float *)d_q, (float *)d_out, 0, nullptr,
                                   nullptr, nullptr, st);
}

size_t linear_workspace_bytes(int32_t n, int32_t in_f, int32_t out_f, int32_t splits) {
  const size_t nt = (size_t)(n + 15) / 16;
  return align256(nt * 16 * in_f * 2) + align256((size_t)splits * n * out_f * 4);
}

hipError_t run_linear(const void *x, const void *w, int32_t dtype, int32_t layout, int32_t n, int32_t in_f,
                      int32_t out_f, int32_t splits, float *y, void *ws, hipStream_t st) {
  if (layout == TR_PACKED) {
    if (n > NP && !(starts_on_16(w) && starts_on_16(ws))) { // the decode kernel, NP rows at a time
      for (int lo = 0; lo < n; lo += NP)
        TR_TRY(run_linear((const bf16_t *)x + (size_t)lo * in_f, w, dtype, layout, n - lo < NP ? n - lo : NP, in_f, out_f, splits,
                          y + (size_t)lo * out_f, ws, st));
      return hipSuccess;
    }
    const int NT = (n + 15) / 16;
    bf16_t *frag = (bf16_t *)ws;
    float *part = (float *)((unsigned char *)ws + align256((size_t)NT * 16 * in_f * 2));
    TR_TRY(launch(k_rows_to_frag, dim3(NT * 16), dim3(256), 0, st, KernelTimer{}, (const bf16_t *)x, n, in_f, NT, frag));
    GemmArgs g{};
    g.a_frag = frag; g.n = n; g.K = in_f;
    g.seg[0] = GemmSeg{(const bf16_t *)w, out_f / 16};
    g.n_seg = 1; g.y = splits > 1 ? part : y; g.ldy = out_f;
    g.split_stride = (size_t)n * out_f; g.mode = GEMM_STORE;
    if (n > NP) { // the prompt-ingestion kernel; it may use fewer splits than allowed
      TR_TRY(launch_gemm_wide(g, splits, &splits, st));
    } else {
      gemm_plan(g, splits, false);
      g.splits = splits; // the caller's split count is used as given
      TR_TRY(launch_gemm_mfma(g, st));
    }
    if (g.y != y) {
      const size_t count = (size_t)n * out_f;
      TR_TRY(launch(k_sum_parts, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, KernelTimer{}, part, splits,
                    (size_t)n * out_f, count, y));
    }
    return hipSuccess;
  }
  RowsArgs p{};
  p.a = x; p.w[0] = w; p.n = n; p.K = in_f; p.O = out_f; p.epilogue = ROWS_STORE; p.y = y; p.ldy = out_f;
  return launch_rows(p, dtype, st);
}

} // namespace tr
