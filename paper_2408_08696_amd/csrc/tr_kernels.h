// Launch interfaces of the bf16 MFMA kernels (gfx950).
#pragma once
#include "tr_internal.h"

namespace tr {

enum GemmMode { GEMM_STORE = 0, GEMM_ROPE = 1 /* GEMM_STORE with GemmRope, picked by the launch */, GEMM_SWIGLU = 2,
                GEMM_RESID = 3 /* GEMM_STORE with GemmResid, likewise */,
                GEMM_PARTS = 4 /* GEMM_STORE over the three matrices of Q/K/V, by launch_gemm_rows8 */ };

// Streaming store for activations that the next kernel reads once: written through as issued, so the
// kernel does not end with dirty L2 lines to write back before its successor may start (the consumers
// mostly sit on other XCDs and read through memory anyway).  Measured per producer; it pays for the
// SwiGLU output and the attention output, not for K-split partial sums or the query / key writes.
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2s;
__device__ inline void store_stream(bf16_t *p, ushort4 v) {
  __builtin_nontemporal_store(u32x2s{(uint32_t)v.x | ((uint32_t)v.y << 16), (uint32_t)v.z | ((uint32_t)v.w << 16)},
                              reinterpret_cast<u32x2s *>(p));
}

// Streaming and written through at once (sc1 nt), base uniform over the wave: for a step's residual kernel, in whose operand 128-byte
// lines take 16 bytes each from eight rows and so from workgroups on eight XCDs.  Left dirty in eight L2s they are written back
// when the kernel ends, and the projection behind it waits.
__device__ inline void store_through(void *base, uint32_t byte, uint4 v) {
  typedef __attribute__((ext_vector_type(4))) uint32_t u4;
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(base, 0, 0xFFFFFFFF, 0x00027000);
  __builtin_amdgcn_raw_buffer_store_b128(u4{v.x, v.y, v.z, v.w}, rsrc, byte, 0, 18);
}

// Two floats rounded to bf16 (nearest even) in one word, by the hardware's packed conversion.
__device__ inline uint32_t bf16_pair(float lo, float hi) {
  typedef __attribute__((ext_vector_type(2))) float f2;
  typedef __attribute__((ext_vector_type(2))) __bf16 b2;
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{lo, hi}, b2));
}
// x / (1 + e^-x), the quotient correctly rounded.  The hardware's reciprocal in its place saves ten instructions, but it is
// one more rounding in float32 and gives 0 from x = -87.3 down, where 1 / (1 + e^-x) is no normal number and the quotient, some
// 1e-36, still is.  e^-x itself is off by up to |x| 2^-24 or so relatively (the rounding of its exponent).
__device__ inline float silu(float x) { return x / (1.0f + __expf(-x)); }

// Fragment order (see tr_gemm_mfma.hip): a tile of 16 rows x 32 k is 64 lane slots of 8 bf16;
// element (row r, k) of an operand with T row tiles lives in tile (k/32, r/16) at lane slot
// (r%16) + 16*((k%32)/8), element k%8.  Weights use tile index (r/16) * (K/32) + k/32 instead.
__host__ __device__ inline size_t act_frag_index(int r, int k, int row_tiles) {
  return ((((size_t)(k >> 5) * row_tiles + (r >> 4)) * 64) + (r & 15) + 16 * ((k & 31) >> 3)) * 8 + (k & 7);
}

// One 1 KiB tile from memory straight into LDS: lane l's 16 bytes at gbase + voff land at lds_off + 16 l.  The
// instruction has no destination register; what it writes becomes readable after wait_tiles() and a barrier.  (The
// builtin for it makes the compiler wait for all such loads before every LDS read.)
__device__ inline void tile_to_lds(uint32_t lds_off, uint32_t voff, uint64_t gbase) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_off), "v"(voff), "s"(gbase)
               : "memory"); // nothing the compiler emits here uses m0
}
// What these loads read has to start on 16 bytes; callers take a kernel with plain loads for blocks that do not.
inline bool starts_on_16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }
// Waits until at most `left` of this wave's tile loads are still under way and all its LDS reads have returned.
template <int left>
__device__ inline void wait_tiles() {
  static_assert(left >= 0 && left < 64, "six bits of vmcnt");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(left) : "memory");
}
__device__ inline void meet_waves() { asm volatile("s_barrier" ::: "memory"); }

struct GemmSeg {
  const bf16_t *w;   // packed weight matrix
  int32_t out_tiles; // its out_features / 16
};

// Optional epilogue of the fused Q/K/V projection (GEMM_STORE, splits == 1, q != nullptr): instead of
// storing y, rotate the query and key features (RoPE) and write queries, keys and values where the
// attention kernel reads them.  Needs wq and wk packed with their rows interleaved per head (feature i and
// i + head_dim/2 adjacent, see launch_pack_weight), so that a rotation pair sits in one lane; queries and
// cached keys then carry that feature order, which the attention dot product does not care about.
struct GemmRope {
  bf16_t *q;             // [n, H, hd] rotated queries; nullptr switches the epilogue off
  bf16_t *k_layer;       // this layer's K block of the cache
  bf16_t *v_layer;       // this layer's V block of the cache
  const float *rope;     // [rows, hd]: cos[hd/2] | sin[hd/2] of every row's position
  const int32_t *d_len;  // committed length L; row r is written at cache position L + r
  int32_t H, Hkv, hd, cap, tiled;
};

// Optional epilogue of the projections that feed the residual stream (GEMM_STORE, splits == 1, x != nullptr): instead of storing y
// for k_add_frag, add it to x and write the next projection's operand and sums of squares.
struct GemmResid {
  float *x;             // [n, ldy] residual stream, read and written
  const bf16_t *gain;   // [ldy] of the normalisation that follows
  bf16_t *xg_frag;      // bf16(x * gain), fragment order over ceil(n / 16) row tiles; rows past n zero
  float *ssq;           // [n, ld_ssq] sums of x^2 over each workgroup's out-tiles, zeros behind the last
  int32_t ld_ssq;       // groups rounded up to a multiple of 4
};

// y[n, O] = a[n, K] * W^T over the concatenation of up to three weight matrices (out-feature axis).
//   GEMM_STORE : y[split][row * ldy + o] = partial sum of that K-split (float32, row-major)
//   GEMM_SWIGLU: h_frag = bf16(silu(a W_gate^T) * (a W_up^T)) in fragment order over (k = o);
//                seg[0] = gate, w2 = up, splits must be 1
struct GemmArgs {
  const bf16_t *a_frag; // activations, fragment order, ceil(n/16) row tiles
  int32_t n, K;
  GemmSeg seg[3];
  int32_t n_seg;
  const bf16_t *w2;
  float *y;
  int32_t ldy;
  int32_t splits;
  size_t split_stride; // floats between consecutive partial results
  bf16_t *h_frag;
  int32_t mode;
  // optional RMS scale applied to output row r: 1/sqrt(sum_c row_ssq[r*n_ssq + c] / norm_dim + eps); in a step n_ssq is a multiple
  // of 4 and row_ssq starts on 16 bytes (sums that a row does not have are zeros)
  const float *row_ssq;
  int32_t n_ssq, norm_dim;
  float eps;
  int32_t total_tiles;  // sum of seg[i].out_tiles
  int32_t tiles_per_wg; // most out-tiles (SWIGLU: gate/up tile pairs) a workgroup handles per pass
  int32_t groups;       // workgroups per K-split; each owns a contiguous ~total_tiles/groups out-tiles
  int32_t part_q, part_rem; // total_tiles / groups and total_tiles % groups (filled by launch_gemm_mfma)
  GemmRope rope;            // Q/K/V epilogue (see above), off when rope.q == nullptr
  GemmResid resid;          // residual epilogue (see above), off when resid.x == nullptr
};

// Fills g.total_tiles, g.tiles_per_wg, g.groups and g.splits (<= max_splits; 1 for GEMM_SWIGLU).  feeds_x: o and down of a step, behind
// which a residual kernel is launched unless they update the residual stream themselves.
void gemm_choose(int32_t n, int32_t K, int32_t total_tiles, bool swiglu, int32_t max_splits, bool feeds_x, int32_t *out_pmax,
                 int32_t *out_groups, int32_t *out_splits);
inline void gemm_plan(GemmArgs &g, int32_t max_splits, bool feeds_x) {
  int32_t total = 0;
  for (int i = 0; i < g.n_seg; ++i) total += g.seg[i].out_tiles;
  g.total_tiles = total;
  gemm_choose(g.n, g.K, total, g.mode == GEMM_SWIGLU, g.mode == GEMM_SWIGLU ? 1 : max_splits, feeds_x, &g.tiles_per_wg,
              &g.groups, &g.splits);
}

// Whether a step's o and down update the residual stream in their own epilogue (GemmResid) instead of leaving partial sums to
// k_add_frag: from whole sums of up to two row tiles, with a workgroup for most compute units.  At 7B width one kernel then costs 0.4 us
// more, as does the one behind it for its 256 sums of squares per row instead of 4, and the launch of 4.6 to 5 us is gone: both o and down
// of a layer, 1 row 34.4 / 25.6 us, 15 rows 34.4 / 25.9.  us a step on the same buffers, k_add_frag / this, 1 and 15 nodes: 8 layers of 7B 747 /
// 720, 795 / 761, 3 of 70B 1209 / 1199, 1202 / 1186, 6 of 6656 1227 / 1211, 1244 / 1225, 12 of 3840 1055 / 1013, 1076 / 1024, of 3328 849 / 837, 912 / 907; 17 to
// 32 rows where gemm_choose keeps o whole for it, and 0.1 to 1.2 % at 8192.  13B's 320 out-tiles make 160 workgroups when whole, which is too
// few: down of one row 23.9 + 4.7 in two shares, 31.2 whole.
// More rows are split over k, and the sums of the shares are no cheaper to bring together inside the launch: 80 rows, 7B o and down 17.0 and
// 26.4 us with k_add_frag, 16.6 and 25.8 with sums that the waves of a group send each other, and 2.6 more in the kernels behind.
constexpr int GEMM_RESID_ROW_TILES = 2;
// partial sums of squares per row that a step's projections take at nt row tiles
constexpr int gemm_most_ssq(int nt) { return nt <= GEMM_RESID_ROW_TILES ? 256 : 8; }
inline bool gemm_updates_residual(int32_t n, int32_t groups, int32_t splits) {
  const int nt = (n + 15) / 16;
  return splits == 1 && nt <= GEMM_RESID_ROW_TILES && groups >= 200 && groups <= gemm_most_ssq(nt);
}
bool gemm_mfma_supported(int32_t n, int32_t K, int32_t O);
hipError_t launch_gemm_mfma(const GemmArgs &g, hipStream_t st, KernelTimer tm = KernelTimer{});
// rope_hd > 0: packed row h*rope_hd + 2j + b takes source row h*rope_hd + j + b*rope_hd/2 (query / key
// matrices: the two features of a rotation pair become neighbours)
// Prompt ingestion: the same contraction and epilogues for up to WIDE_MAX_ROWS rows per launch (tr_gemm_wide.hip);
// a_frag / h_frag span ceil(n / 16) row tiles, rope rows are indexed by row; a plain store may be split over k
// into up to max_splits partial sums split_stride floats apart (*out_splits receives the count used).
constexpr int WIDE_MAX_ROWS = NPW_MOST;
constexpr int WIDE_MAX_SPLITS = 4;
bool gemm_wide_supported(int32_t n, int32_t K, int32_t O);
hipError_t launch_gemm_wide(const GemmArgs &g, int32_t max_splits, int32_t *out_splits, hipStream_t st,
                            KernelTimer tm = KernelTimer{});
// How an ingestion pass of n rows takes o or down: workgroup shape (row tiles x out-tiles), groups of out-tiles, k-splits.  Where neither is
// split they update the residual stream themselves (GemmResid; ld_ssq is filled by the launch).
struct WideProjection {
  int32_t row_tiles, out_tiles, groups, splits;
};
WideProjection wide_plan(int32_t n, int32_t K, int32_t out_tiles);
inline int32_t wide_max_splits(int32_t n) { // as many partial sums of all row tiles as ypart has room for
  const int fit = WIDE_PART_ROWS / ((n + 15) / 16 * 16);
  return fit < WIDE_MAX_SPLITS ? fit : WIDE_MAX_SPLITS;
}
// The same kernel for a tree step's rows (n <= TR_MAX_NODES), where it is the faster one: true and the plan, else
// launch_gemm_mfma is.  Operands have to start on 16 bytes.  max_splits > 1: a plain store without an RMS scale.
struct Rows8Plan {
  int32_t out_tiles, groups, splits; // out-tiles per workgroup, workgroups per K-split
};
bool rows8_plan(int32_t n, int32_t K, int32_t total_tiles, bool swiglu, int32_t max_splits, Rows8Plan *plan);
hipError_t launch_gemm_rows8(const GemmArgs &g, const Rows8Plan &plan, hipStream_t st, KernelTimer tm = KernelTimer{});
// Q/K/V of a step split over k, with a launch behind it that adds the shares, scales, rotates and writes (k_qkv_finish): by size, and
// (operands on 16 bytes) whether a step with this cache and workspace takes it.
bool qkv_split_plan(int32_t n, int32_t K, int32_t total_tiles, Rows8Plan *plan);
bool step_qkv_plan(int32_t n, int32_t d, int32_t H, int32_t Hkv, int32_t hd, int32_t layout, Rows8Plan *plan);
hipError_t launch_pack_weight(const bf16_t *src, bf16_t *dst, int32_t O, int32_t K, int32_t rope_hd, hipStream_t st);

// Shape-generic projections on row-major weights with their prologue and epilogue (tr_rows.hip).
enum RowsEpilogue {
  ROWS_STORE = 0,  // y[row * ldy + o] = v
  ROWS_ADD = 1,    // y[row * ldy + o] += v (residual stream)
  ROWS_SWIGLU = 2, // h[row * O + f] = T(silu(gate) * up); w[0] = gate, w[1] = up, O = features of one of them
  ROWS_ROPE = 3    // Q/K/V: rotate, write queries and this layer's cache entries; w = {q, k, v}, O = all outputs
};
struct RowsArgs {
  const void *a;    // gain != nullptr: float [n, K], the residual stream to normalise; else T [n, K]
  const void *gain; // T [K] or nullptr
  float eps;
  const void *w[3]; // T, row-major [.., K]
  int32_t n, K, O;
  int32_t epilogue;
  float *y;
  int32_t ldy;
  void *h;
  void *q, *k_layer, *v_layer; // ROWS_ROPE
  const float *rope;
  const int32_t *d_len;
  int32_t H, Hkv, hd, cap, tiled;
};
hipError_t launch_rows(const RowsArgs &p, int32_t dtype, hipStream_t st, KernelTimer tm = KernelTimer{});

// Tree attention for head_dim 128, bf16 K/V/Q, split over the key axis with a merge pass.
// len_bound: host upper bound of L + n (sizes the split count only).
// Query heads one workgroup of launch_attn_mfma serves (they share a K/V head), and the key-axis splits it
// uses for H / that many head groups and this bound on committed length + nodes.
int attn_heads_per_wg(int32_t H, int32_t Hkv, int32_t n);
int attn_choose_splits(int32_t head_groups, int32_t len_bound);
// whether workgroups of this many node tiles and heads take their key shares in 64-key steps (k_attn_ring) or tile by tile
bool attn_long_shares(int32_t node_tiles, int32_t hpw, int32_t len_bound, int32_t nsplit);
// true: one launch without key splits or merge pass (short sequences); then the two values above do not apply
bool attn_one_launch(int32_t H, int32_t Hkv, int32_t len_bound);
hipError_t launch_attn_mfma(const bf16_t *q, const bf16_t *Kl, const bf16_t *Vl, int32_t H, int32_t Hkv, int32_t cap,
                            int32_t n, const uint64_t *anc, const int32_t *d_len, int32_t len_bound, float *part_ml,
                            float *part_acc, bf16_t *out, int32_t out_row_tiles, Profiler *prof, hipStream_t st);

// The same for few rows per K/V head (tr_attn_rows.hip; n <= 64, n * H / Hkv <= 128), and whether it is the faster form;
// launch_attn_mfma goes there by itself.  launch_attn_merge: part_rows rows per (split, head) in the partial buffers.
bool attn_rows_better(int32_t H, int32_t Hkv, int32_t n, int32_t len_bound);
int attn_rows_splits(int32_t H, int32_t Hkv, int32_t n, int32_t len_bound); // its key shares (1: no merge launch)
hipError_t launch_attn_rows(const bf16_t *q, const bf16_t *Kl, const bf16_t *Vl, int32_t H, int32_t Hkv, int32_t cap,
                            int32_t n, const uint64_t *anc, const int32_t *d_len, int32_t len_bound, float *part_ml,
                            float *part_acc, bf16_t *out, int32_t out_row_tiles, Profiler *prof, hipStream_t st);
hipError_t launch_attn_merge(const float *part_ml, const float *part_acc, int32_t part_rows, int32_t H, int32_t n, int32_t nsplit,
                             bf16_t *out, int32_t out_row_tiles, KernelTimer tm, hipStream_t st);

// Prompt ingestion (tr_attn_causal.hip): n consecutive rows behind the committed length, row r sees the positions up to
// its own; the keys and values of all of them are cached already.  out in fragment order over out_row_tiles row tiles.
hipError_t launch_attn_causal(const bf16_t *q, const bf16_t *Kl, const bf16_t *Vl, int32_t H, int32_t Hkv, int32_t cap,
                              int32_t n, const int32_t *d_len, bf16_t *out, int32_t out_row_tiles, hipStream_t st);

} // namespace tr
