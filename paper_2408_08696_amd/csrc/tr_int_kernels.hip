// Integer kernels of the Token Recycling step: draft-tree gather, per-row top-k, greedy accept,
// adjacency-matrix scatter and KV compaction.  All single-workgroup or tiny: the work is a few
// KB of dependent L2 accesses, so each kernel is shaped to be one launch with no host round trip.
#include <mutex>

#include "tr_internal.h"

namespace tr {

// ---------------------------------------------------------------------------------------------
// Draft-tree retrieval (Section 3.2, Algorithm 1).  One workgroup; the tree lives in LDS and the
// D-1 dependent gather rounds are separated by workgroup barriers.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(TR_MAX_NODES) void k_build_tree(const int32_t *__restrict__ M, int32_t V,
                                                             int32_t k, const int32_t *__restrict__ parent,
                                                             const int32_t *__restrict__ rank,
                                                             const int32_t *__restrict__ depth, int32_t n_nodes, int32_t n_layers,
                                                             const int32_t *__restrict__ d_root, int32_t *__restrict__ S) {
  __shared__ int32_t s[TR_MAX_NODES];
  const int i = threadIdx.x;
  const bool live = i < n_nodes;
  const int par = live ? parent[i] : -1;
  const int rk = live ? rank[i] : 0;
  const int dep = live ? depth[i] : -1;
  if (i == 0) {
    int r = *d_root;
    s[0] = r < 0 ? 0 : (r >= V ? V - 1 : r);
  }
  for (int d = 1; d < n_layers; ++d) {
    __syncthreads();
    if (dep == d) { // a stored candidate outside [0, V) (a caller-made top-k buffer) is clamped like the root
      const int tk = M[(size_t)s[par] * k + rk];
      s[i] = tk < 0 ? 0 : (tk >= V ? V - 1 : tk);
    }
  }
  __syncthreads();
  if (live) S[i] = s[i];
}

hipError_t launch_build_tree(tr_ctx *c, const int32_t *d_root, int32_t *d_S, hipStream_t st) {
  return launch(k_build_tree, dim3(1), dim3(TR_MAX_NODES), 0, st, c->prof.next(PC_BUILD), c->d_M, c->V, c->k, c->tree.parent,
                c->tree.rank, c->tree.depth, c->tree.n_nodes, c->tree.n_layers, d_root, d_S);
}

// ---------------------------------------------------------------------------------------------
// argtopk (Section 2.1): one workgroup per row, k selection passes.  Pass p finds the first
// element, in the total order (value descending, index ascending), that comes strictly after the
// winner of pass p-1.  Exact for ties and for -0 == +0; no per-thread candidate lists.
// ---------------------------------------------------------------------------------------------
struct Cand {
  float v;
  int32_t i;
};
__device__ inline bool before(const Cand &a, const Cand &b) { // a strictly precedes b
  return a.v > b.v || (a.v == b.v && a.i < b.i);
}

constexpr int TOPK_THREADS = 512;

template <typename T>
__global__ __launch_bounds__(TOPK_THREADS) void k_topk(const T *__restrict__ logits, int32_t V, int32_t k,
                                                        int32_t *__restrict__ out) {
  __shared__ Cand red[TOPK_THREADS / 64];
  __shared__ Cand winner;
  const T *row = logits + (size_t)blockIdx.x * V;
  const int tid = threadIdx.x;
  Cand prev;
  prev.v = __builtin_inff();
  prev.i = -1; // precedes every real element
  for (int p = 0; p < k; ++p) {
    Cand best;
    best.v = -__builtin_inff();
    best.i = 0x7FFFFFFF; // follows every real element
    for (int j = tid; j < V; j += TOPK_THREADS) {
      Cand e;
      e.v = to_f32<T>(row[j]);
      e.i = j;
      if (before(prev, e) && before(e, best)) best = e;
    }
    for (int off = 32; off > 0; off >>= 1) {
      Cand o;
      o.v = __shfl_xor(best.v, off);
      o.i = __shfl_xor(best.i, off);
      if (before(o, best)) best = o;
    }
    if ((tid & 63) == 0) red[tid >> 6] = best;
    __syncthreads();
    if (tid == 0) {
      Cand b = red[0];
      for (int w = 1; w < TOPK_THREADS / 64; ++w)
        if (before(red[w], b)) b = red[w];
      winner = b;
      out[(size_t)blockIdx.x * k + p] = b.i;
    }
    __syncthreads();
    prev = winner;
  }
}

// Threshold variant for k <= TOPK_WAVES.  A workgroup of 16 waves holds one segment (up to TOPK_SEG elements, the whole
// row for most vocabularies) in registers.  The k-th largest of the 16 wave maxima is a value that at least k elements
// reach, so the segment's k best are all among the elements not below it - a dozen or two on ordinary logits.  Those go
// to LDS as 64-bit keys whose unsigned order is the total order of k_topk (the float mapped to an order-preserving
// unsigned, with -0 folded onto +0, in the high word; the complemented index in the low word; key 0 is "nothing"), and
// each finds its place by counting the keys above it.  Per element that is one load, one maximum and no 64-bit
// arithmetic.  Segments whose ties put more than TOPK_LIST elements at or above the threshold are selected by k exact
// passes over the registers instead, and so are segments with a NaN in them, which no threshold can be trusted with.  A
// row of several segments leaves k keys per segment to k_topk_merge.
// Every place of every row is written.  nan_ranks: a NaN takes the place of its bits (before +inf, or behind -inf with the
// sign bit set); else it is no candidate, as in k_topk, and a place nothing is left for holds TOPK_NONE.
// What bounds it: latency (launch, one load round trip, three barriers).  80 rows of 32000 bf16 logits took 12.4 + 5.8 us
// as "every wave selects its own k best by k rounds of 64-bit maxima, a second kernel merges 32 waves per row" (the
// rounds are ~900 clocks of vector ALU each).
constexpr int TOPK_WAVES = 16;
constexpr int TOPK_SEL_THREADS = TOPK_WAVES * 64;
constexpr int TOPK_EPT = 32;                             // elements a thread holds
constexpr int TOPK_SEG = TOPK_SEL_THREADS * TOPK_EPT;
constexpr int TOPK_LIST = 1024;                          // candidates kept in LDS
constexpr int TOPK_MAX_SEGS = 64;
constexpr int TOPK_ROW_SLOTS = TOPK_MAX_SEGS * TOPK_WAVES; // scratch keys per row
constexpr int32_t TOPK_NONE = 0x7FFFFFFF;                // id of a place without a candidate
constexpr int TOPK_NAN_K = 8;                            // NaN ranks for k up to this on rows of TOPK_NAN_K ..
constexpr int TOPK_STATIC_MAX_V = 131072;                // .. TOPK_STATIC_MAX_V elements (what tr.h states)

__device__ inline uint64_t topk_key(float v, int32_t idx) {
  uint32_t u = __float_as_uint(v + 0.0f); // -0 + 0 = +0
  u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return ((uint64_t)u << 32) | (uint32_t)~idx;
}
__device__ inline int32_t topk_id(uint64_t key) { return key == 0 ? TOPK_NONE : (int32_t)~(uint32_t)key; }
// NaN if either is (one instruction: v_maximum3_f32)
__device__ inline float max_or_nan(float a, float b) { return __builtin_elementwise_maximum(a, b); }
// Wave-wide maximum (NaN if any lane's value is) on the vector ALU alone: four data-parallel-primitive exchanges (lane ^ 1, lane ^ 2,
// mirror inside 8 lanes, mirror inside the row of 16) leave every lane with its row's maximum, and the
// four row maxima are read out as scalars.  All 64 lanes must be active.
template <int CTRL>
__device__ inline float dpp_f32(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(x), __float_as_int(x), CTRL, 0xF, 0xF, false));
}
__device__ inline float wave_max_f32(float x) {
  x = max_or_nan(x, dpp_f32<0xB1>(x));  // quad_perm [1,0,3,2]
  x = max_or_nan(x, dpp_f32<0x4E>(x));  // quad_perm [2,3,0,1]
  x = max_or_nan(x, dpp_f32<0x141>(x)); // row_half_mirror
  x = max_or_nan(x, dpp_f32<0x140>(x)); // row_mirror
  auto lane = [&](int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l)); };
  return max_or_nan(max_or_nan(lane(0), lane(16)), max_or_nan(lane(32), lane(48)));
}

// VEC: 16-byte loads (base and row pitch 16-byte aligned, at least one full vector per thread of the workgroup, so
// that every wave has elements); otherwise one element per load.
template <typename T, bool VEC>
__global__ __launch_bounds__(TOPK_SEL_THREADS) void k_topk_select(const T *__restrict__ logits, int32_t V, int32_t k,
                                                                  int32_t seg_len, int32_t nan_ranks,
                                                                  int32_t *__restrict__ out,
                                                                  uint64_t *__restrict__ cand) {
  constexpr int E = VEC ? 16 / (int)sizeof(T) : 1; // elements per load
  __shared__ float wmax[TOPK_WAVES];
  __shared__ uint64_t list[TOPK_LIST];
  __shared__ uint64_t wbest[TOPK_WAVES];
  __shared__ int32_t count;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row = blockIdx.y, seg = blockIdx.x, lo = seg * seg_len;
  const int cnt = V - lo < seg_len ? V - lo : seg_len;
  const T *src = logits + (size_t)row * V + lo;
  auto index_of = [&](int i) { return ((i / E) * TOPK_SEL_THREADS + tid) * E + i % E; }; // of register i, in the segment
  float v[TOPK_EPT];
#pragma unroll
  for (int c = 0; c < TOPK_EPT / E; ++c) {
    const int j = (c * TOPK_SEL_THREADS + tid) * E;
    if constexpr (VEC) {
      uint4 w = uint4{0u, 0u, 0u, 0u};
      const bool on = j < cnt; // a vector is inside or outside as a whole (V and seg_len are multiples of E)
      if (on) w = *reinterpret_cast<const uint4 *>(src + j);
      const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const float x = sizeof(T) == 2 ? bf16_to_f32((bf16_t)(ww[e / 2] >> (16 * (e & 1)))) : __uint_as_float(ww[e % 4]);
        v[c * E + e] = on ? x : -__builtin_inff();
      }
    } else {
      v[c] = j < cnt ? to_f32<T>(src[j]) : -__builtin_inff();
    }
  }
  if (tid == 0) count = 0;
  float m = v[0];
#pragma unroll
  for (int i = 1; i < TOPK_EPT; ++i) m = max_or_nan(m, v[i]);
  const float wm = wave_max_f32(m);
  if (lane == 0) wmax[wave] = wm;
  __syncthreads();
  // threshold: the wave maximum of rank k - 1 (waves without elements count as -inf, which admits every element)
  float thr;
  bool exact; // uniform over the workgroup
  {
    const float mine = wmax[lane & (TOPK_WAVES - 1)];
    exact = __any(mine != mine);
    int rank = 0;
#pragma unroll
    for (int j = 0; j < TOPK_WAVES; ++j) {
      const float o = wmax[j];
      rank += (o > mine || (o == mine && j < (lane & (TOPK_WAVES - 1)))) ? 1 : 0;
    }
    const uint64_t at = __ballot(rank == k - 1);
    thr = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mine), at != 0 ? __builtin_ctzll(at) : 0));
  }
  if (m >= thr && !exact) {
#pragma unroll
    for (int i = 0; i < TOPK_EPT; ++i) {
      const int j = index_of(i);
      if (v[i] >= thr && j < cnt) {
        const int p = atomicAdd(&count, 1);
        if (p < TOPK_LIST) list[p] = topk_key(v[i], lo + j);
      }
    }
  }
  __syncthreads();
  const int n = count;
  auto emit = [&](int rank, uint64_t key) {
    if (cand != nullptr) cand[((size_t)row * gridDim.x + seg) * k + rank] = key;
    else out[(size_t)row * k + rank] = topk_id(key);
  };
  if (cand != nullptr && tid >= cnt && tid < k) emit(tid, 0); // a last segment shorter than k
  if (!exact && n <= TOPK_LIST) {
    if (tid < n) {
      const uint64_t key = list[tid];
      int rank = 0;
#pragma unroll 8
      for (int j = 0; j < n; ++j) rank += list[j] > key ? 1 : 0; // keys are unique: the index is part of them
      if (rank < k) emit(rank, key);
    }
    return;
  }
  uint64_t prev = ~0ull; // n is uniform over the workgroup too
  for (int p = 0; p < k; ++p) {
    uint64_t best = 0;
#pragma unroll
    for (int i = 0; i < TOPK_EPT; ++i) {
      const int j = index_of(i);
      const uint64_t key = j < cnt && (nan_ranks != 0 || v[i] == v[i]) ? topk_key(v[i], lo + j) : 0;
      if (key < prev && key > best) best = key;
    }
    for (int off = 32; off > 0; off >>= 1) {
      const uint64_t o = __shfl_xor(best, off);
      best = o > best ? o : best;
    }
    if (lane == 0) wbest[wave] = best;
    __syncthreads();
    best = wbest[0];
    for (int w = 1; w < TOPK_WAVES; ++w) best = wbest[w] > best ? wbest[w] : best;
    if (tid == 0) emit(p, best);
    prev = best;
    __syncthreads();
  }
}

// one workgroup per row: the k best of n_cand keys by counting the keys above each (keys that are nothing: behind all
// others, in their own order)
__global__ __launch_bounds__(256) void k_topk_merge(const uint64_t *__restrict__ cand, int32_t n_cand, int32_t k,
                                                    int32_t *__restrict__ out) {
  __shared__ uint64_t list[TOPK_ROW_SLOTS];
  const int row = blockIdx.x;
  for (int c = threadIdx.x; c < n_cand; c += 256) list[c] = cand[(size_t)row * n_cand + c];
  __syncthreads();
  for (int c = threadIdx.x; c < n_cand; c += 256) {
    const uint64_t key = list[c];
    int rank = 0;
#pragma unroll 8
    for (int j = 0; j < n_cand; ++j) rank += list[j] > key ? 1 : 0;
    if (key == 0)
      for (int j = 0; j < c; ++j) rank += list[j] == 0 ? 1 : 0;
    if (rank < k) out[(size_t)row * k + rank] = topk_id(key);
  }
}

template <typename T>
static hipError_t topk_select(const T *logits, int32_t rows, int32_t V, int32_t k, int32_t segs, int32_t *out,
                              uint64_t *cand, KernelTimer tm, hipStream_t st) {
  constexpr int E = 16 / (int)sizeof(T);
  const int seg_len = segs == 1 ? V : ((V + segs - 1) / segs + 7) / 8 * 8; // <= TOPK_SEG, which is a multiple of 8
  const int nan_ranks = k <= TOPK_NAN_K && V >= TOPK_NAN_K && V <= TOPK_STATIC_MAX_V;
  // vectors only where each thread gets one: on shorter rows they would leave waves empty and with them no threshold
  if (V % E == 0 && (uintptr_t)logits % 16 == 0 && seg_len >= TOPK_SEL_THREADS * E)
    return launch(k_topk_select<T, true>, dim3(segs, rows), dim3(TOPK_SEL_THREADS), 0, st, tm, logits, V, k, seg_len,
                  nan_ranks, out, cand);
  return launch(k_topk_select<T, false>, dim3(segs, rows), dim3(TOPK_SEL_THREADS), 0, st, tm, logits, V, k, seg_len,
                nan_ranks, out, cand);
}

hipError_t launch_topk(const void *logits, int32_t dtype, int32_t rows, int32_t V, int32_t k, int32_t *d_topk,
                       void *d_cand, Profiler *prof, hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  const size_t esz = dtype_size(dtype);
  const int segs = (V + TOPK_SEG - 1) / TOPK_SEG;
  // A row with fewer waves than k has no threshold: all of it is listed and every element counts every other.  With more
  // rows than compute units k passes over the row are shorter than that (300 rows, k = 9: 400 elements 13.9 us against
  // 19.1, 200 13.4 / 11.1; k = 16: 700 24.9 / 30.7, 512 23.4 / 22.2; up to 128 rows the list always wins).
  const bool passes = k > TOPK_NAN_K && (V + 63) / 64 < k && V > 32 * k && rows > 256;
  if (k <= TOPK_WAVES && segs <= TOPK_MAX_SEGS && (segs == 1 || d_cand != nullptr) && !passes) {
    const int step = segs == 1 ? 65535 : TR_MAX_NODES; // the candidate scratch holds TR_MAX_NODES rows
    for (int r0 = 0; r0 < rows; r0 += step) {
      const int nr = rows - r0 < step ? rows - r0 : step;
      const char *src = (const char *)logits + (size_t)r0 * V * esz;
      int32_t *dst = d_topk + (size_t)r0 * k;
      uint64_t *cand = segs == 1 ? nullptr : (uint64_t *)d_cand;
      const KernelTimer tm = prof_next(prof, PC_TOPK);
      hipError_t e = dtype == TR_BF16 ? topk_select<bf16_t>((const bf16_t *)src, nr, V, k, segs, dst, cand, tm, st)
                                      : topk_select<float>((const float *)src, nr, V, k, segs, dst, cand, tm, st);
      if (e != hipSuccess) return e;
      if (segs > 1) {
        e = launch(k_topk_merge, dim3(nr), dim3(256), 0, st, prof_next(prof, PC_TOPK_MERGE), (const uint64_t *)d_cand,
                   segs * k, k, dst);
        if (e != hipSuccess) return e;
      }
    }
    return hipSuccess;
  }
  if (dtype == TR_BF16)
    return launch(k_topk<bf16_t>, dim3(rows), dim3(TOPK_THREADS), 0, st, prof_next(prof, PC_TOPK), (const bf16_t *)logits,
                  V, k, d_topk);
  return launch(k_topk<float>, dim3(rows), dim3(TOPK_THREADS), 0, st, prof_next(prof, PC_TOPK), (const float *)logits, V,
                k, d_topk);
}

size_t topk_scratch_bytes() { return (size_t)TR_MAX_NODES * TOPK_ROW_SLOTS * sizeof(uint64_t); }

// ---------------------------------------------------------------------------------------------
// argtopk without any allocation: the candidate scratch of rows of several segments is a file-scope device
// array (one copy per GPU, held until the process ends) instead of memory a context allocated.  In host
// code the array's name is only a stand-in: the address the kernels get comes from hipGetSymbolAddress,
// asked once per device with that device current.
// ---------------------------------------------------------------------------------------------
constexpr size_t TOPK_STATIC_BYTES = (size_t)TR_MAX_NODES * TOPK_ROW_SLOTS * sizeof(uint64_t); // 1 MiB
static __device__ __align__(256) unsigned char scratch[TOPK_STATIC_BYTES];

constexpr int MAX_DEVICES = 64;
static void *g_scratch_ptr[MAX_DEVICES];
static std::mutex g_scratch_mutex;

// Device address of this GPU's copy of `scratch`; nullptr (and *err set) if it cannot be had.
static void *static_scratch(hipError_t *err) {
  int dev = -1;
  *err = hipGetDevice(&dev);
  if (*err != hipSuccess) return nullptr;
  if (dev < 0 || dev >= MAX_DEVICES) {
    *err = hipErrorInvalidDevice;
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void *p = nullptr;
    *err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (*err != hipSuccess || p == nullptr) {
      if (*err == hipSuccess) *err = hipErrorInvalidSymbol;
      return nullptr;
    }
    g_scratch_ptr[dev] = p;
  }
  return g_scratch_ptr[dev];
}

bool topk_static_fits(int32_t rows, int32_t V, int32_t k) {
  return rows >= 0 && rows <= TR_MAX_NODES && V >= 8 && V <= TOPK_STATIC_MAX_V && k >= 1 && k <= 8;
}

hipError_t launch_topk_static(const void *logits, int32_t dtype, int32_t rows, int32_t V, int32_t k, int32_t *d_topk,
                              hipStream_t st) {
  if (!topk_static_fits(rows, V, k)) return hipErrorInvalidValue;
  hipError_t e = hipSuccess;
  void *cand = static_scratch(&e);
  if (cand == nullptr) return e;
  // every candidate slot the merge reads is written by the same call, so nothing of the previous call's
  // contents needs clearing
  return launch_topk(logits, dtype, rows, V, k, d_topk, cand, nullptr, st);
}

// ---------------------------------------------------------------------------------------------
// Matrix update (Section 3.3): M[S[i], :] = topk[i, :] for every node.  A token that occurs more
// than once is written by its last occurrence only (Appendix A.5 "Last"), which makes the result
// independent of thread scheduling.
// ---------------------------------------------------------------------------------------------
// mode: TR_UPDATE_LAST / TR_UPDATE_FIRST, which occurrence of a repeated token owns the row.
// sTok: the node tokens in LDS, 16-byte aligned, -1 for nodes that are not to be stored (from n_nodes up to the next
// multiple of 4, and off the accepted path under TR_UPDATE_ACCEPTED_ONLY).
__device__ inline void scatter_rows(int32_t *__restrict__ M, int32_t k, int n_nodes, const int32_t *sTok,
                                    const int32_t *__restrict__ topk, int i, int mode) {
  if (i >= n_nodes) return;
  const int tok = sTok[i];
  if (tok < 0) return;
  if (n_nodes == 1) { // a step of one token: nothing to compare (fetching the code that does: 3.1 us against 2.5)
    for (int c = 0; c < k; ++c) M[(size_t)tok * k + c] = topk[(size_t)i * k + c];
    return;
  }
  int32_t row[8];
  if (k == 8) __builtin_memcpy(row, topk + (size_t)i * 8, 32); // on its way while the occurrences are compared
  int lo = TR_MAX_NODES, hi = -1; // first and last occurrence
#pragma unroll 4
  for (int j0 = 0; j0 < n_nodes; j0 += 4) {
    const int4 t = *reinterpret_cast<const int4 *>(sTok + j0);
    const int tt[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) hi = tt[e] == tok ? j0 + e : hi;
#pragma unroll
    for (int e = 3; e >= 0; --e) lo = (tt[e] == tok && lo > j0 + e) ? j0 + e : lo;
  }
  if (((mode & 1) == TR_UPDATE_FIRST ? lo : hi) != i) return;
  if (k == 8) __builtin_memcpy(M + (size_t)tok * 8, row, 32);
  else
    for (int c = 0; c < k; ++c) M[(size_t)tok * k + c] = topk[(size_t)i * k + c];
}

__global__ __launch_bounds__(TR_MAX_NODES) void k_matrix_update(int32_t *__restrict__ M, int32_t V, int32_t k,
                                                                int32_t n_nodes, const int32_t *__restrict__ S,
                                                                const int32_t *__restrict__ topk, int32_t mode) {
  __shared__ __align__(16) int32_t sS[TR_MAX_NODES];
  const int i = threadIdx.x;
  int t = i < n_nodes ? S[i] : -1;
  if (i < n_nodes) t = t < 0 ? 0 : (t >= V ? V - 1 : t);
  sS[i] = t;
  __syncthreads();
  scatter_rows(M, k, n_nodes, sS, topk, i, mode); // no path here: every node is eligible
}

hipError_t launch_matrix_update(const tr_ctx *c, const int32_t *d_S, const int32_t *d_topk, hipStream_t st) {
  return launch(k_matrix_update, dim3(1), dim3(TR_MAX_NODES), 0, st, KernelTimer{}, c->d_M, c->V, c->k, c->tree.n_nodes,
                d_S, d_topk, c->update_mode);
}

// ---------------------------------------------------------------------------------------------
// KV compaction: the accepted path's keys/values (written by the forward at L + node index) move
// to L + 0..a.  One workgroup of 256 threads per (layer, kv head); all sources are staged in LDS before any
// destination is written, so overlapping source/destination positions are safe.
//   K: [layers][Hkv][cap][hd]   V: [layers][Hkv][hd][cap]
// ---------------------------------------------------------------------------------------------
// blk = layer * Hkv + head; path in LDS; sk: LDS for 2 * TR_MAX_LAYERS * hd elements
template <typename T>
__device__ inline void compact_head(T *__restrict__ K, T *__restrict__ Vt, size_t blk, int32_t cap, int32_t hd, int32_t tiled, int L,
                                    int a, const int32_t *path, T *sk) {
  const int tid = threadIdx.x;
  T *sv = sk + (size_t)TR_MAX_LAYERS * hd;           // [a+1][hd] both
  T *Kb = K + blk * (size_t)cap * hd;
  T *Vb = Vt + blk * (size_t)hd * cap;
  const int total = (a + 1) * hd;
  constexpr int U = 4; // elements of both a thread has in flight
  for (int e0 = tid; e0 < total; e0 += U * 256) {
    T tk[U], tv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * 256 < total ? e0 + u * 256 : e0;
      const int i = e / hd, d = e - i * hd;
      const int src = L + path[i];
      tk[u] = Kb[tiled ? kv_k_index(src, d) : (size_t)src * hd + d];
      tv[u] = Vb[tiled ? kv_v_index(src, d) : (size_t)d * cap + src];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * 256;
      if (e < total) {
        sk[e] = tk[u];
        sv[e] = tv[u];
      }
    }
  }
  __syncthreads();
  for (int e = tid; e < total; e += 256) {
    const int i = e / hd, d = e - i * hd;
    const int dst = L + i;
    Kb[tiled ? kv_k_index(dst, d) : (size_t)dst * hd + d] = sk[e];
    Vb[tiled ? kv_v_index(dst, d) : (size_t)d * cap + dst] = sv[e];
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_compact_kv(T *__restrict__ K, T *__restrict__ Vt, int32_t cap, int32_t hd,
                                                    int32_t tiled, const tr_step_out *__restrict__ out) {
  extern __shared__ unsigned char smem_raw[];
  __shared__ int32_t path[TR_MAX_LAYERS];
  const int a = out->n_accepted, L = out->kv_len - a - 1; // the committed length before the step
  if (threadIdx.x < TR_MAX_LAYERS) path[threadIdx.x] = out->path[threadIdx.x]; // asked for together with the two scalars
  if (a == 0) return;                                                         // root already sits at L
  __syncthreads();
  compact_head<T>(K, Vt, blockIdx.x, cap, hd, tiled, L, a, path, reinterpret_cast<T *>(smem_raw));
}

// ---------------------------------------------------------------------------------------------
// Greedy accept + matrix update in one workgroup (Section 3.3 with the chain rule of Section 2.2).
// match bit i  = draft token i equals the model output at its parent (root: always)
// node i is ok = every bit of its ancestor mask is a match bit
// winner       = deepest ok node, smallest index among equals
// host: the same result in pinned memory of the context, when the caller waits for it: a copy kernel and its staging on the
// host less per step (whole request on the tiny model, 19 steps: 2.11 -> 1.70 ms).
// The kernel also advances *d_len; the compaction kernel that follows takes the length before the step from the published result.
// Where the compaction has few workgroups they are blocks 1 .. of this launch: each finds the winner for itself and takes the length
// with an atomic add that counts it in the bits above LEN_BITS, and the last to do so replaces the count by what was accepted
// (about 20 ns a block).  Nothing of either form stays behind: accepts into different caches may overlap on the device.
// Two waves; what bounds it is the chain load -> barrier -> match -> barrier -> winner -> stores.  Every thread
// places its own node: a node on the winner's path is entry popcount(path bits below it) of the path, and repeated
// tokens are compared four at a time.  With one thread walking the 80 nodes for the path and every thread walking them
// for the repeats the launch took 15.6 us (21.9 at 128 nodes).
// ---------------------------------------------------------------------------------------------
constexpr int LEN_BITS = 25;
template <typename T, bool COMPACT>
__global__ __launch_bounds__(COMPACT ? 256 : TR_MAX_NODES) void k_accept_update(const int32_t *__restrict__ S,
                                                                const int32_t *__restrict__ topk,
                                                                const int32_t *__restrict__ tokens,
                                                                const uint64_t *__restrict__ anc,
                                                                const int32_t *__restrict__ depth,
                                                                const int32_t *__restrict__ parent, int32_t n_nodes, int32_t k,
                                                                int32_t *__restrict__ d_len, int32_t V,
                                                                int32_t *__restrict__ M, tr_step_out *__restrict__ out,
                                                                tr_step_out *__restrict__ host, int32_t mode,
                                                                T *__restrict__ K, T *__restrict__ Vt, int32_t cap, int32_t hd,
                                                                int32_t tiled) {
  __shared__ __align__(16) int32_t sS[TR_MAX_NODES];
  __shared__ int32_t sOut[TR_MAX_NODES];
  __shared__ uint64_t sAnc[TR_MAX_NODES][2];
  __shared__ uint64_t mbits[2];
  __shared__ int32_t wkey[2];
  __shared__ int32_t sL;
  const int i = threadIdx.x;
  const bool live = i < n_nodes;
  // everything that does not depend on the match is loaded up front, in one round trip
  const uint64_t anc0 = live ? anc[2 * i] : 0, anc1 = live ? anc[2 * i + 1] : 0;
  const int dep = live ? depth[i] : 0;
  const int par = live && i > 0 ? parent[i] : 0;
  int L0 = 0;
  uint32_t before = 0; // blocks that took the length before this one
  if (i == 0) {
    if constexpr (COMPACT) {
      const uint32_t got = atomicAdd(reinterpret_cast<uint32_t *>(d_len), 1u << LEN_BITS);
      L0 = (int)(got & ((1u << LEN_BITS) - 1));
      before = got >> LEN_BITS;
    } else {
      L0 = *d_len;
    }
  }
  int tk = -1;
  if (live) {
    tk = S[i];
    // the token the model emits at node i: its argmax, or the caller's draw under temperature sampling
    int ot = tokens != nullptr ? tokens[i] : topk[(size_t)i * k];
    tk = tk < 0 ? 0 : (tk >= V ? V - 1 : tk);
    sOut[i] = ot < 0 ? 0 : (ot >= V ? V - 1 : ot);
  }
  if (!COMPACT || i < TR_MAX_NODES) {
    sS[i] = tk;
    sAnc[i][0] = anc0;
    sAnc[i][1] = anc1;
  }
  if (COMPACT && i == 0) sL = L0;
  __syncthreads();
  const bool match = live && (i == 0 || tk == sOut[par]);
  const uint64_t ballot = __ballot(match);
  if ((i & 63) == 0 && i < TR_MAX_NODES) mbits[i >> 6] = ballot;
  __syncthreads();
  const bool ok = live && ((mbits[0] & anc0) == anc0) && ((mbits[1] & anc1) == anc1);
  int key = ok ? dep * 256 + (255 - i) : -1; // the root is always ok
  for (int off = 32; off > 0; off >>= 1) {
    const int o = __shfl_xor(key, off);
    key = o > key ? o : key;
  }
  if ((i & 63) == 0 && i < TR_MAX_NODES) wkey[i >> 6] = key;
  __syncthreads();
  key = wkey[0] > wkey[1] ? wkey[0] : wkey[1];
  const int w = 255 - (key & 255), a = key >> 8;
  const uint64_t p0 = sAnc[w][0], p1 = sAnc[w][1];
  // ancestors in increasing index order are the path root..winner (breadth-first numbering)
  const bool on_path = live && ((i < 64 ? p0 >> i : p1 >> (i - 64)) & 1ull) != 0;
  const int at = !live ? 0 : i < 64 ? __popcll(p0 & ((1ull << i) - 1)) : __popcll(p0) + __popcll(p1 & ((1ull << (i - 64)) - 1));
  auto publish = [&](tr_step_out *o) {
    if (on_path) {
      o->path[at] = i;
      if (at > 0) o->emitted[at - 1] = tk;
    }
    if (i > a && i < TR_MAX_LAYERS) {
      o->path[i] = -1;
      o->emitted[i] = -1;
    }
    if (i == 0) {
      const int bonus = sOut[w];
      o->emitted[a] = bonus;
      o->n_accepted = a;
      o->n_emitted = a + 1;
      o->winner = w;
      o->next_root = bonus;
      o->kv_len = L0 + a + 1;
    }
  };
  if constexpr (COMPACT) {
    if (i == 0 && before == gridDim.x - 1) atomicAdd(reinterpret_cast<uint32_t *>(d_len), (uint32_t)(a + 1) - (gridDim.x << LEN_BITS));
    if (blockIdx.x > 0) {
      if (a == 0) return; // root already sits at L
      extern __shared__ unsigned char smem_raw[];
      __shared__ int32_t path[TR_MAX_LAYERS];
      if (on_path) path[at] = i;
      __syncthreads();
      compact_head<T>(K, Vt, blockIdx.x - 1, cap, hd, tiled, sL, a, path, reinterpret_cast<T *>(smem_raw));
      return;
    }
  }
  publish(out);
  if (host != nullptr) publish(host);
  if (!COMPACT && i == 0) *d_len = L0 + a + 1;
  if ((mode & TR_UPDATE_ACCEPTED_ONLY) != 0) { // uniform
    __syncthreads();
    if (!on_path && i < TR_MAX_NODES) sS[i] = -1;
    __syncthreads();
  }
  scatter_rows(M, k, n_nodes, sS, topk, i, mode);
}

// ---------------------------------------------------------------------------------------------
// Temperature sampling (Section 5.3): the token drawn at node i is
//   argmax_j ( logits[i][j] * inv_t + noise[L + depth(i) - pos0][j] ),   ties to the smallest j,
// i.e. a draw from softmax(logits / T) when the noise is standard Gumbel.  The two float32 operations
// are kept separate (no fused multiply-add): they decide an integer, and whoever repeats them rounds
// the same way.  One workgroup of 16 waves per node (4 for short rows); a thread has U vectors of both rows in flight, which is what
// counts (every node's compute unit pulls two rows of V floats): 128 nodes x 32000 took 39 us with 4 waves and one
// element of each row in flight, 9.3 now.  VEC: 16-byte loads (V a multiple of 4, both bases aligned).  A NaN is never
// drawn (it is no candidate, so it cannot stand in a thread's or a wave's place either); a row of nothing else gives 0.
// ---------------------------------------------------------------------------------------------
template <bool VEC, int THREADS>
__global__ __launch_bounds__(THREADS) void k_sample_tokens(const float *__restrict__ logits,
                                                                  const float *__restrict__ noise, int32_t V, int32_t pos0,
                                                                  int32_t noise_rows, float inv_t,
                                                                  const int32_t *__restrict__ depth,
                                                                  const int32_t *__restrict__ d_len,
                                                                  int32_t *__restrict__ tokens) {
  constexpr int E = VEC ? 4 : 1, U = 4;
  __shared__ float sv[THREADS / 64];
  __shared__ int32_t si[THREADS / 64];
  const int i = blockIdx.x;
  int row = *d_len + depth[i] - pos0;
  row = row < 0 ? 0 : (row >= noise_rows ? noise_rows - 1 : row); // the host checked the range; never read outside
  const float *lg = logits + (size_t)i * V;
  const float *nz = noise + (size_t)row * V;
  float best = -__builtin_huge_valf();
  int bj = 0x7fffffff;
  for (int j0 = threadIdx.x * E; j0 < V; j0 += THREADS * E * U) {
    float a[U][E], b[U][E];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = j0 + u * THREADS * E;
      const int jc = j < V ? j : j0; // past the end: an element seen before, skipped below
      __builtin_memcpy(a[u], lg + jc, sizeof(a[u]));
      __builtin_memcpy(b[u], nz + jc, sizeof(b[u]));
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int j = j0 + u * THREADS * E + e;
        const float y = __fadd_rn(__fmul_rn(a[u][e], inv_t), b[u][e]);
        if (j < V && (y > best || (bj == 0x7fffffff && y == y))) { // j grows, so on equal values the earlier index stays
          best = y;
          bj = j;
        }
      }
  }
  auto merge = [&](float ov, int oi) {
    if (oi != 0x7fffffff && (bj == 0x7fffffff || ov > best || (ov == best && oi < bj))) {
      best = ov;
      bj = oi;
    }
  };
  for (int off = 32; off > 0; off >>= 1) {
    const float ov = __shfl_xor(best, off);
    const int oi = __shfl_xor(bj, off);
    merge(ov, oi);
  }
  if ((threadIdx.x & 63) == 0) {
    sv[threadIdx.x >> 6] = best;
    si[threadIdx.x >> 6] = bj;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < THREADS / 64; ++w) merge(sv[w], si[w]);
    tokens[i] = bj != 0x7fffffff ? bj : 0;
  }
}

hipError_t launch_sample_tokens(tr_ctx *c, const tr_kv *kv, const float *d_logits, const float *d_noise,
                                int32_t pos0, int32_t noise_rows, float inv_t, int32_t *d_tokens, hipStream_t st) {
  const bool vec = c->V % 4 == 0 && (uintptr_t)d_logits % 16 == 0 && (uintptr_t)d_noise % 16 == 0;
  // short rows: four waves have all of it under way at once, and fewer meet at the end (80 nodes x 1000: 3.7 us against 4.2
  // with 16 waves, x 4096 4.15 / 5.8; the kernel before, four waves with an element each: 3.9 and 5.6)
  const bool few = c->V <= 4096;
  auto kernel = few ? (vec ? k_sample_tokens<true, 256> : k_sample_tokens<false, 256>)
                    : (vec ? k_sample_tokens<true, 1024> : k_sample_tokens<false, 1024>);
  return launch(kernel, dim3(c->tree.n_nodes), dim3(few ? 256 : 1024), 0, st, c->prof.next(PC_SAMPLE), d_logits, d_noise,
                c->V, pos0, noise_rows, inv_t, c->tree.depth, kv->d_len, d_tokens);
}

// Up to this many (layer, kv head) blocks are compacted by the accepting launch itself.  us an accept of 5 drafts (80 nodes) or 3 (15) in a graph of 40, two
// launches / one: 80 nodes, 8 blocks 8.2 / 4.7, 16 blocks 8.6 / 4.7, 32 blocks 8.7 / 4.8; 15 nodes, 8 and 32 blocks 7.0 / 4.0 and 7.4 / 4.5.  A
// step of the tiny model (8 blocks): 15 nodes 71.5 / 69.4, 80 nodes 85.2 / 81.8.  One launch is the faster with 40, 64 and 96 blocks too (8.9 / 4.9,
// 8.9 / 5.1, 9.0 / 5.5); more than 32 have not been compared in whole steps and stay.
constexpr int ACCEPT_COMPACT_BLOCKS = 32;
template <typename T>
static hipError_t launch_accept_t(tr_ctx *c, const tr_kv *kv, const int32_t *d_S, const int32_t *d_topk, const int32_t *d_tokens,
                                  tr_step_out *d_out, tr_step_out *host_out, hipStream_t st) {
  const int blocks = kv->n_layers * kv->n_kv_heads;
  const size_t smem = 2 * (size_t)TR_MAX_LAYERS * kv->head_dim * sizeof(T);
  auto accept = [&](auto kernel, int grid, int threads, size_t lds) {
    return launch(kernel, dim3(grid), dim3(threads), lds, st, c->prof.next(PC_ACCEPT), d_S, d_topk, d_tokens, c->tree.anc, c->tree.depth,
                  c->tree.parent, c->tree.n_nodes, c->k, kv->d_len, c->V, c->d_M, d_out, host_out, c->update_mode, (T *)kv->k,
                  (T *)kv->v, kv->capacity, kv->head_dim, kv->layout);
  };
  static_assert(ACCEPT_COMPACT_BLOCKS + 1 < 1 << (32 - LEN_BITS), "the count of blocks fits above the length");
  if (blocks <= ACCEPT_COMPACT_BLOCKS && smem <= 32768 && kv->capacity < 1 << LEN_BITS)
    return accept(k_accept_update<T, true>, 1 + blocks, 256, smem);
  const hipError_t e = accept(k_accept_update<T, false>, 1, TR_MAX_NODES, 0);
  if (e != hipSuccess) return e;
  return launch(k_compact_kv<T>, dim3(blocks), dim3(256), smem, st, c->prof.next(PC_COMPACT), (T *)kv->k, (T *)kv->v, kv->capacity,
                kv->head_dim, kv->layout, d_out);
}

hipError_t launch_accept_update(tr_ctx *c, const tr_kv *kv, const int32_t *d_S, const int32_t *d_topk,
                                const int32_t *d_tokens, tr_step_out *d_out, tr_step_out *host_out, hipStream_t st) {
  return kv->dtype == TR_BF16 ? launch_accept_t<bf16_t>(c, kv, d_S, d_topk, d_tokens, d_out, host_out, st)
                              : launch_accept_t<float>(c, kv, d_S, d_topk, d_tokens, d_out, host_out, st);
}

// ---------------------------------------------------------------------------------------------
// Plain streaming kernels (measurement aids): a read-only pass and a copy over `slots` 16-byte slots,
// 256 workgroups of 512 threads, 4 independent nontemporal loads per thread in flight.
// ---------------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4s;
__global__ __launch_bounds__(512) void k_stream_read(const u32x4s *__restrict__ src, size_t slots, uint32_t *sink) {
  u32x4s acc = {0u, 0u, 0u, 0u};
  const size_t stride = (size_t)gridDim.x * 512;
  for (size_t i = (size_t)blockIdx.x * 512 + threadIdx.x; i < slots; i += 4 * stride) {
    u32x4s v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = i + u * stride < slots ? __builtin_nontemporal_load(src + i + u * stride) : u32x4s{0u, 0u, 0u, 0u};
#pragma unroll
    for (int u = 0; u < 4; ++u) acc ^= v[u];
  }
  if ((acc.x ^ acc.y ^ acc.z ^ acc.w) == 0x9E3779B9u && sink != nullptr) sink[0] = 1u; // keeps the loads alive
}
__global__ __launch_bounds__(512) void k_stream_copy(const u32x4s *__restrict__ src, u32x4s *__restrict__ dst, size_t slots) {
  const size_t stride = (size_t)gridDim.x * 512;
  for (size_t i = (size_t)blockIdx.x * 512 + threadIdx.x; i < slots; i += 4 * stride) {
    u32x4s v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = i + u * stride < slots ? __builtin_nontemporal_load(src + i + u * stride) : u32x4s{0u, 0u, 0u, 0u};
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i + u * stride < slots) __builtin_nontemporal_store(v[u], dst + i + u * stride);
  }
}
hipError_t launch_stream(const void *src, void *dst, size_t bytes, hipStream_t st) {
  const size_t slots = bytes / 16;
  if (dst == nullptr)
    return launch(k_stream_read, dim3(256), dim3(512), 0, st, KernelTimer{}, (const u32x4s *)src, slots, (uint32_t *)nullptr);
  return launch(k_stream_copy, dim3(256), dim3(512), 0, st, KernelTimer{}, (const u32x4s *)src, (u32x4s *)dst, slots);
}

__global__ void k_advance_len(int32_t *d_len, int32_t by) { *d_len += by; }

hipError_t launch_advance_len(int32_t *d_len, int32_t by, hipStream_t st) {
  return launch(k_advance_len, dim3(1), dim3(1), 0, st, KernelTimer{}, d_len, by);
}

} // namespace tr
