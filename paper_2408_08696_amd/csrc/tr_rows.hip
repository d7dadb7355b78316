// Shape-generic projections on row-major weights, float32 or bf16, any sizes: y[n, O] = a[n, K] * w[O, K]^T with the
// normalisation before it and the activation, rotation or residual add after it in the same launch.  They serve the
// small models (two layers of width 128: 0.5 M weights), whose step is a chain of launches with hardly any work in
// each, so what bounds them is the number of launches and the memory round trips inside one, not bytes or flops.
//
// A workgroup of four waves owns one tile of 16 outputs and RT tiles of 16 rows; the waves take interleaved k-steps of
// 64 bytes of each row (the 16x16 matrix-core product of the element type: 4 x v_mfma_f32_16x16x4_f32 or one
// v_mfma_f32_16x16x32_bf16, A = weights, B = activations, lane l supplying 16 bytes of row l % 16 at k-offset
// 16 (l / 16) bytes of both) and load all they can before the first product, so that a launch is one round trip up to 24
// k-steps with one row tile, 16 with two and 12 with four.  The four partial sums meet in LDS.  Lane l then holds outputs 4 (l / 16) .. + 3 of row l % 16.
// A k-step is summed on its own (float32: its four products in a tree) and added to one of as many running sums as a wave
// loads k-steps ahead, so that no result is the end of a long chain: relative error against float64 at K = 512 / 4096 in
// float32 8.4e-8 / 1.03e-7, with one running sum per wave 2.1e-7 / 5.8e-7 and a wave per output 8.6e-8 / 1.6e-7; the tiny
// model's logits 1.8e-7, 2.5e-7 and 2.1e-7.  It costs up to a third where the products are the time (64 rows, 4096 -> 4096
// 44 -> 61 us; a wave per output 159) and nothing on the tiny model.
//   prologue  RMSNorm: the operand is T(x * gain), the row's scale 1 / sqrt(mean(x^2) + eps) is collected from the same
//             loads and applied to the sums (it is a scalar per row).
//   epilogues store, residual add into x, SwiGLU, and RoPE with the query / cache writes.  For the last two the tile's
//             outputs are chosen in pairs that belong together (gate and up of a feature; the two features a rotation
//             mixes), placed so that a pair is in one lane: outputs 0, 1 of a lane's four are the first members,
//             outputs 2, 3 their partners.
// Against one wave per output with the same 16 rows (each weight loaded once per 16 rows by 64 lanes along k, a
// shuffle reduction per row, normalisation / rotation / activation / q, k and v in launches of their own): a layer of
// the tiny model took 12 launches and 66 us, now 5.
#include "tr_kernels.h"

namespace tr {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr int ROWS_WAVES = 4;

// 16 bytes of a row from element k on; what lies at or beyond K is zero.  Rows start on any element.
template <typename T>
__device__ inline u32x4 load_chunk(const T *row, int k, int K) {
  constexpr int E = 16 / (int)sizeof(T);
  u32x4 v = u32x4{0u, 0u, 0u, 0u};
  if (k + E <= K) {
    __builtin_memcpy(&v, row + k, 16);
  } else if (k < K) {
    T e[E];
#pragma unroll
    for (int i = 0; i < E; ++i) e[i] = k + i < K ? row[k + i] : (T)0;
    __builtin_memcpy(&v, e, 16);
  }
  return v;
}

// the sum of one k-step, on its own
__device__ inline f32x4 product(float, const u32x4 &w, const u32x4 &a) {
  f32x4 c[4];
#pragma unroll
  for (int e = 0; e < 4; ++e)
    c[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w[e]), __uint_as_float(a[e]), f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
  return (c[0] + c[1]) + (c[2] + c[3]);
}
__device__ inline f32x4 product(bf16_t, const u32x4 &w, const u32x4 &a) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, a),
                                                 f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
}

// T(x * gain) of E elements from k on, and the sum of their squares
template <typename T>
__device__ inline u32x4 normed_chunk(const float *x, const T *gain, int k, int K, float &ss) {
  constexpr int E = 16 / (int)sizeof(T);
  const u32x4 gv = load_chunk<T>(gain, k, K);
  T out[E];
  float sq[E];
  if constexpr (sizeof(T) == 4) {
    const u32x4 xv = load_chunk<float>(x, k, K);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float v = __uint_as_float(xv[e]);
      sq[e] = v * v;
      out[e] = v * __uint_as_float(gv[e]);
    }
  } else {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const u32x4 xv = load_chunk<float>(x, k + 4 * h, K);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float v = __uint_as_float(xv[e]);
        const uint32_t gw = gv[(4 * h + e) >> 1];
        sq[4 * h + e] = v * v;
        out[4 * h + e] = f32_to_bf16(v * bf16_to_f32((bf16_t)(e & 1 ? gw >> 16 : gw & 0xFFFFu)));
      }
    }
  }
#pragma unroll
  for (int s = E / 2; s > 0; s /= 2)
#pragma unroll
    for (int e = 0; e < s; ++e) sq[e] += sq[e + s];
  ss += sq[0];
  u32x4 r;
  __builtin_memcpy(&r, out, 16);
  return r;
}

// What the loads need leads the arguments: 14 words, which come in scalar registers with the wave.  n_hd: n, with ROWS_ROPE n + 2^16 hd.
template <typename T, int RT, bool NORM, int EPI>
__global__ __launch_bounds__(ROWS_WAVES * 64) void k_rows(const void *a, const void *gain, const void *w0, const void *w1, const void *w2,
                                                          int32_t K, int32_t O, int32_t n_hd, int32_t H, RowsArgs p) {
  constexpr int E = 16 / (int)sizeof(T), KSTEP = 4 * E;
  constexpr int PF = RT == 1 ? 6 : (RT == 2 ? 4 : 3); // k-steps a wave loads before it multiplies
  __shared__ f32x4 part[ROWS_WAVES][RT][64];
  __shared__ float ssq[ROWS_WAVES][RT * 16];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int r = lane & 15, g = lane >> 4;
  const int tile = blockIdx.x, row0 = blockIdx.y * RT * 16;

  const int n = EPI == ROWS_ROPE ? n_hd & 0xFFFF : n_hd;

  // the weight row this lane loads: output r of the tile (outputs past the end repeat the last one, never stored)
  const T *wrow;
  {
    const int pair = tile * 8 + 2 * (r >> 2) + (r & 1), second = (r >> 1) & 1;
    if (EPI == ROWS_ROPE) {
      const int hd = n_hd >> 16, half = hd / 2, pc = pair < O / 2 ? pair : O / 2 - 1, Hkv = (O / hd - H) / 2;
      const int head = pc / half, i = pc - head * half + second * half;
      const int seg = head < H ? 0 : (head < H + Hkv ? 1 : 2);
      const int base = seg == 0 ? 0 : (seg == 1 ? H : H + Hkv);
      wrow = (const T *)(seg == 0 ? w0 : seg == 1 ? w1 : w2) + (size_t)((head - base) * hd + i) * K;
    } else if (EPI == ROWS_SWIGLU) {
      const int f = pair < O ? pair : O - 1;
      wrow = (const T *)(second ? w1 : w0) + (size_t)f * K;
    } else {
      const int o = tile * 16 + r < O ? tile * 16 + r : O - 1;
      wrow = (const T *)w0 + (size_t)o * K;
    }
  }
  size_t arow[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const int row = row0 + 16 * t + r;
    arow[t] = (size_t)(row < n ? row : n - 1) * K;
  }
  f32x4 acc[PF][RT];
  float ss[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
#pragma unroll
    for (int s = 0; s < PF; ++s) acc[s][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    ss[t] = 0.f;
  }
  for (int k0 = wave * KSTEP; k0 < K; k0 += ROWS_WAVES * PF * KSTEP) {
    u32x4 wq[PF], aq[PF][RT];
#pragma unroll
    for (int j = 0; j < PF; ++j) {
      const int k = k0 + j * ROWS_WAVES * KSTEP + g * E;
      wq[j] = load_chunk<T>(wrow, k, K);
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        if constexpr (NORM) aq[j][t] = normed_chunk<T>((const float *)a + arow[t], (const T *)gain, k, K, ss[t]);
        else aq[j][t] = load_chunk<T>((const T *)a + arow[t], k, K);
      }
    }
#pragma unroll
    for (int j = 0; j < PF; ++j)
#pragma unroll
      for (int t = 0; t < RT; ++t) acc[j][t] += product(T{}, wq[j], aq[j][t]);
  }
#pragma unroll
  for (int t = 0; t < RT; ++t) {
#pragma unroll
    for (int s = 1; s < PF; s *= 2) // pairs, then pairs of those
#pragma unroll
      for (int i = 0; i + s < PF; i += 2 * s) acc[i][t] += acc[i + s][t];
    part[wave][t][lane] = acc[0][t];
    if (NORM) {
      float s = ss[t];
      s += __shfl_xor(s, 16);
      s += __shfl_xor(s, 32);
      if (lane < 16) ssq[wave][t * 16 + lane] = s;
    }
  }
  __syncthreads();

  for (int t = wave; t < RT; t += ROWS_WAVES) {
    const int row = row0 + 16 * t + r;
    if (row >= p.n) continue;
    f32x4 v = (part[0][t][lane] + part[1][t][lane]) + (part[2][t][lane] + part[3][t][lane]);
    if (NORM) {
      const float s = (ssq[0][t * 16 + r] + ssq[1][t * 16 + r]) + (ssq[2][t * 16 + r] + ssq[3][t * 16 + r]);
      v *= 1.0f / sqrtf(s / (float)p.K + p.eps);
    }
    if (EPI == ROWS_STORE || EPI == ROWS_ADD) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int o = tile * 16 + 4 * g + e;
        if (o < p.O) {
          float *dst = p.y + (size_t)row * p.ldy + o;
          *dst = EPI == ROWS_ADD ? *dst + v[e] : v[e];
        }
      }
    } else if (EPI == ROWS_SWIGLU) {
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int f = tile * 8 + 2 * g + e;
        if (f < p.O) ((T *)p.h)[(size_t)row * p.O + f] = from_f32<T>(v[e] / (1.0f + expf(-v[e])) * v[2 + e]);
      }
    } else {
      const int half = p.hd / 2, pos = *p.d_len + row;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int pair = tile * 8 + 2 * g + e;
        if (pair >= p.O / 2) continue;
        const int head = pair / half, i = pair - head * half;
        float a = v[e], b = v[2 + e];
        if (head < p.H + p.Hkv) {
          const float c = p.rope[(size_t)row * p.hd + i], sn = p.rope[(size_t)row * p.hd + half + i];
          const float ra = a * c - b * sn, rb = b * c + a * sn;
          a = ra;
          b = rb;
        }
        const T ta = from_f32<T>(a), tb = from_f32<T>(b);
        if (head < p.H) {
          T *dst = (T *)p.q + ((size_t)row * p.H + head) * p.hd;
          dst[i] = ta;
          dst[i + half] = tb;
        } else if (head < p.H + p.Hkv) {
          T *dst = (T *)p.k_layer + (size_t)(head - p.H) * p.cap * p.hd;
          dst[p.tiled ? kv_k_index(pos, i) : (size_t)pos * p.hd + i] = ta;
          dst[p.tiled ? kv_k_index(pos, i + half) : (size_t)pos * p.hd + i + half] = tb;
        } else {
          T *dst = (T *)p.v_layer + (size_t)(head - p.H - p.Hkv) * p.hd * p.cap;
          dst[p.tiled ? kv_v_index(pos, i) : (size_t)i * p.cap + pos] = ta;
          dst[p.tiled ? kv_v_index(pos, i + half) : (size_t)(i + half) * p.cap + pos] = tb;
        }
      }
    }
  }
}

template <typename T, bool NORM, int EPI>
static hipError_t launch_rows_rt(const RowsArgs &p, hipStream_t st, KernelTimer tm) {
  const int NT = (p.n + 15) / 16;
  if (EPI == ROWS_ROPE && (p.n > 0xFFFF || p.hd > 0x7FFF)) return hipErrorInvalidValue; // a step: at most TR_MAX_NODES rows
  const int32_t n_hd = EPI == ROWS_ROPE ? p.n + (p.hd << 16) : p.n;
  const int tiles = EPI == ROWS_SWIGLU ? (p.O + 7) / 8 : (p.O + 15) / 16;
  // More row tiles a workgroup read a weight less often, but a wave's loads and products per k-step are as many more, and that
  // chain is the launch's time while every workgroup has a compute unit to itself: the fewest that still do so.  float32, 64
  // rows, us with four tiles / one: 512 -> 512 9.5 / 6.5, 2048 -> 512 22.9 / 14.3 (a wave per output: 8.5 and 19.4).
  auto go = [&](auto kernel, int row_blocks) {
    return launch(kernel, dim3(tiles, row_blocks), dim3(ROWS_WAVES * 64), 0, st, tm, p.a, p.gain, p.w[0], p.w[1], p.w[2], p.K, p.O, n_hd,
                  p.H, p);
  };
  if (NT == 1 || tiles * NT <= 256) return go(k_rows<T, 1, NORM, EPI>, NT);
  if (NT == 2 || tiles * ((NT + 1) / 2) <= 256) return go(k_rows<T, 2, NORM, EPI>, (NT + 1) / 2);
  return go(k_rows<T, 4, NORM, EPI>, (NT + 3) / 4);
}

template <typename T>
static hipError_t launch_rows_t(const RowsArgs &p, hipStream_t st, KernelTimer tm) {
  switch (p.epilogue) {
  case ROWS_STORE:
    return p.gain != nullptr ? launch_rows_rt<T, true, ROWS_STORE>(p, st, tm) : launch_rows_rt<T, false, ROWS_STORE>(p, st, tm);
  case ROWS_ADD: return p.gain != nullptr ? hipErrorInvalidValue : launch_rows_rt<T, false, ROWS_ADD>(p, st, tm);
  case ROWS_SWIGLU: return p.gain == nullptr ? hipErrorInvalidValue : launch_rows_rt<T, true, ROWS_SWIGLU>(p, st, tm);
  case ROWS_ROPE: return p.gain == nullptr ? hipErrorInvalidValue : launch_rows_rt<T, true, ROWS_ROPE>(p, st, tm);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_rows(const RowsArgs &p, int32_t dtype, hipStream_t st, KernelTimer tm) {
  if (p.n < 1 || p.K < 1 || p.O < 1) return hipErrorInvalidValue;
  return dtype == TR_BF16 ? launch_rows_t<bf16_t>(p, st, tm) : launch_rows_t<float>(p, st, tm);
}

} // namespace tr
