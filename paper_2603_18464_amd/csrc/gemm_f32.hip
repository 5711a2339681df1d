// float32 GEMM of the float32 configuration:  C[M,N] = A[M,K] * W[N,K]^T  with the layer's elementwise work on both sides
// of the product: RMSNorm of the A rows before it; residual add, SwiGLU, or rotary embedding + KV-cache write after it.
//
// The models of this path are small (K of a few hundred), so a launch is bound by latency: launch ramp, one or two
// rounds of loads, the reduction.  Hence one workgroup per 16 rows x 16 columns (or 16 + 16 paired ones), its four
// waves each take a quarter of K, request all of it at once, and add their partial tiles through LDS in a fixed order.
// The product runs on v_mfma_f32_16x16x4_f32 (full float32, the vector rate): a lane's operands are four consecutive k
// of one row, one 16-byte load, and no LDS staging is needed.  Many rows take 32-row tiles, which halves the weight
// reads from L2; the order of every sum is the same, so a row's bits do not depend on the batch it is in.
// Policy step of the 2-layer model (4 sequences of 32 tokens, 7 tokens out): 3.18 ms with 64 x 64 tiles of scalar FMAs
// (4 workgroups on N = 256, 33 to 78 us a launch) and the norms, rotation, SwiGLU and residual adds as launches of their
// own (11 a layer); 0.40 ms with these (5 a layer); 0.36 with what the epilogues read requested before the product and all
// of a down projection's operands (11 k-steps a wave) in one round instead of two, the attention's keys and values together and
// lane sums in the vector unit.
#include "common.h"

namespace vla {

// Columns of a tile: tile t covers W rows col(t) .. + 15 and, for kNT == 2, + second() .. + 15; store() gets element
// (m, c) of them.  kNT == 2 pairs the columns an elementwise step needs together.  What store() needs from memory is
// requested by index() and fetch() before the product, behind the operands: at the end it would be one or two more
// latencies of a launch that is made of them.
struct F32Resid {
  static constexpr int kNT = 1;
  struct Index {};
  struct Fetched { float x; };
  __device__ Index index(int) const { return {}; }
  __device__ Fetched fetch(int m, int t, int c, const Index&) const { return {x[(size_t)m * ldx + min(t * 16 + c, n - 1)]}; }
  float* x;
  int ldx, n;
  __device__ int col(int t) const { return t * 16; }
  __device__ int second() const { return 0; }
  __device__ int last() const { return n - 1; }
  __device__ void store(int m, int t, int c, const float (&v)[1], const Index&, const Fetched& old) const {
    const int j = t * 16 + c;
    if (j < n) x[(size_t)m * ldx + j] = old.x + v[0];
  }
};

// W = [gate rows | up rows]: act[m][j] = silu(gate j) * up j
struct F32Swiglu {
  static constexpr int kNT = 2;
  struct Index {};
  struct Fetched {};
  __device__ Index index(int) const { return {}; }
  __device__ Fetched fetch(int, int, int, const Index&) const { return {}; }
  float* act;
  int f;
  __device__ int col(int t) const { return t * 16; }
  __device__ int second() const { return f; }
  __device__ int last() const { return f - 1; }
  __device__ void store(int m, int t, int c, const float (&v)[2], const Index&, const Fetched&) const {
    const int j = t * 16 + c;
    if (j < f) act[(size_t)m * f + j] = v[0] / (1.0f + expf(-v[0])) * v[1];
  }
};

// W = [q | k | v] rows, head by head: tile t is 16 rotary pairs (i, i + head_dim/2) of one head of q, k or v
struct F32Qkv {
  static constexpr int kNT = 2;
  struct Index { int pos, slot; };
  struct Fetched { float cs, sn; };
  RopeKv o;
  __device__ Index index(int m) const { return {o.tok_pos[m], o.tok_seq[m]}; }
  __device__ Fetched fetch(int, int t, int c, const Index& x) const {
    const int u = t / tiles_per_head(), at = x.pos * (o.head_dim >> 1) + (t - u * tiles_per_head()) * 16 + c;
    return {o.rope_cos[at], o.rope_sin[at]};
  }
  __device__ int tiles_per_head() const { return o.head_dim >> 5; }
  __device__ int col(int t) const {
    const int u = t / tiles_per_head();
    return u * o.head_dim + (t - u * tiles_per_head()) * 16;
  }
  __device__ int second() const { return o.head_dim >> 1; }
  __device__ int last() const { return 3 * o.d_model - 1; }
  __device__ void store(int m, int t, int c, const float (&v)[2], const Index& x, const Fetched& f) const {
    const int u = t / tiles_per_head(), half = o.head_dim >> 1;
    const int i = (t - u * tiles_per_head()) * 16 + c, which = u / o.n_heads, head = u - which * o.n_heads;
    float a = v[0], b = v[1];
    if (which < 2) rope_pair(v[0], v[1], f.cs, f.sn, a, b);
    float* dst = which == 0 ? (float*)o.q + (size_t)m * o.d_model + head * o.head_dim
                            : (float*)(which == 1 ? o.k_cache : o.v_cache) +
                                  (((size_t)x.slot * o.n_heads + head) * o.max_seq + x.pos) * o.head_dim;
    dst[i] = a;
    dst[i + half] = b;
  }
};

// NORM: the product is of the RMS-normalised rows x * gain / sqrt(mean(x^2) + eps); the gain goes into the operand,
// the row's factor onto the sum.  VEC: K is a multiple of 4, so that every 16-byte load is aligned and inside its row.
// Otherwise (an odd d_ffn) only the last step of a row is loaded element by element; all of them so is what bounds many
// rows: 4000 of d 2048, d_ffn 5631, prefill of 2 layers 21.5 ms (14.6 with d_ffn 5632), with whole steps in one load 14.8.
template <int MT, bool VEC, bool NORM, class Epi>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ A, int lda, const float* __restrict__ W,
                                                       const float* __restrict__ gain, float eps, int M, int K, int tiles, Epi epi) {
  constexpr int NT = Epi::kNT, U = MT == 1 ? (NT == 1 ? 12 : 6) : 4;   // k-steps (16 k) requested together
  __shared__ float red[4][MT * NT][256];
  __shared__ float s_ss[4][MT * 16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, g = lane >> 4;                  // operand row, k group (4 k of each step)
  const int tile = blockIdx.x % tiles, m0 = blockIdx.x / tiles * 16 * MT;
  const int steps = (K + 15) >> 4;
  const int s_begin = wave * steps / 4, s_end = (wave + 1) * steps / 4;

  const float* a_row[MT];
  const float* w_row[NT];
#pragma unroll
  for (int i = 0; i < MT; ++i) a_row[i] = A + (size_t)min(m0 + i * 16 + r, M - 1) * lda;
#pragma unroll
  for (int j = 0; j < NT; ++j) w_row[j] = W + (size_t)(min(epi.col(tile) + r, epi.last()) + j * epi.second()) * K;
  auto load = [&](const float* row, int s) {               // 4 k of a row, zero past K
    const int k = s * 16 + g * 4;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if constexpr (VEC) {
      if (k < K) v = *(const f32x4*)(row + k);
    } else if (s * 16 + 16 <= K) {                         // whole step (uniform): 16-byte loads need 4-byte alignment only
      typedef f32x4 f32x4u __attribute__((aligned(4)));
      v = *(const f32x4u*)(row + k);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (k + e < K) v[e] = row[k + e];
    }
    return v;
  };

  f32x4 acc[MT][NT];
  float ss[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    ss[i] = 0.f;
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  f32x4 a[U][MT], w[U][NT], gn[NORM ? U : 1];
  auto request = [&](int s0) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (s0 + u < s_end) {                                // uniform across the wave
#pragma unroll
        for (int i = 0; i < MT; ++i) a[u][i] = load(a_row[i], s0 + u);
#pragma unroll
        for (int j = 0; j < NT; ++j) w[u][j] = load(w_row[j], s0 + u);
        if constexpr (NORM) gn[u] = load(gain, s0 + u);
      }
  };
  const int t = threadIdx.x, row = t >> 4, c = t & 15;     // the output element(s) of this thread
  typename Epi::Index index[MT];
  typename Epi::Fetched fetched[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) index[i] = epi.index(min(m0 + i * 16 + row, M - 1));
  request(s_begin);
#pragma unroll
  for (int i = 0; i < MT; ++i) fetched[i] = epi.fetch(min(m0 + i * 16 + row, M - 1), tile, c, index[i]);
  __builtin_amdgcn_sched_barrier(0);
  for (int s0 = s_begin; s0 < s_end; s0 += U) {
    if (s0 > s_begin) request(s0);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (s0 + u < s_end) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < MT; ++i) {
            float x = a[u][i][e];
            if constexpr (NORM) {
              ss[i] = fmaf(x, x, ss[i]);
              x *= gn[u][e];
            }
#pragma unroll
            for (int j = 0; j < NT; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, w[u][j][e], acc[i][j], 0, 0, 0);
          }
      }
  }
  // accumulator element e of a lane is row 4 * (lane >> 4) + e, column lane & 15
#pragma unroll
  for (int i = 0; i < MT; ++i) {
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) red[wave][i * NT + j][(4 * g + e) * 16 + r] = acc[i][j][e];
    if constexpr (NORM) {
      const float s = lanes_sum<16, 32>(ss[i]);
      if (g == 0) s_ss[wave][i * 16 + r] = s;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const int m = m0 + i * 16 + row;
    if (m >= M) break;
    float inv = 1.f;
    if constexpr (NORM) {
      const int q = i * 16 + row;
      inv = 1.0f / sqrtf(((s_ss[0][q] + s_ss[1][q]) + (s_ss[2][q] + s_ss[3][q])) / (float)K + eps);
    }
    float v[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j)
      v[j] = ((red[0][i * NT + j][t] + red[1][i * NT + j][t]) + (red[2][i * NT + j][t] + red[3][i * NT + j][t])) * inv;
    epi.store(m, tile, c, v, index[i], fetched[i]);
  }
}

template <bool NORM, class Epi>
static void launch(const float* A, int lda, const float* W, const float* gain, float eps, int M, int tiles, int K,
                   const Epi& epi, hipStream_t st) {
  // 32-row tiles once 16-row ones would be more than about four workgroups per compute unit
  const bool wide = (long long)((M + 15) / 16) * tiles > 1024;
#define VLA_F32_LAUNCH(MTV, VECV)                                                                                    \
  hipLaunchKernelGGL((gemm_f32_kernel<MTV, VECV, NORM, Epi>), dim3(tiles * ((M + 16 * MTV - 1) / (16 * MTV))), dim3(256), \
                     0, st, A, lda, W, gain, eps, M, K, tiles, epi)
  if (K % 4 == 0) {
    if (wide) VLA_F32_LAUNCH(2, true);
    else VLA_F32_LAUNCH(1, true);
  } else {                                                 // an odd d_ffn: rows of W and of the activations are not aligned
    if (wide) VLA_F32_LAUNCH(2, false);
    else VLA_F32_LAUNCH(1, false);
  }
#undef VLA_F32_LAUNCH
}

void gemm_f32_qkv(const float* x, const float* gain, float eps, const float* W, int M, const RopeKv& o, hipStream_t st) {
  launch<true>(x, o.d_model, W, gain, eps, M, 3 * o.d_model / 32, o.d_model, F32Qkv{o}, st);
}
void gemm_f32_swiglu(const float* x, const float* gain, float eps, const float* W, float* act, int M, int d, int f,
                     hipStream_t st) {
  launch<true>(x, d, W, gain, eps, M, (f + 15) / 16, d, F32Swiglu{act, f}, st);
}
void gemm_f32_resid(const float* A, const float* W, float* x, int M, int d, int K, hipStream_t st) {
  launch<false>(A, K, W, nullptr, 0.f, M, d / 16, K, F32Resid{x, d, d}, st);
}

}  // namespace vla
