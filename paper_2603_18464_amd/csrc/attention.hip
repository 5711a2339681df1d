// Causal attention against the KV cache: the float32 rows kernel, flash attention of the 16-bit prefill, and the decode
// kernel of the 16-bit path.
//
// attention_rows (float32): one wave per (token, head).  Keys and values of a (slot, head) are contiguous
// [position][head_dim] rows in the cache; HD / 4 lanes share a row, 16 bytes each, so an instruction reads 64 * 4 / HD whole
// rows and a score is a butterfly over the lanes of its row.  A few dozen keys: bound by its chain of latencies, so the rows
// of two groups of G instructions are in flight, a group requested again as soon as its registers are free, and the first
// values with the keys, before there is a score.  Groups by a context's use of them: six instructions, four where these are
// eight rows each.  us a decode step of two layers of d 512, groups of twelve one after the other / these: one sequence of
// 1000 keys, heads of 64 154 / 128, of 256 438 / 307; a prefill of 64 prefixes of 33, heads of 32, 604 / 568.
#include <type_traits>

#include "common.h"

namespace vla {

template <int HD>
__global__ __launch_bounds__(256) void attention_rows_kernel(
    const float* __restrict__ q, const float* __restrict__ k_cache, const float* __restrict__ v_cache,
    const int32_t* __restrict__ tok_seq, const int32_t* __restrict__ tok_pos, float* __restrict__ out, int n_items,
    int n_heads, int max_seq) {
  extern __shared__ float smem[];                    // [4 waves][max_seq] scores
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int item = blockIdx.x * 4 + wave;            // (token, head)
  if (item >= n_items) return;                       // whole wave leaves; no block barrier is used
  float* sc = smem + (size_t)wave * max_seq;
  constexpr int LPR = HD / 4, RPI = 64 / LPR, G = HD == 32 ? 4 : 6, STEP = G * RPI;
  const int c = lane % LPR, sub = lane / LPR;
  const int tok = item / n_heads, head = item - tok * n_heads;
  const int slot = tok_seq[tok], pos = tok_pos[tok];
  const f32x4 qv = *(const f32x4*)(q + (size_t)item * HD + c * 4);
  const size_t blk = ((size_t)slot * n_heads + head) * max_seq * HD + c * 4;
  const float *kbase = k_cache + blk, *vbase = v_cache + blk;
  const float scale = rsqrtf((float)HD);
  f32x4 kv[2][G], vv[2][G];
  auto request = [&](f32x4 (&r)[G], const float* base, int key0) {
#pragma unroll
    for (int u = 0; u < G; ++u) r[u] = *(const f32x4*)(base + (size_t)min(key0 + u * RPI + sub, pos) * HD);   // keys 0..pos
  };
  float mx = -INFINITY, sum = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  auto scores = [&](const f32x4 (&k)[G], int key0) __attribute__((always_inline)) {
    float s[G];
#pragma unroll
    for (int u = 0; u < G; ++u) s[u] = fmaf(qv[3], k[u][3], fmaf(qv[2], k[u][2], fmaf(qv[1], k[u][1], qv[0] * k[u][0])));
#pragma unroll
    for (int u = 0; u < G; ++u) s[u] = lanes_sum<1, LPR / 2>(s[u]);
#pragma unroll
    for (int u = 0; u < G; ++u) {
      const int key = key0 + u * RPI + sub;
      s[u] *= scale;
      mx = fmaxf(mx, s[u]);                                // (a clamped row repeats key pos: the same maximum)
      if (c == 0 && key <= pos) sc[key] = s[u];
    }
  };
  auto values = [&](const f32x4 (&v)[G], int key0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < G; ++u) {
      const int key = key0 + u * RPI + sub;
      if (key <= pos) {
        const float p = __expf(sc[key] - mx);
        sum += p;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = fmaf(p, v[u][e], acc[e]);
      }
    }
  };
  // one pass over the rows; the first two groups are requested
  auto pass = [&](f32x4 (&r)[2][G], const float* base, auto&& consume) __attribute__((always_inline)) {
    int key0 = 0;
    for (; key0 + 2 * STEP <= pos; key0 += 2 * STEP) {
      consume(r[0], key0);
      request(r[0], base, key0 + 2 * STEP);
      consume(r[1], key0 + STEP);
      request(r[1], base, key0 + 3 * STEP);
    }
    consume(r[0], key0);
    if (key0 + STEP <= pos) consume(r[1], key0 + STEP);
  };
  request(kv[0], kbase, 0);
  request(kv[1], kbase, STEP);
  request(vv[0], vbase, 0);
  request(vv[1], vbase, STEP);
  __builtin_amdgcn_sched_barrier(0);
  pass(kv, kbase, scores);
  if constexpr (LPR < 64) mx = lanes_max<LPR, 32>(mx);
  __builtin_amdgcn_wave_barrier();
  pass(vv, vbase, values);
  if constexpr (LPR < 64) {
    sum = lanes_sum<LPR, 32>(sum);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = lanes_sum<LPR, 32>(acc[e]);
  }
  const float inv = 1.0f / sum;
  if (sub == 0) *(f32x4*)(out + (size_t)item * HD + c * 4) = acc * inv;
}

// ---- prefill: causal flash attention on the matrix cores --------------------------------------------
// One workgroup = 4 waves = 128 consecutive query positions of one (sequence, head); each wave owns
// 32 queries.  Keys/values are walked in tiles of 64 positions staged in LDS.
//   S^T = K Q^T  : A operand = K rows (key-major, straight from the cache layout, XOR-swizzled 16-byte
//                  chunks in LDS), B operand = the wave's Q rows kept in registers.  In the 32x32
//                  accumulator layout every lane then owns ONE query (column l & 31) and 16 of the 32
//                  keys of a sub-tile, so the softmax statistics are per-lane scalars plus one exchange
//                  with lane ^ 32.
//   O^T += V^T P^T: B operand = P^T taken directly from the S^T accumulators (the contraction index
//                  may be permuted freely as long as both operands agree), A operand = V^T read from an
//                  LDS tile that was transposed while staging, with the key order inside each group of
//                  16 arranged so that a lane's 8 keys are contiguous.
// Bound by latency: a workgroup lives for three key tiles on average (prefixes of 290) and starts with two dependent
// rounds of loads.  Per layer, 64 prefixes of 290, 32 heads of 128: 169 us with a head's tiles on one XCD (180 with them
// dealt over three), 32 prefixes, 12 heads of 64: 20.6 us with four workgroups per compute unit (23.0 with two); with the output in
// fragment order, where a store of 32 rows is 512 bytes in a row instead of 64 pieces of 8, 155 and 19.4 (low terms 369 -> 340).
// TWO (two-term mode): queries, keys and values each come as hi + lo terms (the low terms of the queries in half
// precision at column lo_off of the same rows, those of the cache as bytes, lo8 = bf8(16 * lo), in k_lo / v_lo
// with the cache's indexing; they are widened exactly to half precision while the tile is staged), the
// scores are K_hi Q_hi + K_lo Q_hi + K_hi Q_lo, the output sum takes V_hi + V_lo, and the output rows are written
// with both terms as well.  The staging tiles double, so one workgroup runs per compute unit instead of two.
// The LDS serves a 16-byte read in groups of 16 lanes that here are 16 keys whose numbers differ in their low four bits:
// the swizzle puts their chunks in 16 different slots of the 64 banks (two rows of 64 dimensions share the banks).
template <int HD>
__device__ __forceinline__ int k_swizzle(int kk) { return HD == 128 ? kk & 15 : (kk >> 1) & 7; }
template <int HD, bool TWO>
__global__ __launch_bounds__(256, !TWO && HD == 64 ? 4 : 2) void flash_prefill_kernel(
    const f16* __restrict__ q, int ldq, const f16* __restrict__ k_cache, const f16* __restrict__ v_cache,
    const unsigned char* __restrict__ k_lo, const unsigned char* __restrict__ v_lo,
    const int32_t* __restrict__ cu_patch,
    const int32_t* __restrict__ cu_instr, const int32_t* __restrict__ slot_map, f16* __restrict__ out, int ldo,
    int n_qt, int B, int n_heads, int max_seq, int lo_off, int out_lo8) {
  constexpr int KS = HD / 16;          // k-steps of the QK^T contraction
  constexpr int DT = HD / 32;          // 32-row tiles of O^T
  constexpr int KCH = HD / 8;          // 16-byte chunks per key row
  constexpr int VPITCH = 64 + 8;       // halves per V^T row (padding keeps b128 reads conflict free)
  constexpr int NP = TWO ? 2 : 1;      // planes: hi (and lo)
  __shared__ __attribute__((aligned(16))) f16 Ks[NP][64 * HD];
  __shared__ __attribute__((aligned(16))) f16 Vt[NP][HD * VPITCH];

  // Workgroups are dealt to the eight XCDs in turn: give each XCD a contiguous run of (sequence, head, query tile), query
  // tiles innermost, so that the tiles of a head find its keys and values in one L2.
  const int pid = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const int qt = pid % n_qt, bh = pid / n_qt;
  if (bh >= B * n_heads) return;
  const int b = bh % B, head = bh / B;
  const int row0 = cu_patch[b] + cu_instr[b];
  const int S = cu_patch[b + 1] + cu_instr[b + 1] - row0;
  // Query tiles of 128 are aligned to the END of the sequence (the first tile is the short one): a tile needs the
  // keys up to its last query, so a prefix of 290 costs 1 + 3 + 5 key tiles instead of 2 + 4 + 5.
  const int nq = (S + 127) / 128;
  if (qt >= nq) return;
  const int q0 = S - 128 * (nq - qt);        // negative for a short first tile: those lanes are idle
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int half = lane >> 5, col = lane & 31;
  const int qpos = q0 + wave * 32 + col;                 // this lane's query position (< S; idle if negative)
  const int qrow = row0 + max(qpos, 0);                   // clamped: idle lanes are never stored
  const int slot = slot_map ? slot_map[b] : b;
  const size_t blk = ((size_t)slot * n_heads + head) * max_seq * HD;
  const f16* kbase = k_cache + blk;
  const f16* vbase = v_cache + blk;
  const unsigned char* kbase8 = TWO ? k_lo + blk : nullptr;   // low terms of the cache: one byte per element
  const unsigned char* vbase8 = TWO ? v_lo + blk : nullptr;

  // The wave's query fragments (low terms too in two-term mode) stay in registers.
  f16x8 qreg[NP][KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
#pragma unroll
    for (int pl = 0; pl < NP; ++pl)
      qreg[pl][ks] = *(const f16x8*)(q + (size_t)qrow * ldq + pl * lo_off + head * HD + (ks * 2 + half) * 8);

  f32x16 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[dt][e] = 0.f;
  // Softmax statistics are kept in the base-2 domain: scores are scaled by log2(e) / sqrt(HD) once, and every
  // exponential is a bare exp2.  m_run is a reference point, not necessarily the running maximum: it is moved up
  // (and the accumulators rescaled) only when some query of the wave has found a score more than kLazy above it,
  // so most tiles skip the rescaling; probabilities relative to it stay below 2^kLazy, well inside half precision.
  // l_run is this lane's share: the two halves of a query are added at the end.
  float m_run = -INFINITY, l_run = 0.f;
  const float scale2 = rsqrtf((float)HD) * 1.44269504088896341f;
  constexpr float kLazy = 8.0f;

  const int kend = q0 + 128;                              // keys needed by this workgroup (<= S)
  const int wave_last = q0 + wave * 32 + 31;              // last query position of this wave
  // The next tile's keys and values are fetched into registers while the current tile is being consumed, so
  // the global-memory latency of a tile hides under the MFMAs and the softmax of the one before.
  constexpr int KI = 64 * KCH / 256, VI = 32 * KCH / 256;
  typedef __attribute__((ext_vector_type(2))) int i32x2;
  u32x4 kreg[KI];
  f16x8 vreg[VI][2];
  i32x2 kreg8[TWO ? KI : 1], vreg8[TWO ? VI : 1][2];       // the same items of the low-term planes, 8 bytes each
  auto fetch = [&](int k0) {                               // high terms of the tile at k0
#pragma unroll
    for (int i = 0; i < KI; ++i) {
      const int item = t + 256 * i;
      const int c = item % KCH, kk = item / KCH;
      const int kp = min(k0 + kk, S - 1);
      kreg[i] = *(const u32x4*)(kbase + (size_t)kp * HD + c * 8);
    }
#pragma unroll
    for (int i = 0; i < VI; ++i) {
      const int item = t + 256 * i;
      const int u = item & 31, c = item >> 5;
      const int ka = min(k0 + 2 * u, S - 1), kb = min(k0 + 2 * u + 1, S - 1);
      vreg[i][0] = *(const f16x8*)(vbase + (size_t)ka * HD + c * 8);
      vreg[i][1] = *(const f16x8*)(vbase + (size_t)kb * HD + c * 8);
    }
  };
  auto fetch8 = [&](int k0) {                              // low terms of the tile at k0
#pragma unroll
    for (int i = 0; i < KI; ++i) {
      const int item = t + 256 * i;
      const int c = item % KCH, kk = item / KCH;
      const int kp = min(k0 + kk, S - 1);
      kreg8[i] = *(const i32x2*)(kbase8 + (size_t)kp * HD + c * 8);
    }
#pragma unroll
    for (int i = 0; i < VI; ++i) {
      const int item = t + 256 * i;
      const int u = item & 31, c = item >> 5;
      const int ka = min(k0 + 2 * u, S - 1), kb = min(k0 + 2 * u + 1, S - 1);
      vreg8[i][0] = *(const i32x2*)(vbase8 + (size_t)ka * HD + c * 8);
      vreg8[i][1] = *(const i32x2*)(vbase8 + (size_t)kb * HD + c * 8);
    }
  };
  auto widen8 = [&](const i32x2& w) {                      // 8 low-term bytes -> half precision (exact)
    f16x8 h;
    h[0] = (f16)unpack_lo8(w[0], 0); h[1] = (f16)unpack_lo8(w[0], 1); h[2] = (f16)unpack_lo8(w[0], 2); h[3] = (f16)unpack_lo8(w[0], 3);
    h[4] = (f16)unpack_lo8(w[1], 0); h[5] = (f16)unpack_lo8(w[1], 1); h[6] = (f16)unpack_lo8(w[1], 2); h[7] = (f16)unpack_lo8(w[1], 3);
    return h;
  };
  fetch(0);
  for (int k0 = 0; k0 < kend; k0 += 64) {
    // Two-term: only the high terms are prefetched a tile ahead (the registers do not hold both); the low terms
    // are requested here, and the other workgroup on the compute unit covers their latency.
    if constexpr (TWO) fetch8(k0);
    __syncthreads();                                      // previous tile fully consumed
#pragma unroll
    for (int pl = 0; pl < NP; ++pl) {
      // K tile: 64 keys x KCH chunks, chunk c of key kk stored at slot c ^ k_swizzle(kk)
#pragma unroll
      for (int i = 0; i < KI; ++i) {
        const int item = t + 256 * i;
        const int c = item % KCH, kk = item / KCH;
        u32x4 v = kreg[i];
        if constexpr (TWO) {
          if (pl == 1) v = __builtin_bit_cast(u32x4, widen8(kreg8[i]));
        }
        *(u32x4*)(Ks[pl] + kk * HD + ((c ^ k_swizzle<HD>(kk)) << 3)) = v;
      }
      // V tile, transposed: Vt[dim][pos(key)], two keys per 32-bit store
#pragma unroll
      for (int i = 0; i < VI; ++i) {
        const int item = t + 256 * i;
        const int u = item & 31, c = item >> 5;
        const int g = (2 * u) & 15;                       // position of the key inside its group of 16
        const int pos = ((2 * u) & ~15) + ((g >> 2) & 1) * 8 + (g >> 3) * 4 + (g & 3);
        f16x8 va = vreg[i][0], vb = vreg[i][1];
        if constexpr (TWO) {
          if (pl == 1) {
            va = widen8(vreg8[i][0]);
            vb = widen8(vreg8[i][1]);
          }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
          f16x2 pr;
          pr[0] = va[j];
          pr[1] = vb[j];
          *(f16x2*)(Vt[pl] + (c * 8 + j) * VPITCH + pos) = pr;
        }
      }
    }
    __syncthreads();
    if (k0 + 64 < kend) fetch(k0 + 64);                   // uniform across the workgroup
    if (k0 > wave_last || wave_last < 0) continue;        // tile above this wave's diagonal, or no live query in the wave

    // S^T for the two 32-key sub-tiles
    f32x16 sacc[2];
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int e = 0; e < 16; ++e) sacc[st][e] = 0.f;
    // k-step outermost: one query fragment serves both key sub-tiles, and the two accumulator chains alternate
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const f16x8 qfr = qreg[0][ks];
#pragma unroll
      for (int st = 0; st < 2; ++st) {
        const int kk = st * 32 + col;
        const int koff = kk * HD + (((ks * 2 + half) ^ k_swizzle<HD>(kk)) << 3);
        const f16x8 kf = *(const f16x8*)(Ks[0] + koff);
        sacc[st] = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf, qfr, sacc[st], 0, 0, 0);
        if constexpr (TWO) {
          const f16x8 kl = *(const f16x8*)(Ks[NP - 1] + koff);
          sacc[st] = __builtin_amdgcn_mfma_f32_32x32x16_f16(kl, qfr, sacc[st], 0, 0, 0);
          sacc[st] = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf, qreg[NP - 1][ks], sacc[st], 0, 0, 0);
        }
      }
    }
    // scale, causal mask (only the tiles that reach past the wave's first query need one; a key position is below
    // S whenever it is at most the position of a live query), tile maximum
    float m_tile = -INFINITY;
    if (k0 + 63 > q0 + wave * 32) {
      // element (st, e) is key k0 + 4 * half + [st * 32 + 8 * (e >> 2) + (e & 3)]: visible iff [..] <= lim
      const int lim = qpos - k0 - 4 * half;
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const float v = (st * 32 + 8 * (e >> 2) + (e & 3) <= lim) ? sacc[st][e] * scale2 : -INFINITY;
          sacc[st][e] = v;
          m_tile = fmaxf(m_tile, v);
        }
    } else {
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          sacc[st][e] *= scale2;
          m_tile = fmaxf(m_tile, sacc[st][e]);
        }
    }
    m_tile = fmaxf(m_tile, __shfl_xor(m_tile, 32, 64));
    if (__any(m_tile > m_run + kLazy)) {                    // (-inf + kLazy = -inf: true on the first live tile)
      const float m_new = fmaxf(m_run, m_tile);
      const float m_use = m_new == -INFINITY ? 0.f : m_new;  // fully masked so far: keep everything at zero
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_use);   // exp2(-inf) = 0 on the first live tile
      l_run *= alpha;
      m_run = m_new;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[dt][e] *= alpha;
    }
    const float m_ref = m_run == -INFINITY ? 0.f : m_run;
    float l_tile = 0.f;
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const float p = __builtin_amdgcn_exp2f(sacc[st][e] - m_ref);
        sacc[st][e] = p;
        l_tile += p;
      }
    l_run += l_tile;
    // O^T += V^T P^T   (two-term mode: P too is split, P_hi V_hi + P_hi V_lo + P_lo V_hi)
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int ip = 0; ip < 2; ++ip) {
        f16x8 pf, pl8;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          pf[j] = (f16)sacc[st][8 * ip + j];
          if constexpr (TWO) pl8[j] = (f16)(sacc[st][8 * ip + j] - (float)pf[j]);
        }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          const int voff = (dt * 32 + col) * VPITCH + st * 32 + ip * 16 + half * 8;
          const f16x8 vf = *(const f16x8*)(Vt[0] + voff);
          o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf, pf, o[dt], 0, 0, 0);
          if constexpr (TWO) {
            const f16x8 vl = *(const f16x8*)(Vt[NP - 1] + voff);
            o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vl, pf, o[dt], 0, 0, 0);
            o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf, pl8, o[dt], 0, 0, 0);
          }
        }
      }
  }
  l_run += __shfl_xor(l_run, 32, 64);
  if (qpos >= 0) {
    const float inv = 1.0f / l_run;
    const int m = row0 + qpos;                             // rows of fragment order, 16 bytes apart: an instruction writes 512 in a row
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        typedef __attribute__((ext_vector_type(4))) _Float16 f16x4;
        f16x4 w, we;
        float e[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float v = o[dt][4 * i + r] * inv;
          w[r] = from_f32<f16>(v);
          e[r] = v - (float)w[r];
          we[r] = from_f32<f16>(e[r]);
        }
        const int k = head * HD + dt * 32 + 8 * i + 4 * half;
        *(f16x4*)(out + act_index(m, k, ldo)) = w;
        if constexpr (TWO) {
          if (out_lo8)                                     // 8-bit low terms, behind the lo_off high terms
            *(int*)((unsigned char*)out + act_lo8_index(m, k, ldo, lo_off)) = pack_lo8(e[0], e[1], e[2], e[3]);
          else
            *(f16x4*)(out + act_index(m, lo_off + k, ldo)) = we;
        }
      }
  }
}

// k_lo / v_lo != nullptr selects the two-term kernel: q rows are [hi | lo] of pitch ldq with the low terms at
// column lo_off = d_model, and so the output (fragment order, ldo halves a row), unless out_lo8 asks for 8-bit low terms.
void flash_prefill(const f16* q, int ldq, const f16* k_cache, const f16* v_cache, const unsigned char* k_lo,
                   const unsigned char* v_lo, const int32_t* cu_patch, const int32_t* cu_instr, const int32_t* slot_map,
                   f16* out, int ldo, bool out_lo8, int B, int max_len, int n_heads, int head_dim, int max_seq,
                   hipStream_t st) {
  const int n_qt = (max_len + 127) / 128;
  const dim3 grid((n_qt * B * n_heads + 7) / 8 * 8);
  const int lo_off = n_heads * head_dim;
#define VLA_FLASH(HDV, TWOV)                                                                                       \
  hipLaunchKernelGGL((flash_prefill_kernel<HDV, TWOV>), grid, dim3(256), 0, st, q, ldq, k_cache, v_cache, k_lo, v_lo, \
                     cu_patch, cu_instr, slot_map, out, ldo, n_qt, B, n_heads, max_seq, lo_off, out_lo8 ? 1 : 0)
  if (k_lo) {
    if (head_dim == 128) VLA_FLASH(128, true);
    else VLA_FLASH(64, true);
  } else {
    if (head_dim == 128) VLA_FLASH(128, false);
    else VLA_FLASH(64, false);
  }
#undef VLA_FLASH
}

// ---- decode: one new query per (sequence, head) against the whole cache -------------------------------
// HBM-bound at large batches, bound by its chain of latencies at small ones: the keys and values of a (slot, head) are
// one contiguous [position][HD] block each, and the kernel streams them once with 16-byte-per-lane loads (a wave
// instruction covers 64*16/(2*HD) whole rows).  One workgroup = 8 waves per (sequence, head); wave w takes every 8th
// group of rows.  A lane owns 8 head dimensions of one row at a time: scores are added up over the HD/8 lanes of a row
// in the vector unit, the probability-weighted values stay in 8 per-lane accumulators, and the partial softmax
// statistics and outputs of the waves are merged through LDS at the end.
//
// The query and the new key / value row of this (sequence, head) are not read from memory but formed here from
// the split-K partial sums of the QKV GEMM (summed in plane order, RoPE applied; the query stays in float32, the
// key / value row is rounded as the cache holds it); the new row is appended to the cache for the following steps
// and used from LDS in this one: a group that reaches past the cached rows takes it into its registers first.
// One wave each forms the query, the key and the value, its partial sums and rotary factors requested before any
// cache row (answers come back in the order of the requests, and the partial sums need no context length), behind them the
// first group of rows and, of a context that has one, the second, and every group's successor as soon as its registers are
// free.  us a launch at one row and 290 positions: 12 heads of 64 5.95 -> 5.27 (low terms 6.7 -> 6.2), 32 heads of 128 8.2 ->
// 7.3 (10.0 -> 9.4), against one wave that formed all three behind the requests of the cache rows and a branch a row for the
// new one.
//
// Rows past the cached ones are not requested: the loads are bounded by a buffer descriptor of the group's rows that exist.
// Clamped to the last row they cost little while its line stays in the L1; read as data that does not come again it does not
// stay, and with blocks of about a power of two bytes the last rows of all of them lie on a few channels.  us a step of 4 layers
// of d 2048 (heads of 64, single-term) at 512 sequences, normal and clamped / once and clamped / once and bounded: 60 positions in
// blocks of 127 1169 / 1578 / 1140, 100 in blocks of 127 1276 / 1542 / 1229, 60 in blocks of 201 1149 / 1138 / 1126; normal and
// bounded is as normal and clamped (+-1 %).  A row's low terms are requested with its high ones: behind those of the whole group
// they made a step of two-term layers at 256 sequences of 300 and 500 positions 5 and 9 % longer.
struct QkvPartials {
  const float* part;       // [ksplit][rows][3 * d_model]
  int ksplit, rows;
  const float* rope_cos;   // [max_seq, HD/2]
  const float* rope_sin;
};

// Elements from `at` on of the first `rows` rows of ROW elements behind base (uniform, as rows is); zeros, and no request, for
// those of later rows.  ONCE: as data that is not read again.
template <class V, bool ONCE, int ROW, class E>
__device__ __forceinline__ V load_row(const E* base, int rows, unsigned at) {
#if defined(__HIP_DEVICE_COMPILE__)
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, rows * (int)(ROW * sizeof(E)), 0x00027000);
  if constexpr (sizeof(V) == 16) return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(rsrc, at * sizeof(E), 0, ONCE ? 2 : 0));
  else return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(rsrc, at * sizeof(E), 0, ONCE ? 2 : 0));
#else
  return V{};
#endif
}

// TWO (two-term mode): the cache holds every key / value as a half-precision high term plus a one-byte low term
// (k_lo / v_lo, same indexing, bf8(16 * lo)); both are streamed and added in float32; the output is written as hi
// and lo fragments (out_frag_lo).
// ONCE: the step's keys, values and weights together do not stay in the 256 MB last-level cache until the next step (see
// kv_read_once), so the rows are requested as data that is not read again.  They then leave the caches to what is.
template <int HD, bool TWO, bool ONCE>
__global__ __launch_bounds__(512, 4) void decode_attention_kernel(
    f16* __restrict__ k_cache, f16* __restrict__ v_cache,
    unsigned char* __restrict__ k_lo, unsigned char* __restrict__ v_lo, const int32_t* __restrict__ tok_seq,
    const int32_t* __restrict__ tok_pos,
    f16* __restrict__ out_frag, f16* __restrict__ out_frag_lo, int d_model, int n_heads, int max_seq,
    QkvPartials qp) {
  constexpr int LPR = HD / 8;            // lanes per row
  constexpr int RPI = 64 / LPR;          // rows per wave instruction
  constexpr int NW = 8;                  // waves
  constexpr int G = TWO ? 3 : 4;         // instructions of a group (what the registers hold twice)
  __shared__ float s_m[NW], s_l[NW];
  __shared__ float s_o[NW][HD];
  __shared__ __attribute__((aligned(16))) float s_q[HD];               // the query, unrounded
  __shared__ __attribute__((aligned(16))) f16 s_new[2][HD];            // the new key and value row, as the cache holds them
  __shared__ __attribute__((aligned(8))) unsigned char s_new_lo[2][TWO ? HD : 8];
  const int b = blockIdx.x, head = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int sub = lane / LPR, c = lane % LPR;          // row inside the instruction, 8-dim chunk
  const int ctx = tok_pos[b] + 1;                      // >= 2 in a decode step: the prefix holds a position
  const int slot = tok_seq[b];
  const size_t blk = ((size_t)slot * n_heads + head) * max_seq * HD;
  f16* kb = k_cache + blk;
  f16* vb = v_cache + blk;
  unsigned char* kbl = TWO ? k_lo + blk : nullptr;     // low terms: one byte per element, bf8(16 * lo)
  unsigned char* vbl = TWO ? v_lo + blk : nullptr;
  const int last_global = ctx - 2;                     // last row that is read from the cache

  typedef __attribute__((ext_vector_type(2))) int i32x2;
  f16x8 kv[2][G], vv[2][G];
  i32x2 kl[2][TWO ? G : 1], vl[2][TWO ? G : 1];         // low terms of the same rows: 8 bytes per lane
  const int n_it = (ctx + NW * RPI - 1) / (NW * RPI);   // instructions of a wave
  auto row_of = [&](int it) { return (it * NW + wave) * RPI + sub; };
  auto request = [&](auto S, int it0) {
    constexpr int s = decltype(S)::value;
    const int r0 = it0 * NW * RPI, rows = min(ctx - 1 - r0, G * NW * RPI);   // uniform; rows >= 0: it0 < n_it
    const size_t from = (size_t)r0 * HD;
    unsigned at0 = (unsigned)row_of(0) * HD + c * 8;
    hold32(at0);                                       // the offsets are formed here, an addition a load, and not kept
#pragma unroll
    for (int u = 0; u < G; ++u) {
      const unsigned at = at0 + u * NW * RPI * HD;
      kv[s][u] = load_row<f16x8, ONCE, HD>(kb + from, rows, at);
      vv[s][u] = load_row<f16x8, ONCE, HD>(vb + from, rows, at);
      if constexpr (TWO) {
        kl[s][u] = load_row<i32x2, ONCE, HD>(kbl + from, rows, at);
        vl[s][u] = load_row<i32x2, ONCE, HD>(vbl + from, rows, at);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  constexpr std::integral_constant<int, 0> s0{};
  constexpr std::integral_constant<int, 1> s1{};
  // waves 0, 1, 2: the new query, key, value; a lane has the rotary pair i, i + HD / 2 (HD 64: lanes 32.. repeat the others)
  constexpr int HALF = HD / 2;
  const int i = lane % HALF, pos = ctx - 1;
  float p[kMaxKSplit][2];
  float cs = 0.f, sn = 0.f;
  if (wave < 3) {
    const int c0 = wave * d_model + head * HD + i;
#pragma unroll
    for (int ks = 0; ks < kMaxKSplit; ++ks) {           // all planes in flight; planes past the last repeat it, unused
      const float* pp = qp.part + ((size_t)min(ks, qp.ksplit - 1) * qp.rows + b) * 3 * (size_t)d_model;
      p[ks][0] = pp[c0];
      p[ks][1] = pp[c0 + HALF];
    }
    cs = qp.rope_cos[pos * HALF + i];
    sn = qp.rope_sin[pos * HALF + i];
  }
  float qf[8];
  auto new_row = [&]() __attribute__((always_inline)) {   // forms and stores the new row, and leaves this lane's part of the query
    if (wave < 3) {
      float v0 = p[0][0], v1 = p[0][1];
#pragma unroll
      for (int ks = 1; ks < kMaxKSplit; ++ks) {
        v0 = ks < qp.ksplit ? v0 + p[ks][0] : v0;
        v1 = ks < qp.ksplit ? v1 + p[ks][1] : v1;
      }
      if (wave < 2) {
        float r0, r1;
        rope_pair(v0, v1, cs, sn, r0, r1);
        v0 = r0;
        v1 = r1;
      }
      if (lane < HALF) {
        if (wave == 0) {                                // the query never leaves float32
          s_q[i] = v0;
          s_q[i + HALF] = v1;
        } else {
          const size_t at = (size_t)pos * HD + i;
          const f16 h0 = from_f32<f16>(v0), h1 = from_f32<f16>(v1);
          f16* rows = wave == 1 ? kb : vb;
          rows[at] = h0;
          rows[at + HALF] = h1;
          s_new[wave - 1][i] = h0;
          s_new[wave - 1][i + HALF] = h1;
          if constexpr (TWO) {
            const int e = pack_lo8(v0 - (float)h0, v1 - (float)h1, 0.f, 0.f);
            const unsigned char e0 = (unsigned char)(e & 0xff), e1 = (unsigned char)((e >> 8) & 0xff);
            unsigned char* rows_lo = wave == 1 ? kbl : vbl;
            rows_lo[at] = e0;
            rows_lo[at + HALF] = e1;
            s_new_lo[wave - 1][i] = e0;
            s_new_lo[wave - 1][i + HALF] = e1;
          }
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; ++j) qf[j] = s_q[c * 8 + j];
  };
  // A context that one group covers has no second one (its requests, clamped to the last row, made 74 us of 256 sequences of 60
  // positions, 32 heads of 64, low terms, 88).  The branches meet behind the new row, the short one with nothing in flight,
  // so that the waits that follow count on the second group's requests (without that the first group waits for both: 1 % of a
  // launch at 290 positions, 5 % of some).
  request(s0, 0);
  if (__builtin_expect(n_it > G, 1)) {                  // uniform
    request(s1, G);
    new_row();
  } else {
    new_row();
    __builtin_amdgcn_s_waitcnt(0x0f70);                 // vmcnt(0), for the compiler to see
  }
  const float scale = rsqrtf((float)HD);

  // One pass with a running maximum per lane: the key rows and the value rows of a group are requested together, so
  // twice as many bytes are in flight as with a score pass followed by a value pass, and no scores have to be kept.  The
  // maximum moves once per group.
  float m_run = -INFINITY, lsum = 0.f;
  float acc[8] = {};
  auto consume = [&](auto S, int it0) {
    constexpr int s = decltype(S)::value;
    float sc[G];
    float m_new = m_run;
    if (((it0 + G - 1) * NW + wave + 1) * RPI > ctx - 1) {         // (uniform) rows the cache did not hold: the new one and,
      const f16x8 kn = *(const f16x8*)&s_new[0][c * 8], vn = *(const f16x8*)&s_new[1][c * 8];   // masked below, those past it
#pragma unroll
      for (int u = 0; u < G; ++u) {
        const bool in = row_of(it0 + u) > last_global;
        kv[s][u] = in ? kn : kv[s][u];
        vv[s][u] = in ? vn : vv[s][u];
      }
      if constexpr (TWO) {
        const i32x2 kln = *(const i32x2*)&s_new_lo[0][c * 8], vln = *(const i32x2*)&s_new_lo[1][c * 8];
#pragma unroll
        for (int u = 0; u < G; ++u) {
          const bool in = row_of(it0 + u) > last_global;
          kl[s][u] = in ? kln : kl[s][u];
          vl[s][u] = in ? vln : vl[s][u];
        }
      }
    }
#pragma unroll
    for (int u = 0; u < G; ++u) {
      float t = 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        float kf = (float)kv[s][u][j];
        if constexpr (TWO) kf += unpack_lo8(kl[s][u][j >> 2], j & 3);
        t = fmaf(qf[j], kf, t);
      }
      sc[u] = t;
    }
#pragma unroll
    for (int u = 0; u < G; ++u) sc[u] = lanes_sum<1, LPR / 2>(sc[u]);
#pragma unroll
    for (int u = 0; u < G; ++u) {
      sc[u] = row_of(it0 + u) < ctx ? sc[u] * scale : -INFINITY;   // uniform over the LPR lanes of a row
      m_new = fmaxf(m_new, sc[u]);
    }
    const float m_use = m_new == -INFINITY ? 0.f : m_new;          // no live row so far: everything stays zero
    const float alpha = __expf(m_run - m_use);                     // exp(-inf) = 0 on the lane's first live group
    m_run = m_new;
    lsum *= alpha;
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] *= alpha;
#pragma unroll
    for (int u = 0; u < G; ++u) {
      const float p = __expf(sc[u] - m_use);
      lsum += p;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        float vf = (float)vv[s][u][j];
        if constexpr (TWO) vf += unpack_lo8(vl[s][u][j >> 2], j & 3);
        acc[j] = fmaf(p, vf, acc[j]);
      }
    }
  };
  for (int it0 = 0; it0 < n_it; it0 += 2 * G) {
    consume(s0, it0);
    if (it0 + 2 * G < n_it) request(s0, it0 + 2 * G);              // uniform
    if (it0 + G < n_it) {
      consume(s1, it0 + G);
      if (it0 + 3 * G < n_it) request(s1, it0 + 3 * G);
    }
  }
  // bring the lanes of the wave to a common maximum, then add the row groups
  const float mx = lanes_max<LPR, 32>(m_run);
  {
    const float f = m_run == -INFINITY ? 0.f : __expf(m_run - mx);
    lsum *= f;
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] *= f;
  }
  lsum = lanes_sum<LPR, 32>(lsum);
#pragma unroll
  for (int j = 0; j < 8; ++j) acc[j] = lanes_sum<LPR, 32>(acc[j]);
  if (sub == 0) {
#pragma unroll
    for (int j = 0; j < 8; ++j) s_o[wave][c * 8 + j] = acc[j];
    if (c == 0) { s_m[wave] = mx; s_l[wave] = lsum; }
  }
  __syncthreads();
  if (threadIdx.x < HD) {
    const int col = threadIdx.x;
    float m = s_m[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) m = fmaxf(m, s_m[w]);
    float l = 0.f, o = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float f = s_m[w] == -INFINITY ? 0.f : __expf(s_m[w] - m);
      l += s_l[w] * f;
      o += s_o[w][col] * f;
    }
    const int k = head * HD + col;
    const size_t at = ((size_t)(b >> 5) * (d_model >> 4) + (k >> 4)) * 512 + ((b & 31) + 32 * ((k >> 3) & 1)) * 8 + (k & 7);
    const float r = o / l;
    const f16 r16 = from_f32<f16>(r);
    out_frag[at] = r16;
    if constexpr (TWO) out_frag_lo[at] = from_f32<f16>(r - (float)r16);
  }
}

// Row b of the step lives in cache slot tok_seq[b]; the query and the new cache row come from the QKV GEMM's partial
// sums part[ksplit][part_rows][3 * d_model].  k_lo != nullptr selects two-term mode.
void decode_attention_fused(const float* part, int ksplit, int part_rows, const float* rope_cos, const float* rope_sin,
                            f16* k_cache, f16* v_cache, unsigned char* k_lo, unsigned char* v_lo, const int32_t* tok_seq,
                            const int32_t* tok_pos, f16* out_frag, f16* out_frag_lo, int B, int d_model, int n_heads,
                            int head_dim, int max_seq, bool kv_once, hipStream_t st) {
  const dim3 grid(B, n_heads);
  const QkvPartials qp{part, ksplit, part_rows, rope_cos, rope_sin};
#define VLA_DEC_ATT_ONCE(HDV, TWOV, ONCEV)                                                                         \
  hipLaunchKernelGGL((decode_attention_kernel<HDV, TWOV, ONCEV>), grid, dim3(512), 0, st, k_cache, v_cache,       \
                     k_lo, v_lo, tok_seq, tok_pos, out_frag, out_frag_lo, d_model, n_heads, max_seq, qp)
#define VLA_DEC_ATT(HDV, TWOV)                      \
  do {                                              \
    if (kv_once) VLA_DEC_ATT_ONCE(HDV, TWOV, true); \
    else VLA_DEC_ATT_ONCE(HDV, TWOV, false);        \
  } while (0)
  if (k_lo) {
    if (head_dim == 128) VLA_DEC_ATT(128, true);
    else VLA_DEC_ATT(64, true);
  } else {
    if (head_dim == 128) VLA_DEC_ATT(128, false);
    else VLA_DEC_ATT(64, false);
  }
#undef VLA_DEC_ATT
#undef VLA_DEC_ATT_ONCE
}

void attention_rows_f32(const float* q, const float* k_cache, const float* v_cache, const int32_t* tok_seq,
                        const int32_t* tok_pos, float* out, int n_tok, int n_heads, int head_dim, int max_seq,
                        hipStream_t st) {
  const int n_items = n_tok * n_heads;
  const int blocks = (n_items + 3) / 4;
  const size_t smem = attention_rows_lds(max_seq);
#define VLA_ATTN_CASE(HD)                                                                                   \
  case HD:                                                                                                  \
    hipLaunchKernelGGL((attention_rows_kernel<HD>), dim3(blocks), dim3(256), smem, st, q, k_cache, v_cache, \
                       tok_seq, tok_pos, out, n_items, n_heads, max_seq);                                   \
    break;
  switch (head_dim) {
    VLA_ATTN_CASE(32)
    VLA_ATTN_CASE(64)
    VLA_ATTN_CASE(128)
    VLA_ATTN_CASE(256)
    default: break;   // rejected by vla_create
  }
#undef VLA_ATTN_CASE
}
}  // namespace vla
