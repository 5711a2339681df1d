// Decode-step GEMMs: C[M,N] = A[M,K] * W[N,K]^T with M = batch (<= 128 rows), bound by streaming the
// weights from HBM once.  No LDS and no barriers in the streaming loop: every wave is an independent
// stream.
//
//   * A wave owns two 32-row weight blocks (64 output columns) over one slice of K.  Per k-step of 16
//     it loads two weight fragments (1 KiB each, fully coalesced, straight from the packed layout into
//     MFMA operand registers) and M/32 activation fragments, and issues 2*M/32 MFMAs.
//   * Activations are kept in the same fragment order as the weights ([m/32][k/16][lane][8], written
//     that way by the producing kernels), so their loads are coalesced 1 KiB reads that hit in L2.
//   * Loads run D k-steps ahead of the MFMAs through a register ring (static indices after unrolling),
//     which keeps D * (2 + M/32) KiB per wave in flight.
//   * K is split into 4 * kgroups slices to put enough waves on the chip.  The four waves of a
//     workgroup add their partial tiles through LDS; one plane part[kg][M][N] is written per group and
//     the following reduce kernel adds the planes in a fixed order (deterministic) and applies the
//     layer's elementwise step: RoPE + KV append, residual add + RMSNorm for the next GEMM, or SwiGLU.
#include <type_traits>

#include "common.h"

namespace vla {

// Element (m, k) of an [M, K] operand in fragment order.
__device__ __forceinline__ size_t frag_index(int m, int k, int K) {
  return ((size_t)(m >> 5) * (K >> 4) + (k >> 4)) * 512 + ((m & 31) + 32 * ((k >> 3) & 1)) * 8 + (k & 7);
}

// acc += a * b, the sum in the registers of acc: left to itself the compiler gives products separate source and result
// registers, and from two blocks of rows on it spills and moves accumulators in the streaming loop.  It does not know the
// latency of the statement: settle() before anything but another of these touches the accumulators.
__device__ __forceinline__ void mfma_in_place(f32x16& acc, const f16x8& a, const f16x8& b) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
#endif
}
// The wait on both sides of a run of such products (12 issue slots behind a product, 2 in front of one; 32 given).  It
// takes the accumulators and gives them back, so whatever reads them, register copies included, depends on it.
template <int MT>
__device__ __forceinline__ void settle(f32x16 (&p)[MT], f32x16 (&q)[MT]) {
  static_assert(MT >= 1 && MT <= 4, "one statement names every accumulator");
#if defined(__HIP_DEVICE_COMPILE__)
#define VLA_SETTLE(...) asm volatile("s_nop 15\n\ts_nop 15" : __VA_ARGS__)
  if constexpr (MT == 1) VLA_SETTLE("+v"(p[0]), "+v"(q[0]));
  else if constexpr (MT == 2) VLA_SETTLE("+v"(p[0]), "+v"(q[0]), "+v"(p[1]), "+v"(q[1]));
  else if constexpr (MT == 3) VLA_SETTLE("+v"(p[0]), "+v"(q[0]), "+v"(p[1]), "+v"(q[1]), "+v"(p[2]), "+v"(q[2]));
  else VLA_SETTLE("+v"(p[0]), "+v"(q[0]), "+v"(p[1]), "+v"(q[1]), "+v"(p[2]), "+v"(q[2]), "+v"(p[3]), "+v"(q[3]));
#undef VLA_SETTLE
#endif
}

// launch(two, once) with the flags as compile-time values.  once: the weights are read as data that does not come again (see
// weights_read_once).
template <class F>
static void by_flags(bool two, bool once, F&& launch) {
  if (two && once) launch(std::true_type{}, std::true_type{});
  else if (two) launch(std::true_type{}, std::false_type{});
  else if (once) launch(std::false_type{}, std::true_type{});
  else launch(std::false_type{}, std::false_type{});
}

// ---- RMS statistics of a float32 row ---------------------------------------------------------------------------
// Every kernel of the decode path that normalises a row adds its squares in one order, so that the bits do not depend on
// which of them a batch takes: pieces of four elements; groups of 16, (p0 + p1) + (p2 + p3); spans of 64, (g0 + g1) +
// (g2 + g3); lane j of sixteen adds spans j, j + 16, ...; a butterfly over the sixteen, narrowest stride first.
__device__ __forceinline__ float sum4_squares(const f32x4& v) {
  return fmaf(v[3], v[3], fmaf(v[2], v[2], fmaf(v[1], v[1], v[0] * v[0])));
}
// ss: a lane's spans; lanes 16 i .. 16 i + 15 hold one row.
__device__ __forceinline__ float norm_factor(float ss, int d, float eps) {
  ss = lanes_sum<1, 8>(ss);
  return 1.0f / sqrtf(ss / (float)d + eps);
}

// The same behind products the compiler knows, whose waits over a chain of branches are a slot short of the longest case.
__device__ __forceinline__ void settle(f32x16& p) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_nop 15" : "+v"(p));
#endif
}

// y * factor as one or two terms.  The product is rounded to float32 here: left to itself the compiler makes one instruction of
// product and conversion in some kernels and two in others, with other bits.
__device__ __forceinline__ float norm_scaled(float y, float factor) {
  float h = y * factor;
  asm("" : "+v"(h));
  return h;
}

// One wave's share of the product: k-blocks kb_begin .. kb_end - 1 (16 k each) of column pair nbp, all MT * 32 rows.
// TWO: two-term activations.  Af_lo holds the low terms in the same fragment order; every weight fragment is
// used for the hi and the lo activation fragments (weights are read once, the MFMA work doubles).
// D: ring depth.  Rows of A past M - 1 are read from row M - 1: their results are not used, and a few rows then cost the
// L2 a few lines per fragment instead of sixteen.
template <int MT, int D, bool TWO, bool ONCE>
__device__ __forceinline__ void stream_slice(const f16* __restrict__ Af, const f16* __restrict__ Af_lo,
                                             const f16* __restrict__ Wp, int nbp, int kb_begin, int kb_end, int KB16,
                                             int M, f32x16 (&acc0)[MT], f32x16 (&acc1)[MT]) {
  // bases are the same for the whole wave (scalar registers), a lane adds its 16 bytes of a fragment
  const unsigned lane = threadIdx.x & 63, at_lane = lane * 8;
  const unsigned at_last = (min(lane & 31, (unsigned)(M - 1 - 32 * (MT - 1))) + (lane & 32)) * 8;   // last block of rows
  const f16* w0 = Wp + ((size_t)(2 * nbp) * KB16) * 512;
  const f16* w1 = w0 + (size_t)KB16 * 512;

#pragma unroll
  for (int i = 0; i < MT; ++i) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      acc0[i][e] = 0.f;
      acc1[i][e] = 0.f;
    }
  }
  settle<MT>(acc0, acc1);                                  // the zeros are written

  // Each wave walks its slice from a different starting point (rotated by its column pair).  The rows of
  // the packed matrix are a power-of-two number of bytes apart for K = 4096, so waves marching through k
  // in lockstep would all hit the same memory channels at the same time.
  const int len = kb_end - kb_begin;
  const int rot = (nbp * 5) % len;
  auto kb_of = [&](int i) {                                // i-th step of this wave, clamped to the slice
    const int j = min(i, len - 1) + rot;
    return (size_t)(kb_begin + (j >= len ? j - len : j));
  };
  constexpr int NA = TWO ? 2 * MT : MT;                    // activation fragments per k-step: hi (then lo)
  f16x8 wq[D][2], aq[D][NA];
  auto load_stage = [&](int s, size_t kb) {
    wq[s][0] = load_once<ONCE>((const f16x8*)(w0 + kb * 512 + at_lane));
    wq[s][1] = load_once<ONCE>((const f16x8*)(w1 + kb * 512 + at_lane));
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const size_t at = ((size_t)mt * KB16 + kb) * 512;
      aq[s][mt] = *(const f16x8*)(Af + at + (mt == MT - 1 ? at_last : at_lane));
      if constexpr (TWO) aq[s][MT + mt] = *(const f16x8*)(Af_lo + at + (mt == MT - 1 ? at_last : at_lane));
    }
  };
  auto mfma_stage = [&](int s) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      mfma_in_place(acc0[mt], aq[s][mt], wq[s][0]);
      mfma_in_place(acc1[mt], aq[s][mt], wq[s][1]);
      if constexpr (TWO) {
        mfma_in_place(acc0[mt], aq[s][MT + mt], wq[s][0]);
        mfma_in_place(acc1[mt], aq[s][MT + mt], wq[s][1]);
      }
    }
  };
#pragma unroll
  for (int s = 0; s < D; ++s) load_stage(s, kb_of(s));
  // Full groups of D k-steps: straight-line body (no branches, so the load counter is tracked exactly and
  // each MFMA waits only for its own stage); every consumed stage is refilled D steps ahead, clamped to the
  // last step of the slice.  The remaining steps (< D) sit in the first stages after the last group.
  const int n_full = len / D;
  for (int g = 0; g < n_full; ++g) {
    const int base = g * D;
#pragma unroll
    for (int s = 0; s < D; ++s) {
      mfma_stage(s);
      load_stage(s, kb_of(base + s + D));
      __builtin_amdgcn_sched_barrier(0);   // keep the refills in stage order, or the oldest stage's wait
                                           // degenerates into a wait for every outstanding load
    }
  }
  const int rem = len - n_full * D;
#pragma unroll
  for (int s = 0; s < D; ++s)
    if (s < rem) mfma_stage(s);
  settle<MT>(acc0, acc1);
}

// Accumulators to / from LDS slot `slot` of [slots][MT * 32 registers][64 lanes].
template <int MT>
__device__ __forceinline__ void put_acc(float* red, int slot, const f32x16 (&acc0)[MT], const f32x16 (&acc1)[MT]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      red[(((size_t)slot * MT + mt) * 32 + e) * 64 + lane] = acc0[mt][e];
      red[(((size_t)slot * MT + mt) * 32 + 16 + e) * 64 + lane] = acc1[mt][e];
    }
}
template <int MT>
__device__ __forceinline__ void add_acc(const float* red, int slot, f32x16 (&acc0)[MT], f32x16 (&acc1)[MT]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      acc0[mt][e] += red[(((size_t)slot * MT + mt) * 32 + e) * 64 + lane];
      acc1[mt][e] += red[(((size_t)slot * MT + mt) * 32 + 16 + e) * 64 + lane];
    }
}

// Where element (m, c) of the 64-column tile lies in a slot: row 32 mt + r is register 4 * (r >> 3) + (r & 3) of the lanes
// of half (r >> 2) & 1, column c is lane c & 31 of the half, columns 32 .. 63 are registers 16 .. 31.
__device__ __forceinline__ int acc_at(int m, int c) {
  const int r = m & 31;
  return ((m >> 5) * 32 + (c >> 5) * 16 + 4 * (r >> 3) + (r & 3)) * 64 + 32 * ((r >> 2) & 1) + (c & 31);
}

// Output rows: the M rows of this launch are rows row0 .. row0 + M - 1 of planes of plane_rows rows each.
template <int MT, int D, bool TWO, bool ONCE>
__global__ __launch_bounds__(256, (MT <= 2 || !TWO) ? 2 : 1) void skinny_gemm_kernel(const f16* __restrict__ Af, const f16* __restrict__ Af_lo,
                                                          const f16* __restrict__ Wp, float* __restrict__ part, int M,
                                                          int N, int K, int kgroups, int plane_rows, int row0) {
  // Workgroup = one pair of 32-row weight blocks (64 output columns) x one group of 4 K slices; wave w
  // streams slice 4*kg + w.  The four partial tiles are added through LDS in the fixed order
  // (w0 + w2) + (w1 + w3), so one plane part[kg] is written per group, deterministically.
  extern __shared__ float red[];                          // [2][MT*32 regs][64 lanes]
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int NP = N >> 6;
  const int nbp = blockIdx.x % NP, kg = blockIdx.x / NP;
  const int KB16 = K >> 4;
  const int slices = 4 * kgroups, sl = 4 * kg + wave;
  const int kb_begin = (int)((long long)sl * KB16 / slices);
  const int kb_end = (int)((long long)(sl + 1) * KB16 / slices);   // non-empty: slices <= KB16

  // two arrays (one per 32-column block) rather than one: the compiler splits an array into scalars only up to a
  // bounded number of accesses, and an unsplit accumulator array would live in scratch memory
  f32x16 acc0[MT], acc1[MT];
  stream_slice<MT, D, TWO, ONCE>(Af, Af_lo, Wp, nbp, kb_begin, kb_end, KB16, M, acc0, acc1);
  if (wave >= 2) put_acc<MT>(red, wave - 2, acc0, acc1);
  __syncthreads();
  if (wave < 2) add_acc<MT>(red, wave, acc0, acc1);         // w0 += w2, w1 += w3
  __syncthreads();
  if (wave < 2) put_acc<MT>(red, wave, acc0, acc1);
  __syncthreads();
  // all threads add the last two and write 16-byte row pieces
  float* out = part + ((size_t)kg * plane_rows + row0) * N + nbp * 64;
  for (int i = threadIdx.x; i < MT * 32 * 16; i += 256) {
    const int m = i >> 4, c = (i & 15) * 4;
    if (m >= M) break;
    const float* p = red + acc_at(m, c);
    const f32x4 p0 = *(const f32x4*)p, p1 = *(const f32x4*)(p + MT * 32 * 64);
    *(f32x4*)(out + (size_t)m * N + c) = (p0 + p1) * (1.0f / kWeightScale);
  }
}

// The end of the gate/up products: the eight waves' tiles are added through LDS ([4][MT*32 regs][64 lanes]) as ((w0 + w2) +
// (w1 + w3)) + ((w4 + w6) + (w5 + w7)), which is the order two planes of four waves and a sum over the planes would have.
template <int MT>
__device__ __forceinline__ void swiglu_finish(float* red, int wave, f32x16 (&acc0)[MT], f32x16 (&acc1)[MT],
                                              f16* __restrict__ act_frag, f16* __restrict__ act_frag_lo, int M, int f, int nbp) {
  const int pair = (wave >> 2) * 2 + (wave & 1);          // slot of waves {0, 2}, {1, 3}, {4, 6}, {5, 7}
  if (wave & 2) put_acc<MT>(red, pair, acc0, acc1);
  __syncthreads();
  if (!(wave & 2)) add_acc<MT>(red, pair, acc0, acc1);
  __syncthreads();
  if (!(wave & 2)) put_acc<MT>(red, pair, acc0, acc1);
  __syncthreads();
  // a thread finishes four consecutive outputs of a row
  for (int i = threadIdx.x; i < MT * 32 * 8; i += 512) {
    const int m = i >> 3, c = (i & 7) * 4;
    if (m >= M) break;
    f32x4 s[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const float* p = red + acc_at(m, j * 32 + c);         // gates, ups
      constexpr int slot = MT * 32 * 64;
      const f32x4 p0 = *(const f32x4*)p, p1 = *(const f32x4*)(p + slot), p4 = *(const f32x4*)(p + 2 * slot),
                  p5 = *(const f32x4*)(p + 3 * slot);
#pragma unroll
      for (int e = 0; e < 4; ++e) s[j][e] = (p0[e] + p1[e]) * (1.0f / kWeightScale) + (p4[e] + p5[e]) * (1.0f / kWeightScale);
    }
    typedef __attribute__((ext_vector_type(4))) _Float16 f16x4;
    f16x4 o, oe;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float a = s[0][e] / (1.0f + __expf(-s[0][e])) * s[1][e];
      o[e] = from_f32<f16>(a);
      oe[e] = from_f32<f16>(a - (float)o[e]);
    }
    const size_t to = frag_index(m, nbp * 32 + c, f);
    *(f16x4*)(act_frag + to) = o;
    if (act_frag_lo) *(f16x4*)(act_frag_lo + to) = oe;
  }
}

// The gate/up product with its elementwise step: a column pair is 32 gates and the matching 32 ups, so a workgroup that
// covers all of K has both sums at hand and writes silu(gate) * up as fragments, with no partial planes in memory and no
// launch behind it.  Eight waves, slice w each.
// Two workgroups per compute unit up to 32 rows, and with single-term operands up to 64 (the register budget behind the
// ring depths): all 344 of the 7B matrix are then resident at once.  From 65 rows on the LDS (96 or 128 KiB) holds one,
// and 344 of them are two rounds on 256 compute units: single-term 45.5 us at 64 rows (43.5 with ONCE), 66.7 at 128.
template <int MT, int D, bool TWO, bool ONCE>
__global__ __launch_bounds__(512, MT == 1 || (MT == 2 && !TWO) ? 4 : 2) void skinny_swiglu_kernel(const f16* __restrict__ Af,
                                                                             const f16* __restrict__ Af_lo,
                                                                             const f16* __restrict__ Wp,
                                                                             f16* __restrict__ act_frag,
                                                                             f16* __restrict__ act_frag_lo, int M, int f,
                                                                             int K) {
  extern __shared__ float red[];                          // [4][MT*32 regs][64 lanes]
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nbp = blockIdx.x, KB16 = K >> 4;
  const int kb_begin = (int)((long long)wave * KB16 / 8);
  const int kb_end = (int)((long long)(wave + 1) * KB16 / 8);      // non-empty: K >= 128
  f32x16 acc0[MT], acc1[MT];
  stream_slice<MT, D, TWO, ONCE>(Af, Af_lo, Wp, nbp, kb_begin, kb_end, KB16, M, acc0, acc1);
  swiglu_finish<MT>(red, wave, acc0, acc1, act_frag, act_frag_lo, M, f, nbp);
}

// M <= kSkinnyMaxRows rows (fragment blocks start at the first of them); Wp: the fused gate/up matrix [2 f, K].
// act_frag_lo may be given with single-term operands and the other way round.
void skinny_swiglu(const f16* Afrag, const f16* Afrag_lo, const f16* Wp, f16* act_frag, f16* act_frag_lo, int M, int f,
                   int K, bool w_once, hipStream_t st) {
  const dim3 grid(f / 32), block(512);
  const int MT = (M + 31) / 32;
#define VLA_SKINNY_LAUNCH(MTV, DV, TWOV, ONCEV)                                                                   \
  {                                                                                                               \
    auto kern = skinny_swiglu_kernel<MTV, DV, TWOV, ONCEV>;                                                       \
    constexpr size_t smem = (size_t)4 * MTV * 32 * 64 * sizeof(float);                                            \
    static bool attr_set = false;                                                                                 \
    if (!attr_set) {                                                                                              \
      (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);        \
      attr_set = true;                                                                                            \
    }                                                                                                             \
    hipLaunchKernelGGL(kern, grid, block, smem, st, Afrag, Afrag_lo, Wp, act_frag, act_frag_lo, M, f, K);         \
  }
#define VLA_SKINNY_CASE(MTV, DV, DV2)                            \
  case MTV:                                                      \
    if (Afrag_lo && w_once) VLA_SKINNY_LAUNCH(MTV, DV2, true, true) \
    else if (Afrag_lo) VLA_SKINNY_LAUNCH(MTV, DV2, true, false)  \
    else if (w_once) VLA_SKINNY_LAUNCH(MTV, DV, false, true)     \
    else VLA_SKINNY_LAUNCH(MTV, DV, false, false)                \
    break;
  switch (MT) {
    VLA_SKINNY_CASE(1, 6, 4)
    VLA_SKINNY_CASE(2, 3, 4)
    VLA_SKINNY_CASE(3, 5, 3)
    VLA_SKINNY_CASE(4, 4, 2)
    default: break;                                        // callers keep M <= kSkinnyMaxRows
  }
#undef VLA_SKINNY_CASE
#undef VLA_SKINNY_LAUNCH
}

// ---- few rows: norm in front, residual add behind ----------------------------------------------------------------
// A decode step of a few rows is a chain of short launches, each of which costs 2.4 us before it does anything, and the
// launches that only sum planes and normalise move next to no data (4.7 us each at d = 4096, two of them a layer).  So
// there the O and down products finish the residual rows themselves and the QKV and gate/up products normalise them: five
// launches a layer instead of seven.  What passes between them are the rows times the next norm's gain, y, in float32 and in
// fragment order, and the sums of their squares over groups of 16 columns: a lane of a fragment holds one row, so a consumer
// needs one factor a lane, and everything it does for the norm happens under its weight loads.
struct NormRows {
  const float* y;        // x * gain, [k / 16][lane][8] (32 rows a block)
  const float* sums;     // [M][d / 16] sums of squares of x
  float eps;
  int M, d;
};

// The norm factor of row (lane & 31) clamped to M - 1.  factors: 32 floats of LDS.  between() runs after the first loads of
// the sums have been issued: loads return in order, so what it requests does not delay them.
template <class Between>
__device__ __forceinline__ float row_factor(const NormRows& in, float* factors, Between&& between) {
  const int j = threadIdx.x & 15, spans = in.d >> 6;
  constexpr int H = 4;                                     // spans of a lane requested at once (all of them to d = 4096)
  f32x4 q[H];
  auto request = [&](int row) {
#pragma unroll
    for (int i = 0; i < H; ++i)
      if (row < in.M && j + 16 * i < spans) q[i] = *(const f32x4*)(in.sums + (size_t)row * (in.d >> 4) + (j + 16 * i) * 4);
  };
  auto finish = [&](int row) {
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < H; ++i)
      if (row < in.M && j + 16 * i < spans) ss += (q[i][0] + q[i][1]) + (q[i][2] + q[i][3]);
    if (row < in.M)
      for (int sp = j + 16 * H; sp < spans; sp += 16) {
        const f32x4 r = *(const f32x4*)(in.sums + (size_t)row * (in.d >> 4) + sp * 4);
        ss += (r[0] + r[1]) + (r[2] + r[3]);
      }
    const float f = norm_factor(ss, in.d, in.eps);
    if (row < in.M && j == 0) factors[row] = f;
  };
  request(threadIdx.x >> 4);
  __builtin_amdgcn_sched_barrier(0);
  between();
  __builtin_amdgcn_sched_barrier(0);
  finish(threadIdx.x >> 4);
  for (int row0 = blockDim.x >> 4; row0 < in.M; row0 += blockDim.x >> 4) {
    request(row0 + (threadIdx.x >> 4));
    finish(row0 + (threadIdx.x >> 4));
  }
  __syncthreads();
  return factors[min((int)threadIdx.x & 31, in.M - 1)];
}

// stream_slice for at most 32 rows that are normalised on the way: a lane's eight elements of a k-block are read as float32,
// scaled by its row's factor and rounded.  D: ring depth.
template <int D, bool TWO, bool ONCE>
__device__ __forceinline__ void norm_stream_slice(const NormRows& in, const f16* __restrict__ Wp, int nbp, int kb_begin,
                                                  int kb_end, float* factors, f32x16& acc0, f32x16& acc1) {
  const unsigned lane = threadIdx.x & 63, at_lane = lane * 8;
  const unsigned at_row = (min(lane & 31, (unsigned)(in.M - 1)) + (lane & 32)) * 8;
  const int KB16 = in.d >> 4;
  const f16* w0 = Wp + ((size_t)(2 * nbp) * KB16) * 512;
  const f16* w1 = w0 + (size_t)KB16 * 512;
  const int len = kb_end - kb_begin;
  const int rot = (nbp * 5) % len;                         // as in stream_slice: the same order of the products
  auto kb_of = [&](int i) {
    const int j = min(i, len - 1) + rot;
    return (size_t)(kb_begin + (j >= len ? j - len : j));
  };
  f16x8 wq[D][2];
  f32x4 yq[D][2];
  auto load_stage = [&](int s, int i) {
    const size_t at = kb_of(i) * 512;
    wq[s][0] = load_once<ONCE>((const f16x8*)(w0 + at + at_lane));
    wq[s][1] = load_once<ONCE>((const f16x8*)(w1 + at + at_lane));
    yq[s][0] = *(const f32x4*)(in.y + at + at_row);
    yq[s][1] = *(const f32x4*)(in.y + at + at_row + 4);
  };
  const float inv = row_factor(in, factors, [&] {
#pragma unroll
    for (int s = 0; s < D; ++s) load_stage(s, s);
  });
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    acc0[e] = 0.f;
    acc1[e] = 0.f;
  }
  auto mfma_stage = [&](int s) {
    f16x8 hi, lo;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float h = norm_scaled(yq[s][j >> 2][j & 3], inv);
      hi[j] = from_f32<f16>(h);
      if constexpr (TWO) lo[j] = from_f32<f16>(h - (float)hi[j]);
    }
    acc0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(hi, wq[s][0], acc0, 0, 0, 0);
    acc1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(hi, wq[s][1], acc1, 0, 0, 0);
    if constexpr (TWO) {
      acc0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(lo, wq[s][0], acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(lo, wq[s][1], acc1, 0, 0, 0);
    }
  };
  const int n_full = len / D;
  for (int g = 0; g < n_full; ++g) {
#pragma unroll
    for (int s = 0; s < D; ++s) {
      mfma_stage(s);
      load_stage(s, g * D + s + D);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  const int rem = len - n_full * D;
#pragma unroll
  for (int s = 0; s < D; ++s)
    if (s < rem) mfma_stage(s);
  settle(acc0);
  settle(acc1);
}

// skinny_gemm_kernel for at most 32 rows with the norm of its rows in front.
template <int D, bool TWO, bool ONCE>
__global__ __launch_bounds__(256, 2) void skinny_norm_gemm_kernel(NormRows in, const f16* __restrict__ Wp,
                                                                  float* __restrict__ part, int N, int kgroups) {
  __shared__ float red[2 * 32 * 64];
  __shared__ float factors[32];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int NP = N >> 6, KB16 = in.d >> 4, M = in.M;
  const int nbp = blockIdx.x % NP, kg = blockIdx.x / NP;
  const int slices = 4 * kgroups, sl = 4 * kg + wave;
  f32x16 acc0[1], acc1[1];
  norm_stream_slice<D, TWO, ONCE>(in, Wp, nbp, (int)((long long)sl * KB16 / slices), (int)((long long)(sl + 1) * KB16 / slices),
                               factors, acc0[0], acc1[0]);
  if (wave >= 2) put_acc<1>(red, wave - 2, acc0, acc1);
  __syncthreads();
  if (wave < 2) add_acc<1>(red, wave, acc0, acc1);         // w0 += w2, w1 += w3
  __syncthreads();
  if (wave < 2) put_acc<1>(red, wave, acc0, acc1);
  __syncthreads();
  float* out = part + (size_t)kg * M * N + nbp * 64;
  for (int i = threadIdx.x; i < M * 16; i += 256) {
    const int m = i >> 4, c = (i & 15) * 4;
    const float* p = red + acc_at(m, c);
    const f32x4 p0 = *(const f32x4*)p, p1 = *(const f32x4*)(p + 32 * 64);
    *(f32x4*)(out + (size_t)m * N + c) = (p0 + p1) * (1.0f / kWeightScale);
  }
}

// skinny_swiglu_kernel for at most 32 rows with the norm of its rows in front.  Two workgroups per compute unit.
template <int D, bool TWO, bool ONCE>
__global__ __launch_bounds__(512, 4) void skinny_norm_swiglu_kernel(NormRows in, const f16* __restrict__ Wp,
                                                                    f16* __restrict__ act_frag, f16* __restrict__ act_frag_lo,
                                                                    int f) {
  __shared__ float red[4 * 32 * 64];
  __shared__ float factors[32];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int KB16 = in.d >> 4;
  f32x16 acc0[1], acc1[1];
  norm_stream_slice<D, TWO, ONCE>(in, Wp, blockIdx.x, (int)((long long)wave * KB16 / 8), (int)((long long)(wave + 1) * KB16 / 8),
                               factors, acc0[0], acc1[0]);
  swiglu_finish<1>(red, wave, acc0, acc1, act_frag, act_frag_lo, in.M, f, blockIdx.x);
}

// Lanes 16 .. 31 and 48 .. 63 of v, in lanes 0 .. 15 and 32 .. 47 (the others: anything).
__device__ __forceinline__ f16x8 odd_sixteens(const f16x8& v) {
#if defined(__HIP_DEVICE_COMPILE__)
  const u32x4 a = __builtin_bit_cast(u32x4, v);
  u32x4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    unsigned c = a[i];
    asm("" : "+v"(c));                                     // (of a swap of a value with itself the compiler makes a copy)
    r[i] = __builtin_amdgcn_permlane16_swap(a[i], c, false, false)[1];
  }
  return __builtin_bit_cast(f16x8, r);
#else
  return v;
#endif
}

// x += A * W^T for at most 32 rows, and with a gain y = x * gain and the sums of squares for the next product.  A workgroup
// covers 16 columns over all of K, one wave a slice (4 * planes of them, as skinny_gemm_kernel cuts them), so the residual
// rows are finished here, in the order of that kernel's planes.  16 columns because 32 would leave half of the compute units
// of the N = 4096 products without work.  The product takes 32 columns a k-block, of which 16 are used; a load takes 16
// columns of two k-blocks, lanes l and l + 16 (l + 32 and l + 48), and the second k-block's are moved over when they are
// due.  FEW: at most 16 rows, whose fragments are loaded the same way.  (A load instruction occupies a compute unit's address
// path for 16 cycles whatever its lanes have in common: with a load of 512 bytes and one of activations a k-block that alone
// is 3.9 us of the N = K = 4096 product, 10.5 us at K = 11008.)  us at 1 row, cold weights, with the reduce kernel's work /
// the planes and the reduce kernel: N 4096 K 4096 8.7 / 12.4, K 11008 17.4 / 20.4, N 768 K 768 3.4 / 5.9, K 2048 4.4 / 6.4; at
// 32 rows 10.8 / 12.9, 22.8 / 21.4, 3.7 / 6.8, 5.1 / 7.1.
// D: pairs of k-blocks in flight a wave.
template <int D, bool TWO, bool FEW, bool ONCE>
__global__ __launch_bounds__(1024) void skinny_resid_kernel(const f16* __restrict__ Af, const f16* __restrict__ Af_lo,
                                                            const f16* __restrict__ Wp, float* __restrict__ x,
                                                            const float* __restrict__ gain, float* __restrict__ y,
                                                            float* __restrict__ sums, int M, int N, int K) {
  extern __shared__ float red[];                          // [waves][16 regs][64 lanes]
  const unsigned lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), slices = blockDim.x >> 6;
  const int n0 = blockIdx.x * 16, nbp = n0 >> 6, KB16 = K >> 4;
  const int kb_begin = (int)((long long)wave * KB16 / slices), kb_end = (int)((long long)(wave + 1) * KB16 / slices);
  // a thread finishes outputs threadIdx.x and threadIdx.x + blockDim.x of [M][16] (blockDim.x >= 256)
  float old[2], g = 0.f;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int i = min((int)(threadIdx.x + j * blockDim.x), M * 16 - 1);
    old[j] = x[(size_t)(i >> 4) * N + n0 + (i & 15)];
  }
  if (gain) g = gain[n0 + (threadIdx.x & 15)];
  const int len = kb_end - kb_begin, odd = (lane >> 4) & 1;
  const int rot = (nbp * 5) % len;                         // as in stream_slice: the same order of the products
  const f16* w0 = Wp + ((size_t)(n0 >> 5) * KB16 + kb_begin) * 512;
  const f16* a0 = Af + (size_t)kb_begin * 512;
  const f16* l0 = TWO ? Af_lo + (size_t)kb_begin * 512 : nullptr;
  const unsigned at_w = ((lane & 15) + (n0 & 16) + (lane & 32)) * 8;
  const unsigned at_a = (min(lane & (FEW ? 15 : 31), (unsigned)(M - 1)) + (lane & 32)) * 8;
  auto kb_at = [&](int i) {                                // i-th k-block of this wave, clamped to the slice
    const int j = min(i, len - 1) + rot;
    return (unsigned)(j >= len ? j - len : j) * 512u;
  };
  f16x8 wq[D], aq[D][FEW ? 1 : 2], al[TWO ? D : 1][FEW ? 1 : 2];
  auto load_pair = [&](int s, int p) {
    const unsigned at = kb_at(2 * p + odd);
    wq[s] = load_once<ONCE>((const f16x8*)(w0 + at + at_w));
#pragma unroll
    for (int h = 0; h < (FEW ? 1 : 2); ++h) {
      const unsigned k = (FEW ? at : kb_at(2 * p + h)) + at_a;
      aq[s][h] = *(const f16x8*)(a0 + k);
      if constexpr (TWO) al[s][h] = *(const f16x8*)(l0 + k);
    }
  };
  f32x16 acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  auto mfma_even = [&](int s) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(aq[s][0], wq[s], acc, 0, 0, 0);
    if constexpr (TWO) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(al[s][0], wq[s], acc, 0, 0, 0);
  };
  auto mfma_odd = [&](int s, bool there) {                 // there: false past the end of a slice of odd length
    const f16x8 w = odd_sixteens(wq[s]), none = {};
    const f16x8 a = FEW ? odd_sixteens(aq[s][0]) : aq[s][FEW ? 0 : 1];
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(there ? a : none, w, acc, 0, 0, 0);
    if constexpr (TWO) {
      const f16x8 l = FEW ? odd_sixteens(al[s][0]) : al[s][FEW ? 0 : 1];
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(there ? l : none, w, acc, 0, 0, 0);
    }
  };
#pragma unroll
  for (int s = 0; s < D; ++s) load_pair(s, s);
  const int pairs = len >> 1, n_full = pairs / D;
  for (int t = 0; t < n_full; ++t) {
#pragma unroll
    for (int s = 0; s < D; ++s) {
      mfma_even(s);
      mfma_odd(s, true);
      load_pair(s, t * D + s + D);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  const int rem = ((len + 1) >> 1) - n_full * D;
#pragma unroll
  for (int s = 0; s < D; ++s)
    if (s < rem) {
      mfma_even(s);
      mfma_odd(s, s < rem - (len & 1));
    }
  settle(acc);
#pragma unroll
  for (int e = 0; e < 16; ++e) red[(wave * 16 + e) * 64 + lane] = acc[e];
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int i = threadIdx.x + j * blockDim.x, m = i >> 4, c = i & 15;
    if (i - (int)lane >= M * 16) break;                    // whole waves: the sums below take all lanes
    const float* p = red + (4 * (m >> 3) + (m & 3)) * 64 + 32 * ((m >> 2) & 1) + c;
    float v = old[j];
    for (int kg = 0; kg < slices; kg += 4, p += 4 * 16 * 64)
      v += ((p[0] + p[2 * 16 * 64]) + (p[16 * 64] + p[3 * 16 * 64])) * (1.0f / kWeightScale);
    if (m < M) x[(size_t)m * N + n0 + c] = v;
    if (gain) {
      if (m < M) y[frag_index(m, n0 + c, N)] = v * g;
      f32x4 e;                                             // the four elements of this lane's piece
      e[0] = dpp<kQuad0>(v);
      e[1] = dpp<kQuad1>(v);
      e[2] = dpp<kQuad2>(v);
      e[3] = dpp<kQuad3>(v);
      float ss = combine_step<4>(sum4_squares(e), Add());
      ss = combine_step<8>(ss, Add());
      if (m < M && c == 0) sums[(size_t)m * (N >> 4) + blockIdx.x] = ss;
    }
  }
}

void skinny_norm_gemm(const float* y, const float* sums, float eps, bool two, const f16* Wp, float* part, int M, int N, int d,
                      int kgroups, bool w_once, hipStream_t st) {
  const NormRows in{y, sums, eps, M, d};
  const dim3 grid((N / 64) * kgroups), block(256);
  auto launch = [&](auto TWO, auto ONCE) {
    hipLaunchKernelGGL((skinny_norm_gemm_kernel<6, decltype(TWO)::value, decltype(ONCE)::value>), grid, block, 0, st, in, Wp, part,
                       N, kgroups);
  };
  by_flags(two, w_once, launch);
}
void skinny_norm_swiglu(const float* y, const float* sums, float eps, bool two, const f16* Wp, f16* act_frag, f16* act_frag_lo,
                        int M, int f, int d, bool w_once, hipStream_t st) {
  const NormRows in{y, sums, eps, M, d};
  const dim3 grid(f / 32), block(512);
  auto launch = [&](auto TWO, auto ONCE) {
    hipLaunchKernelGGL((skinny_norm_swiglu_kernel<3, decltype(TWO)::value, decltype(ONCE)::value>), grid, block, 0, st, in, Wp,
                       act_frag, act_frag_lo, f);
  };
  by_flags(two, w_once, launch);
}
template <int D, bool TWO, bool FEW>
static void launch_resid(bool w_once, const f16* Afrag, const f16* Afrag_lo, const f16* Wp, float* x, const float* gain, float* y, float* sums,
                         int M, int N, int K, int kgroups, hipStream_t st) {
  auto kern = w_once ? skinny_resid_kernel<D, TWO, FEW, true> : skinny_resid_kernel<D, TWO, FEW, false>;
  hipLaunchKernelGGL(kern, dim3(N / 16), dim3(256 * kgroups), (size_t)4 * kgroups * 16 * 64 * sizeof(float), st, Afrag, Afrag_lo, Wp, x,
                     gain, y, sums, M, N, K);
}
// Slices of up to eight k-blocks (the products of a small model) take two pairs in flight, which start sooner: N 768 K 768
// 3.3 us with two, 3.5 with four, K 2048 4.3 and 4.5; others four (three where the registers hold 32 rows of both terms).
void skinny_resid(const f16* Afrag, const f16* Afrag_lo, const f16* Wp, float* x, const float* gain, float* y, float* sums, int M,
                  int N, int K, int kgroups, bool w_once, hipStream_t st) {
  const bool brief = K / 16 <= 4 * kgroups * 8;
#define VLA_RESID(D, TWO, FEW) launch_resid<D, TWO, FEW>(w_once, Afrag, Afrag_lo, Wp, x, gain, y, sums, M, N, K, kgroups, st)
  if (M <= 16) {
    if (Afrag_lo) { if (brief) VLA_RESID(2, true, true); else VLA_RESID(4, true, true); }
    else { if (brief) VLA_RESID(2, false, true); else VLA_RESID(4, false, true); }
  } else {
    if (Afrag_lo) { if (brief) VLA_RESID(2, true, false); else VLA_RESID(3, true, false); }
    else { if (brief) VLA_RESID(2, false, false); else VLA_RESID(4, false, false); }
  }
#undef VLA_RESID
}

#ifndef VLA_SKINNY_UNITS
#define VLA_SKINNY_UNITS 1536    // independent streams (waves) a decode GEMM is cut into, at least
#endif
// Number of partial planes (groups of 4 K slices) for an [N, K] weight matrix.
int skinny_ksplit(int N, int K) {
  const int NP = N / 64;
  int kg = (VLA_SKINNY_UNITS + 4 * NP - 1) / (4 * NP);
  if (kg < 1) kg = 1;
  if (kg > kMaxKSplit) kg = kMaxKSplit;
  while (kg > 1 && 4 * kg > K / 16) --kg;
  return kg;
}

// M <= kSkinnyMaxRows rows (fragment blocks Afrag / Afrag_lo start at the first of them); Afrag_lo != nullptr: two-term.
void skinny_gemm(const f16* Afrag, const f16* Afrag_lo, const f16* Wp, float* part, int M, int N, int K, int kgroups,
                 int plane_rows, int row0, bool w_once, hipStream_t st) {
  // (read once, matrices in MB, 32 to 64 rows: 14 11.4 -> 12.0 us, 25 12.5 -> 13.2 and 14.6 -> 15.6, 34 19.1 -> 19.9, 56 18.9 ->
  // 18.7, 90 32.2 -> 30.4, 101 34.6 -> 33.9, 141 60.4 -> 56.5)
  w_once = w_once && 2LL * N * K >= 64'000'000;
  const dim3 grid((N / 64) * kgroups), block(256);
  const int MT = (M + 31) / 32;
  const size_t smem = (size_t)2 * MT * 32 * 64 * sizeof(float);
#define VLA_SKINNY_LAUNCH(MTV, DV, TWOV, ONCEV)                                                                   \
  {                                                                                                               \
    auto kern = skinny_gemm_kernel<MTV, DV, TWOV, ONCEV>;                                                         \
    static bool attr_set = false;                                                                                 \
    if (!attr_set) {                                                                                              \
      (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);        \
      attr_set = true;                                                                                            \
    }                                                                                                             \
    hipLaunchKernelGGL(kern, grid, block, smem, st, Afrag, Afrag_lo, Wp, part, M, N, K, kgroups, plane_rows, row0); \
  }
#define VLA_SKINNY_CASE(MTV, DV, DV2)                            \
  case MTV:                                                      \
    if (Afrag_lo && w_once) VLA_SKINNY_LAUNCH(MTV, DV2, true, true) \
    else if (Afrag_lo) VLA_SKINNY_LAUNCH(MTV, DV2, true, false)  \
    else if (w_once) VLA_SKINNY_LAUNCH(MTV, DV, false, true)     \
    else VLA_SKINNY_LAUNCH(MTV, DV, false, false)                \
    break;
  switch (MT) {     // ring depth: as deep as the registers allow (weights 2 + activations MT or 2 MT fragments per stage)
    VLA_SKINNY_CASE(1, 8, 6)
    VLA_SKINNY_CASE(2, 6, 4)
    VLA_SKINNY_CASE(3, 4, 3)
    VLA_SKINNY_CASE(4, 3, 2)
    default: break;                                        // callers keep M <= kSkinnyMaxRows
  }
#undef VLA_SKINNY_CASE
#undef VLA_SKINNY_LAUNCH
}

// ---- reduce + elementwise kernels ---------------------------------------------------------------------
// x[m,:] += sum_ks part[ks][m,:]; if gain: hn (fragment order) = f16(x * gain / rms(x)), and with hn_frag_lo the
// low terms f16(h - hi) as well.  Row m of the launch is row prow0 + m of each plane (plane_rows rows per plane) and
// row row0 + m of x and hn.  Bound by latency (one row is 16 KiB a plane at d = 4096): up to 1024 threads a row, so that
// all of a row's loads are one round, and the sums stay in registers between the statistics and the output.
template <int VPT>                                         // float4 per thread
__global__ __launch_bounds__(1024) void reduce_resid_norm_kernel(const float* __restrict__ part, int ksplit,
                                                                 int plane_rows, int prow0, int d,
                                                                 float* __restrict__ x, const float* __restrict__ gain,
                                                                 float eps, f16* __restrict__ hn_frag,
                                                                 f16* __restrict__ hn_frag_lo, int row0) {
  __shared__ float red[VPT * 64];
  const int m = blockIdx.x;
  float* row = x + (size_t)(row0 + m) * d;
  f32x4 v[VPT], g[VPT];
#pragma unroll
  for (int it = 0; it < VPT; ++it) {
    const int i = (threadIdx.x + it * blockDim.x) * 4;
    if (i < d) {
      f32x4 p[kMaxKSplit];
      v[it] = *(const f32x4*)(row + i);
#pragma unroll
      for (int ks = 0; ks < kMaxKSplit; ++ks)              // all loads in flight first; summed in slice order
        p[ks] = ks < ksplit ? *(const f32x4*)(part + ((size_t)ks * plane_rows + prow0 + m) * d + i)
                            : f32x4{0.f, 0.f, 0.f, 0.f};
      if (gain) g[it] = *(const f32x4*)(gain + i);
#pragma unroll
      for (int ks = 0; ks < kMaxKSplit; ++ks)
#pragma unroll
        for (int j = 0; j < 4; ++j) v[it][j] += p[ks][j];
      *(f32x4*)(row + i) = v[it];
    }
    if (gain) {                                            // a span of 64 columns is 16 lanes
      float ss = i < d ? sum4_squares(v[it]) : 0.f;
      ss = lanes_sum<1, 8>(ss);
      if (i < d && (threadIdx.x & 15) == 0) red[i >> 6] = ss;
    }
  }
  if (!gain) return;
  __syncthreads();
  float ss = 0.f;
  for (int sp = threadIdx.x & 15; sp < (d >> 6); sp += 16) ss += red[sp];
  const float inv = norm_factor(ss, d, eps);
#pragma unroll
  for (int it = 0; it < VPT; ++it) {
    const int i = (threadIdx.x + it * blockDim.x) * 4;
    if (i < d) {
      typedef __attribute__((ext_vector_type(4))) _Float16 f16x4;
      f16x4 o, oe;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float h = norm_scaled(v[it][j] * g[it][j], inv);
        o[j] = from_f32<f16>(h);
        oe[j] = from_f32<f16>(h - (float)o[j]);
      }
      const size_t at = frag_index(row0 + m, i, d);
      *(f16x4*)(hn_frag + at) = o;
      if (hn_frag_lo) *(f16x4*)(hn_frag_lo + at) = oe;
    }
  }
}

void reduce_resid_norm(const float* part, int ksplit, int plane_rows, int prow0, int M, int d, float* x,
                       const float* gain, float eps, f16* hn_frag, f16* hn_frag_lo, int row0, hipStream_t st) {
  const int n4 = d / 4, threads = n4 >= 1024 ? 1024 : (n4 + 63) / 64 * 64;     // d <= 16384 (configuration checks)
#define VLA_REDUCE(V)                                                                                                 \
  hipLaunchKernelGGL(reduce_resid_norm_kernel<V>, dim3(M), dim3(threads), 0, st, part, ksplit, plane_rows, prow0, d, x, \
                     gain, eps, hn_frag, hn_frag_lo, row0)
  if (n4 <= 1024) VLA_REDUCE(1);
  else if (n4 <= 2048) VLA_REDUCE(2);
  else VLA_REDUCE(4);
#undef VLA_REDUCE
}

// Start of a decode step, one workgroup per row: the token's embedding becomes row b of the residual stream, the row's
// cache slot and position are noted for the layers and the sequence grows by one; with a gain (16-bit path) the row goes on
// to the first layer, as y and sums of squares (see NormRows) or, if y is null, normalised in fragment order.  (One launch:
// four of them, a few us each, are a tenth of a step of a small model.)
template <class T>
__global__ __launch_bounds__(256) void decode_begin_kernel(const int32_t* __restrict__ ids, const T* __restrict__ embed,
                                                           int vocab, int32_t* seq_len,
                                                           const int32_t* __restrict__ slot_map,
                                                           int32_t* __restrict__ tok_seq, int32_t* __restrict__ tok_pos,
                                                           float* __restrict__ x, int d, const float* __restrict__ gain,
                                                           float eps, float* __restrict__ y, float* __restrict__ sums,
                                                           f16* __restrict__ hn_frag, f16* __restrict__ hn_frag_lo) {
  __shared__ float red[256];                               // spans of 64 (d <= 16384)
  const int m = blockIdx.x;
  if (threadIdx.x == 0) {
    const int slot = slot_map ? slot_map[m] : m;
    const int pos = seq_len[slot];
    tok_seq[m] = slot;
    tok_pos[m] = pos;
    seq_len[slot] = pos + 1;
  }
  int id = ids[m];
  id = id < 0 ? 0 : (id >= vocab ? vocab - 1 : id);   // ids come from device memory: stay in bounds
  const T* src = embed + (size_t)id * d;
  float* row = x + (size_t)m * d;
  auto load = [&](int i) {
    f32x4 v;
    if constexpr (sizeof(T) == 2) {
      const bf16x4 e = *(const bf16x4*)(src + i);
      v = f32x4{(float)e[0], (float)e[1], (float)e[2], (float)e[3]};
    } else {
      v = *(const f32x4*)(src + i);
    }
    return v;
  };
  typedef __attribute__((ext_vector_type(4))) _Float16 f16x4;
  for (int i0 = 0; i0 < d; i0 += 1024) {                   // (whole waves: the sums of squares take all lanes)
    const int i = i0 + threadIdx.x * 4;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (i < d) {
      v = load(i);
      *(f32x4*)(row + i) = v;
    }
    if (gain) {
      float ss = sum4_squares(v);
      ss = lanes_sum<1, 2>(ss);
      if (y) {
        if (i < d) {
          *(f32x4*)(y + frag_index(m, i, d)) = v * *(const f32x4*)(gain + i);
          if ((threadIdx.x & 3) == 0) sums[(size_t)m * (d >> 4) + (i >> 4)] = ss;
        }
      } else {
        ss = combine_step<8>(combine_step<4>(ss, Add()), Add());
        if (i < d && (threadIdx.x & 15) == 0) red[i >> 6] = ss;
      }
    }
  }
  if (!gain || y) return;
  __syncthreads();
  float ss = 0.f;
  for (int sp = threadIdx.x & 15; sp < (d >> 6); sp += 16) ss += red[sp];
  const float inv = norm_factor(ss, d, eps);
  for (int i = threadIdx.x * 4; i < d; i += 1024) {
    const f32x4 v = load(i), g = *(const f32x4*)(gain + i);
    f16x4 o, oe;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float h = norm_scaled(v[j] * g[j], inv);
      o[j] = from_f32<f16>(h);
      oe[j] = from_f32<f16>(h - (float)o[j]);
    }
    const size_t at = frag_index(m, i, d);
    *(f16x4*)(hn_frag + at) = o;
    if (hn_frag_lo) *(f16x4*)(hn_frag_lo + at) = oe;
  }
}
template <class T>
void decode_begin(const int32_t* ids, const T* embed, int vocab, int32_t* seq_len, const int32_t* slot_map,
                  int32_t* tok_seq, int32_t* tok_pos, float* x, int M, int d, const float* gain, float eps, float* y,
                  float* sums, f16* hn_frag, f16* hn_frag_lo, hipStream_t st) {
  hipLaunchKernelGGL(decode_begin_kernel<T>, dim3(M), dim3(256), 0, st, ids, embed, vocab, seq_len, slot_map, tok_seq,
                     tok_pos, x, d, gain, eps, y, sums, hn_frag, hn_frag_lo);
}
template void decode_begin<float>(const int32_t*, const float*, int, int32_t*, const int32_t*, int32_t*, int32_t*, float*,
                                  int, int, const float*, float, float*, float*, f16*, f16*, hipStream_t);
template void decode_begin<bf16>(const int32_t*, const bf16*, int, int32_t*, const int32_t*, int32_t*, int32_t*, float*,
                                 int, int, const float*, float, float*, float*, f16*, f16*, hipStream_t);

// act (fragment order, [M, f]) = silu(gate) * up, gate/up summed over the K slices.  The fused
// gate-up columns are interleaved in blocks of 32: gate j at (j/32)*64 + j%32, up 32 further.
__global__ __launch_bounds__(256) void reduce_swiglu_kernel(const float* __restrict__ part, int ksplit, int plane_rows,
                                                            int prow0, int f, f16* __restrict__ act_frag,
                                                            f16* __restrict__ act_frag_lo, int row0) {
  const int m = blockIdx.y;
  const int j0 = (blockIdx.x * 256 + threadIdx.x) * 4;      // 4 consecutive outputs (same 32-block)
  if (j0 >= f) return;
  const int col = (j0 >> 5) * 64 + (j0 & 31);
  f32x4 gp[kMaxKSplit], up[kMaxKSplit];
#pragma unroll
  for (int ks = 0; ks < kMaxKSplit; ++ks)                    // all loads in flight first; summed in slice order
    if (ks < ksplit) {
      const float* p = part + ((size_t)ks * plane_rows + prow0 + m) * (2 * (size_t)f) + col;
      gp[ks] = *(const f32x4*)p;
      up[ks] = *(const f32x4*)(p + 32);
    }
  f32x4 g = {0.f, 0.f, 0.f, 0.f}, u = g;
#pragma unroll
  for (int ks = 0; ks < kMaxKSplit; ++ks)
    if (ks < ksplit) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        g[j] += gp[ks][j];
        u[j] += up[ks][j];
      }
    }
  typedef __attribute__((ext_vector_type(4))) _Float16 f16x4;
  f16x4 o, oe;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float a = g[j] / (1.0f + __expf(-g[j])) * u[j];
    o[j] = from_f32<f16>(a);
    oe[j] = from_f32<f16>(a - (float)o[j]);
  }
  const size_t at = frag_index(row0 + m, j0, f);
  *(f16x4*)(act_frag + at) = o;
  if (act_frag_lo) *(f16x4*)(act_frag_lo + at) = oe;
}
void reduce_swiglu(const float* part, int ksplit, int plane_rows, int prow0, int M, int f, f16* act_frag,
                   f16* act_frag_lo, int row0, hipStream_t st) {
  hipLaunchKernelGGL(reduce_swiglu_kernel, dim3((f / 4 + 255) / 256, M), dim3(256), 0, st, part, ksplit, plane_rows,
                     prow0, f, act_frag, act_frag_lo, row0);
}

}  // namespace vla
