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

// One wave's share of the product: k-blocks kb_begin .. kb_end - 1 (16 k each) of column pair nbp, all MT * 32 rows.
// TWO: two-term activations.  Af_lo holds the low terms in the same fragment order; every weight fragment is
// used for the hi and the lo activation fragments (weights are read once, the MFMA work doubles).
// D: ring depth.  Rows of A past M - 1 are read from row M - 1: their results are not used, and a few rows then cost the
// L2 a few lines per fragment instead of sixteen.
template <int MT, int D, bool TWO>
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
    wq[s][0] = *(const f16x8*)(w0 + kb * 512 + at_lane);
    wq[s][1] = *(const f16x8*)(w1 + kb * 512 + at_lane);
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
template <int MT, int D, bool TWO>
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
  stream_slice<MT, D, TWO>(Af, Af_lo, Wp, nbp, kb_begin, kb_end, KB16, M, acc0, acc1);
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

// The gate/up product with its elementwise step: a column pair is 32 gates and the matching 32 ups, so a workgroup that
// covers all of K has both sums at hand and writes silu(gate) * up as fragments, with no partial planes in memory and no
// launch behind it.  Eight waves, slice w each; the partial tiles are added as ((w0 + w2) + (w1 + w3)) + ((w4 + w6) +
// (w5 + w7)), which is the order two planes of four waves and a sum over the planes would have.
// Two workgroups per compute unit up to 32 rows, and with single-term operands up to 64 (the register budget behind the
// ring depths): all 344 of the 7B matrix are then resident at once.  From 65 rows on the LDS (96 or 128 KiB) holds one,
// and 344 of them are two rounds on 256 compute units: single-term 45.5 us at 64 rows, 66.7 at 128.
template <int MT, int D, bool TWO>
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
  stream_slice<MT, D, TWO>(Af, Af_lo, Wp, nbp, kb_begin, kb_end, KB16, M, acc0, acc1);
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

// M <= kSkinnyMaxRows rows (fragment blocks start at the first of them); Wp: the fused gate/up matrix [2 f, K].
// act_frag_lo may be given with single-term operands and the other way round.
void skinny_swiglu(const f16* Afrag, const f16* Afrag_lo, const f16* Wp, f16* act_frag, f16* act_frag_lo, int M, int f,
                   int K, hipStream_t st) {
  const dim3 grid(f / 32), block(512);
  const int MT = (M + 31) / 32;
#define VLA_SKINNY_LAUNCH(MTV, DV, TWOV)                                                                          \
  {                                                                                                               \
    auto kern = skinny_swiglu_kernel<MTV, DV, TWOV>;                                                              \
    constexpr size_t smem = (size_t)4 * MTV * 32 * 64 * sizeof(float);                                            \
    static bool attr_set = false;                                                                                 \
    if (!attr_set) {                                                                                              \
      (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);        \
      attr_set = true;                                                                                            \
    }                                                                                                             \
    hipLaunchKernelGGL(kern, grid, block, smem, st, Afrag, Afrag_lo, Wp, act_frag, act_frag_lo, M, f, K);         \
  }
#define VLA_SKINNY_CASE(MTV, DV, DV2)                  \
  case MTV:                                            \
    if (Afrag_lo) VLA_SKINNY_LAUNCH(MTV, DV2, true)    \
    else VLA_SKINNY_LAUNCH(MTV, DV, false)             \
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
                 int plane_rows, int row0, hipStream_t st) {
  const dim3 grid((N / 64) * kgroups), block(256);
  const int MT = (M + 31) / 32;
  const size_t smem = (size_t)2 * MT * 32 * 64 * sizeof(float);
#define VLA_SKINNY_LAUNCH(MTV, DV, TWOV)                                                                          \
  {                                                                                                               \
    auto kern = skinny_gemm_kernel<MTV, DV, TWOV>;                                                                \
    static bool attr_set = false;                                                                                 \
    if (!attr_set) {                                                                                              \
      (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);        \
      attr_set = true;                                                                                            \
    }                                                                                                             \
    hipLaunchKernelGGL(kern, grid, block, smem, st, Afrag, Afrag_lo, Wp, part, M, N, K, kgroups, plane_rows, row0); \
  }
#define VLA_SKINNY_CASE(MTV, DV, DV2)                  \
  case MTV:                                            \
    if (Afrag_lo) VLA_SKINNY_LAUNCH(MTV, DV2, true)    \
    else VLA_SKINNY_LAUNCH(MTV, DV, false)             \
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
__device__ __forceinline__ float block_sum_256d(float v, float* red) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

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
  __shared__ float red[16];
  const int m = blockIdx.x;
  float* row = x + (size_t)(row0 + m) * d;
  f32x4 v[VPT], g[VPT];
  float ss = 0.f;
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
      ss += v[it][0] * v[it][0] + v[it][1] * v[it][1] + v[it][2] * v[it][2] + v[it][3] * v[it][3];
    }
  }
  if (!gain) return;
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  ss = 0.f;
  for (int w = 0; w < (int)(blockDim.x >> 6); ++w) ss += red[w];
  const float inv = 1.0f / sqrtf(ss / (float)d + eps);
#pragma unroll
  for (int it = 0; it < VPT; ++it) {
    const int i = (threadIdx.x + it * blockDim.x) * 4;
    if (i < d) {
      typedef __attribute__((ext_vector_type(4))) _Float16 f16x4;
      f16x4 o, oe;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float h = v[it][j] * inv * g[it][j];
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
// cache slot and position are noted for the layers and the sequence grows by one; with a gain (16-bit path) the first
// layer's normalised row goes to fragment order too.  (One launch: four of them, a few us each, are a tenth of a step of
// a small model.)
template <class T>
__global__ __launch_bounds__(256) void decode_begin_kernel(const int32_t* __restrict__ ids, const T* __restrict__ embed,
                                                           int vocab, int32_t* seq_len,
                                                           const int32_t* __restrict__ slot_map,
                                                           int32_t* __restrict__ tok_seq, int32_t* __restrict__ tok_pos,
                                                           float* __restrict__ x, int d, const float* __restrict__ gain,
                                                           float eps, f16* __restrict__ hn_frag,
                                                           f16* __restrict__ hn_frag_lo) {
  __shared__ float red[4];
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
  float ss = 0.f;
  for (int i = threadIdx.x * 4; i < d; i += 1024) {
    const f32x4 v = load(i);
    *(f32x4*)(row + i) = v;
    ss += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
  }
  if (!gain) return;
  ss = block_sum_256d(ss, red);
  const float inv = 1.0f / sqrtf(ss / (float)d + eps);
  typedef __attribute__((ext_vector_type(4))) _Float16 f16x4;
  for (int i = threadIdx.x * 4; i < d; i += 1024) {
    const f32x4 v = load(i), g = *(const f32x4*)(gain + i);
    f16x4 o, oe;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float h = v[j] * inv * g[j];
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
                  int32_t* tok_seq, int32_t* tok_pos, float* x, int M, int d, const float* gain, float eps, f16* hn_frag,
                  f16* hn_frag_lo, hipStream_t st) {
  hipLaunchKernelGGL(decode_begin_kernel<T>, dim3(M), dim3(256), 0, st, ids, embed, vocab, seq_len, slot_map, tok_seq,
                     tok_pos, x, d, gain, eps, hn_frag, hn_frag_lo);
}
template void decode_begin<float>(const int32_t*, const float*, int, int32_t*, const int32_t*, int32_t*, int32_t*, float*,
                                  int, int, const float*, float, f16*, f16*, hipStream_t);
template void decode_begin<bf16>(const int32_t*, const bf16*, int, int32_t*, const int32_t*, int32_t*, int32_t*, float*,
                                 int, int, const float*, float, f16*, f16*, hipStream_t);

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
