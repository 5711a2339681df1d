// Half-precision MFMA GEMM  C[M,N] = A[M,K] * W[N,K]^T  for gfx950, with the layer's elementwise
// work fused into the epilogue (residual add; SwiGLU; rotary embedding + KV-cache write).
//
// Operand layouts
//   A   [M, K] f16 in fragment order like the weights, lda halves a row: blocks of 32 rows, in each its slabs of 64 k (4 KiB: four
//       blocks of 16 k), behind those of the high terms those of the low ones (act_index, act_lo8_index).  A row-major A costs
//       the same bytes as 128-byte pieces of eight rows an instruction instead of one KiB, and an address a lane.
//   Wp  weights (bf16 at the boundary, re-encoded exactly as f16 * kWeightScale) repacked once at
//       load time into MFMA fragment order: the 32x16 block
//       (rows n0..n0+31, k0..k0+15) is stored as 64 lanes x 8 halves = 1 KiB, lane l holding
//       row n0 + (l & 31), k = k0 + 8*(l >> 5) .. +7; blocks are ordered [n/32][k/16].  A wave
//       reads one block with a single fully coalesced 16-byte-per-lane load, from global memory or
//       from LDS, with no bank conflicts and no swizzle.
#include <cmath>
#include <type_traits>
#include <utility>

#include "common.h"

namespace vla {

// ---- epilogues ------------------------------------------------------------------------------------
// A wave (or a pair of waves side by side, where a wave's columns do not cover the span an epilogue needs) writes
// 32 rows of accumulators to LDS in row-major order and hands them to consume(), which reads them back as float4 row
// chunks, so that global memory sees 16-byte accesses that cover whole 128- to 512-byte row segments instead of
// scattered 2- and 4-byte ones.
//   consume<COLS, PITCH, ROWS>(tile, m_base, nb, lane, M): rows m_base .. + ROWS - 1 and columns nb .. + COLS - 1 of
//   the product, element (r, c) at tile[r * PITCH + c].
//   kSpan: columns that have to be handed over together.

struct EpiResid {
  static constexpr int kSpan = 32;
  float* x;
  int ldx;
  // x += tile / kWeightScale: all loads of the rows are issued before the first store (a store followed by a load of
  // the same array would otherwise serialise on the memory latency); rows past M are read from row M-1, not stored
  template <int COLS, int PITCH, int ROWS>
  __device__ __forceinline__ void consume(const float* tile, int m_base, int nb, int lane, int M) const {
    constexpr int LPR = COLS / 4, RPI = 64 / LPR, IT = ROWS / RPI;
    const int r0 = lane / LPR, c4 = (lane % LPR) * 4;
    f32x4 v[IT], old[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int r = it * RPI + r0;
      v[it] = *(const f32x4*)(tile + r * PITCH + c4);
      old[it] = *(const f32x4*)(x + (size_t)min(m_base + r, M - 1) * ldx + nb + c4);
    }
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int m = m_base + it * RPI + r0;
      if (m < M) *(f32x4*)(x + (size_t)m * ldx + nb + c4) = old[it] + v[it] * (1.0f / kWeightScale);
    }
  }
};

// Split-K form (decode steps of large batches): the tile's partial sums over one K slice go, with the weight scale
// divided out, to plane `kz` of part[ksplit][plane_rows][N]; the reduce kernels of the decode path add the planes.
struct EpiPartial {
  static constexpr int kSpan = 32;
  float* part;          // plane 0; the kernel moves it to its slice's plane
  int plane_rows, row0, N;
  const f16* a_lo;      // low-term activation fragments (two-term operands), or nullptr
  template <int COLS, int PITCH, int ROWS>
  __device__ __forceinline__ void consume(const float* tile, int m_base, int nb, int lane, int M) const {
    constexpr int LPR = COLS / 4, RPI = 64 / LPR;
    const int r0 = lane / LPR, c4 = (lane % LPR) * 4;
#pragma unroll
    for (int it = 0; it < ROWS / RPI; ++it) {
      const int r = it * RPI + r0, m = m_base + r;
      const f32x4 v = *(const f32x4*)(tile + r * PITCH + c4);
      if (m < M) *(f32x4*)(part + (size_t)(row0 + m) * N + nb + c4) = v * (1.0f / kWeightScale);
    }
  }
};

// silu(g) * u for accumulator values G = g * kWeightScale, U = u * kWeightScale, with the scale folded into the
// constants: (G * U / scale^2) / (1 + 2^(-G * log2(e) / scale)).
__device__ __forceinline__ float swiglu_scaled(float G, float U) {
  constexpr float c1 = 1.44269504088896341f / kWeightScale, c2 = 1.0f / (kWeightScale * kWeightScale);
  return (G * U * c2) * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-(G * c1)));
}

// Fused gate/up weights are interleaved in blocks of 32 rows: [gate 0..31, up 0..31, gate 32..63, ...]
// so that every 64 columns of the product are 32 gates followed by the matching 32 ups.
struct EpiSwiglu {
  static constexpr int kSpan = 64;
  f16* act;
  int ld;
  int f;        // number of outputs per row
  int lo_mode;  // 0: single-term; 1: half-precision low terms of output j at column f + j; 2: bytes (act_lo8_index)
  // A lane finishes eight outputs of a row, 16 bytes of a fragment; the lanes of an instruction are 32 (16) rows by 2 (4) such.
  template <int COLS, int PITCH, int ROWS>
  __device__ __forceinline__ void consume(const float* tile, int m_base, int nb, int lane, int M) const {
    typedef __attribute__((ext_vector_type(2))) int i32x2;
    constexpr int PIECES = COLS / 16, PPI = 64 / ROWS;     // of a row; of a row and instruction
    static_assert(PIECES % PPI == 0, "whole instructions");
    const int r = lane % ROWS, m = m_base + r;
#pragma unroll
    for (int it = 0; it < PIECES / PPI; ++it) {
      const int p = it * PPI + lane / ROWS, c = (p >> 2) * 64 + (p & 3) * 8, k = nb / 2 + p * 8;
      float a[8], e[8];
      f16x8 o;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const f32x4 g = *(const f32x4*)(tile + r * PITCH + c + 4 * h);
        const f32x4 u = *(const f32x4*)(tile + r * PITCH + c + 32 + 4 * h);
#pragma unroll
        for (int j = 0; j < 4; ++j) a[4 * h + j] = swiglu_scaled(g[j], u[j]);
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) o[j] = from_f32<f16>(a[j]);
      if (m < M) {
        *(f16x8*)(act + act_index(m, k, ld)) = o;
        if (lo_mode != 0) {                  // (uniform) low terms only where the layer carries them
#pragma unroll
          for (int j = 0; j < 8; ++j) e[j] = a[j] - (float)o[j];
          if (lo_mode == 1) {
            f16x8 oe;
#pragma unroll
            for (int j = 0; j < 8; ++j) oe[j] = from_f32<f16>(e[j]);
            *(f16x8*)(act + act_index(m, f + k, ld)) = oe;
          } else {
            *(i32x2*)((unsigned char*)act + act_lo8_index(m, k, ld, f)) = i32x2{pack_lo8(e[0], e[1], e[2], e[3]), pack_lo8(e[4], e[5], e[6], e[7])};
          }
        }
      }
    }
  }
};

// Columns [0,d) are queries, [d,2d) keys, [2d,3d) values.  The columns handed over are whole heads of one section, so
// the rotary partner (i, i + hd/2) of every column is at hand.
template <int HD>
struct EpiQkv {
  static constexpr int kSpan = HD;
  RopeKv o;
  template <int COLS, int PITCH, int ROWS>
  __device__ __forceinline__ void consume(const float* tile, int m_base, int nb, int lane, int M) const {
    typedef __attribute__((ext_vector_type(4))) _Float16 f16x4;
    constexpr int HALF = HD / 2, LPH = HD / 8;      // lanes per head
    constexpr int LPR = COLS / 8, RPI = 64 / LPR, IT = ROWS / RPI;
    const int rs = lane / LPR, q = lane % LPR, hh = q / LPH, c4 = (q % LPH) * 4;
    const int d = o.d_model;
    const int sect = nb / d;
    const int head = (nb - sect * d) / HD + hh;
    // Positions, slots and rotary factors of all row groups are fetched up front (rows past M clamped), so
    // the two dependent global loads per row overlap instead of forming serial chains.
    int pos[IT], slot[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int m = min(m_base + it * RPI + rs, M - 1);
      pos[it] = o.tok_pos[m];
      slot[it] = o.tok_seq[m];
    }
    f32x4 cs[IT], sn[IT];
    if (sect < 2) {
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        cs[it] = *(const f32x4*)(o.rope_cos + (size_t)pos[it] * HALF + c4);
        sn[it] = *(const f32x4*)(o.rope_sin + (size_t)pos[it] * HALF + c4);
      }
    }
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int r = it * RPI + rs, m = m_base + r;
      f32x4 lo = *(const f32x4*)(tile + r * PITCH + hh * HD + c4) * (1.0f / kWeightScale);
      f32x4 hi = *(const f32x4*)(tile + r * PITCH + hh * HD + HALF + c4) * (1.0f / kWeightScale);
      f16* dst;
      f16* dst_lo = nullptr;                 // two-term mode: low terms of the queries (half precision, column d + ...)
      unsigned char* dst_lo8 = nullptr;      // ... and of the cached keys / values (one byte each)
      if (sect == 0) {
        dst = (f16*)o.q + (size_t)min(m, M - 1) * o.ldq + (size_t)head * HD;
        if (o.k_lo) dst_lo = dst + d;
      } else {
        const size_t at = (((size_t)slot[it] * o.n_heads + head) * o.max_seq + pos[it]) * HD;
        dst = (f16*)(sect == 1 ? o.k_cache : o.v_cache) + at;
        if (o.k_lo) dst_lo8 = (unsigned char*)(sect == 1 ? o.k_lo : o.v_lo) + at;
      }
      if (sect < 2) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float a, b;
          rope_pair(lo[j], hi[j], cs[it][j], sn[it][j], a, b);
          lo[j] = a;
          hi[j] = b;
        }
      }
      f16x4 l4, h4;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        l4[j] = from_f32<f16>(lo[j]);
        h4[j] = from_f32<f16>(hi[j]);
      }
      if (m < M) {
        *(f16x4*)(dst + c4) = l4;
        *(f16x4*)(dst + HALF + c4) = h4;
        if (o.k_lo) {                        // (uniform) low terms only in two-term layers
          float le[4], he[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            le[j] = lo[j] - (float)l4[j];
            he[j] = hi[j] - (float)h4[j];
          }
          if (dst_lo) {
            f16x4 l4e, h4e;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              l4e[j] = from_f32<f16>(le[j]);
              h4e[j] = from_f32<f16>(he[j]);
            }
            *(f16x4*)(dst_lo + c4) = l4e;
            *(f16x4*)(dst_lo + HALF + c4) = h4e;
          }
          if (dst_lo8) {
            *(int*)(dst_lo8 + c4) = pack_lo8(le[0], le[1], le[2], le[3]);
            *(int*)(dst_lo8 + HALF + c4) = pack_lo8(he[0], he[1], he[2], he[3]);
          }
        }
      }
    }
  }
};

// ---- 8-bit low terms --------------------------------------------------------------------------------------
// Two-term activations may carry their low term as one byte: lo8 = bf8(16 * (a - f16(a))) (1-5-2 format), behind the
// Kw high terms of a block of 32 rows (act_lo8_index).  The low-term product then runs
// on v_mfma_f32_16x16x128 in 8-bit formats (twice the rate of the half-precision instruction) against a second
// copy of the weights, W8 = fp8(w * 16) (1-4-3 format, saturating at +-448, i.e. |w| = 28), so that
// lo8 * W8 = 2^8 * lo * w lands in the same accumulator as hi * (w * 2^8).  The correction term only has to be good
// to a few percent (it is itself 2^-12 of the result), which three and two mantissa bits give.
// Layout: 128 k of lo8 have the geometry of 64 k of hi (4 KiB of 32 rows): the 16-byte chunk c (16 k) of a row lies where
// the 16-byte chunk c (8 k) of the row lies in the halves, and W8 is packed likewise; a lane's operand of the 128-deep product is
// its 16 bytes of k-step 0 followed by its 16 bytes of k-step 1, for both operands.
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(8))) int i32x8;
__device__ __forceinline__ f32x4 mfma_lo8(const f16x8& a0, const f16x8& a1, const f16x8& b0, const f16x8& b1,
                                          const f32x4& c) {
#if defined(__HIP_DEVICE_COMPILE__)
  const i32x8 a = __builtin_shufflevector(__builtin_bit_cast(i32x4, a0), __builtin_bit_cast(i32x4, a1), 0, 1, 2, 3, 4, 5, 6, 7);
  const i32x8 b = __builtin_shufflevector(__builtin_bit_cast(i32x4, b0), __builtin_bit_cast(i32x4, b1), 0, 1, 2, 3, 4, 5, 6, 7);
  // A: bf8 (format 1), B: fp8 (format 0), no block scales
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 1, 0, 0, 0, 0, 0);
#else
  return c;
#endif
}

// ---- the kernel ---------------------------------------------------------------------------------------------
// One kernel template for every size: a workgroup of WGM x WGN waves computes a BM x BN tile (a wave WM x WN of it).
//
// * Slabs of PK k of A and W go straight from global memory into LDS (global_load_lds_dwordx4: lane l of a wave
//   instruction deposits its 16 bytes at the wave-uniform LDS base + 16*l), S slabs of A and SW of W ahead of the MFMAs,
//   through a ring of stages each; one barrier per slab publishes the landed slab and frees the one everybody has in
//   registers.  A comes from the L2 and W, in a launch of few tiles, from HBM: where the 160 KiB do not hold another stage of
//   both they hold a third one of W.  Against two stages of each: 192x256 at 290 rows 79 -> 62 us (qkv), 84 -> 68 (gate/up),
//   191 -> 142 (down), at 18560 rows 1811 -> 1652, 2846 -> 2656, 1760 -> 1493; 256x256 at 290 rows 88 -> 75, 94 -> 82,
//   212 -> 180, at 18560 rows down 1443 -> 1377 and with low terms 2381 -> 2315, 3988 -> 3900, 2125 -> 1987.
// * SPREAD: the weights of a slab are requested a k-step after its activations, so that the loads go out evenly.
// * Both slabs are in fragment order, so that a load is one KiB from one place, with a scalar offset, and a read of the LDS has no
//   bank conflicts.  A row-major A took an address a lane and eight pieces of 128 bytes a load: us, 18560 rows, that / this,
//   gate/up 2450 / 2372, down 1336 / 1314, o 548 / 535, with low terms 4 % (gate/up) and 2.5 % (qkv) less, qkv 0 to 2 % more
//   (1377 / 1404, 1412 / 1427, 1396 / 1394 on three cards); 2338 rows
//   gate/up 346 / 336, down 176 / 173.  On operands of zeros, where the clock does not drop, 1834 / 1741, 1113 / 977, 465 / 434:
//   most of what it saves goes into the power limit.
// * Four waves of 128x128 for the residual add's 256x256 tiles: a third fewer reads of the LDS than eight of 64x128, down 1314 ->
//   1269, o 535 -> 530.  The accumulators are the 256 registers of the accumulation half.  With the other epilogues and with low
//   terms, which two waves a SIMD cover better, gate/up 2372 -> 2450, qkv 1388 -> 1441, qkv with low terms 2190 -> 2349.
// * What bounds the large launches: without the loads of the main loop gate/up takes 2120 of 2546 us (row-major A), without its
//   reads of the LDS too 1568; barriers cost nothing; how the loads are spread over the k-steps makes no difference.
// * Fragments are double buffered in registers: while the MFMAs of one k-step run, the reads of the next
//   are in flight, slotted one by one between the MFMAs.  The compiler cannot tell the stages apart and would wait
//   for ALL outstanding LDS loads before any LDS read, so the reads are inline assembly and the waits explicit.
// * The instruction: 16x16x32.  On real operands the matrix cores are limited by power, not issue: an MFMA-only loop on
//   weight bits (vla_probe) sustains 1.76 PFLOP/s with 16x16x32 (half the accumulator traffic per product) against 1.59
//   with 32x32x16.  In this kernel that is 2.59 ms instead of 2.85 (gate/up, 18560 x 22016 x 4096),
//   1.40 instead of 1.48 (down), 0.56 instead of 0.61 (o).
// * DEEP: the fragments are read a whole slab ahead, for launches of at most 256 of the smallest tiles, where a k-step of four
//   products a wave is shorter than the reads of the next one take.  With eight waves of 32x32 instead of four of 32x64 and
//   four stages (whose number costs instructions where it is not a power of two) a slab of the 64x128 tile is 0.25 us instead
//   of 0.33: 290 rows, N 768: K 2048 12.7 -> 9.6 us, K 768 7.3 -> 6.2; N 4096 K 4096 from the caches 25 -> 20, with weights
//   from HBM 27 and 28 (K 11008 67 and 67).  Larger tiles gain nothing (128x256 at 290 and 2338 rows +-1 %).
// * A pass of 8-bit low terms (LO8) follows on 16x16x128: both k-steps of a slab are one product, so the two register
//   buffers hold one slab and there is none to spare for the next.  Each register is refilled as soon as its last
//   product has issued instead: a slab runs as two halves of the wave's rows, the first half's A fragments are refilled
//   during the second half, a column's B fragments behind their last product there, and the second half's A fragments
//   at its end, so that every refill has half a slab of products to arrive under.
//   Against 4 waves of 128x128 with 32x32x16 and 32x32x64 the 7B policy step of 64 takes 244.5 instead of 247.5 ms (its
//   4 two-term layers are a sixth of it), of 8 54.0 instead of 54.2, the 12-layer model's of 32 6.24 instead of 6.29;
//   with 128x256 tiles at every size 247.9, 54.3 and 6.22.
// * Every variant runs the same sequence of MFMAs per output element (k ascending, one chain), so a sequence's bits do
//   not depend on which tile its batch selects.

// 16 bytes per lane from global memory straight into LDS at lds_wave_base + 16 * lane.  base and soff (bytes) are the same
// for the whole wave and live in scalar registers, off is the lane's offset in bytes: a buffer load takes the three as
// they are, where a 64-bit address per lane would cost an addition and two registers a load (with the pass of low terms
// those registers spilled).  The builtins only exist in the device pass; the host pass just needs the kernel's stub.
__device__ __forceinline__ void load_to_lds_16(const f16* base, unsigned off, unsigned soff, f16* lds_wave_base) {
#if defined(__HIP_DEVICE_COMPILE__)
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, -1, 0x00027000);   // raw, 4 GiB
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)lds_wave_base, 16, off, soff, 0, 0);
#else
  (void)base;
  (void)off;
  (void)soff;
  (void)lds_wave_base;
#endif
}
// One fragment read with a compile-time byte offset (no wait: the register must not be touched before wait_lds() and
// hold() have been executed).
template <int OFF>
__device__ __forceinline__ void read_frag_asm(f16x8& dst, unsigned addr) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF) : "memory");
#endif
}
// Until at most N of the reads issued so far are outstanding (they return in order; a scalar load in flight counts as
// well, which can only make the wait longer).
template <int N = 0>
__device__ __forceinline__ void wait_lds() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N < 15 ? N : 15) : "memory");
#endif
}
// Ties a fragment to the wait before it: nothing that uses it can be scheduled above.
__device__ __forceinline__ void hold(f16x8& v) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(v));
#endif
}
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
#endif
}
#define VLA_INLINE __attribute__((always_inline))    // the kernel's lambdas: a call would put the captured arrays in memory
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  [&]<int... I>(std::integer_sequence<int, I...>) VLA_INLINE { (f(std::integral_constant<int, I>{}), ...); }
  (std::make_integer_sequence<int, N>{});
}

// acc += a * b, the sum in the registers of acc.  With two loops over the same accumulators the compiler gives the
// products of the first separate source and result registers, and the 256 of a wave run out (12 spilled, reloaded in
// the loop with a wait for every load in flight).  The compiler does not know the latency of the statement: settle()
// before anything but another of these touches the accumulators.
// AGPR: the accumulators are in the accumulation half of the register file (a wave of 128x128 has 256 of them, which is all of
// it; left to itself the compiler moves them back and forth).
template <bool AGPR>
__device__ __forceinline__ void mfma_in_place(f32x4& acc, const f16x8& a, const f16x8& b) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (AGPR) asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
  else asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
#endif
}
// The wait on both sides of a run of such products (8 issue slots behind a product, 2 in front of one; 32 given), eight
// accumulators a statement.  It takes them and gives them back, so whatever reads them, register copies included,
// depends on it.
template <bool AGPR, int MT, int NT>
__device__ __forceinline__ void settle(f32x4 (&acc)[MT][NT]) {
  static_assert(MT * NT % 4 == 0, "whole groups of eight, and one of four");
#if defined(__HIP_DEVICE_COMPILE__)
#define VLA_ACC(c, j) "+" c(acc[(g + j) / NT][(g + j) % NT])
#define VLA_SETTLE4(c) asm volatile("s_nop 15\n\ts_nop 15" : VLA_ACC(c, 0), VLA_ACC(c, 1), VLA_ACC(c, 2), VLA_ACC(c, 3))
#define VLA_SETTLE8(c)                                                                                                            \
  asm volatile("s_nop 15\n\ts_nop 15" : VLA_ACC(c, 0), VLA_ACC(c, 1), VLA_ACC(c, 2), VLA_ACC(c, 3), VLA_ACC(c, 4), VLA_ACC(c, 5), \
               VLA_ACC(c, 6), VLA_ACC(c, 7))
  constexpr int EIGHTS = MT * NT / 8 * 8;
#pragma unroll
  for (int g = 0; g < EIGHTS; g += 8) {
    if constexpr (AGPR) VLA_SETTLE8("a");
    else VLA_SETTLE8("v");
  }
  if constexpr (EIGHTS < MT * NT) {
    constexpr int g = EIGHTS;
    if constexpr (AGPR) VLA_SETTLE4("a");
    else VLA_SETTLE4("v");
  }
#undef VLA_SETTLE8
#undef VLA_SETTLE4
#undef VLA_ACC
#endif
}

constexpr int PK = 64;                                 // k of a slab (a slab of low terms is one 128-deep product)

template <class Epi> __device__ __forceinline__ const f16* epi_a_lo(const Epi&) { return nullptr; }
__device__ __forceinline__ const f16* epi_a_lo(const EpiPartial& e) { return e.a_lo; }

// The accumulators of a wave's 16 MT x 16 NT, rows m_wave .. and column group wn of a tile's columns n0 .., through LDS to the
// epilogue.
template <int MT, int NT, int WGN, class Epi>
__device__ __forceinline__ void store_tile(f32x4 (&acc)[MT][NT], const Epi& epi, unsigned char* smem, int wave, int wn, int lane,
                                           int m_wave, int n0, int M) {
  // The pitch keeps the stores of a 32-row group conflict free: the four row groups a store instruction covers start 16
  // banks apart.
  constexpr bool PAIR = 16 * NT < Epi::kSpan;               // two waves side by side share a staging tile
  static_assert(!PAIR || (WGN % 2 == 0 && 32 * NT >= Epi::kSpan), "an epilogue's span is one or two wave tiles");
  constexpr int COLS = PAIR ? 32 * NT : 16 * NT, PITCH = COLS + 4, ROWS = PAIR ? 16 : 32;
  float* tile = (float*)smem + (PAIR ? wave >> 1 : wave) * 32 * PITCH;
  const int side = PAIR ? wn & 1 : 0;
#pragma unroll
  for (int mb = 0; mb < MT / 2; ++mb) {
    if constexpr (PAIR) {
      if (mb > 0) __syncthreads();                     // the partner has read the previous rows
    }
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          tile[(mi * 16 + 4 * (lane >> 4) + e) * PITCH + side * 16 * NT + nt * 16 + (lane & 15)] = acc[mb * 2 + mi][nt][e];
    if constexpr (PAIR) __syncthreads();
    epi.template consume<COLS, PITCH, ROWS>(tile + side * ROWS * PITCH, m_wave + mb * 32 + side * ROWS,
                                            n0 + (PAIR ? wn >> 1 : wn) * COLS, lane, M);
  }
  if constexpr (MT % 2 != 0) {                         // the last 16 rows
    if constexpr (PAIR) __syncthreads();
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        tile[(4 * (lane >> 4) + e) * PITCH + side * 16 * NT + nt * 16 + (lane & 15)] = acc[MT - 1][nt][e];
    if constexpr (PAIR) __syncthreads();
    epi.template consume<COLS, PITCH, ROWS / 2>(tile + side * (ROWS / 2) * PITCH, m_wave + (MT - 1) * 16 + side * (ROWS / 2),
                                                n0 + (PAIR ? wn >> 1 : wn) * COLS, lane, M);
  }
}

// LO8: the launch has slabs of 8-bit low terms (W8 != nullptr): K == 1.5 * Kw, A row = [hi: Kw halves | lo8: Kw bytes].
// Otherwise K == Kw, or K == 2 * Kw (half-precision low terms behind the high terms: the weight slabs wrap).
// SPLITK (with EpiPartial; one row of tiles, M <= BM): the low terms of two-term operands are in a second buffer of the order of
// the first, tiles_m is the number of K slices, and workgroup (tile column tn, slice kz) accumulates slice kz of K only.
template <int WGM, int WGN, int WM, int WN, int S, int SW, int OCC, bool DEEP, bool SPREAD, class Epi, bool LO8, bool SPLITK>
__global__ __launch_bounds__(WGM* WGN * 64, OCC) void gemm_f16_kernel(const f16* __restrict__ A, int lda,
                                                                   const f16* __restrict__ Wp,
                                                                   const f16* __restrict__ W8, int M, int K, int Kw,
                                                                   int tiles_m, int tiles_n, Epi epi_in) {
  constexpr int NW = WGM * WGN, BM = WGM * WM, BN = WGN * WN, MT = WM / 16, NT = WN / 16;
  constexpr bool AGPR = MT * NT == 64;
  static_assert(!AGPR || !LO8, "the products of low terms leave their accumulators to the compiler");
  constexpr int KS = PK / 32, KS16 = PK / 16;          // k-steps of a slab; 16-k blocks of a slab
  // KiB pieces per wave and slab.  Where those of A do not divide among the waves (REST of them are left for the last round),
  // piece i of a wave is piece i * NW + wave of the slab, and the last round's are loaded by several waves: the same bytes to
  // the same place, so that every wave counts the same loads (160 rows: 56 pieces a slab for 52, 224 rows: 64 for 60; what the
  // four cost has not been timed apart).
  constexpr int A_ALL = BM * PK / 512, AP = (A_ALL + NW - 1) / NW, WP = BN * PK / 512 / NW, LPS = AP + WP;
  constexpr int REST = A_ALL % NW;
  static_assert(A_ALL * 512 == BM * PK && WP * NW * 512 == BN * PK, "slab must divide among the waves");
  static_assert(BM % 32 == 0, "whole blocks of A");
  // Rings of one depth are one ring of [A slab | W slab], with one offset a stage (two rings: 128x256 tiles 0.6 % slower,
  // 128x128 0.3 %); else they follow one another.
  constexpr int A_HALVES = BM * PK, W_HALVES = BN * PK, A_STAGE = A_HALVES + (SW == S ? W_HALVES : 0);
  constexpr int W_STAGE = SW == S ? A_STAGE : W_HALVES, W0_HALVES = SW == S ? A_HALVES : S * A_HALVES;
  static_assert(SW == S || SW == S + 1, "the counts of loads in flight below");
  static_assert(!SPREAD || (SW == S + 1 && !DEEP && !LO8), "as counted below");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  f16* lds = (f16*)smem;                               // [S][A slab | W slab], or [S][A slab], [SW][W slab]

  // XCD-aware tile order: consecutive workgroup ids land on different XCDs, so give each XCD a contiguous run of
  // tiles, walked in groups of GM row-tiles that share the same weight columns (4 and 8 measure alike for the small
  // tiles and for those of 224 rows, 26 products within +-1.2 % and one 2.4 % better with 8; the 256-row tile is 4 % slower with 8
  // at 18560 rows, where the L2 then holds too few weight columns).
  const int nblk = tiles_m * tiles_n;
  const int per_xcd = gridDim.x >> 3;
  const int pid = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (pid >= nblk) return;
  int tm, tn, kz = 0;
  if constexpr (SPLITK) {                              // consecutive workgroups of an XCD share a K slice (the A slabs)
    tm = 0;
    tn = pid % tiles_n;
    kz = pid / tiles_n;
  } else {
    constexpr int GM = BM >= 256 ? 4 : 8;
    const int per_group = GM * tiles_n;
    const int grp = pid / per_group;
    const int first_m = grp * GM;
    const int gm = min(tiles_m - first_m, GM);
    const int in_grp = pid - grp * per_group;
    tm = first_m + in_grp % gm;
    tn = in_grp / gm;
  }
  const int m0 = tm * BM, n0 = tn * BN;
  Epi epi = epi_in;

  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  const int KB16 = Kw >> 4;
  int KT = K / PK, KTw = Kw / PK;                      // slabs; of which the first KTw are high terms
  size_t kb0 = 0;                                      // first 16-k block of this workgroup's K range
  if constexpr (SPLITK) {
    const int u0 = (int)((long long)kz * KTw / tiles_m), u1 = (int)((long long)(kz + 1) * KTw / tiles_m);
    kb0 = (size_t)u0 * KS16;
    KTw = u1 - u0;
    KT = K > Kw ? 2 * KTw : KTw;                       // the low-term slabs of the slice follow its high-term slabs
    epi.part += (size_t)kz * epi.plane_rows * epi.N;
  }

  const unsigned lane16 = (unsigned)lane * 16u;        // lane offset in an operand in fragment order
  const f16* a_base = A + (size_t)m0 * lda + kb0 * 512;
  const f16* a_lo_base = SPLITK && epi_a_lo(epi) ? epi_a_lo(epi) + kb0 * 512 : a_base;
  const f16* w_base = Wp + ((size_t)(n0 / 32) * KB16 + kb0) * 512;
  const f16* w8_base = LO8 ? W8 + (size_t)(n0 / 32) * KB16 * 256 : w_base;
  const unsigned a_block = 64u * (unsigned)lda;        // bytes of a block of 32 rows of A
  const int a_last = (M - 1 - m0) >> 5;                // last block there is (a launch's rows are allocated in whole blocks)
  // The lanes of rows past M ask for what others do, so that a last tile of few rows has few lines of A to wait for: its workgroup
  // runs ahead of the others of the same columns and XCD, which find the weights in the L2.  us with whole blocks / this, cold
  // weights, N 4096: 580 rows K 4096 41.2 / 38.7, K 11008 94 / 88, with low terms 137 / 127; 1160 rows 61 / 57.6, 138 / 133.
  const unsigned lane_last = (unsigned)(min(lane & 31, (M - 1 - m0) & 31) + (lane & 32)) * 16u;      // in block a_last
  const int a_back = REST ? wave - wave % (REST ? REST : 1) : 0;     // pieces a wave's last one is moved back by
  auto issue_one = [&](int kt, auto I) VLA_INLINE {    // piece I of this wave's share of slab kt (clamped), A first
    constexpr int i = decltype(I)::value;
    const int ks = min(kt, KT - 1), kw = ks >= KTw ? ks - KTw : ks;
    if constexpr (i < AP) {                            // piece j of the slab: block row j / KS16 (clamped), 16-k block j % KS16
      const int j = REST ? i * NW + wave - (i == AP - 1 ? a_back : 0) : wave * AP + i;
      const unsigned blk = (unsigned)min(j / KS16, a_last) * a_block + (unsigned)(j % KS16) * 1024u;
      const bool low = SPLITK && ks >= KTw;
      load_to_lds_16(low ? a_lo_base : a_base, j / KS16 < a_last ? lane16 : j / KS16 == a_last ? lane_last : 0u, blk + 1024u * KS16 * (unsigned)(SPLITK ? kw : ks), lds + (kt % S) * A_STAGE + j * 512);
    } else {
      const int j = wave * WP + i - AP;                // piece of the slab: block row j / KS16, 16-k block j % KS16
      const bool low = LO8 && ks >= KTw;
      const unsigned blk = (unsigned)(j / KS16 * KB16) * (low ? 512u : 1024u) + (unsigned)(j % KS16) * 1024u;
      load_to_lds_16(low ? w8_base : w_base, lane16, blk + 1024u * KS16 * (unsigned)kw, lds + W0_HALVES + (kt % SW) * W_STAGE + j * 512);
    }
  };

  auto issue_next = [&](int kt, auto I) VLA_INLINE {   // piece I of what takes the stages of slab kt
    issue_one(decltype(I)::value < AP ? kt + S : kt + SW, I);
  };

  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // LDS byte addresses of this lane's fragments inside stage 0.  A lane of a fragment is (row l % 16, k group
  // l / 16 of 8 k); in fragment order its 16 bytes are at 16 * (row & 31) + 512 * (group & 1) of 16-k block group / 2.
  const unsigned lds0 = (unsigned)(size_t)((__attribute__((address_space(3))) unsigned char*)smem);
  const int fgrp = lane >> 4;
  const unsigned in_block = (unsigned)(fgrp >> 1) * 1024u + (unsigned)(fgrp & 1) * 512u + (unsigned)(lane & 15) * 16u;
  // first fragment of A of this wave, and what is added for every second one: of wave tiles of an odd number of fragments the
  // second begins in the middle of a block
  const int a_frag = wm * MT;
  const unsigned a_even = lds0 + (unsigned)(a_frag >> 1) * (KS16 * 1024u) + (unsigned)(a_frag & 1) * 256u + in_block;
  const unsigned a_odd = MT % 2 ? a_even + (a_frag & 1 ? KS16 * 1024u - 512u : 0u) : a_even;
  const unsigned w_b = lds0 + 2u * (unsigned)(W0_HALVES + wn * (WN / 32) * KS16 * 512) + in_block;

  constexpr int NBUF = DEEP ? 2 * KS : 2;              // register buffers, a k-step each
  f16x8 af[NBUF][MT], bf[NBUF][NT];
  constexpr int R = MT + NT, MF = MT * NT;             // reads and products of a k-step
  struct Stages { unsigned a, b; };                    // byte offsets of a slab's stages
  auto stages_of = [&](int kt) VLA_INLINE {
    return Stages{(unsigned)(kt % S) * (2u * A_STAGE), (unsigned)(kt % SW) * (2u * W_STAGE)};
  };
  // fragment reads of k-step ss of the slab in stages so (block j of an operand in fragment order: 32 rows hold two
  // fragments)
  auto read_a = [&](Stages so, f16x8& dst, auto SS, auto J) VLA_INLINE {
    constexpr int ss = decltype(SS)::value, j = decltype(J)::value;
    read_frag_asm<(j / 2 * KS16 + 2 * ss) * 1024 + (j & 1) * 256>(dst, (j & 1 ? a_odd : a_even) + so.a);
  };
  auto read_b = [&](Stages so, f16x8& dst, auto SS, auto J) VLA_INLINE {
    constexpr int ss = decltype(SS)::value, j = decltype(J)::value;
    read_frag_asm<(j / 2 * KS16 + 2 * ss) * 1024 + (j & 1) * 256>(dst, w_b + so.b);
  };
  auto read_one = [&](Stages so, int f, auto SS, auto I) VLA_INLINE {   // I-th fragment read of a k-step
    constexpr int x = decltype(I)::value;
    if constexpr (x < MT) read_a(so, af[f][x], SS, I);
    else read_b(so, bf[f][x - MT], SS, std::integral_constant<int, x - MT>{});
  };
  auto arrived = [&](int f) VLA_INLINE {
    wait_lds();
#pragma unroll
    for (int i = 0; i < MT; ++i) hold(af[f][i]);
#pragma unroll
    for (int j = 0; j < NT; ++j) hold(bf[f][j]);
  };
  // One k-step of slab kt: the MFMAs, and between them fragment reads (in the first three quarters, so that they have
  // landed at the end) and the loads that take slab kt's stages (A of slab kt + S, W of slab kt + SW).
  // Read ahead by a k-step: the k-steps alternate between two buffers, P is the slab's first one.  The reads of the last
  // k-step belong to slab kt + 1, which must have landed, and slab kt is in everybody's registers: its stage takes the loads.
  // DEEP, read ahead by a slab: P is the half of the buffers slab kt is in, and all of this holds from its first k-step on.
  auto step = [&](int kt, auto P, auto SS) VLA_INLINE {
    constexpr int p = decltype(P)::value, ss = decltype(SS)::value;
    constexpr bool last = ss == KS - 1, next = DEEP || last;        // next: the reads are of slab kt + 1
    constexpr int f = DEEP ? p * KS + ss : (p + ss) & 1, g = DEEP ? (p ^ 1) * KS + ss : f ^ 1;
    constexpr int n_rd = MF * 3 / 4 > 0 ? MF * 3 / 4 : 1;
    if constexpr (DEEP ? ss == 0 : last) {
      wait_vmcnt<(S - 2) * LPS + (SW - S) * WP>();
      __builtin_amdgcn_s_barrier();
    }
    const Stages so = stages_of(kt + (next ? 1 : 0));
    static_for<MF>([&](auto I) VLA_INLINE {
      constexpr int i = decltype(I)::value, mt = i / NT, nt = i % NT;
      if constexpr (LO8 || AGPR) mfma_in_place<AGPR>(acc[mt][nt], af[f][mt], bf[f][nt]);
      else acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af[f][mt], bf[f][nt], acc[mt][nt], 0, 0, 0);
      constexpr int r0 = i < n_rd ? i * R / n_rd : R, r1 = i < n_rd ? (i + 1) * R / n_rd : R;
      static_for<r1 - r0>([&](auto J) VLA_INLINE {
        read_one(so, g, std::integral_constant<int, DEEP ? ss : (last ? 0 : ss + 1)>{}, std::integral_constant<int, r0 + decltype(J)::value>{});
      });
      if constexpr (SPREAD) {                          // last k-step: A; the next one: W
        constexpr int n = last ? AP : WP, l0 = i * n / MF, l1 = (i + 1) * n / MF;
        static_for<l1 - l0>([&](auto J) VLA_INLINE {
          issue_next(last ? kt : kt - 1, std::integral_constant<int, (last ? 0 : AP) + l0 + decltype(J)::value>{});
        });
      } else if constexpr (next) {
        constexpr int at = DEEP ? ss * MF + i : i, of = DEEP ? KS * MF : MF;
        constexpr int l0 = at * LPS / of, l1 = (at + 1) * LPS / of;
        static_for<l1 - l0>([&](auto J) VLA_INLINE { issue_next(kt, std::integral_constant<int, l0 + decltype(J)::value>{}); });
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (!DEEP) arrived(g);
    else if constexpr (last) static_for<KS>([&](auto J) VLA_INLINE { arrived((p ^ 1) * KS + decltype(J)::value); });
  };
  auto slab = [&](int kt, auto P) VLA_INLINE {
    static_for<KS>([&](auto SS) VLA_INLINE { step(kt, P, SS); });
  };
  constexpr std::integral_constant<int, 0> c0{};
  constexpr std::integral_constant<int, 1> c1{};
  constexpr std::integral_constant<int, DEEP ? 1 : 0> cn{};       // P of an odd slab
  static_for<S>([&](auto I) VLA_INLINE { static_for<LPS>([&](auto J) VLA_INLINE { issue_one(decltype(I)::value, J); }); });
  if constexpr (!SPREAD)
    static_for<SW - S>([&](auto I) VLA_INLINE {
      static_for<WP>([&](auto J) VLA_INLINE { issue_one(S + decltype(I)::value, std::integral_constant<int, AP + decltype(J)::value>{}); });
    });
  wait_vmcnt<(S - 1) * LPS + (SPREAD ? 0 : (SW - S) * WP)>();
  __builtin_amdgcn_s_barrier();
  static_for<DEEP ? KS : 1>([&](auto SS) VLA_INLINE {
    static_for<R>([&](auto I) VLA_INLINE { read_one(stages_of(0), decltype(SS)::value, SS, I); });
  });
  static_for<DEEP ? KS : 1>([&](auto SS) VLA_INLINE { arrived(decltype(SS)::value); });
  const int KTh = LO8 ? KTw : KT;
  int kt = 0;
  if constexpr (LO8 || AGPR) settle<AGPR>(acc);        // the zeros are written
  if constexpr (LO8) {
    if constexpr (DEEP) {
      for (; kt + 1 < KTh; kt += 2) {
        slab(kt, c0);
        slab(kt + 1, cn);
      }
      if (kt < KTh) slab(kt++, c0);
    } else {
      for (; kt < KTh; ++kt) slab(kt, c0);
    }
    settle<AGPR>(acc);
    // Fragments of one slab, k-steps 0 and 1: variables of their own, read afresh, since the product wants the two in
    // adjacent registers and the loop above must not be bound by that.  Reads are issued in the order: first-half A
    // fragments, B fragments column by column, second-half A fragments.
    constexpr int H = MT / 2;
    f16x8 al[2][MT], bl[2][NT];
    auto refill_a = [&](Stages so, auto J) VLA_INLINE {
      read_a(so, al[0][decltype(J)::value], c0, J);
      read_a(so, al[1][decltype(J)::value], c1, J);
    };
    auto refill_b = [&](Stages so, auto J) VLA_INLINE {
      read_b(so, bl[0][decltype(J)::value], c0, J);
      read_b(so, bl[1][decltype(J)::value], c1, J);
    };
    auto hold_a = [&](int i) VLA_INLINE {
      hold(al[0][i]);
      hold(al[1][i]);
    };
    auto product = [&](auto MI, auto NI) VLA_INLINE {
      constexpr int mt = decltype(MI)::value, nt = decltype(NI)::value;
      acc[mt][nt] = mfma_lo8(al[0][mt], al[1][mt], bl[0][nt], bl[1][nt], acc[mt][nt]);
    };
    auto low_slab = [&](int t) VLA_INLINE {
      static_for<NT>([&](auto NI) VLA_INLINE {         // rows of the first half
        constexpr int nt = decltype(NI)::value;
        wait_lds<2 * (NT - 1 - nt) + 2 * (MT - H)>();
        if constexpr (nt == 0) {
#pragma unroll
          for (int i = 0; i < H; ++i) hold_a(i);
        }
        hold(bl[0][nt]);
        hold(bl[1][nt]);
        static_for<H>([&](auto MI) VLA_INLINE { product(MI, NI); });
        __builtin_amdgcn_sched_barrier(0);
      });
      wait_lds();
#pragma unroll
      for (int i = H; i < MT; ++i) hold_a(i);
      wait_vmcnt<(S - 2) * LPS + (SW - S) * WP>();                     // slab t + 1 has landed, slab t is in everybody's registers
      __builtin_amdgcn_s_barrier();
      const Stages so = stages_of(t + 1);
      static_for<NT>([&](auto NI) VLA_INLINE {         // rows of the second half
        constexpr int nt = decltype(NI)::value;
        static_for<MT - H>([&](auto MI) VLA_INLINE {
          product(std::integral_constant<int, H + decltype(MI)::value>{}, NI);
          if constexpr (decltype(MI)::value == 0) {
            if constexpr (nt == 0) static_for<H>([&](auto J) VLA_INLINE { refill_a(so, J); });
            else refill_b(so, std::integral_constant<int, nt - 1>{});
          }
        });
        constexpr int l0 = nt * LPS / NT, l1 = (nt + 1) * LPS / NT;
        static_for<l1 - l0>([&](auto J) VLA_INLINE { issue_next(t, std::integral_constant<int, l0 + decltype(J)::value>{}); });
        __builtin_amdgcn_sched_barrier(0);
      });
      refill_b(so, std::integral_constant<int, NT - 1>{});
      static_for<MT - H>([&](auto J) VLA_INLINE { refill_a(so, std::integral_constant<int, H + decltype(J)::value>{}); });
    };
    const Stages so0 = stages_of(kt);
    static_for<H>([&](auto J) VLA_INLINE { refill_a(so0, J); });
    static_for<NT>([&](auto J) VLA_INLINE { refill_b(so0, J); });
    static_for<MT - H>([&](auto J) VLA_INLINE { refill_a(so0, std::integral_constant<int, H + decltype(J)::value>{}); });
    for (; kt < KT; ++kt) low_slab(kt);
    wait_lds();                                        // the last slab's refills
#pragma unroll
    for (int i = 0; i < MT; ++i) hold_a(i);
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      hold(bl[0][j]);
      hold(bl[1][j]);
    }
  } else {
    for (; kt + 1 < KTh; kt += 2) {
      slab(kt, c0);
      slab(kt + 1, cn);
    }
    if (kt < KTh) slab(kt, c0);
  }
  if constexpr (AGPR) settle<AGPR>(acc);
  wait_vmcnt<0>();                                     // the clamped tail loads still target this workgroup's LDS
  __syncthreads();                                     // every wave is done with the slabs: LDS becomes epilogue staging

  store_tile<MT, NT, WGN>(acc, epi, smem, wave, wn, lane, m0 + wm * WM, n0, M);
}

template <int WGM, int WGN, int WM, int WN, int S, int SW, int OCC, bool DEEP, bool SPREAD, bool LO8, bool SPLITK, class Epi>
static void launch_tiles(const f16* A, int lda, const f16* Wp, const f16* W8, int M, int K, int Kw, int tiles_m,
                         int tiles_n, const Epi& epi, hipStream_t st) {
  const int grid = (tiles_m * tiles_n + 7) / 8 * 8;
  constexpr size_t slabs = ((size_t)S * WGM * WM + (size_t)SW * WGN * WN) * PK * sizeof(f16);
  constexpr bool pair = WN < Epi::kSpan;
  constexpr size_t stage = (size_t)WGM * WGN / (pair ? 2 : 1) * 32 * ((pair ? 2 : 1) * WN + 4) * sizeof(float);
  constexpr size_t smem = slabs > stage ? slabs : stage;
  auto kern = gemm_f16_kernel<WGM, WGN, WM, WN, S, SW, OCC, DEEP, SPREAD, Epi, LO8, SPLITK>;
  static bool attr_set = false;
  if (!attr_set) {
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    attr_set = true;
  }
  hipLaunchKernelGGL(kern, dim3(grid), dim3(WGM * WGN * 64), smem, st, A, lda, Wp, W8, M, K, Kw, tiles_m, tiles_n, epi);
}
template <int WGM, int WGN, int WM, int WN, int S, int SW, int OCC, bool DEEP, bool SPREAD, bool LO8, class Epi>
static void launch(const GemmF16& g, const Epi& epi, hipStream_t st) {
  launch_tiles<WGM, WGN, WM, WN, S, SW, OCC, DEEP, SPREAD, LO8, false>(g.A, g.lda, g.Wp, g.W8, g.M, g.K, g.Kw,
                                                               (g.M + WGM * WM - 1) / (WGM * WM), g.N / (WGN * WN), epi, st);
}

// Decode GEMM of a large batch: partial sums of `ksplit` K slices, see EpiPartial and the SPLITK form of the kernel.
// Afrag / Afrag_lo: activation fragments of rows row0 .. row0 + M - 1 (their block row 0 = row row0, a multiple of 32).
bool splitk_gemm_fits(int M, int N, int K) { return M <= 256 && N % 256 == 0 && K % 64 == 0 && K >= 128; }
int splitk_ksplit(int N, int K) {
  int ks = 256 / (N / 256);                  // about one workgroup per compute unit
  if (ks > kMaxKSplit) ks = kMaxKSplit;
  while (ks > 1 && K / 64 < 4 * ks) --ks;    // at least 4 slabs per slice
  return ks < 1 ? 1 : ks;
}
void splitk_gemm(const f16* Afrag, const f16* Afrag_lo, const f16* Wp, float* part, int M, int N, int K, int ksplit,
                 int plane_rows, int row0, hipStream_t st) {
  const f16* no8 = nullptr;
  const EpiPartial epi{part, plane_rows, row0, N, Afrag_lo};
  const int k = Afrag_lo ? 2 * K : K;
  // 256 columns a workgroup re-read the activations least, but a matrix of 4096 columns would occupy 64 compute units: 64
  // columns then.  256 rows, K = 4096 / 11008: 17 / 39 us (256 columns 46 / 83, two weight-streaming launches 45 / 72).
  if (N / 256 * ksplit >= 128) launch_tiles<4, 2, 64, 128, 2, 3, 1, false, false, false, true>(Afrag, K, Wp, no8, M, k, K, ksplit, N / 256, epi, st);
  else launch_tiles<4, 2, 64, 32, 4, 4, 1, false, false, false, true>(Afrag, K, Wp, no8, M, k, K, ksplit, N / 64, epi, st);
}


// ---- few rows ---------------------------------------------------------------------------------------------------
// x += A * W^T of a few hundred rows.  A compute unit has some 64 KiB of loads in flight, which come back in order: where its
// weights come from HBM (1.1 us) it takes in 58 GB/s whatever the depth of its rings, activations that are in the L2 included.
// So a tile is 64 columns (four waves of 16 MT x 16), which shares the products out over the most compute units, and with `ahead`
// a workgroup more for each 64 columns does nothing but read their weights, which the workgroups of the row tiles, on the same
// XCD, then find in its L2.  A wave's weights go straight to its registers, four U k-steps ahead, A in slabs of 128 k through S
// stages of LDS, in pieces of a fragment (16 rows x 32 k, one KiB, which half a block of fragment order makes as well), and its
// fragments are read two k-steps ahead.  The sequence of products per element is that of gemm_f16_kernel.
// us, that kernel's 64x128 tiles / this without / with reading ahead, cold weights, N 4096: 230 rows K 4096 26.2 / 22.1 / 17.2,
// K 11008 69.9 / 54.9 / 40.9; 165 rows K 11008 70.5 / 41.0 / 34.9; with low terms 290 rows 99.9 / 76 / 68; N 768, 290 rows (weights
// from the last-level cache) K 768 5.8 / 4.1, K 2048 9.9 / 6.4, with low terms 7.9 / 4.7 and 14.8 / 8.5.
// (More stages, 16 or 32 k-steps of weights ahead, waves of their own for the loads of A: 53 to 55 us of the 54.9.  Reading ahead
// beside the tiles of gemm_f16_kernel does little for QKV and gate/up: 128x256 at 290 rows 57 -> 54, 160x256 70 -> 70.)
template <int MT, int S, int U, bool LO8>
__global__ __launch_bounds__(256, 1) void gemm_few_kernel(const f16* __restrict__ A, int lda, const f16* __restrict__ Wp,
                                                          const f16* __restrict__ W8, int M, int Kw, int tiles_m, int tiles_n,
                                                          int ahead, EpiResid epi) {
  constexpr int D = 4 * U, AP = MT, STAGE = MT * 4 * 1024;           // weight fragments and pieces of A of a wave; bytes of a stage
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  // the row tiles of 64 columns one after the other: their weights come to one L2
  const int pid = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const int per_n = tiles_m + ahead;
  if (pid >= per_n * tiles_n) return;
  const int tn = pid / per_n, tm = pid - tn * per_n - ahead, m0 = max(tm, 0) * 16 * MT, n0 = tn * 64;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int KTh = Kw / 128, KT = LO8 ? KTh + Kw / 256 : KTh;         // slabs of high terms, and with the low ones (256 k each)
  // a lane's 16 bytes of a fragment: row lane % 16, k group lane / 16 of 8 k
  const unsigned in_block = (unsigned)(lane >> 5) * 1024u + (unsigned)((lane >> 4) & 1) * 512u + (unsigned)(lane & 15) * 16u;
  const f16* a_base = A + (size_t)(m0 >> 5) * 32 * lda;
  const unsigned a_block = 64u * (unsigned)lda;
  const int h0 = (m0 >> 4) & 1, h_last = ((M - 1) >> 4) - ((m0 >> 5) << 1);     // half blocks, from the tile's first block on
  auto issue_a = [&](int kt, unsigned stage, auto I) VLA_INLINE {    // a wave's k-step of the slab, fragment I
    constexpr int i = decltype(I)::value;
    const int h = min(i + h0, h_last);
    const unsigned off = (unsigned)(h >> 1) * a_block + (unsigned)(h & 1) * 256u + (unsigned)wave * 2048u + 8192u * (unsigned)min(kt, KT - 1);
    load_to_lds_16(a_base, in_block, off, (f16*)(smem + stage + (i * 4 + wave) * 1024));
  };
  const int blk = (n0 >> 5) + (wave >> 1);
  const f16* w_base = Wp + (size_t)blk * Kw * 32 + (wave & 1) * 128;
  const f16* w8_base = LO8 ? W8 + (size_t)blk * Kw * 16 + (wave & 1) * 128 : w_base;
  f16x8 wq[D];
  auto load_w = [&](const f16* base, int q, int n, int s) VLA_INLINE {         // k-step q of n (clamped)
#if defined(__HIP_DEVICE_COMPILE__)
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, -1, 0x00027000);
    wq[s] = __builtin_bit_cast(f16x8, __builtin_amdgcn_raw_buffer_load_b128(rsrc, in_block, 2048u * (unsigned)min(q, n - 1), 0));
#endif
  };
  f32x4 acc[MT][1];
#pragma unroll
  for (int i = 0; i < MT; ++i) acc[i][0] = f32x4{0.f, 0.f, 0.f, 0.f};
  const unsigned a_rd = (unsigned)(size_t)((__attribute__((address_space(3))) unsigned char*)smem) + (unsigned)lane * 16u;
  f16x8 af[4][MT];                                     // fragments of a slab's k-steps
  auto read_a = [&](unsigned so, auto SS, auto J) VLA_INLINE {
    constexpr int ss = decltype(SS)::value, j = decltype(J)::value;
    read_frag_asm<(j * 4 + ss) * 1024>(af[ss][j], a_rd + so);
  };
  auto hold_all = [&](int ss) VLA_INLINE {
#pragma unroll
    for (int i = 0; i < MT; ++i) hold(af[ss][i]);
  };
  // Loads newer than those of the next slab when it is waited for, at least: A of the S - 2 slabs behind it, and the weights of the
  // k-steps since, which are 4 S - 5 where it was requested in the fourth k-step of the slab S - 1 before this one, and in the
  // first slabs, whose A was requested in front of all weights, D + 2 and more.  To the compiler the weights are ordinary loads,
  // which it moves to where they are used and drops where they are not: only those count that a turn of the main loop leaves to
  // the next one, and those in front of it, which it always takes.  Slabs behind the loop (number T, -1: in it) request none, so
  // that 2 and 4 a slab fewer are in flight, and those of low terms behind theirs, which may be the only ones, count none.
  constexpr int W_LOOP = 4 * S - 6 < D + 2 ? 4 * S - 6 : D + 2;
  auto next_landed = [&](auto W) VLA_INLINE {          // W: weights among them; and this slab is in everybody's registers
    wait_lds();
    wait_vmcnt<(S - 2) * AP + decltype(W)::value>();
    __builtin_amdgcn_s_barrier();
  };
  static_assert((S - 1) * AP + D <= 63, "the counter of loads in flight");
  constexpr int BAR = MT / 2;                          // product of the third k-step in front of which the barrier stands
  auto step = [&](int kt, unsigned so, unsigned nx, auto SS, auto RS, auto T) VLA_INLINE {
    constexpr int ss = decltype(SS)::value, s = decltype(RS)::value, tail = decltype(T)::value;
    constexpr int newer = tail < 0 ? W_LOOP : 4 * S - 8 - 4 * tail;
    wait_lds<MT>();                                    // read two k-steps ago; newer: the last one's reads
    hold_all(ss);
    static_for<MT>([&](auto I) VLA_INLINE {
      constexpr int i = decltype(I)::value;
      if constexpr (ss == 2 && i == BAR) next_landed(std::integral_constant<int, (newer > 0 ? newer : 0)>{});
      acc[i][0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af[ss][i], wq[s], acc[i][0], 0, 0, 0);
      constexpr int f0 = ss == 2 ? BAR : 0, x0 = i < f0 ? 0 : (i - f0) * MT / (MT - f0), x1 = i < f0 ? 0 : (i - f0 + 1) * MT / (MT - f0);
      static_for<x1 - x0>([&](auto J) VLA_INLINE {
        read_a(ss >= 2 ? nx : so, std::integral_constant<int, (ss + 2) & 3>{}, std::integral_constant<int, x0 + decltype(J)::value>{});
      });
      if constexpr (ss == 3) issue_a(kt + S, so, I);   // (its stage is free behind the barrier)
      if constexpr (i == MT - 1 && tail < 0) load_w(w_base, kt * 4 + ss + D, 4 * KTh, s);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  if (tm < 0) {                                        // reads the columns' weights into the L2
    auto pass = [&](const f16* base, int n) VLA_INLINE {
      static_for<D>([&](auto I) VLA_INLINE { load_w(base, decltype(I)::value, n, decltype(I)::value); });
      for (int q = D; q < n + D; q += D)
        static_for<D>([&](auto I) VLA_INLINE {
          hold(wq[decltype(I)::value]);
          if (q < n) load_w(base, q + decltype(I)::value, n, decltype(I)::value);
          __builtin_amdgcn_sched_barrier(0);
        });
    };
    pass(w_base, 4 * KTh);
    if constexpr (LO8) pass(w8_base, 2 * KTh);
    return;
  }
  static_for<S>([&](auto I) VLA_INLINE {
    static_for<AP>([&](auto J) VLA_INLINE { issue_a(decltype(I)::value, decltype(I)::value * STAGE, J); });
    __builtin_amdgcn_sched_barrier(0);                 // (the counts of loads in flight rely on this order)
  });
  static_for<D>([&](auto I) VLA_INLINE { load_w(w_base, decltype(I)::value, 4 * KTh, decltype(I)::value); });
  __builtin_amdgcn_sched_barrier(0);
  wait_vmcnt<(S - 1) * AP + D>();
  __builtin_amdgcn_s_barrier();
  static_for<MT>([&](auto J) VLA_INLINE { read_a(0, std::integral_constant<int, 0>{}, J); });
  static_for<MT>([&](auto J) VLA_INLINE { read_a(0, std::integral_constant<int, 1>{}, J); });
  unsigned so = 0;
  auto after = [&](unsigned o) VLA_INLINE { return o + STAGE == STAGE * S ? 0u : o + STAGE; };
  auto slab = [&](int kt, auto X, auto T) VLA_INLINE {
    const unsigned nx = after(so);
    static_for<4>([&](auto SS) VLA_INLINE { step(kt, so, nx, SS, std::integral_constant<int, 4 * decltype(X)::value + decltype(SS)::value>{}, T); });
    so = nx;
  };
  int kt = 0;
  do {                                                 // (at least U slabs: few_tiles)
    static_for<U>([&](auto X) VLA_INLINE { slab(kt + decltype(X)::value, X, std::integral_constant<int, -1>{}); });
    kt += U;
  } while (kt + U <= KTh);
  const int rest = KTh - kt;
  static_for<U - 1>([&](auto X) VLA_INLINE { if ((int)decltype(X)::value < rest) slab(kt + decltype(X)::value, X, X); });
  if constexpr (LO8) {                                 // a product takes two pieces of A and of W: 128 k of low terms
    static_for<D>([&](auto I) VLA_INLINE { load_w(w8_base, decltype(I)::value, 2 * KTh, decltype(I)::value); });
    auto low_slab = [&](int t, int q0, auto X, auto LOOP) VLA_INLINE {
      constexpr bool loop = decltype(LOOP)::value;
      const unsigned nx = after(so);
      static_for<2>([&](auto PR) VLA_INLINE {
        constexpr int pr = decltype(PR)::value, s = 4 * decltype(X)::value + 2 * pr;
        if constexpr (pr == 1) next_landed(std::integral_constant<int, loop ? W_LOOP : 0>{});
        else wait_lds();
        hold_all(2 * pr);
        hold_all(2 * pr + 1);
        static_for<MT>([&](auto I) VLA_INLINE {
          constexpr int i = decltype(I)::value;
          acc[i][0] = mfma_lo8(af[2 * pr][i], af[2 * pr + 1][i], wq[s], wq[s + 1], acc[i][0]);
          read_a(pr ? nx : so, std::integral_constant<int, 2 - 2 * pr>{}, I);
          read_a(pr ? nx : so, std::integral_constant<int, 3 - 2 * pr>{}, I);
          if constexpr (pr == 1) issue_a(t + S, so, I);
          __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (loop) {
          load_w(w8_base, q0 + 2 * pr + D, 2 * KTh, s);
          load_w(w8_base, q0 + 2 * pr + 1 + D, 2 * KTh, s + 1);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      so = nx;
    };
    int q0 = 0;
    for (kt = KTh; kt + U <= KT; kt += U, q0 += D)
      static_for<U>([&](auto X) VLA_INLINE { low_slab(kt + decltype(X)::value, q0 + 4 * decltype(X)::value, X, std::true_type{}); });
    const int last = KT - kt;
    static_for<U - 1>([&](auto X) VLA_INLINE { if ((int)decltype(X)::value < last) low_slab(kt + decltype(X)::value, q0 + 4 * decltype(X)::value, X, std::false_type{}); });
  }
  wait_lds();                                          // the reads ahead of the end, and the clamped loads, before the LDS is staging
  static_for<4>([&](auto SS) VLA_INLINE { hold_all(decltype(SS)::value); });
  wait_vmcnt<0>();
  __syncthreads();
  store_tile<MT, 1, 4>(acc, epi, smem, wave, wave, lane, m0, n0, M);
}
template <int MT, int S, bool LO8>
static void launch_few(const GemmF16& g, int ahead, const EpiResid& epi, hipStream_t st) {
  const int tiles_m = (g.M + 16 * MT - 1) / (16 * MT), tiles_n = g.N / 64;
  constexpr size_t smem = (size_t)S * MT * 4096;
  auto kern = gemm_few_kernel<MT, S, 4, LO8>;
  static bool attr_set = false;
  if (!attr_set) {
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    attr_set = true;
  }
  hipLaunchKernelGGL(kern, dim3(((tiles_m + ahead) * tiles_n + 7) / 8 * 8), dim3(256), smem, st, g.A, g.lda, g.Wp, g.W8, g.M, g.Kw, tiles_m,
                     tiles_n, ahead, epi);
}

// ---- tile choice ------------------------------------------------------------------------------------------------
// The time of a launch is modelled from two figures per tile, measured on 7B shapes with weights that come from HBM:
// what a workgroup takes on a chip that is not full (bound by the latency and rate of its LDS fills: fixed + per_k *
// K / 1024), and the rate of a chip full of them (bound by power and the L2).  Full rounds of 256 workgroups cost the
// larger of the two, the last partial round likewise for its share.  us at K = 4096 / 11008, and PFLOP/s:
//   64x128 27.9 / 67.6, 0.68; 128x128 33.8 / 83.6, 0.92; 64x256 44 / 107, 0.80; 128x256 50 / 128, 1.15; 192x256
//   59 / 143, 1.25; 256x256 73 / 180, 1.30.
// The constants of the last two are a little above these times (62.8 / 155, 75.3 / 184): they stand for every width, and in a
// model of matrices that come from the caches the third weight stage gives these tiles less.  Over 1084 products (the four
// matrices of models of d 256 to 5120 at 64 to 37120 rows, single- and two-term, each tile forced in turn) the pick is the
// fastest in 1015 and 0.30 % slower in the mean; constants that meet the two columns make it 0.38 %, and 0.57 instead of 0.19 %
// over the 7B matrices among them; the best of a search over both tiles' constants 0.25 %.
// us single-term, the model's pick (192 and 256 rows are balanced afterwards, tile_rows) and others: 290 rows qkv 50 (64x256;
// 192x256 64), gate/up 69 (192x256; 64x256 92), o 28 (64x128; 73) and down 68 (64x128; 180), which gemm_few_kernel runs; 580 rows gate/up 112 (128x256; 256x256 163), down 84 (128x128; 191); 870 rows qkv 78
// (192x256; 256x256 90); 2320 rows gate/up 378 (256x256; 128x256 389), o 86 (192x256; 256x256 101), down 197 (192x256;
// 256x256 236); 9216 rows of d 768 gate/up 62 (192x256; 128x256 69).
// Where it is off most: qkv at 580 rows of d 5120 116 (256x256; 192x256 99), gate/up at 13920 rows of d 768 112 (128x256;
// 256x256 102), down at 3480 rows of d 3072 184 (256x256; 192x256 159), the matrices of d 512 and less at 7000 rows and more by
// 4 to 20 %, qkv at 37120 rows of d 1536 515 (192x256; 256x256 486).
enum Tile { T_64x128, T_128x128, T_64x256, T_128x256, T_192x256, T_256x256, T_COUNT };
struct TileCost { int bm, bn; float fixed, per_k, rate; };
constexpr TileCost kTileCost[T_COUNT] = {{64, 128, 3.9f, 5.9f, 0.68f}, {128, 128, 4.3f, 7.4f, 0.92f},
                                         {64, 256, 6.8f, 9.3f, 0.80f}, {128, 256, 4.2f, 11.4f, 1.15f}, {192, 256, 8.0f, 13.7f, 1.25f},
                                         {256, 256, 10.9f, 16.1f, 1.30f}};
struct TilePick { Tile tile; long long tiles; };
static TilePick pick_tile(int M, int N, int K) {
  TilePick best{T_64x128, 0};
  float best_us = 1e30f;
  for (int t = 0; t < T_COUNT; ++t) {
    const TileCost& c = kTileCost[t];
    if (N % c.bn) continue;
    const long long tiles = (long long)((M + c.bm - 1) / c.bm) * (N / c.bn);
    const float alone = c.fixed + c.per_k * (float)K / 1024.0f;
    const float per_tile = 2.0f * (float)c.bm * (float)c.bn * (float)K / (c.rate * 1e9f);      // us, full chip
    const long long rounds = tiles / 256, rest = tiles % 256;
    const float us = (float)rounds * fmaxf(alone, 256.0f * per_tile) + (rest ? fmaxf(alone, (float)rest * per_tile) : 0.f);
    if (us < best_us) {
      best_us = us;
      best = TilePick{(Tile)t, tiles};
    }
  }
  return best;
}

// Rings are as deep as the LDS allows: cold weights take longer than two slabs to arrive (64x128 with 6 stages 28 and
// 68 us for o and down at 290 rows, with 3 stages and two workgroups per compute unit 30 and 73), except
// * where several rounds of 64x128 tiles share the compute units (3 stages, two workgroups), and in the eight-wave form of a
//   launch of few of them, whose four stages do; an epilogue that needs 128 columns of a row together (span 128) cannot have
//   that form's wave tiles of 32 columns and keeps four waves and six stages;
// * 256x256: the residual epilogue (four waves of 128x128) and single-term launches of fewer than three rounds, or whose weights
//   stay in the caches between the tile rows that read them, request the weights a k-step after the activations (SPREAD); the
//   others request them together, and so do low terms.  The line lies where the weights and half of the activations reach 170 MB of the
//   256 MB last-level cache.  SPREAD / together, in % of two stages of both, weights + activations in MB: gate/up 46 + 38 (d
//   2048, 9280 rows) 0.0 / +0.4, 71 + 95 -0.3 / +0.1, 101 + 114 (d 3072) -0.3 / -0.1, 180 + 38 (7B, 4640 rows) -0.8 / -0.6, 180 + 57
//   -2.1 / -2.3, 180 + 76 -3.0 / -3.5, 180 + 152 -3.1 / -3.3, 283 + 190 -3.5 / -4.4; qkv 25 + 76 -0.2 / +0.6, 57 + 57 -0.4 / +0.2,
//   101 + 76 (7B, 9280 rows) -0.9 / -0.3, 101 + 152 -0.1 / 0.0 (on other cards +0.9 / 0.0 and +1.0 / +0.3), 157 + 95 -2.4 / -3.7,
//   157 + 190 -1.6 / -4.0.  Residual adds gain by it (18560 rows down 1337 against 1348 us, o 590 against 595).
// (Slabs of 32 k throughout, in four stages of both operands, against slabs of 64 k in two and three: down 203 and 201 us at
// 2338 rows, 536 and 525 at 6960, 1435 and 1377 at 18560; o 86 and 85, 211 and 206, 570 and 548.)
constexpr int kFewHeights = 7;                            // gemm_few_kernel's tiles: 32, 48, ... 128 rows
enum Variant {
  V_FEW, V_FEW_AHEAD = V_FEW + kFewHeights,              // (the first of each; ahead: with workgroups that read the weights ahead)
  V_64x128_8W = V_FEW_AHEAD + kFewHeights, V_64x128, V_64x128_ROUNDS, V_128x128, V_64x256, V_128x256, V_160x256, V_192x256,
  V_224x256, V_256x256, V_256x256_SPREAD, V_COUNT
};
const char* const kGemmF16Variants[] = {
    "32x64", "48x64", "64x64", "80x64", "96x64", "112x64", "128x64",
    "32x64 ahead", "48x64 ahead", "64x64 ahead", "80x64 ahead", "96x64 ahead", "112x64 ahead", "128x64 ahead",
    "64x128 8 waves", "64x128 6 stages", "64x128 3 stages", "128x128", "64x256", "128x256", "160x256", "192x256",
    "224x256", "256x256", "256x256 spread"};
static_assert(sizeof(kGemmF16Variants) / sizeof(char*) == V_COUNT, "a name each");

// Rows of the tiles a launch runs.  Where the model picks 192 or 256 rows, the rounds are balanced: the last one costs a whole
// tile's time however few workgroups it has, and that is proportional to a tile's rows + 90 (a slab of weights, the fill and the
// end of a tile cost the same for each), so of 160, 192, 224 and 256 rows those are taken that need the least rounds x (rows +
// 90), if that is 2.5 % less than the model's.  us with the model's rows / these, 7B: 780 rows qkv 80 / 73, gate/up 143 / 132;
// 2208 rows gate/up 361 / 330, down 180 / 173, o 77.7 / 74.9; 2368 rows gate/up 364 / 343, down 185 / 181; 4100 rows down
// 368 / 340, o 154 / 142, qkv 370 / 350; 6960 rows down 509 / 488, o 213 / 204; 9400 rows down 762 / 705; 14000 rows down 1032 / 978;
// with low terms 5 to 10 % likewise.  Over the 354 products that it changes among those of d 768 to 5120 at 290 to 23200 rows,
// with and without low terms, 5.2 % less in the mean; the worst are qkv with low terms at 9280 rows of d 3072, 644 / 650, and
// without at 1450, 76.5 / 77.2.
static long long rounds_cost(int M, int N, int rows) {
  return (((long long)(M + rows - 1) / rows * (N / 256) + 255) / 256) * (rows + 90);
}
static int tile_rows(const TilePick& pick, int M, int N) {
  const int picked = kTileCost[pick.tile].bm;
  if (picked < 192) return picked;
  auto cost = [&](int rows) { return rounds_cost(M, N, rows); };
  int best = picked;
  for (int rows = 160; rows <= 256; rows += 32)
    if (cost(rows) < cost(best) && 40 * cost(rows) < 39 * cost(picked)) best = rows;
  return best;
}
// gemm_few_kernel's tiles where a launch runs them (rows 0: it does not): residual adds (no wider than their contraction, which
// gate/up and QKV products of these sizes are) of whole slabs.  The tiles are the lowest that leave the weights of every 64 columns
// a workgroup of their own on a chip of 256 (a last tile of a fragment's rows is as good), and if none do, the lowest that fit.
// The line: rows x (columns + 1200) up to 2^21, from where gemm_f16_kernel's launch fills as many compute units with tiles that
// read less.  us, that kernel / this: N 512 K 1536 870 rows 8.5 / 5.4, 1224 K 2048 10.0 / 10.3; N 768 K 768 580 rows 5.8 / 4.1,
// 1065 6.4 / 5.5, 1450 6.5 / 6.4, K 2048 580 9.9 / 6.5, 1065 10.9 / 10.6, 1450 11.4 / 12.9; N 1536 K 4096 700 rows 24.4 / 19.2;
// N 2048 K 5632 580 rows 35 / 27, 870 36 / 34; N 4096 K 11008 385 rows 68 / 64, 480 71 / 73, 580 88 / 90.  Over 498 products
// between 385 rows and the line (N 512 to 4096, K of one to eight N, with and without low terms) 1.38 times as fast in the mean;
// the worst N 1536 K 1536 at 766 rows, 0.97, and the above at 1224, 0.97.
// Where one tile holds all rows and the columns are many, reading ahead only doubles the reads (80 rows of N 8192 40 us, without 33).
struct FewTiles { int rows, ahead; };
static FewTiles few_tiles(int M, int N, int K, int Kw) {
  const bool lo8 = 2 * K == 3 * Kw;
  if (N > Kw || N < 512 || (long long)M * (N + 1200) > 1 << 21 || (K != Kw && !lo8) || Kw % (lo8 ? 256 : 128)) return {0, 0};
  for (int ahead = 1; ahead >= 0; --ahead)
    for (int rows = 32; rows <= (ahead ? 128 : 96); rows += 16) {
      const int tiles = (M + rows - 1) / rows, brief = ahead && tiles > 1 && (M - 1) % rows < 16;
      if ((tiles + ahead - brief) * (N / 64) <= 256 && (!ahead || tiles > 1 || N <= 4096)) return {rows, ahead - brief};
    }
  return {0, 0};
}
int gemm_f16_tile_rows(int M, int N, int K, int Kw, int span) {
  const int few = span == EpiResid::kSpan ? few_tiles(M, N, K, Kw).rows : 0;
  return few ? few : tile_rows(pick_tile(M, N, K), M, N);
}
int gemm_f16_variant(int M, int N, int K, int Kw, bool lo8, int span) {
  const FewTiles few = span == EpiResid::kSpan ? few_tiles(M, N, K, Kw) : FewTiles{0, 0};
  if (few.rows) return (few.ahead ? V_FEW_AHEAD : V_FEW) + few.rows / 16 - 2;
  const TilePick p = pick_tile(M, N, K);
  switch (p.tile) {
    case T_64x128: return p.tiles > 256 ? V_64x128_ROUNDS : span <= 64 ? V_64x128_8W : V_64x128;
    case T_128x128: return V_128x128;
    case T_64x256: return V_64x256;
    case T_128x256: return V_128x256;
    default: break;
  }
  switch (tile_rows(p, M, N)) {
    case 160: return V_160x256;
    case 192: return V_192x256;
    case 224: return V_224x256;
    default: break;
  }
  if (lo8) return V_256x256;
  const bool few_rounds = (long long)((M + 255) / 256) * (N / 256) < 768;
  return span == EpiResid::kSpan || few_rounds || (2LL * N + M) * Kw <= 170'000'000 ? V_256x256_SPREAD : V_256x256;
}

// Rows that go into a first launch of whole rounds where the rest of them costs less in a launch of its own, with lower tiles,
// than as the last round of all: 0 where it does not.  The second launch costs some 5 us (its own, and the end of the first's
// last round), and by the model the two have to come to 2.5 % less, those of QKV and gate/up to 4 %.
// us from the first launch's start to the last one's end, 7B, 18560 rows (73 x 16 tiles of 256 rows: 4.56 rounds; now four whole
// ones, and 14 x 16 tiles of 160), before the 128x128 waves, with them, and in two launches: down 1311, 1269, 1217; o 537, 530, 515.
// One launch over two, 261 products of d 768 to 5120 at 1500 to 25000 rows that 2.5 % splits: residual adds 1.023 in the mean and
// 0.994 at worst, with low terms 1.040 and 1.010; QKV and gate/up that the model gives 4 % 1.026 and 0.983 (QKV of d 4096 at 4806
// rows), with low terms 1.037 and 1.009, those that it gives less 1.010 and 0.965 (QKV of d 5120 at 12259 rows), 1.015 and 0.981.
int gemm_f16_first_rows(int M, int N, int K, int span) {
  const auto cost_of = [&](int rows) -> long long {        // 0: not a launch of such tiles
    const TilePick p = pick_tile(rows, N, K);
    return kTileCost[p.tile].bm < 192 ? 0 : rounds_cost(rows, N, tile_rows(p, rows, N));
  };
  const long long one = cost_of(M);
  if (one <= 2 * 346) return 0;                            // (a round of 256 rows and another)
  const float us_per_cost = (kTileCost[T_256x256].fixed + kTileCost[T_256x256].per_k * (float)K / 1024.0f) / 346.0f;
  const long long launch = (long long)(5.0f / us_per_cost);
  long long best = span == EpiResid::kSpan ? one * 39 / 40 : one * 25 / 26;
  int first = 0;
  for (int rows = 160; rows <= 256; rows += 32) {
    const int rounds = (int)(((long long)(M / rows) * (N / 256)) / 256);           // whole ones there are
    for (int r = rounds; r > 0 && r > rounds - 2; --r) {
      const int m = (int)((long long)r * 256 / (N / 256)) * rows;
      if (m <= 0 || m >= M) continue;
      const long long a = cost_of(m), b = cost_of(M - m);
      if (a && b && a + b + launch < best) {
        best = a + b + launch;
        first = m;
      }
    }
  }
  return first;
}

template <bool LO8, class Epi>
static void dispatch_lo(const GemmF16& g, const Epi& epi, hipStream_t st) {
  constexpr int span = Epi::kSpan;
  constexpr bool resid = span == EpiResid::kSpan;
  const int variant = gemm_f16_variant(g.M, g.N, g.K, g.Kw, LO8, span);
  if constexpr (resid) {
    const int ahead = variant >= V_FEW_AHEAD;
    switch (variant - (ahead ? V_FEW_AHEAD : V_FEW)) {
      case 0: return launch_few<2, 8, LO8>(g, ahead, epi, st);
      case 1: return launch_few<3, 6, LO8>(g, ahead, epi, st);
      case 2: return launch_few<4, 5, LO8>(g, ahead, epi, st);
      case 3: return launch_few<5, 4, LO8>(g, ahead, epi, st);
      case 4: return launch_few<6, 4, LO8>(g, ahead, epi, st);
      case 5: return launch_few<7, 4, LO8>(g, ahead, epi, st);
      case 6: return launch_few<8, 4, LO8>(g, ahead, epi, st);
      default: break;
    }
  }
  switch (variant) {
    case V_64x128_8W:
      if constexpr (span <= 64) launch<2, 4, 32, 32, 4, 4, 1, true, false, LO8>(g, epi, st);
      break;
    case V_64x128:
      if constexpr (span > 64) launch<2, 2, 32, 64, 6, 6, 1, false, false, LO8>(g, epi, st);
      break;
    case V_64x128_ROUNDS: launch<2, 2, 32, 64, 3, 3, 2, false, false, LO8>(g, epi, st); break;
    case V_128x128: launch<4, 2, 32, 64, 4, 4, 1, false, false, LO8>(g, epi, st); break;
    case V_64x256: launch<2, 4, 32, 64, 4, 4, 1, false, false, LO8>(g, epi, st); break;
    case V_128x256: launch<2, 4, 64, 64, 3, 3, 1, false, false, LO8>(g, epi, st); break;
    case V_160x256: launch<2, 4, 80, 64, 3, 3, 1, false, false, LO8>(g, epi, st); break;
    case V_192x256: launch<2, 4, 96, 64, 2, 3, 1, false, false, LO8>(g, epi, st); break;
    case V_224x256: launch<2, 4, 112, 64, 2, 3, 1, false, false, LO8>(g, epi, st); break;
    case V_256x256:
      if constexpr (LO8 || !resid) launch<4, 2, 64, 128, 2, 3, 1, false, false, LO8>(g, epi, st);
      break;
    default:
      if constexpr (!LO8 && resid) launch<2, 2, 128, 128, 2, 3, 1, false, true, LO8>(g, epi, st);
      else if constexpr (!LO8) launch<4, 2, 64, 128, 2, 3, 1, false, true, LO8>(g, epi, st);
  }
}
// An epilogue for rows m .. of its operands (m a multiple of 32).
static EpiResid rows_from(const EpiResid& e, int m) { return EpiResid{e.x + (size_t)m * e.ldx, e.ldx}; }
static EpiSwiglu rows_from(const EpiSwiglu& e, int m) { return EpiSwiglu{e.act + (size_t)m * e.ld, e.ld, e.f, e.lo_mode}; }
template <int HD>
static EpiQkv<HD> rows_from(EpiQkv<HD> e, int m) {
  e.o.q = (f16*)e.o.q + (size_t)m * e.o.ldq;
  e.o.tok_seq += m;
  e.o.tok_pos += m;
  return e;
}
template <class Epi>
static void dispatch_whole(const GemmF16& g, const Epi& epi, hipStream_t st) {
  if (g.W8) dispatch_lo<true>(g, epi, st);
  else dispatch_lo<false>(g, epi, st);
}
template <class Epi>
static void dispatch(const GemmF16& g, const Epi& epi, hipStream_t st) {
  if (const int m = gemm_f16_first_rows(g.M, g.N, g.K, Epi::kSpan)) {
    GemmF16 a = g, b = g;
    a.M = m;
    b.M = g.M - m;
    b.A += (size_t)m * g.lda;
    dispatch_whole(a, epi, st);
    dispatch_whole(b, rows_from(epi, m), st);
  } else {
    dispatch_whole(g, epi, st);
  }
}

void gemm_f16_resid(const GemmF16& g, float* x, int ldx, hipStream_t st) { dispatch(g, EpiResid{x, ldx}, st); }
void gemm_f16_swiglu(const GemmF16& g, f16* act, int ldact, int lo_mode, hipStream_t st) {
  dispatch(g, EpiSwiglu{act, ldact, g.N / 2, lo_mode}, st);
}
void gemm_f16_qkv(const GemmF16& g, const RopeKv& o, hipStream_t st) {
  if (o.head_dim == 128) dispatch(g, EpiQkv<128>{o}, st);
  else dispatch(g, EpiQkv<64>{o}, st);
}

// ---- weight repacking -------------------------------------------------------------------------------
// Converts `rows` bf16 source rows [rows, K] to f16 * kWeightScale (exact: a power-of-two scale moves
// the exponent only, and f16 has more mantissa bits than bf16; values beyond +-255 saturate) and
// stores them in fragment order starting at packed row `row0`.  interleave_mode 0: packed row =
// row0 + r.  1 (gate) / 2 (up): rows go to the even / odd 32-row blocks of the fused gate-up matrix.
// One workgroup re-encodes 32 source rows x 512 k: 128-byte row segments are read coalesced, transposed through
// LDS, and each 1 KiB fragment block is written by one wave in one piece.
// range_flag (device int): bit 0 is set if a weight is too large for the re-encoding (|w| > 255) or not finite.
// (At the other end nothing is reported: 0 < |w| < 2^-25 falls between half-precision subnormals and is rounded
// with an absolute error below 2^-33, which is far below what any tolerance can see; random weights contain
// such values.)
// dst8 != nullptr: the same 32 x 64 spans also go, as fp8(w * 16) saturated at +-448, to the 8-bit copy
// [n/32][k/64][2 KiB]: piece j (1 KiB) of a span holds, for lane (n, g), the 16 bytes k = 32 j + 16 g .. + 15.
__global__ __launch_bounds__(256) void pack_weight_kernel(const bf16* __restrict__ src, int K,
                                                          f16* __restrict__ dst, unsigned char* __restrict__ dst8,
                                                          int row0, int mode, int* __restrict__ range_flag) {
  __shared__ u32x4 tile[32 * 8];
  const int r0 = blockIdx.x * 32;                       // first source row of this workgroup
  const int nb = mode == 0 ? (row0 + r0) >> 5 : (r0 >> 5) * 2 + (mode == 2 ? 1 : 0);
  const int t = threadIdx.x, rr = t >> 3, cc = t & 7;   // load role: row, 16-byte chunk of a 64-k span
  const int blk = t >> 6, lane = t & 63;                // store role: fragment block of the span, lane
  const int k_end = min(K, (int)(blockIdx.y + 1) * 512);
  int bad = 0;
  for (int k0 = blockIdx.y * 512; k0 < k_end; k0 += 64) {
    const bf16x8 v = *(const bf16x8*)(src + (size_t)(r0 + rr) * K + k0 + cc * 8);
    f16x8 o;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float w = (float)v[j], a = fabsf(w);
      if (!(a <= 255.0f)) bad |= 1;                     // also true for NaN
      o[j] = from_f32<f16>(w * kWeightScale);
    }
    __syncthreads();                                    // the previous span has been read out
    tile[rr * 8 + (cc ^ (rr & 7))] = __builtin_bit_cast(u32x4, o);
    __syncthreads();
    const int sr = lane & 31, sc = 2 * blk + (lane >> 5);
    *(u32x4*)(dst + ((size_t)nb * (K >> 4) + (k0 >> 4) + blk) * 512 + lane * 8) = tile[sr * 8 + (sc ^ (sr & 7))];
    if (dst8) {
#if defined(__HIP_DEVICE_COMPILE__)
      const int j8 = t >> 7, l8 = (t >> 1) & 63, h8 = t & 1;       // piece, lane, 8-byte half of the lane's 16 bytes
      const int n8 = l8 & 31, c8 = 4 * j8 + 2 * (l8 >> 5) + h8;    // row, 8-k chunk of the span
      const f16x8 w8 = __builtin_bit_cast(f16x8, tile[n8 * 8 + (c8 ^ (n8 & 7))]);
      float v8[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v8[j] = fminf(fmaxf((float)w8[j] * (kLo8Scale / kWeightScale), -448.0f), 448.0f);
      int p0 = __builtin_amdgcn_cvt_pk_fp8_f32(v8[0], v8[1], 0, false);
      p0 = __builtin_amdgcn_cvt_pk_fp8_f32(v8[2], v8[3], p0, true);
      int p1 = __builtin_amdgcn_cvt_pk_fp8_f32(v8[4], v8[5], 0, false);
      p1 = __builtin_amdgcn_cvt_pk_fp8_f32(v8[6], v8[7], p1, true);
      int* o8 = (int*)(dst8 + ((size_t)nb * (K >> 6) + (k0 >> 6)) * 2048 + j8 * 1024 + l8 * 16 + h8 * 8);
      o8[0] = p0;
      o8[1] = p1;
#endif
    }
  }
  if (bad) atomicOr(range_flag, bad);
}

void pack_weight_f16(const bf16* src, int rows, int K, f16* dst, unsigned char* dst8, int row0, int interleave_mode,
                     int* range_flag, hipStream_t st) {
  // rows, row0 multiples of 32 and K a multiple of 64: guaranteed by the configuration checks
  hipLaunchKernelGGL(pack_weight_kernel, dim3((unsigned)(rows / 32), (unsigned)((K + 511) / 512)), dim3(256), 0, st,
                     src, K, dst, dst8, row0, interleave_mode, range_flag);
}

}  // namespace vla
