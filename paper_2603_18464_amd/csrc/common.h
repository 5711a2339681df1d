// Shared device helpers and the host-side launcher declarations of the VLA policy library.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace vla {

typedef __bf16 bf16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef _Float16 f16;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

constexpr int kWave = 64;

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16 v) { return (float)v; }
__device__ __forceinline__ float to_f32(f16 v) { return (float)v; }
template <class T> __device__ __forceinline__ T from_f32(float v);
// float -> half, IEEE round to nearest even: a value beyond the half-precision range becomes an infinity and a
// NaN stays a NaN, so an overflow or a non-finite input reaches the logits and the log-probs as NaN instead of
// being clamped to something plausible.
template <> __device__ __forceinline__ f16 from_f32<f16>(float v) { return (f16)v; }
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16 from_f32<bf16>(float v) { return (bf16)v; }

// ---- values across the lanes of a wave ------------------------------------------------------------------------
// combine<LO, HI>(v, op): v combined over the lanes that differ in strides LO, 2 LO, .. HI, narrowest first, the result in all
// of them.  In the vector unit: a step is one instruction behind the operand's, where a shuffle goes through the LDS and takes
// some hundred cycles, and the kernels of a decode step are chains of such steps.  LO is 1, 8, 16 or 32 (a stride of 4 is
// done by a mirror, which needs lanes that already agree in strides 1 and 2).
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
#else
  return v;
#endif
}
constexpr int kQuad0 = 0x00, kQuad1 = 0x55, kQuad2 = 0xAA, kQuad3 = 0xFF;       // lane 0 .. 3 of a quad to all of it
template <int STRIDE, class Op>
__device__ __forceinline__ float combine_step(float v, Op op) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (STRIDE == 1) return op(v, dpp<0xB1>(v));                        // quad_perm 1 0 3 2
  if constexpr (STRIDE == 2) return op(v, dpp<0x4E>(v));                        // quad_perm 2 3 0 1
  if constexpr (STRIDE == 4) return op(v, dpp<0x141>(v));                       // row_half_mirror
  if constexpr (STRIDE == 8) return op(v, dpp<0x128>(v));                       // row_ror 8
  if constexpr (STRIDE >= 16) {                                                 // both halves of the pair in both its lanes
    unsigned a = __builtin_bit_cast(unsigned, v), c = a;
    asm("" : "+v"(c));                                     // (of a swap of a value with itself the compiler makes a copy)
    const auto s = [&] {
      if constexpr (STRIDE == 16) return __builtin_amdgcn_permlane16_swap(a, c, false, false);
      else return __builtin_amdgcn_permlane32_swap(a, c, false, false);
    }();
    a = s[0];
    c = s[1];
    asm("" : "+v"(a), "+v"(c));                            // (... and takes its two results for one)
    return op(__builtin_bit_cast(float, a), __builtin_bit_cast(float, c));
  }
#endif
  return v;
}
template <int LO, int HI, class Op>
__device__ __forceinline__ float combine(float v, Op op) {
  static_assert(LO == 1 || LO >= 8, "see above");
  if constexpr (LO <= 1 && HI >= 1) v = combine_step<1>(v, op);
  if constexpr (LO <= 2 && HI >= 2) v = combine_step<2>(v, op);
  if constexpr (LO <= 4 && HI >= 4) v = combine_step<4>(v, op);
  if constexpr (LO <= 8 && HI >= 8) v = combine_step<8>(v, op);
  if constexpr (LO <= 16 && HI >= 16) v = combine_step<16>(v, op);
  if constexpr (LO <= 32 && HI >= 32) v = combine_step<32>(v, op);
  return v;
}
struct Add { __device__ __forceinline__ float operator()(float a, float b) const { return a + b; } };
struct Max { __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); } };
template <int LO, int HI> __device__ __forceinline__ float lanes_sum(float v) { return combine<LO, HI>(v, Add()); }
template <int LO, int HI> __device__ __forceinline__ float lanes_max(float v) { return combine<LO, HI>(v, Max()); }
__device__ __forceinline__ float wave_sum(float v) { return lanes_sum<1, 32>(v); }
__device__ __forceinline__ float wave_max(float v) { return lanes_max<1, 32>(v); }

// ---- kernel families timed by the profiling hooks ----------------------------------------------
enum Family {
  FAM_GEMM_QKV_PREFILL = 0,
  FAM_GEMM_O_PREFILL,
  FAM_GEMM_GATEUP_PREFILL,
  FAM_GEMM_DOWN_PREFILL,
  FAM_ATTN_PREFILL,
  FAM_GEMM_QKV_DECODE,
  FAM_GEMM_O_DECODE,
  FAM_GEMM_GATEUP_DECODE,
  FAM_GEMM_DOWN_DECODE,
  FAM_ATTN_DECODE,
  FAM_NORM,
  FAM_HEAD,
  FAM_MISC,
  FAM_TAIL,      // last prefill layer restricted to the rows that feed the head
  FAM_GEMM_QKV_TWO_PREFILL,      // the prefill GEMMs of two-term layers (with their low-term pass), same order
  FAM_GEMM_O_TWO_PREFILL,
  FAM_GEMM_GATEUP_TWO_PREFILL,
  FAM_GEMM_DOWN_TWO_PREFILL,
  FAM_COUNT
};

// ---- launcher arguments ---------------------------------------------------------------------------
struct RopeKv {
  void* q;               // [T, ldq] storage dtype, rotated queries (two-term mode: columns [d_model, 2 d_model) hold the low terms)
  void* k_cache;         // layer base: [slot][head][position][head_dim]
  void* v_cache;
  void* k_lo;            // two-term mode: low terms of the cached keys / values, same indexing, one byte per element
  void* v_lo;            //   (bf8(16 * lo)); nullptr otherwise
  int ldq;               // row pitch of q in elements
  const int32_t* tok_seq;   // [T] slot of each packed token
  const int32_t* tok_pos;   // [T] position of each packed token inside its sequence
  const float* rope_cos;    // [max_seq, head_dim/2]
  const float* rope_sin;
  int n_heads, head_dim, max_seq, d_model;   // max_seq: positions per (slot, head) block of the cache (its pitch)
};

// The 16-bit path keeps weights as bfloat16 at the boundary but feeds the matrix cores in half
// precision: bf16 -> f16 is exact once the weights are scaled by a power of two (kWeightScale keeps
// |w| up to 255 finite and everything above 2^-25 exact), activations rounded to f16 carry 8x less
// rounding error than bf16 at the same MFMA rate, and the scale is divided out in the epilogue.
constexpr float kWeightScale = 256.0f;
constexpr int kMaxKSplit = 4;   // most partial planes (groups of 4 K slices) a decode GEMM writes

// Element (m, k) of an operand of ld halves a row in MFMA fragment order: blocks of 32 rows, in each [k / 16][lane][8] where lane
// l holds row l & 31 and k = 8 * (l >> 5) .. + 7.  32 rows of 64 k are 4 KiB, so a slab of a product is loaded in pieces of
// one KiB, and rows that follow one another lie 16 bytes apart, so a kernel that holds many of them writes whole lines.
__device__ __forceinline__ size_t act_index(int m, int k, int ld) {
  return (size_t)(m >> 5) * 32 * ld + (size_t)(k >> 4) * 512 + ((m & 31) + 32 * ((k >> 3) & 1)) * 8 + (k & 7);
}
// Byte of its 8-bit low terms: they follow the Kw high terms of a block, [k / 32][lane][16], lane l: row l & 31, k = 16 * (l >> 5) ..
__device__ __forceinline__ size_t act_lo8_index(int m, int k, int ld, int Kw) {
  return (size_t)(m >> 5) * 64 * ld + (size_t)64 * Kw + (size_t)(k >> 5) * 1024 + ((m & 31) + 32 * ((k >> 4) & 1)) * 16 + (k & 15);
}

// Two-term activations: a value a is carried as hi = f16(a) and lo = f16(a - hi) (together about 22 significant
// bits).  Operands keep them side by side, A = [hi | lo] with K = 2 * Kw columns; since the weights
// are exact, A * W^T = hi * W^T + lo * W^T is one contraction over 2 * Kw in which the weight index wraps.
struct GemmF16 {
  const f16* A;    // [M, K] activations in fragment order, allocated to a multiple of 32 rows (see act_index)
  int lda;         // halves a row
  const f16* Wp;   // [N, Kw] weights * kWeightScale in MFMA fragment order (see pack_weight_f16)
  int M, N, K;     // K = Kw (single-term A), 2 * Kw (two-term A, half-precision low terms) or, with W8, 1.5 * Kw
  int Kw;          //   (two-term A whose low terms are bytes: row = [hi: Kw halves | lo8: Kw bytes]; Kw % 128 == 0)
  const f16* W8;   // 8-bit copy of the weights for 8-bit low terms (see gemm_f16.hip), or nullptr
};
// 8-bit low terms (see gemm_f16.hip): lo8 = bf8(16 * (a - f16(a))), four at a time.
constexpr float kLo8Scale = 16.0f;
__device__ __forceinline__ int pack_lo8(float e0, float e1, float e2, float e3) {
#if defined(__HIP_DEVICE_COMPILE__)
  int p = __builtin_amdgcn_cvt_pk_bf8_f32(e0 * kLo8Scale, e1 * kLo8Scale, 0, false);
  return __builtin_amdgcn_cvt_pk_bf8_f32(e2 * kLo8Scale, e3 * kLo8Scale, p, true);
#else
  return 0;
#endif
}
__device__ __forceinline__ float unpack_lo8(int word, int byte) {   // byte must be a compile-time constant 0..3
#if defined(__HIP_DEVICE_COMPILE__)
  float v;
  switch (byte) {
    case 0: v = __builtin_amdgcn_cvt_f32_bf8(word, 0); break;
    case 1: v = __builtin_amdgcn_cvt_f32_bf8(word, 1); break;
    case 2: v = __builtin_amdgcn_cvt_f32_bf8(word, 2); break;
    default: v = __builtin_amdgcn_cvt_f32_bf8(word, 3); break;
  }
  return v * (1.0f / kLo8Scale);
#else
  return 0.f;
#endif
}

// Rotation of one pair by (cos, sin), written with explicit roundings: every kernel that applies it (the two
// epilogue forms of the QKV GEMM, the decode step) then produces the same float32 bits, which two-term outputs
// make visible.
__device__ __forceinline__ void rope_pair(float lo, float hi, float cs, float sn, float& a, float& b) {
  a = __fmaf_rn(lo, cs, -__fmul_rn(hi, sn));
  b = __fmaf_rn(hi, cs, __fmul_rn(lo, sn));
}

// *p, and with ONCE as data that is not read again before the caches have turned over: it is the first to leave them.
template <bool ONCE, class V>
__device__ __forceinline__ V load_once(const V* p) {
  if constexpr (ONCE) return __builtin_nontemporal_load(p);
  else return *p;
}

// Keeps what is computed from v from being computed ahead of a loop and kept in registers.
__device__ __forceinline__ void hold32(unsigned& v) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(v));
#endif
}

// C = A * W^T with fused epilogues (f16 MFMA, fp32 accumulation).
void gemm_f16_resid(const GemmF16& g, float* x, int ldx, hipStream_t st);           // x += C
// silu(gate)*up; lo_mode 1: also half-precision low terms at column f + j; 2: 8-bit low terms (act_lo8_index)
void gemm_f16_swiglu(const GemmF16& g, f16* act, int ldact, int lo_mode, hipStream_t st);
void gemm_f16_qkv(const GemmF16& g, const RopeKv& o, hipStream_t st);               // RoPE + cache
// range_flag: device int, bits are OR-ed in when a weight cannot be re-encoded exactly (see pack_weight_kernel);
// dst8 != nullptr: also the 8-bit copy fp8(w * 16) for 8-bit low terms (K % 64 == 0)
// The variant of the kernel a launch takes (an index into the names), by the product's size (Kw: its contraction; K: that and
// its low terms, 1.5 or 2 * Kw), whether it has slabs of 8-bit low terms, and its epilogue: the columns of a row that this needs
// together, 32 (residual add), 64 (gate/up, QKV of heads of 64) or 128 (QKV of heads of 128).
extern const char* const kGemmF16Variants[];
int gemm_f16_variant(int M, int N, int K, int Kw, bool lo8, int span);
int gemm_f16_tile_rows(int M, int N, int K, int Kw, int span);    // rows of that launch's tiles
int gemm_f16_first_rows(int M, int N, int K, int span);    // rows of the first of a product's two launches, 0: it is one
void pack_weight_f16(const bf16* src, int rows, int K, f16* dst, unsigned char* dst8, int row0, int interleave_mode,
                     int* range_flag, hipStream_t st);

// float32 path: W [N, K] row-major; the q/k/v and gate/up products take the RMSNorm of the x rows [M, d_model] with them.
void gemm_f32_qkv(const float* x, const float* gain, float eps, const float* W, int M, const RopeKv& o, hipStream_t st);
void gemm_f32_swiglu(const float* x, const float* gain, float eps, const float* W /* [gate | up] */, float* act, int M,
                     int d, int f, hipStream_t st);
void gemm_f32_resid(const float* A, const float* W, float* x, int M, int d, int K, hipStream_t st);   // x += A * W^T

// Row-wise kernels.
void rmsnorm(const float* x, const float* gain, f16* out, int rows, int d, float eps,
             int lo_mode /* out in fragment order, 0: rows of d; 1: [hi | lo] of 2 d; 2: [hi | lo8] of 1.5 d */, hipStream_t st);
template <class T>
void assemble_prefix(const T* patch_emb, const int32_t* instr_ids, const T* embed,
                     const int32_t* tok_src, float* x, int T_tokens, int d, int vocab, hipStream_t st);
// Attention: one query row per (token, head) against the cache; its LDS holds the scores of four of them.
inline size_t attention_rows_lds(int max_seq) { return 4 * (size_t)max_seq * sizeof(float); }
void attention_rows_f32(const float* q, const float* k_cache, const float* v_cache, const int32_t* tok_seq,
                        const int32_t* tok_pos, float* out, int n_tok, int n_heads, int head_dim, int max_seq,
                        hipStream_t st);

// Prefill attention for the 16-bit path: causal flash attention over whole prefixes (MFMA).
// cu_patch / cu_instr are the device copies of the cumulative offsets; max_len = longest prefix; slot_map
// (device, [B], or nullptr for the identity) gives the cache slot of each sequence of the call.
// k_lo / v_lo (low terms of the cache) != nullptr: two-term mode, q rows are [hi | lo] with the low terms at column
// d_model; the output is in fragment order (act_index, ldo halves a row), low terms at column d_model too, or (out_lo8) as bytes.
void flash_prefill(const f16* q, int ldq, const f16* k_cache, const f16* v_cache, const unsigned char* k_lo,
                   const unsigned char* v_lo, const int32_t* cu_patch, const int32_t* cu_instr, const int32_t* slot_map,
                   f16* out, int ldo, bool out_lo8, int B, int max_len, int n_heads, int head_dim, int max_seq,
                   hipStream_t st);

// Decode-step GEMMs (M <= 128): weight-streaming split-K kernel writing partial sums, and the kernels
// that add the partials in a fixed order and apply the elementwise step that follows each GEMM.
// Activations named *_frag are [M, K] in MFMA fragment order: [m/32][k/16][lane][8].
int skinny_ksplit(int N, int K);
constexpr int kSkinnyMaxRows = 128;   // most rows of one weight-streaming GEMM launch
// Two-term mode: *_lo arguments hold the low terms f16(a - f16(a)) in the same fragment order (nullptr: single-term).
// The M rows of a launch are rows prow0 .. prow0 + M - 1 of partial planes of plane_rows rows each.
// w_once: the weights do not stay in the caches until they are read again.
void skinny_gemm(const f16* Afrag, const f16* Afrag_lo, const f16* Wp, float* part, int M, int N, int K, int ksplit,
                 int plane_rows, int prow0, bool w_once, hipStream_t st);
// The gate/up product of at most kSkinnyMaxRows rows with its elementwise step, straight to fragments (K >= 128).
void skinny_swiglu(const f16* Afrag, const f16* Afrag_lo, const f16* Wp, f16* act_frag, f16* act_frag_lo, int M, int f,
                   int K, bool w_once, hipStream_t st);
// The same products for at most kNormRows rows that take the RMSNorm of their rows with them (two: as two terms), from y = x *
// gain (float32, fragment order) and sums of squares [M][d / 16]; and the O / down product that adds to the residual rows x
// [M, N] itself, with the sums of skinny_gemm with kgroups planes and reduce_resid_norm, and with a gain leaves y and sums.
constexpr int kNormRows = 32;
void skinny_norm_gemm(const float* y, const float* sums, float eps, bool two, const f16* Wp, float* part, int M, int N, int d,
                      int kgroups, bool w_once, hipStream_t st);
void skinny_norm_swiglu(const float* y, const float* sums, float eps, bool two, const f16* Wp, f16* act_frag, f16* act_frag_lo,
                        int M, int f, int d, bool w_once, hipStream_t st);
void skinny_resid(const f16* Afrag, const f16* Afrag_lo, const f16* Wp, float* x, const float* gain, float* y, float* sums, int M,
                  int N, int K, int kgroups, bool w_once, hipStream_t st);
// The same product for up to 256 rows on the tiled kernel (256 rows x 256 or 64 columns a workgroup), split over `ksplit`
// K slices (one partial plane each): activations go through LDS once per workgroup instead of once per wave, which is what
// a large batch needs to stream every weight once at full rate.  Needs N % 256 == 0 and K % 64 == 0 (splitk_gemm_fits).
bool splitk_gemm_fits(int M, int N, int K);
int splitk_ksplit(int N, int K);
void splitk_gemm(const f16* Afrag, const f16* Afrag_lo, const f16* Wp, float* part, int M, int N, int K, int ksplit,
                 int plane_rows, int prow0, hipStream_t st);
void reduce_resid_norm(const float* part, int ksplit, int plane_rows, int prow0, int M, int d, float* x,
                       const float* gain, float eps, f16* hn_frag, f16* hn_frag_lo, int row0, hipStream_t st);
// Start of a decode step: x rows from the embedding table, tok_seq / tok_pos of the step, lengths + 1, and with a gain the
// first norm in fragment order, or with y != nullptr y and sums as above.  slot_map: device [M] cache slot of each row, nullptr = identity.
template <class T>
void decode_begin(const int32_t* ids, const T* embed, int vocab, int32_t* seq_len, const int32_t* slot_map,
                  int32_t* tok_seq, int32_t* tok_pos, float* x, int M, int d, const float* gain, float eps, float* y,
                  float* sums, f16* hn_frag, f16* hn_frag_lo, hipStream_t st);
void reduce_swiglu(const float* part, int ksplit, int plane_rows, int prow0, int M, int f, f16* act_frag,
                   f16* act_frag_lo, int row0, hipStream_t st);

// Decode attention of the 16-bit path (one query per row of the step); output in fragment order.  k_lo / v_lo
// != nullptr: two-term mode (low terms of the cache, output also as low-term fragments out_frag_lo).
// kv_once: the cached rows do not stay in the last-level cache until the next step reads them.
void decode_attention_fused(const float* part, int ksplit, int part_rows, const float* rope_cos, const float* rope_sin,
                            f16* k_cache, f16* v_cache, unsigned char* k_lo, unsigned char* v_lo, const int32_t* tok_seq,
                            const int32_t* tok_pos, f16* out_frag, f16* out_frag_lo, int B, int d_model, int n_heads,
                            int head_dim, int max_seq, bool kv_once, hipStream_t st);

// Action head: final RMSNorm + action rows of the LM head -> logits [B, A] float32.
template <class T>
void head_logits(const float* x, const int32_t* row_index, const float* gain, const T* w_head,
                 float* logits, int ld_logits, int B, int d, int A, float eps, hipStream_t st);
void select_tokens(const float* logits, int ld_logits, int B, int A, float temperature, const float* gumbel, int k,
                   int n_tokens, const float* act_scale, const float* act_offset, int action_dim,
                   int32_t* tokens_out, float* logp_out, float* actions_out, int out_stride,
                   int32_t* next_ids, int id0, hipStream_t st);

// Value head (attention pooling over the rows that feed the action head, step embedding, GELU MLP).
void value_accumulate(const float* x, const int32_t* row_index, const float* gain, float eps, const float* attn_w,
                      const float* attn_b, int B, int d, bool first, float* vz, float* vml, hipStream_t st);
template <class T>
void value_finish(const float* vz, const float* vml, const T* step_emb, int n_steps, const int32_t* step_t,
                  const T* w1, const float* b1, const float* w2, const float* b2, int B, int d, float* vu, float* vh,
                  float* values, hipStream_t st);

// Last prefill layer, compact rows: gather attention output (to fragment order) and residual rows, scatter back.
// att_frag_lo != nullptr: att (fragment order, ld_att halves a row) has low terms (lo8: bytes), which go to att_frag_lo as half
// precision
void gather_tail(const f16* att, int ld_att, bool lo8, const float* x, const int32_t* need, int n, int d,
                 f16* att_frag, f16* att_frag_lo, float* x_c, hipStream_t st);
void scatter_tail(const float* x_c, const int32_t* need, int n, int d, float* x, hipStream_t st);

// Chunk pass (all K action rows in one forward): merged id stream, fed-token buffer, emitting rows, scoring.
void merge_tail_ids(const int32_t* instr_ids, const int32_t* cu2_dev, const int32_t* tail, int B, int n_tail,
                    int total, int32_t* out, hipStream_t st);
void tail_ids(const int32_t* tokens, int B, int K, int id0, int A, int placeholder, int32_t* tail, hipStream_t st);
void chunk_rows(const int32_t* last_row, int B, int K, int32_t* rows, hipStream_t st);
void score_rows(const float* logits, int rows, int A, float temperature, const int32_t* tokens, const float* mu,
                float sigma, float* logp_out, float* ratio_out, float* weight_out, hipStream_t st);

// Ceiling probes (see vla_probe): an MFMA-only loop on weight bits and a plain streaming read.
void probe_mfma(const f16* w, size_t n_frag, int n_wg, int iters, float* sink, hipStream_t st);
double probe_mfma_flops(int n_wg, int iters);
void probe_stream(const void* src, size_t bytes, int n_wg, unsigned* sink, hipStream_t st);

// Small utilities.
void rope_table(float* cos_t, float* sin_t, int max_seq, int head_dim, float theta, hipStream_t st);
// slot_map: device [B] cache slot of each sequence of the call, nullptr = identity; seq_len is indexed by slot.
void build_token_maps(const int32_t* cu_patch_dev, const int32_t* cu_instr_dev, const int32_t* slot_map, int B,
                      int T_tokens, int32_t* tok_seq, int32_t* tok_pos, int32_t* tok_src, int32_t* last_row,
                      int32_t* seq_len, hipStream_t st);
template <class T>
void convert_copy(const T* src, float* dst, size_t n, hipStream_t st);   // gains -> float32
template <class T>
void plain_copy(const T* src, T* dst, size_t n, hipStream_t st);

}  // namespace vla
