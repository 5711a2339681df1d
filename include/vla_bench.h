/*
 * vla_bench.h — measurement support of the VLA policy library (include/vla.h): the practical ceilings of the
 * device and per-kernel-family timing.  Not part of the policy path; used by bench.py only.
 */
#ifndef VLA_BENCH_H
#define VLA_BENCH_H

#include "vla.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Practical ceilings of the device the context runs on, for reporting next to the vendor peaks (benchmark
 * support, not part of the policy path; unlike every other call it waits for its own kernels).  Needs loaded
 * weights on the 16-bit path.
 *   kind 0: an MFMA-only loop (32 independent 16x16x32 half-precision MFMAs per iteration and wave, the prefill
 *           GEMMs' instruction; two waves per SIMD, operands = real weight fragments held in registers)
 *                                                                                        -> *value_out in TFLOP/s
 *   kind 1: a plain 16-byte-per-lane streaming read of all layer weights                -> *value_out in GB/s
 * Best of three timed runs after a warm-up. */
int vla_probe(vla_ctx* ctx, int32_t kind, double* value_out, void* hip_stream);

/* Rows of the first launch of a prefill product [rows, k] x [n, k]^T that takes two, one of whole rounds of tiles and one of the
 * rest; 0 where it takes one, and for sizes the 16-bit path does not have.  Host only.  two_term: operands of a two-term layer;
 * span: 32 for the output projection and the down projection, 64 for gate/up and for the QKV product of heads of 64, 128 for that
 * of heads of 128 (the columns of a row that the product's last step needs together). */
int32_t vla_gemm_first_rows(int32_t rows, int32_t n, int32_t k, int32_t two_term, int32_t span);

/* Which variant of the prefill GEMM a launch over `rows` rows of such a product runs ("128x256", ...: rows x columns of a tile,
 * and its form where there are several): a static text, "" for sizes the 16-bit path does not have.  Of a product of two launches
 * ask for the rows of each.  Host only. */
const char* vla_gemm_variant(int32_t rows, int32_t n, int32_t k, int32_t two_term, int32_t span);

/* Rows of the tiles that this launch runs: 32 to 128 for residual adds of rows x (n + 1200) <= 2^21, of products no wider
 * than their contraction (tiles of 64 columns).  Where the cost model picks tiles of 192 or 256 rows, of 160, 192, 224 and
 * 256 those are taken that need the least rounds of 256 workgroups x (rows + 90), if that is 2.5 % less than the model's.  0 for
 * sizes the 16-bit path does not have.  Host only. */
int32_t vla_gemm_tile_rows(int32_t rows, int32_t n, int32_t k, int32_t two_term, int32_t span);

/* What a decode step of `rows` sequences with `positions` cached positions (all of them together) reads as data that does not
 * come again: bit 0 the weights (products that leave partial sums for the next launch: only matrices of 64 MB and more), bit 1
 * the keys and values.  0 on the float32 path, for a NULL context and for sizes that no step has.  Host only. */
int32_t vla_decode_reads_once(vla_ctx* ctx, int32_t rows, int64_t positions);

/* Timing hooks for the benchmark: duration of the launches of one kernel family, measured with
 * HIP events recorded on the launch stream around each launch.  vla_prof_enable(ctx, mask) clears
 * what was collected and then times the families whose bit (1 << index) is set in mask (0 = off).
 * vla_prof_read synchronises the recorded events (host-blocking) and reports, for family index i
 * (0 <= i < vla_prof_count()), its name, number of launches and total milliseconds.  Families are
 * named by the read-out itself: the four GEMMs (qkv, o, gate-up, down) and the attention of prefill
 * and of decode, rmsnorm, head_select, misc. */
int vla_prof_enable(vla_ctx* ctx, int32_t mask);
int vla_prof_count(void);
int vla_prof_read(vla_ctx* ctx, int32_t i, const char** name, int64_t* launches, double* total_ms);

#ifdef __cplusplus
}
#endif
#endif /* VLA_BENCH_H */
