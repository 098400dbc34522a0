/*
 * regione_bench.h - measurement aids of the RegionE library (NOT part of the method's ABI in regione.h): forced
 * kernel plans for same-process comparisons, per-kernel-class timing with HIP events, and a register-only probe of
 * what the chip's matrix cores sustain.  Used by the benchmark and by tests that sweep kernel plans.
 */
#ifndef REGIONE_BENCH_H
#define REGIONE_BENCH_H

#include "regione.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Tuning knob for experiments: forces the tile (1..6: six tiles from 64 x 64 to 256 x 256; larger numbers are the tile
 * codes of csrc/gemm_tiles.h, any other is refused) and the number of K splits of every later GEMM of this context; 0 leaves
 * either to the library.  K splits without a tile split the tile that the product gets by itself.  A product fails that
 * has no such tile (some are bf16 or E4M3 only) or whose split does not fit the workspace. */
int regione_tune_gemm(regione_ctx* ctx, int32_t wave_tile_blocks, int32_t k_splits);

/* The tile and the number of K splits that a product of m rows, n columns and k elements gets by itself, with a K-split workspace
 * of that many bytes (a context has 128 MiB, half of it while text and image rows run side by side).  A pure host function.  *tile
 * is a tile code of csrc/gemm_tiles.h, or 0 for the kernel of few bf16 rows and of narrow bf16 results (at most 64 columns).
 * REGIONE_GEMM_BF16_STORED: the bf16 projection that writes K and V in a storing forward (REGIONE_FLAG_STORE), whose tiles are chosen apart so
 * that the same rows give the same stored bits from one version of the library to the next. */
enum { REGIONE_GEMM_BF16 = 0, REGIONE_GEMM_E4M3 = 1, REGIONE_GEMM_BF16_STORED = 2 };
int regione_gemm_plan_host(int32_t m, int32_t n, int32_t k, int32_t kind, int64_t workspace_bytes, int32_t* tile, int32_t* k_splits);

/* How many lanes (streams) the projections of a double-stream block run on with that many fresh text and image rows: 2 where the two groups run
 * side by side, else 1.  While per-class timing is on, and in the 8-bit form, it is always one.  A pure host function. */
int regione_block_lanes_host(int32_t n_txt, int32_t n_img, int32_t hidden, int32_t mlp, int32_t compute_dtype, int32_t* lanes);

/* Tuning knob for experiments: forces the number of key-range splits (1..32) of every later
 * attention call of this context; 0 restores the automatic choice. */
int regione_tune_attention(regione_ctx* ctx, int32_t key_splits);

/* How an attention of n_q queries on n_keys keys is dealt to workgroups in this bf16 context, with its workspace and what
 * regione_tune_attention forces, for keys in one array, in two (fresh rows, then cache rows) or named by an index list: *key_splits equal key ranges per
 * query tile, or, where *range_tiles > 0, even ranges of that many key tiles (64 keys) each behind the first *whole_query_tiles query tiles
 * (counted in 128 queries) of every head, which stay unsplit; workgroups of 256 queries take them in pairs and leave an odd last one to the
 * ranges.  A forced number of equal ranges is taken in workgroups of 128 queries.  Host only. */
enum { REGIONE_KEYS_CONTIGUOUS = 0, REGIONE_KEYS_TWO = 1, REGIONE_KEYS_INDEXED = 2 };
int regione_attention_plan(regione_ctx* ctx, int32_t n_q, int32_t n_keys, int32_t heads, int32_t d, int32_t source, int32_t* key_splits,
                           int32_t* range_tiles, int32_t* whole_query_tiles);

/* Tuning knob for experiments: the kind of workgroups and of key ranges that later attention calls of this context take where they have such; 0 leaves either to the
 * library.  form: workgroups of 128 or 256 queries in two wave groups (head dimension 128), of 32 queries whose keys are dealt to the waves, or of 128 queries in
 * waves that run freely.  ranges: equal ones, even ones for all query tiles, or even ones behind unsplit query tiles (the last two for head dimension
 * 128).  A number of equal ranges that regione_tune_attention forces is taken in that form.  The ranges of wide 8-bit blocks stay as they are. */
enum { REGIONE_ATTN_TILES_128 = 1, REGIONE_ATTN_TILES_256 = 2, REGIONE_ATTN_DEALT = 3, REGIONE_ATTN_FREE = 4 };
enum { REGIONE_RANGES_EQUAL = 1, REGIONE_RANGES_EVEN = 2, REGIONE_RANGES_EVEN_BEHIND = 3 };
int regione_tune_attention_form(regione_ctx* ctx, int32_t form, int32_t ranges);

/* The kind of workgroups (REGIONE_ATTN_*) that regione_attention_plan's call gets, with its *key_splits and *range_tiles.  One more source: the keys of an 8-bit
 * double-stream block wider than 1024, whose key ranges are chosen apart.  Host only. */
enum { REGIONE_KEYS_WIDE_8BIT = 3 };
int regione_attention_workgroups(regione_ctx* ctx, int32_t n_q, int32_t n_keys, int32_t heads, int32_t d, int32_t source, int32_t* form, int32_t* key_splits,
                                 int32_t* range_tiles);

/* Per-kernel-class timing for benchmarks (not part of the method).  While enabled, every
 * kernel launch group of the context is bracketed by a HIP event pair on its stream (at most
 * 8192 pairs between two reads).  regione_profile_read waits for the stream, adds the elapsed
 * milliseconds and the number of launch groups of each class into the two host arrays of
 * n_classes entries (index = REGIONE_PROF_*), and clears the recorded pairs. */
enum { REGIONE_PROF_PARTITION = 0, REGIONE_PROF_ROWS = 1, REGIONE_PROF_LAYERNORM = 2, REGIONE_PROF_GEMM = 3,
       REGIONE_PROF_ATTENTION = 4, REGIONE_PROF_VELOCITY = 5, REGIONE_PROF_CLASSES = 6 };
int regione_profile_enable(regione_ctx* ctx, int32_t on);
int regione_profile_read(regione_ctx* ctx, double* total_ms_host, int64_t* launches_host, int32_t n_classes);

/* Matrix-core peak probe for benchmarks (not part of the method): what the MFMA units of THIS
 * chip sustain at the clock it holds under load, to read the achieved TFLOP/s against.  Every
 * wave runs `iters` rounds of four independent register-only MFMAs (format 0: bf16
 * v_mfma_f32_32x32x16_bf16; 1: E4M3 v_mfma_f32_32x32x64_f8f6f4) on pseudo-random finite
 * operands and stores one float per lane so the work cannot be dropped.  n_workgroups
 * workgroups of 256 threads; out: float32 [n_workgroups * 256].  The launch is timed under
 * REGIONE_PROF_GEMM; *flops_host receives the work of the launch (n_workgroups * 4 waves *
 * iters * 4 * 2 * 32 * 32 * K, K = 16 or 64). */
int regione_mfma_peak_probe(regione_ctx* ctx, int32_t format, int32_t iters, int32_t n_workgroups, float* out, double* flops_host);

#ifdef __cplusplus
}
#endif
#endif /* REGIONE_BENCH_H */
