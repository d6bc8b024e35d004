/*
 * rls - aids for benchmarks and tests.  NOT part of the library's interface proper (rls.h) and not part of the
 * paper's method: a benchmark program uses rls_profile_* to time the fused assign + update pass that dominates the
 * k-means calls of Algorithm 1 (Sec. 4.2) on the stream the library launches it on.
 *
 * Unlike everything in rls.h rls_profile_* keep process-wide state (a flag and a pool of HIP events the
 * library creates on first use); a mutex guards that state.  While enabled, every sweep of every host thread
 * records into the one pool, so the figures only mean something when one thread is sweeping.  Leave it
 * disabled (the default) anywhere else: a sweep that is being recorded into a HIP graph must not record events.
 */
#ifndef RLS_BENCH_H
#define RLS_BENCH_H

#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

/* on != 0: rls_kmeans_sweep[_batched] records a pair of events around every launch of the Lloyd step kernel. */
int32_t rls_profile_enable(int32_t on);
/* Waits for the recorded events; returns the number of launches timed and their summed duration in
 * milliseconds, and forgets them.  RLS_ERR_NULL / RLS_ERR_HIP as in rls.h. */
int32_t rls_profile_read(int32_t *n_launches, double *total_ms);
/* The seeding chain of up to about a million points runs in one launch whose workgroups wait for each other; one that has
 * waited too long (2 ms for all of them to be there, 0.1 ms in the parts of a batch after one that gave up, 50 ms later on) gives up, and a
 * second kernel, whose workgroups need not run at the same time, does the chain again.  This sets these limits, in ticks of the 100 MHz clock, for the calls of the
 * host thread that sets it.  0 makes every launch with more than one workgroup take that second path, for tests; a negative
 * value restores the default. */
int32_t rls_seed_wait_limit(int64_t ticks);
/* The same for the workgroups of a space from `first_workgroup` on; the ones before it wait the default time. */
int32_t rls_seed_wait_limit_from(int32_t first_workgroup, int64_t ticks);
/* How the seeding chains of up to 64 spaces of a batch are drawn on a chip with so many compute units: the number of spaces per launch
 * (`batch`: all together; fewer: in parts), or 0 where they are walked in memory, with launches for every centre.  `quads` != 0: the rows of
 * every space can be read 16 bytes at a time. */
int32_t rls_seed_spaces_at_once(int64_t N, int32_t d, int32_t batch, int32_t k_max, int32_t quads, int32_t compute_units);
/* Where in its workspace a sweep of one space over rows in spatial order keeps the tile lists of its last round, for tests of what
 * lists occur: byte offset and number of 32-bit words (0: the sweep takes the points as they come).  Per group with lists and
 * unit of points 16 words; the four highest bits of each of the first eight are the number of tiles the unit meets, less one. */
int32_t rls_sweep_tile_lists(int64_t N, int32_t d, int32_t k_min, int32_t k_max, int64_t *offset_out, int64_t *words_out);
/* How rls_gbt_score_batched scores with forests of one shape: configurations of a tile, trees walked side by side, trees of a chunk, and whether
 * one part of a workgroup's threads adds leaf values while the others move the next chunk. */
int32_t rls_score_plan(int64_t N, int32_t d, int32_t batch, int32_t n_trees, int32_t depth, int32_t *tile_out, int32_t *side_out,
                       int32_t *trees_per_chunk_out, int32_t *apart_out);
/* Lanes that rls_snap_to_valid_batched puts on a (centroid, knob): 64, or 1 where there are many of them. */
int32_t rls_snap_lanes(int32_t batch, int32_t k, int32_t n_knobs);
/* `n` single matrix instructions (32 x 32 x 16, fp16 or bf16 operands, fp32 accumulators) on operands as the kernels hold them, for
 * tests of what the instruction leaves out of a sum:
 *   a_dev, b_dev  [n][64 lanes][8] 16-bit elements: lane l holds those of row (column) l % 32, k = 8 (l / 32) .. + 7; 16-byte aligned
 *   acc_dev       [n][64][16] fp32 (acc_out_dev: the same, may be acc_dev): entry 4 q + e of lane l is row 8 q + 4 (l / 32) + e, column l % 32 */
int32_t rls_matrix_step(int32_t bf16, const void *a_dev, const void *b_dev, const float *acc_dev, float *acc_out_dev, int32_t n,
                        void *stream);

#ifdef __cplusplus
}
#endif
#endif /* RLS_BENCH_H */
