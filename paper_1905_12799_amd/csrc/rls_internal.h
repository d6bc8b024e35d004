// Internal declarations shared by the host entry points and the kernel files.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rls.h"
#include "rls_bench.h"

namespace rls {

// last failing hipError_t on this thread
void set_hip_error(hipError_t e);

#define RLS_HIP_TRY(expr)                      \
    do {                                       \
        hipError_t rls_e_ = (expr);            \
        if (rls_e_ != hipSuccess) {            \
            ::rls::set_hip_error(rls_e_);      \
            return RLS_ERR_HIP;                \
        }                                      \
    } while (0)

inline int64_t align_up(int64_t v, int64_t a) { return (v + a - 1) / a * a; }

// ---------------------------------------------------------------------------------------------
// Sweep plan: how the runs (one per k) of a sweep are packed into workgroup-sized groups.
//
// An MFMA tile has 32 centroid rows = 8 quads of 4 rows.  Quad `slot` (0..7) of every tile of a
// group belongs to one run for the whole group, so the running (best, second best) of a point
// never leaves its lane.  A group holds R = 8 / S runs, each owning S slots.
// Centroid j of run r sits in tile (j/4)/S, slot r*S + (j/4)%S, row-in-quad j%4.
struct GroupDesc {
    int16_t run0;      // index of the first run (k = k_min + run0)
    int16_t n_runs;    // real runs in this group (<= 8 / S)
    int16_t S;         // slots per run: 1, 2, 4 or 8
    int16_t n_tiles;   // 32-row tiles
    int16_t copies;    // copies of the LDS accumulators (a power of two up to 16)
    int16_t lab0;      // run slots (8 / S each) of all earlier groups: where this group's label bytes begin, in units of N rounded up to 16
    int32_t tile0;     // tiles of all earlier groups (offset of this group's operand block)
    int32_t n_chunks;  // chunks the points are cut into for this group
    int32_t chunk_len; // points per chunk (a multiple of 64)
    int32_t wg0;       // chunks of all earlier groups
    int32_t list0;     // groups with tile lists before this one; -1: every unit meets every tile
    int32_t part0;     // per-chunk centroid rows of all earlier groups (n_chunks times rows each): where this group's deltas begin
};

constexpr int kMaxGroups = 64;       // (44 is the most any range of k and number of features needs)

struct SweepPlan {
    int32_t n_groups;
    int32_t n_runs;      // k_max - k_min + 1
    int32_t k_min;
    int32_t total_tiles;
    int32_t lab_slots;   // sum over the groups of their 8 / S run slots
    int32_t total_rows;  // sum of k over the runs
    int32_t n_wgs;       // chunks of all groups: workgroups of a step launch per space
    int32_t loss_wgs;    // the same of the plan by which the losses are added up: that of the sweep without an order of the points
    int32_t n_parts;     // per-chunk centroid rows of all groups
    int32_t n_lists;     // groups with tile lists
    int32_t chunk_block; // > 0: every group has the same chunks, and the step kernel's workgroup order takes this many at a time (all
                         // groups of a block of chunks, then the next block); 0: the groups have chunks of their own, of equal cost
    int32_t dp;          // padded feature count: 8, 16 or 32
    int32_t ordered;     // 1: rounds after the first run on a spatially ordered copy of the points (kmeans_order.hip), whose blocks
                         // meet only the tiles of centroids that can win there
    GroupDesc g[kMaxGroups];
    uint8_t sched[kMaxGroups];   // launch order: group indices by falling cost
};

// rows of runs k_min .. k_min+run-1
__host__ __device__ inline int32_t rows_before(int32_t k_min, int32_t run) {
    return run * k_min + run * (run - 1) / 2;
}

struct LloydGeometry {
    int threads;      // workgroup size
    int tile_points;  // points per tile
    int lds_budget;   // bytes of LDS one workgroup may use
};
LloydGeometry lloyd_geometry(int dp);
int padded_d(int d);
// LDS bytes of a group: operand tiles + centroid copy + exact-sum accumulators + fixed part
int64_t lloyd_group_lds_bytes(int dp, int d, int n_tiles, int real_rows, int copies, bool ordered);
// whether sweeps over k_min .. k_max (the waves of a sweep until the knee: the whole range) are worth an order of the points
bool sweep_wants_order(int64_t N, int32_t d, int32_t k_min, int32_t k_max, int32_t batch);
// `batch`: spaces swept by the same launches (sizes the chunks so that the whole batch gives ~512 workgroups)
int32_t make_sweep_plan(int64_t N, int32_t d, int32_t k_min, int32_t k_max, int32_t batch, bool ordered, SweepPlan *plan);

// Workspace carving for one sweep (all offsets in bytes from the workspace base, per batch element
// unless noted).  Filled by sweep_layout().
struct SweepLayout {
    int64_t colstat_part;   // per-block partial column statistics
    int64_t mind;           // fp64 [N] squared distance to the nearest chosen centre
    int64_t bsum;           // fp64 [seed blocks] block sums of mind
    int64_t near;           // uint8 [N] chain position of the nearest chosen centre
    int64_t seedthr;        // fp64 [k_max] per chosen centre: the bound below which a point's distance cannot improve
    int64_t colinfo;        // mean[32] fp32, shift[32] int32, wide[33] int32
    int64_t chain;          // int64 [k_max] seeding chain
    int64_t opA;            // per 32-row tile: fp16 pieces of the centred, -2-scaled centroids and the bf16 bias slot, in MFMA operand order
    int64_t cnmax;          // fp32 [n_runs][parts of a run] maximum of cn over the centroids of a part
    int64_t psum;           // int64 per group [n_chunks][rows of the group][d]: per-chunk changes of the fixed-point sums
    int64_t pcnt;           // int32 per group [n_chunks][rows of the group]: per-chunk changes of the member counts
    int64_t pj;             // fp64 [chunks of all groups (loss_wgs)][8] partial losses
    int64_t losum;          // int64 [total_rows][d] low-order fixed-point sums of wide columns (running)
    int64_t tot;            // int64 [total_rows][d][2] running 128-bit fixed-point sums (hi, lo)
    int64_t totcnt;         // int64 [total_rows][d] running member counts (one copy per feature)
    int64_t prev;           // uint8 per group [N rounded up to 16][8 / S]: label of every point in the last round (0xff: none yet)
    int64_t xp;             // prepared copy of the points: per block of 32, the matrix operands and squared norms (kmeans_lloyd.hip)
    // with an order of the points (plan.ordered); xp is in that order, and so are the labels of the last round
    int64_t keyinfo;        // KeyInfo
    int64_t perm, inv;      // int32 [N] place -> point, point -> place
    int64_t xs;             // fp32 [N rounded up to 64][dp] rows in that order, zero past the last feature (before: the scratch of the ordering)
    int64_t centres;        // prepared copy of the units' centres, as xp
    int64_t radius;         // fp32 [units rounded up to 32] upper bound of a unit's radius, in scaled units
    int64_t rowpos;         // uint16 [total_rows] place of a centroid among the rows of its group
    int64_t rowidx;         // uint8 [total_rows] centroid of its run that has a place
    int64_t lists;          // uint32 per group [units][16]: the tiles that a unit meets (see tile lists, kmeans_lloyd.hip)
    int64_t per_batch;      // bytes per batch element (multiple of 256)
    int64_t total;          // per_batch * batch
    int32_t seed_blocks;
    int32_t stat_blocks;
};
void sweep_layout(const SweepPlan &plan, int64_t N, int32_t d, int32_t k_max, int32_t batch, SweepLayout *L);
// words of the tile lists of all groups, as they lie in the workspace of an ordered sweep
int64_t tile_list_words(const SweepPlan &plan, int64_t N);

// the column statistics' partial results come after the seeding chain: their place serves the chain's exchange area
constexpr int kSeedExchangeBytes = 256 * 32 * 40;
constexpr int kSeedBlock = 1024;   // points per block of the seeding kernels
constexpr int kStatBlocks = 256;   // blocks of the column-statistics kernel

// ---------------------------------------------------------------------------------------------
// kernel launchers (each enqueues on `s` and returns a HIP status)
struct ForestArgs {
    int32_t n_trees, depth;
    float base;
    const int32_t *feat;
    const float *thr;
    const float *leaf;
};
hipError_t launch_gbt_score(const ForestArgs *forests_host, int32_t batch, const float *X, int64_t N, int32_t d,
                            int64_t ldx, int64_t x_batch_stride, float *score, hipStream_t s);
// what such a call of forests of one shape would take: configurations per tile, trees side by side, trees per chunk; returns whether one slice of the threads
// adds while the others move the next chunk
bool score_plan(int64_t N, int32_t d, int32_t batch, int32_t n_trees, int32_t depth, int32_t *tile, int32_t *side, int32_t *trees_per_chunk);

struct DomainArgs {
    int32_t n_knobs;
    const int32_t *offsets;
    const float *values;
};
hipError_t launch_snap(const DomainArgs *domains_host, int32_t batch, const float *C, int32_t k, int32_t d, int64_t ldc,
                       int64_t c_batch_stride, int32_t *cfg, hipStream_t s);
int32_t snap_lanes(int32_t batch, int32_t k, int32_t n_knobs);     // lanes per (centroid, knob): 64 or 1

hipError_t launch_knob_modes(const float *X, int64_t N, int64_t ldx, const DomainArgs &dm, int32_t n_total,
                             int32_t *mode_cfg, int32_t *hist, hipStream_t s);
hipError_t launch_replace_visited(int32_t *cfg, int32_t k, int32_t n_knobs, const int32_t *visited, int64_t n_visited,
                                  const int32_t *mode_cfg, int32_t *replaced, hipStream_t s);

hipError_t launch_apply_actions(const int32_t *cfg, const signed char *action, int64_t m, const DomainArgs &dm,
                                int32_t *cfg_out, float *features, int64_t ldf, hipStream_t s);

hipError_t launch_seed_chain(const float *X, int64_t N, int32_t d, int64_t ldx, int64_t x_batch_stride, int32_t batch,
                             int32_t k_max, const uint64_t *seeds_host, int64_t *chain, int64_t chain_batch_stride,
                             char *ws, const SweepLayout &L, hipStream_t s, int32_t j_begin = 0);

// spaces per launch of a chain of `spaces` (at most 64) on a chip with `cus` compute units; 0: walked in memory.  `quads`: rows can be read 16 bytes at a time
int seed_spaces_at_once(int64_t N, int32_t d, int spaces, bool quads, int k_max, int cus);
// how long the workgroups (from `first_workgroup` of each space on) of the chains launched by this host thread wait for
// each other, in ticks of the 100 MHz clock; negative: the default (see rls_bench.h)
void set_seed_wait_ticks(int32_t first_workgroup, long long ticks);

struct SweepArgs {
    const float *X;
    int64_t N;
    int32_t d;
    int64_t ldx;
    int64_t x_batch_stride;
    int32_t batch;
    int32_t iters;
    const int64_t *init_idx;      // [batch][k_max]
    int64_t init_batch_stride;
    int32_t *labels;              // [batch][n_runs][N] or null
    float *centroids;             // [batch][total_rows * d]
    double *inertia;              // [batch][n_runs]
    double *trace;                // [batch][n_runs][iters+1] or null
    int32_t *status;              // [batch]
    char *ws;                     // workspace base
    // A sweep over the same rows with the same workspace has run before (the waves of a sweep that stops at the knee):
    // the column information, and the prepared copy of the points, are still in place and are not made again.
    int32_t reuse_colstats;
    int32_t reuse_prepared;
};
// benchmark timing of the Lloyd step kernel (see rls_bench.h)
bool profile_enabled();
hipError_t profile_mark(hipStream_t s, bool begin);

hipError_t launch_sweep(const SweepPlan &plan, const SweepLayout &L, const SweepArgs &a, hipStream_t s);

// sweeps of few points: one workgroup per run, one launch (kmeans_small.hip)
bool sweep_is_small(const SweepPlan &plan, int64_t N, int32_t batch, int32_t iters, bool trace);
hipError_t launch_small_sweep(const SweepPlan &plan, const SweepLayout &L, const SweepArgs &a, hipStream_t s);

// ---- spatial order of the points (kmeans_order.hip)
constexpr int kKeyBits = 24, kKeyColBits = 10;      // of a key, and of one column at most
struct KeyInfo {
    int32_t n_cols;                          // columns that have bits of the key
    int32_t col[RLS_MAX_D], bits[RLS_MAX_D];
    int32_t first[RLS_MAX_D];                // cells of all columns before
    float lo[RLS_MAX_D], mul[RLS_MAX_D];     // cell of a value: (x - lo) mul, cut off
    unsigned char place[RLS_MAX_D][12];      // where a column's bits go, the first is the cell's highest
};
// Whole units (of 2^unit_shift places) are dealt out: unit u of the sorted sequence is unit u * step mod n_full of the order
struct OrderSpread {
    int32_t unit_shift;
    uint32_t n_full, step, back;             // back: the inverse of step
};
OrderSpread order_spread(int64_t N, int unit_shift);
int64_t order_scratch_bytes(int64_t N);
hipError_t launch_order(const float *X, int64_t N, int32_t d, int64_t ldx, int64_t x_batch_stride, int32_t batch, const int32_t *status, char *ws,
                        int64_t ws_bs, int64_t off_keyinfo, int64_t off_perm, int64_t off_inv, int64_t off_scratch, int unit_shift, hipStream_t s);
// whether the rounds after the first of such a sweep read the prepared copy of the points
bool sweep_uses_prepared(const SweepPlan &plan, int32_t iters, bool trace);

}  // namespace rls
