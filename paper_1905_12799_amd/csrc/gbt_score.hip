// Tree-ensemble scoring of a trajectory of configurations (cost-model query, Sec. 4.1 of the paper).
//
// A workgroup of 1024 threads keeps a tile of P configurations in LDS, feature-major (xs[f][p]): the walk reads
// xs[feat][lane], whose bank depends on the lane alone, so these gathers never conflict.  The internal nodes of the
// forest are streamed through LDS in chunks of whole trees, each packed as (LDS address of the feature's row,
// threshold bits); the leaves stay in global memory: a tree's leaf is one 4-byte gather per configuration out of a
// block of at most 16 KB that the first-level cache holds, and it is only added a group of trees later.
//
// Large inputs take P = 1024, one configuration per thread.  Every workgroup streams the whole forest, so that is the
// cheapest tile per configuration - but 2000 configurations would fill two compute units.  Smaller inputs take tiles of
// 512 ... 64 configurations and split the trees of a chunk over the 1024 / P slices of the workgroup; the leaf values
// then meet in LDS, where one slice adds them.  Either way a configuration's leaves are added in fp32 in tree order, so
// the result does not depend on the launch shape.  (Measured: 2000 x 8, 64 trees of depth 6: 23.9 -> 9.0 us a call with
// 32 workgroups instead of two; 65,536 x 8, 256 of depth 8: 112 -> 43 us with tiles of 256; leaves in global memory
// instead of LDS, which alone bound the large ones: 8M x 32, 512 of depth 10: 14.9 -> 11.9 ms.)
//
// A step of the walk is two dependent LDS reads and four vector instructions: the walk keeps the node's LDS
// address a (node n of a tree at byte b sits at b + 8 n) and moves to child 2n + 1 + c by a <- 2 a + (8 + 8 c - b).
#include <algorithm>
#include <mutex>

#include "rls_internal.h"

namespace rls {

namespace {

constexpr int kScoreThreads = 1024;
constexpr int kScoreLds = 160 * 1024;
constexpr int kChunkNodes = 12 * kScoreThreads;                        // nodes of a chunk at most (96 KB)
// Where four slices share the trees, the first one adds the leaf values of a chunk while the others move the next chunk's nodes, if a chunk
// has many trees.  (When all moved nodes and the first then added, the others waited for it: 65,536 x 8, 256 trees of depth 8, 48 a chunk 41.2 ->
// 39.9 us, 60,000 x 16 41.9 -> 40.9; chunks of few trees are more to move than to add: 50,000 x 32, depth 10, 8 a chunk 67.6 -> 71.6.  With two
// slices one of them moves too slowly, 100,003 x 32 of depth 10 114 -> 130; with eight or more the others gain nothing, 30,000 x 32 34.9 -> 37.1.)
constexpr int kApartTile = 256, kApartTrees = 32;
// (a kernel of its own: with the choice at run time the chunks of few trees were 3% slower)
// groups of four nodes a thread carries in registers for the next chunk
constexpr int stage_quads_of(bool apart) { return apart ? 4 : 3; }
static_assert(4 * 3 * kScoreThreads >= kChunkNodes && 4 * 4 * (kScoreThreads - kApartTile) >= kChunkNodes, "a chunk fits the registers of those that move it");
constexpr int kScoreBatch = 64;                                        // forests per launch (they travel as kernel arguments)

struct ForestBatch {
    ForestArgs f[kScoreBatch];
};

// LDS is addressed by 32-bit byte addresses that the walk computes itself (the start of the dynamic block is folded into
// them once: as a pointer offset it is a link-time constant and would cost an addition per read)
typedef __attribute__((address_space(3))) unsigned char lds_byte;
__device__ inline unsigned lds_address(const void *p) { return (unsigned)(uintptr_t)(lds_byte *)p; }
typedef unsigned uint2v __attribute__((ext_vector_type(2)));
typedef unsigned uint4v __attribute__((ext_vector_type(4)));
__device__ inline uint2v lds_read_u2(unsigned a) { return *(const __attribute__((address_space(3))) uint2v *)(uintptr_t)a; }
__device__ inline float lds_read_f(unsigned a) { return *(const __attribute__((address_space(3))) float *)(uintptr_t)a; }
__device__ inline void lds_write_u2(unsigned a, uint2v v) { *(__attribute__((address_space(3))) uint2v *)(uintptr_t)a = v; }
__device__ inline void lds_write_u4(unsigned a, uint4v v) { *(__attribute__((address_space(3))) uint4v *)(uintptr_t)a = v; }

// P configurations per tile, 1024 / P slices of the trees, W trees walked side by side by a thread.
// `quads`: the forests' node arrays start at multiples of 16 bytes and the chunks at multiples of four trees, so that a
// chunk of a multiple of four trees is moved four nodes at a time.
template <int P, int W, bool APART = false>
__global__ void __launch_bounds__(kScoreThreads) gbt_score_kernel(ForestBatch fb, const float *__restrict__ Xall, int64_t N, int d, int64_t ldx,
                                                                  int64_t x_bs, float *__restrict__ score, int trees_per_chunk, int quads)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int SL = kScoreThreads / P;
    const ForestArgs f = fb.f[blockIdx.y];
    const float *const X = Xall + (int64_t)blockIdx.y * x_bs;
    const int n_int = (1 << f.depth) - 1;
    const int n_leaf = 1 << f.depth;
    float *xs = reinterpret_cast<float *>(smem);                                // [d][P]
    const unsigned xs_bytes = (unsigned)d * (unsigned)P * 4u;
    const unsigned lv_bytes = SL > 1 ? (unsigned)trees_per_chunk * (unsigned)P * 4u : 0u;

    const int tid = threadIdx.x;
    const int cfg = tid & (P - 1);
    const int slice = SL > 1 ? __builtin_amdgcn_readfirstlane(tid / P) : 0;      // P is a multiple of the wave size
    const unsigned lds0 = lds_address(smem);
    const unsigned lv_at = lds0 + xs_bytes;                                      // leaf values of a chunk [tree][P] (several slices)
    const unsigned nodes_at = lv_at + lv_bytes;                                  // nodes of a chunk [tree][n_int]
    const int64_t row = (int64_t)blockIdx.x * P + cfg;
    const bool valid = row < N;
    {
        const float *x = X + (valid ? row : 0) * ldx;
        if ((d % 4 == 0) && (ldx % 4 == 0) && ((reinterpret_cast<uintptr_t>(X) & 15) == 0)) {
            const float4 *x4 = reinterpret_cast<const float4 *>(x);
            for (int c = slice; c < d / 4; c += SL) {
                const float4 v = x4[c];
                xs[(4 * c + 0) * P + cfg] = v.x;
                xs[(4 * c + 1) * P + cfg] = v.y;
                xs[(4 * c + 2) * P + cfg] = v.z;
                xs[(4 * c + 3) * P + cfg] = v.w;
            }
        } else {
            for (int c = slice; c < d; c += SL) xs[c * P + cfg] = x[c];
        }
    }

    // The next chunk of the forest travels in registers while the current one is walked: its loads are issued
    // before the walk (offsets clamped to the chunk) and written to LDS after it.  Every offset is a 32-bit byte
    // offset from the chunk's start in its array; staging costs a few instructions per node.
    constexpr int Q = stage_quads_of(APART), E = 4 * Q, M = APART ? kScoreThreads - P : kScoreThreads;
    const int mover = APART ? tid - P : tid;                                    // (negative: a thread of the slice that adds)
    int st_feat[E];
    float st_thr[E];
    auto fetch_chunk = [&](int t0, int tc) {
        if (APART && mover < 0) return;
        const unsigned n_nodes = (unsigned)(tc * n_int);
        const char *const fc = reinterpret_cast<const char *>(f.feat + (size_t)t0 * n_int);
        const char *const hc = reinterpret_cast<const char *>(f.thr + (size_t)t0 * n_int);
        if (quads && (tc & 3) == 0) {
            const unsigned last_n = n_nodes * 4u - 16u;
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                if ((unsigned)(4 * i * M) >= n_nodes) break;        // same for the whole workgroup
                const unsigned on = min((unsigned)(mover + i * M) * 16u, last_n);
                const int4 a = *reinterpret_cast<const int4 *>(fc + on);
                const float4 h = *reinterpret_cast<const float4 *>(hc + on);
                st_feat[4 * i + 0] = a.x; st_feat[4 * i + 1] = a.y; st_feat[4 * i + 2] = a.z; st_feat[4 * i + 3] = a.w;
                st_thr[4 * i + 0] = h.x; st_thr[4 * i + 1] = h.y; st_thr[4 * i + 2] = h.z; st_thr[4 * i + 3] = h.w;
            }
        } else {
            const unsigned last_n = n_nodes * 4u - 4u;
#pragma unroll
            for (int i = 0; i < E; ++i) {
                if ((unsigned)(i * M) >= n_nodes) break;
                const unsigned on = min((unsigned)(mover + i * M) * 4u, last_n);
                st_feat[i] = *reinterpret_cast<const int *>(fc + on);
                st_thr[i] = *reinterpret_cast<const float *>(hc + on);
            }
        }
    };
    // a node in LDS: (LDS address of its feature's row of the tile, threshold bits)
    auto row_of = [&](int ft) { return lds0 + (unsigned)min(max(ft, 0), d - 1) * (unsigned)(P * 4); };
    auto store_chunk = [&](int tc) {
        if (APART && mover < 0) return;
        const unsigned nodes_end = (unsigned)(tc * n_int) * 8u;
        if (quads && (tc & 3) == 0) {
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                const unsigned g = (unsigned)(mover + i * M);
                if (g * 32u < nodes_end) {
                    uint4v lo, hi;
                    lo.x = row_of(st_feat[4 * i + 0]); lo.y = __float_as_uint(st_thr[4 * i + 0]);
                    lo.z = row_of(st_feat[4 * i + 1]); lo.w = __float_as_uint(st_thr[4 * i + 1]);
                    hi.x = row_of(st_feat[4 * i + 2]); hi.y = __float_as_uint(st_thr[4 * i + 2]);
                    hi.z = row_of(st_feat[4 * i + 3]); hi.w = __float_as_uint(st_thr[4 * i + 3]);
                    lds_write_u4(nodes_at + g * 32u, lo);
                    lds_write_u4(nodes_at + g * 32u + 16u, hi);
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < E; ++i) {
                const unsigned e = (unsigned)(mover + i * M);
                if (e * 8u < nodes_end) {
                    uint2v n;
                    n.x = row_of(st_feat[i]); n.y = __float_as_uint(st_thr[i]);
                    lds_write_u2(nodes_at + e * 8u, n);
                }
            }
        }
    };

    float sum = f.base;
    // The leaf values of the group of trees walked last, on their way: a walk is a chain of dependent LDS reads, so W
    // trees go side by side, and their leaves are picked up only when the next group has been walked.
    float pend[W];
    int pend_n = 0, pend_t = 0;                                                  // how many, and the first tree's place in the chunk
    auto take_pending = [&]() {
#pragma unroll
        for (int w = 0; w < W; ++w) {
            if (w >= pend_n) break;
            if constexpr (SL == 1) sum = sum + pend[w];
            else *(__attribute__((address_space(3))) float *)(uintptr_t)(lv_at + (unsigned)((pend_t + w) * P + cfg) * 4u) = pend[w];
        }
    };
    const unsigned cfg4 = (unsigned)cfg * 4u;
    auto walk_chunk = [&](int t0, int tc) {
        const char *const lc = reinterpret_cast<const char *>(f.leaf + (size_t)t0 * n_leaf);
        for (int t = slice * W; t < tc; t += SL * W) {
            unsigned base[W], a[W], k_left[W], k_right[W];
#pragma unroll
            for (int w = 0; w < W; ++w) {
                base[w] = nodes_at + (unsigned)min(t + w, tc - 1) * (unsigned)n_int * 8u;
                a[w] = base[w];
                k_left[w] = 8u - base[w];      // x < threshold: child 2n + 1
                k_right[w] = 16u - base[w];    // otherwise: child 2n + 2
                asm volatile("" : "+v"(k_left[w]), "+v"(k_right[w]));   // keep both as they are: one select per step
            }
            for (int lev = 0; lev < f.depth; ++lev) {
                uint2v nd[W];
#pragma unroll
                for (int w = 0; w < W; ++w) nd[w] = lds_read_u2(a[w]);
                float xv[W];
#pragma unroll
                for (int w = 0; w < W; ++w) xv[w] = lds_read_f(nd[w].x + cfg4);
#pragma unroll
                for (int w = 0; w < W; ++w) a[w] = 2u * a[w] + ((xv[w] < __uint_as_float(nd[w].y)) ? k_left[w] : k_right[w]);
            }
            take_pending();
            // leaf l of tree t + w: the walk ends at a = base + 8 (n_int + l), the leaf is element (t + w) n_leaf + l of the
            // chunk, at byte a / 2 + (4 (t + w) n_leaf - 4 n_int - base / 2): one shift and one add of a scalar
#pragma unroll
            for (int w = 0; w < W; ++w)
                pend[w] = *reinterpret_cast<const float *>(lc + ((a[w] >> 1) + (4u * (unsigned)(min(t + w, tc - 1) * n_leaf - n_int) - (base[w] >> 1))));
            pend_n = min(W, tc - t);
            pend_t = t;
        }
    };
    const int tpc = trees_per_chunk;
    fetch_chunk(0, min(tpc, f.n_trees));
    store_chunk(min(tpc, f.n_trees));
    __syncthreads();   // first chunk and xs in place
    for (int t0 = 0; t0 < f.n_trees; t0 += tpc) {
        const int tc = min(tpc, f.n_trees - t0);
        const int tc_next = min(tpc, f.n_trees - (t0 + tpc));
        if (tc_next > 0) fetch_chunk(t0 + tpc, tc_next);
        walk_chunk(t0, tc);
        if constexpr (SL > 1) {
            take_pending();
            pend_n = 0;
        }
        __syncthreads();   // every wave is done with this chunk
        if (tc_next > 0) store_chunk(tc_next);
        if constexpr (SL > 1) {
            if (slice == 0) {
                const unsigned at = lv_at + cfg4;
                // (eight reads under way at a time, added in tree order: one by one every tree waited for its read, 70 ns)
                constexpr int U = 8;
                for (int t = 0; t < tc; t += U) {
                    float v[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) v[u] = lds_read_f(at + (unsigned)(min(t + u, tc - 1) * P) * 4u);
#pragma unroll
                    for (int u = 0; u < U; ++u) sum = sum + (t + u < tc ? v[u] : -0.0f);       // (-0 changes no sum)
                }
            }
        }
        __syncthreads();
    }
    if constexpr (SL == 1) take_pending();
    if (valid && slice == 0) score[(int64_t)blockIdx.y * N + row] = sum;
}

using Kernel = void (*)(ForestBatch, const float *, int64_t, int, int64_t, int64_t, float *, int, int);

// the tiles, and the kernels of each for 8 (the largest tile only), 4, 2, 1 trees side by side
struct TileKernels {
    int tile;
    Kernel kernel[4];
};
template <int P>
constexpr TileKernels tile_kernels()
{
    return TileKernels{P, {gbt_score_kernel<P, P == kScoreThreads ? 8 : 4>, gbt_score_kernel<P, 4>, gbt_score_kernel<P, 2>, gbt_score_kernel<P, 1>}};
}
static_assert(RLS_MAX_D * kScoreThreads * 4 + ((1 << RLS_MAX_DEPTH) - 1) * 8 <= kScoreLds,
              "the deepest tree fits beside the largest tile at the largest number of features");

const TileKernels tiles[] = {tile_kernels<1024>(), tile_kernels<512>(), tile_kernels<256>(), tile_kernels<128>(), tile_kernels<64>()};

struct ScorePlan {
    const TileKernels *tile;
    int side, tpc;           // trees side by side, trees per chunk
    bool apart;              // a slice that adds while the others move the next chunk
    size_t lds;
};

// The tile: a workgroup pays for moving the whole forest through LDS and for the walks of its tile, and there are
// as many turns as the workgroups fill the 256 compute units.  Times in ns per tree, fitted to depths 4 to 10 with
// tiles of 64 to 1024: 0.15 per node moved, 70 for a tree whatever the tile, 0.032 per configuration and level
// walked, and a walk of one group of trees takes at least 100 per level.  (141,494 x 8, 145 trees of depth 7: one
// turn of 1024 takes 50 us, three of 256 take 64.)
ScorePlan plan_score(int64_t N, int32_t d, int nb, int n_trees, int depth)
{
    const int64_t n_int = ((int64_t)1 << depth) - 1;
    ScorePlan best{nullptr, 0, 0, false, 0};
    double best_ns = 0.0;
    for (const TileKernels &t : tiles) {
        const int P = t.tile, SL = kScoreThreads / P;
        const int64_t space = kScoreLds - (int64_t)d * P * 4;
        int64_t fit = std::min<int64_t>(space / (n_int * 8 + (SL > 1 ? P * 4 : 0)), kChunkNodes / n_int);
        if (fit < 1) continue;
        if (fit > n_trees) fit = n_trees;
        // (eight side by side hide more of the chains' latency where a thread walks whole chunks: 1M x 16, 512 trees of depth 5
        // 508 -> 482 us, of depth 8 794 -> 782; split over slices they leave more of a chunk's last round idle,
        // and chunks of 8 trees where 12 fit cost more than that: 6.8M x 16, 67 trees of depth 10 1141 -> 1255 us)
        const int side = SL == 1 && fit >= 8 && fit % 8 < 4 ? 8 : (fit >= 4 * SL ? 4 : (fit >= 2 * SL ? 2 : 1));
        int tpc = (int)fit;
        if (tpc > side * SL) tpc -= tpc % (side * SL);      // whole rounds of the slices ...
        if (tpc > 4) tpc -= tpc % 4;                        // ... and chunks that start at a multiple of four trees
        if (tpc < n_trees && tpc > 4 && tpc % 4 != 0) continue;
        const double turns = (double)(((N + P - 1) / P * nb + 255) / 256);
        const int busy = std::min(SL, (tpc + side - 1) / side);
        const double walk = 70.0 + std::max(0.032 * P * depth, 100.0 * depth / (busy * side));
        const double ns = turns * n_trees * (0.15 * (double)(n_int + 1) + walk);
        if (best.tile == nullptr || ns < best_ns) {
            const bool apart = P == kApartTile && side == 4 && tpc >= kApartTrees && tpc < n_trees;
            best = ScorePlan{&t, side, tpc, apart, (size_t)d * P * 4 + (size_t)tpc * (n_int * 8 + (SL > 1 ? P * 4 : 0))};
            best_ns = ns;
        }
    }
    return best;
}

}  // namespace

bool score_plan(int64_t N, int32_t d, int32_t batch, int32_t n_trees, int32_t depth, int32_t *tile, int32_t *side, int32_t *trees_per_chunk)
{
    const ScorePlan p = plan_score(N, d, std::min(batch, (int32_t)kScoreBatch), n_trees, depth);
    *tile = p.tile ? p.tile->tile : 0;
    *side = p.side;
    *trees_per_chunk = p.tpc;
    return p.apart;
}

hipError_t launch_gbt_score(const ForestArgs *forests_host, int32_t batch, const float *X, int64_t N, int32_t d,
                            int64_t ldx, int64_t x_batch_stride, float *score, hipStream_t s)
{
    static std::once_flag attr_once;
    static hipError_t attr_status = hipSuccess;
    std::call_once(attr_once, [] {
        for (const TileKernels &t : tiles)
            for (const Kernel k : t.kernel)
                if (attr_status == hipSuccess)
                    attr_status = hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, kScoreLds);
        if (attr_status == hipSuccess)
            attr_status = hipFuncSetAttribute(reinterpret_cast<const void *>(gbt_score_kernel<kApartTile, 4, true>),
                                              hipFuncAttributeMaxDynamicSharedMemorySize, kScoreLds);
    });
    if (attr_status != hipSuccess) return attr_status;
    for (int32_t b0 = 0; b0 < batch;) {
        // one launch for the spaces that follow each other with forests of one shape
        const int n_trees = forests_host[b0].n_trees, depth = forests_host[b0].depth;
        int nb = 1;
        while (b0 + nb < batch && nb < kScoreBatch && forests_host[b0 + nb].n_trees == n_trees && forests_host[b0 + nb].depth == depth) ++nb;
        ForestBatch fb;
        uintptr_t bits = 0;
        for (int i = 0; i < kScoreBatch; ++i) {
            fb.f[i] = forests_host[b0 + (i < nb ? i : 0)];
            bits |= reinterpret_cast<uintptr_t>(fb.f[i].feat) | reinterpret_cast<uintptr_t>(fb.f[i].thr);
        }
        const ScorePlan best = plan_score(N, d, nb, n_trees, depth);
        if (best.tile == nullptr) return hipErrorInvalidValue;     // depth <= 12: cannot happen
        const int quads = (best.tpc % 4 == 0 || best.tpc == n_trees) && (bits & 15) == 0;
        const Kernel kernel = best.apart ? gbt_score_kernel<kApartTile, 4, true>
                                         : best.tile->kernel[best.side == 8 ? 0 : (best.side == 4 ? 1 : (best.side == 2 ? 2 : 3))];
        const unsigned grid = (unsigned)((N + best.tile->tile - 1) / best.tile->tile);
        hipLaunchKernelGGL(kernel, dim3(grid, (unsigned)nb), dim3(kScoreThreads), best.lds, s, fb, X + (int64_t)b0 * x_batch_stride, N, (int)d,
                           ldx, x_batch_stride, score + (int64_t)b0 * N, best.tpc, quads);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        b0 += nb;
    }
    return hipSuccess;
}

}  // namespace rls
