// An order of the points in which neighbours in memory are neighbours in space, made once per sweep.
//
// The step kernel of the sweep (kmeans_lloyd.hip) looks at 32 or 64 points at a time.  Taken from the input as it comes, such
// points lie anywhere, and every centroid of a run is the nearest of some of them; taken in this order they lie close together,
// and a ball test against their common centre leaves a few centroids.  The order has no influence on any result - labels are
// decided exactly, sums are integer sums - so it may be approximate, and it is:
//   key      a Morton key of kKeyBits bits: the bits go, one at a time, to the column whose cells are still the widest against
//            its spread (colstats_final_kernel leaves the allocation), cells are equal parts of the column's range
//   buckets  by the first kBucketBits bits: counts per slice of the points in LDS, one scan, points put down by bucket
//   pieces   of kPiece points of that sequence are sorted in LDS (bitonic).  A bucket
//            longer than a piece is sorted in parts, each of which covers the whole bucket: coarser blocks, nothing else.
//   spread   whole units are then dealt out with a constant step, so that any stretch of the order - a workgroup's chunk -
//            holds units from all over: what a unit costs (points that change their cluster, close calls, units that meet many
//            tiles) depends on where it lies, and workgroups with a region each finished at very different times.
// No global atomics (millions of them on a few thousand cells of knob data would queue up), no order left to chance but
// which points of a long bucket share a piece.
#include <numeric>
#include <type_traits>

#include "rls_internal.h"

namespace rls {

namespace {

constexpr int kBucketBits = 10;
constexpr int kBuckets = 1 << kBucketBits;
constexpr int kPiece = 4096;
constexpr int kOrderThreads = 1024;
constexpr int kMaxSlices = 256, kSlice = 1024;     // slices, and points of one at least
constexpr int kCells = 2 * (1 << kKeyColBits) + (1 << (kKeyBits - 2 * kKeyColBits));     // cells of all columns, at most

__host__ __device__ inline int slices_of(int64_t N)
{
    const int64_t s = (N + kSlice - 1) / kSlice;
    return (int)(s < kMaxSlices ? s : kMaxSlices);
}

struct OrderArgs {
    const float *X;
    int64_t N, ldx, x_bs;
    int32_t d;
    const int32_t *status;
    char *ws;
    int64_t ws_bs, off_keyinfo, off_perm, off_inv, off_pairs, off_counts;
    int32_t unit_shift;          // a unit is 2^unit_shift places
    uint32_t n_full, spread;     // whole units, and the step at which they are dealt out
};

// Keys, and how many points of each slice fall into each bucket.  The bits of a cell are spread by a table of all cells of
// all columns (at most kCells words).
__global__ void __launch_bounds__(kOrderThreads) order_count_kernel(OrderArgs a)
{
    __shared__ unsigned hist[kBuckets];
    __shared__ unsigned spread[kCells];
    __shared__ KeyInfo ki;
    __shared__ __align__(16) float4 col[RLS_MAX_D];      // per column of the rows: lowest value, cells per unit, last cell (-1: none), first cell
    const int b = blockIdx.y, tid = threadIdx.x;
    if (a.status[b] != 0) return;
    char *wsb = a.ws + (int64_t)b * a.ws_bs;
    const float *Xb = a.X + (int64_t)b * a.x_bs;
    hist[tid] = 0u;
    if (tid < (int)(sizeof(KeyInfo) / 4)) reinterpret_cast<int *>(&ki)[tid] = reinterpret_cast<const int *>(wsb + a.off_keyinfo)[tid];
    __syncthreads();
    for (int e = tid; e < kCells && ki.n_cols > 0; e += kOrderThreads) {
        int c = 0;
        while (c + 1 < ki.n_cols && ki.first[c + 1] <= e) ++c;
        const int nb = ki.bits[c], q = e - ki.first[c];
        unsigned key = 0u;
        for (int i = 0; i < nb; ++i) key |= (((unsigned)q >> (nb - 1 - i)) & 1u) << ki.place[c][i];
        spread[e] = key;
    }
    if (tid < RLS_MAX_D) col[tid] = make_float4(0.0f, 0.0f, __int_as_float(-1), 0.0f);
    __syncthreads();
    if (tid < ki.n_cols) col[ki.col[tid]] = make_float4(ki.lo[tid], ki.mul[tid], __int_as_float((1 << ki.bits[tid]) - 1), __int_as_float(ki.first[tid]));
    __syncthreads();
    unsigned *keys = reinterpret_cast<unsigned *>(wsb + a.off_perm);
    const int64_t per = (a.N + gridDim.x - 1) / gridDim.x, p0 = (int64_t)blockIdx.x * per, p1 = min(a.N, p0 + per);
    const int n_cols = __builtin_amdgcn_readfirstlane(ki.n_cols);
    // A row of 64 or 128 bytes is a line of the cache: read column by column, every load of a wave asked for 64 lines.  Rows that can be are
    // read 16 bytes at a time, all columns.  (1M x 16 39 -> 22.5 us.)
    if ((a.d & 3) == 0 && (a.ldx & 3) == 0 && (reinterpret_cast<uintptr_t>(Xb) & 15) == 0) {
        for (int64_t p = p0 + tid; p < p1; p += kOrderThreads) {
            const float4 *row = reinterpret_cast<const float4 *>(Xb + p * a.ldx);
            unsigned key = 0u;
            constexpr int U = 4;               // quads in flight at a time
            for (int q0 = 0; q0 < a.d / 4; q0 += U) {
                float4 v[U];
#pragma unroll
                for (int u = 0; u < U; ++u) v[u] = row[min(q0 + u, a.d / 4 - 1)];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (q0 + u >= a.d / 4) break;            // (same for all threads)
                    const float x[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float4 k = col[4 * (q0 + u) + i];
                        const int last = __float_as_int(k.z);
                        if (__builtin_amdgcn_readfirstlane(last) < 0) continue;
                        key |= spread[__float_as_int(k.w) + min(max((int)((x[i] - k.x) * k.y), 0), last)];
                    }
                }
            }
            keys[p] = key;
            atomicAdd(&hist[key >> (kKeyBits - kBucketBits)], 1u);
        }
    } else
    for (int64_t p = p0 + tid; p < p1; p += kOrderThreads) {
        const float *row = Xb + p * a.ldx;
        unsigned key = 0u;
        constexpr int U = 8;                   // columns in flight at a time
        for (int c0 = 0; c0 < n_cols; c0 += U) {
            float x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = row[ki.col[min(c0 + u, n_cols - 1)]];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = min(c0 + u, n_cols - 1);      // (a column taken again gives the same bits again)
                key |= spread[ki.first[c] + min(max((int)((x[u] - ki.lo[c]) * ki.mul[c]), 0), (1 << ki.bits[c]) - 1)];
            }
        }
        keys[p] = key;
        atomicAdd(&hist[key >> (kKeyBits - kBucketBits)], 1u);
    }
    __syncthreads();
    reinterpret_cast<unsigned *>(wsb + a.off_counts)[tid * kMaxSlices + (int)blockIdx.x] = hist[tid];
}

// one wave per bucket: its counts per slice become the points of the bucket in earlier slices; and their total
__global__ void __launch_bounds__(256) order_scan_kernel(OrderArgs a, int slices)
{
    const int b = blockIdx.y, lane = threadIdx.x & 63, bucket = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (a.status[b] != 0) return;
    unsigned *counts = reinterpret_cast<unsigned *>(a.ws + (int64_t)b * a.ws_bs + a.off_counts);
    unsigned *at = counts + bucket * kMaxSlices + 4 * lane;
    static_assert(kMaxSlices == 4 * 64, "four slices per lane");
    unsigned v[4], sum = 0u;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = 4 * lane + i < slices ? at[i] : 0u;
#pragma unroll
    for (int i = 0; i < 4; ++i) { const unsigned t = v[i]; v[i] = sum; sum += t; }
    unsigned incl = sum;
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned o = (unsigned)__shfl_up((int)incl, off, 64);
        if (lane >= off) incl += o;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (4 * lane + i < slices) at[i] = incl - sum + v[i];
    if (lane == 63) counts[kBuckets * kMaxSlices + bucket] = incl;
}

__global__ void __launch_bounds__(kOrderThreads) order_place_kernel(OrderArgs a)
{
    static_assert(kBuckets == kOrderThreads, "one thread per bucket");
    __shared__ unsigned next[kBuckets], wtot[kOrderThreads / 64];
    const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (a.status[b] != 0) return;
    char *wsb = a.ws + (int64_t)b * a.ws_bs;
    const unsigned *counts = reinterpret_cast<const unsigned *>(wsb + a.off_counts);
    const unsigned total = counts[kBuckets * kMaxSlices + tid], before = counts[tid * kMaxSlices + (int)blockIdx.x];
    unsigned incl = total;
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned o = (unsigned)__shfl_up((int)incl, off, 64);
        if (lane >= off) incl += o;
    }
    if (lane == 63) wtot[wave] = incl;
    __syncthreads();
    unsigned base = incl - total + before;
    for (int w = 0; w < wave; ++w) base += wtot[w];
    next[tid] = base;
    __syncthreads();
    const unsigned *keys = reinterpret_cast<const unsigned *>(wsb + a.off_perm);
    unsigned long long *pairs = reinterpret_cast<unsigned long long *>(wsb + a.off_pairs);
    const int64_t per = (a.N + gridDim.x - 1) / gridDim.x, p0 = (int64_t)blockIdx.x * per, p1 = min(a.N, p0 + per);
    for (int64_t p = p0 + tid; p < p1; p += kOrderThreads) {
        const unsigned key = keys[p];
        pairs[atomicAdd(&next[key >> (kKeyBits - kBucketBits)], 1u)] = ((unsigned long long)key << 32) | (unsigned)p;
    }
}

// bitonic sort: stage(size, stride) for size = SIZE .. kPiece and stride = size / 2 .. 1, unrolled
template <int SIZE, int STRIDE, class Stage>
__device__ __forceinline__ void merge_strides(Stage &stage)
{
    stage(std::integral_constant<int, SIZE>{}, std::integral_constant<int, STRIDE>{});
    if constexpr (STRIDE > 1) merge_strides<SIZE, STRIDE / 2>(stage);
}
template <int SIZE, class Stage>
__device__ __forceinline__ void merge_stages(Stage &stage)
{
    merge_strides<SIZE, SIZE / 2>(stage);
    if constexpr (SIZE < kPiece) merge_stages<2 * SIZE>(stage);
}

// One piece: its pairs in ascending order of the key's first 20 bits, as words (key, place within the piece); perm: place ->
// point, inv: point -> place.  A wave holds 256 neighbouring words, four per lane: exchanges over 64 and 128 places stay in a
// lane, shorter ones go through the wave's own part of LDS, without a barrier.
__global__ void __launch_bounds__(kOrderThreads) order_sort_kernel(OrderArgs a)
{
    static_assert(kPiece == 4 * kOrderThreads && kPiece <= 4096 && kKeyBits >= 20, "four words per thread, twelve bits for the place");
    __shared__ unsigned v[kPiece], point[kPiece];
    const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, w0 = (tid >> 6) * 256;
    if (a.status[b] != 0) return;
    char *wsb = a.ws + (int64_t)b * a.ws_bs;
    const unsigned long long *pairs = reinterpret_cast<const unsigned long long *>(wsb + a.off_pairs);
    const int64_t base = (int64_t)blockIdx.x * kPiece;
    unsigned x[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = w0 + 64 * e + lane;
        const unsigned long long pr = base + i < a.N ? pairs[base + i] : ~0ull;            // past the end: behind everything
        point[i] = (unsigned)pr;
        x[e] = base + i < a.N ? (unsigned)(pr >> (32 + kKeyBits - 20)) << 12 | (unsigned)i : 0xffffffffu;
    }
    auto stage = [&](auto size_c, auto stride_c) {
        constexpr int size = decltype(size_c)::value, stride = decltype(stride_c)::value;
        unsigned y[4];
        if constexpr (stride >= 256) {
            __syncthreads();
#pragma unroll
            for (int e = 0; e < 4; ++e) v[w0 + 64 * e + lane] = x[e];
            __syncthreads();
#pragma unroll
            for (int e = 0; e < 4; ++e) y[e] = v[(w0 + 64 * e + lane) ^ stride];
        } else if constexpr (stride >= 64) {
#pragma unroll
            for (int e = 0; e < 4; ++e) y[e] = x[e ^ (stride >> 6)];
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) y[e] = (unsigned)__shfl_xor((int)x[e], stride, 64);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = w0 + 64 * e + lane;
            const bool low = ((i & stride) == 0) == ((i & size) == 0);
            x[e] = low ? min(x[e], y[e]) : max(x[e], y[e]);
        }
    };
    merge_stages<2>(stage);
    int32_t *perm = reinterpret_cast<int32_t *>(wsb + a.off_perm), *inv = reinterpret_cast<int32_t *>(wsb + a.off_inv);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        int64_t at = base + w0 + 64 * e + lane;
        if (at < a.N) {
            const uint32_t unit = (uint32_t)(at >> a.unit_shift);
            if (unit < a.n_full)
                at = ((int64_t)((uint64_t)unit * a.spread % a.n_full) << a.unit_shift) | (at & ((1 << a.unit_shift) - 1));
            const unsigned p = point[x[e] & (kPiece - 1)];
            perm[at] = (int32_t)p;
            inv[p] = (int32_t)at;
        }
    }
}

}  // namespace

int64_t order_scratch_bytes(int64_t N) { return align_up(N * 8, 256) + (int64_t)kBuckets * (kMaxSlices + 1) * 4; }

OrderSpread order_spread(int64_t N, int unit_shift)
{
    OrderSpread s;
    s.unit_shift = unit_shift;
    s.n_full = (uint32_t)(N >> unit_shift);
    s.step = s.back = 1u;
    if (s.n_full < 2u) return s;
    // a step near the golden section of the number of units, without a common divisor with it
    s.step = (uint32_t)(0.6180339887498949 * (double)s.n_full) | 1u;
    while (std::gcd(s.step, s.n_full) > 1u) s.step += 2u;
    s.step %= s.n_full;
    // its inverse modulo that number (Euclid's algorithm)
    int64_t r0 = s.n_full, r1 = s.step, t0 = 0, t1 = 1;
    while (r1 > 1) {
        const int64_t q = r0 / r1, r = r0 - q * r1, t = t0 - q * t1;
        r0 = r1; r1 = r; t0 = t1; t1 = t;
    }
    s.back = (uint32_t)((t1 % (int64_t)s.n_full + s.n_full) % s.n_full);
    return s;
}

hipError_t launch_order(const float *X, int64_t N, int32_t d, int64_t ldx, int64_t x_batch_stride, int32_t batch, const int32_t *status, char *ws,
                        int64_t ws_bs, int64_t off_keyinfo, int64_t off_perm, int64_t off_inv, int64_t off_scratch, int unit_shift, hipStream_t s)
{
    OrderArgs a;
    a.X = X; a.N = N; a.d = d; a.ldx = ldx; a.x_bs = x_batch_stride;
    a.status = status; a.ws = ws; a.ws_bs = ws_bs;
    a.off_keyinfo = off_keyinfo; a.off_perm = off_perm; a.off_inv = off_inv;
    a.off_pairs = off_scratch; a.off_counts = off_scratch + align_up(N * 8, 256);
    const OrderSpread sp = order_spread(N, unit_shift);
    a.unit_shift = unit_shift; a.n_full = sp.n_full; a.spread = sp.step;
    const int slices = slices_of(N);
    const unsigned pieces = (unsigned)((N + kPiece - 1) / kPiece);
    hipLaunchKernelGGL(order_count_kernel, dim3(slices, batch), dim3(kOrderThreads), 0, s, a);
    hipLaunchKernelGGL(order_scan_kernel, dim3(kBuckets / 4, batch), dim3(256), 0, s, a, slices);
    hipLaunchKernelGGL(order_place_kernel, dim3(slices, batch), dim3(kOrderThreads), 0, s, a);
    hipLaunchKernelGGL(order_sort_kernel, dim3(pieces, batch), dim3(kOrderThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace rls
