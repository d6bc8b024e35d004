// Centroids -> valid configurations ("NextSamples = Centroids", Algorithm 1 of the paper).
// Of a knob's domain the value nearest to the centroid's coordinate, comparing |c - v| in fp64; of equal ones the lower index wins.
// A few centroids are as long as their chain of dependent reads, and a wave takes one (centroid, knob): its lanes share the domain, 256
// values under way together.  Many centroids are work, of which a wave of 64 lanes over a domain of two values does 64 times too
// much: there a thread takes one (centroid, knob), eight values under way.
#include <algorithm>

#include "rls_internal.h"

namespace rls {

namespace {

constexpr int kSnapBatch = 64;   // spaces per launch (domain descriptors travel as kernel arguments)

struct SnapArgs {
    DomainArgs dom[kSnapBatch];
};

constexpr int kSnapThreads = 256;

__global__ void __launch_bounds__(kSnapThreads) snap_kernel(SnapArgs a, const float *__restrict__ C, int k, int64_t ldc, int64_t c_batch_stride,
                                                            int32_t *__restrict__ cfg, int n_knobs_out)
{
    const DomainArgs dm = a.dom[blockIdx.y];
    const int lane = threadIdx.x & 63;
    const int e = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (kSnapThreads / 64) + (threadIdx.x >> 6)));
    if (e >= k * dm.n_knobs) return;
    const int i = e / dm.n_knobs, j = e % dm.n_knobs;
    const double c = (double)C[(int64_t)blockIdx.y * c_batch_stride + (int64_t)i * ldc + j];
    const int lo = dm.offsets[j], hi = dm.offsets[j + 1];
    double best = INFINITY;
    int arg = 0x7fffffff;                    // (none: a coordinate that is no number, or infinitely far from all values)
    constexpr int U = 4;
    for (int v0 = lo; v0 < hi; v0 += 64 * U) {
        float val[U];
#pragma unroll
        for (int u = 0; u < U; ++u) val[u] = dm.values[min(v0 + 64 * u + lane, hi - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int v = v0 + 64 * u + lane;
            const double gap = fabs(c - (double)val[u]);
            if (v < hi && gap < best) { best = gap; arg = v - lo; }      // (the lane's indices ascend)
        }
    }
    for (int off = 32; off >= 1; off >>= 1) {
        const double other = __shfl_xor(best, off, 64);
        const int oarg = __shfl_xor(arg, off, 64);
        if (other < best || (other == best && oarg < arg)) { best = other; arg = oarg; }
    }
    if (lane == 0) cfg[((int64_t)blockIdx.y * k + i) * n_knobs_out + j] = arg == 0x7fffffff ? 0 : arg;
}

// A workgroup takes as many rows at a time as it has threads for, a thread one knob of a row.
__global__ void __launch_bounds__(kSnapThreads) snap_rows_kernel(SnapArgs a, const float *__restrict__ C, int64_t k, int64_t ldc,
                                                                 int64_t c_batch_stride, int32_t *__restrict__ cfg, int n_knobs)
{
    const DomainArgs dm = a.dom[blockIdx.y];
    const int rows = kSnapThreads / n_knobs, j = threadIdx.x % n_knobs, at = threadIdx.x / n_knobs;
    if (at >= rows) return;
    const int lo = dm.offsets[j], hi = dm.offsets[j + 1];
    for (int64_t i = (int64_t)blockIdx.x * rows + at; i < k; i += (int64_t)gridDim.x * rows) {
        const double c = (double)C[(int64_t)blockIdx.y * c_batch_stride + i * ldc + j];
        double best = INFINITY;
        int arg = 0, v = lo;
        auto look = [&](float val, int place) {
            const double gap = fabs(c - (double)val);
            if (gap < best) { best = gap; arg = place - lo; }
        };
        constexpr int U = 8;
        for (; v + U <= hi; v += U) {
            float val[U];
#pragma unroll
            for (int u = 0; u < U; ++u) val[u] = dm.values[v + u];
#pragma unroll
            for (int u = 0; u < U; ++u) look(val[u], v + u);
        }
        for (; v < hi; ++v) look(dm.values[v], v);
        cfg[((int64_t)blockIdx.y * k + i) * n_knobs + j] = arg;
    }
}

// Up to this many (centroid, knob) pairs of a launch a wave takes one, beyond a thread does.  Calls with rows of 8 knobs, a thread | a wave, domains
// of 220, 40, 40, 10, 2, 2, 3, 2 values: 32 rows 11.2 | 2.8 us, 1024 14.2 | 4.5, 4096 12.9 | 10.6, 8192 11.9 | 18.8, 1M 376 | 2120; of 1000 values each
// 4096 31 | 17, 8192 31 | 30, 1M 2390 | 3510; of two 32 2.1 | 2.8, 1024 2.4 | 4.5, 4096 2.4 | 10.6, 1M 29 | 2120.  (The host does not know the domains.
// A thread that takes one value at a time: 32 rows 20 us, 1M 500.)  With a wave each 2^26 pairs would be a launch of 2^32 threads, which there is not.
constexpr int64_t kSnapWaves = 1 << 15;
constexpr unsigned kSnapBlocks = 1u << 16;       // workgroups of threads per space at most: 2^24 pairs, more are taken in turns

}  // namespace

int32_t snap_lanes(int32_t batch, int32_t k, int32_t n_knobs)
{
    return (int64_t)std::min(batch, kSnapBatch) * k * n_knobs <= kSnapWaves ? 64 : 1;
}

hipError_t launch_snap(const DomainArgs *domains_host, int32_t batch, const float *C, int32_t k, int32_t d, int64_t ldc,
                       int64_t c_batch_stride, int32_t *cfg, hipStream_t s)
{
    (void)d;
    for (int32_t b0 = 0; b0 < batch; b0 += kSnapBatch) {
        const int nb = batch - b0 < kSnapBatch ? batch - b0 : kSnapBatch;
        SnapArgs a;
        for (int b = 0; b < kSnapBatch; ++b) a.dom[b] = domains_host[b0 + (b < nb ? b : 0)];
        const int n_knobs = domains_host[b0].n_knobs;   // all spaces of a batch share n_knobs (checked by the caller)
        const float *const Cb = C + (int64_t)b0 * c_batch_stride;
        int32_t *const cb = cfg + (int64_t)b0 * k * n_knobs;
        if (snap_lanes(nb, k, n_knobs) == 64) {
            const int waves = kSnapThreads / 64;
            hipLaunchKernelGGL(snap_kernel, dim3((unsigned)((k * n_knobs + waves - 1) / waves), nb), dim3(kSnapThreads), 0, s, a, Cb, (int)k, ldc,
                               c_batch_stride, cb, n_knobs);
        } else {
            const int rows = kSnapThreads / n_knobs;
            const unsigned blocks = std::min((unsigned)(((int64_t)k + rows - 1) / rows), kSnapBlocks);
            hipLaunchKernelGGL(snap_rows_kernel, dim3(blocks, nb), dim3(kSnapThreads), 0, s, a, Cb, (int64_t)k, ldc, c_batch_stride, cb, n_knobs);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace rls
