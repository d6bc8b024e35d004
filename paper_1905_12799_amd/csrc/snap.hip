// Centroids -> valid configurations ("NextSamples = Centroids", Algorithm 1 of the paper).
// One wave per (centroid, knob): its lanes share the knob's domain and look for the value nearest to the centroid's
// coordinate, comparing |c - v| in fp64; of equal ones the lower index wins.  A call is as long as its chain of dependent reads: one
// thread per (centroid, knob), which walked the domain value by value, took 16 us for 32 centroids over domains of up to 165 values
// (4.4 now), whose 256 reads a wave has under way together.
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

}  // namespace

hipError_t launch_snap(const DomainArgs *domains_host, int32_t batch, const float *C, int32_t k, int32_t d, int64_t ldc,
                       int64_t c_batch_stride, int32_t *cfg, hipStream_t s)
{
    (void)d;
    for (int32_t b0 = 0; b0 < batch; b0 += kSnapBatch) {
        const int nb = batch - b0 < kSnapBatch ? batch - b0 : kSnapBatch;
        SnapArgs a;
        int max_knobs = 0;
        for (int b = 0; b < nb; ++b) {
            a.dom[b] = domains_host[b0 + b];
            if (a.dom[b].n_knobs > max_knobs) max_knobs = a.dom[b].n_knobs;
        }
        for (int b = nb; b < kSnapBatch; ++b) a.dom[b] = a.dom[0];
        const int n_knobs = domains_host[b0].n_knobs;   // all spaces of a batch share n_knobs (checked by the caller)
        const int threads = kSnapThreads, waves = threads / 64;
        const unsigned gx = (unsigned)((k * max_knobs + waves - 1) / waves);
        hipLaunchKernelGGL(snap_kernel, dim3(gx, nb), dim3(threads), 0, s, a, C + (int64_t)b0 * c_batch_stride, (int)k, ldc,
                           c_batch_stride, cfg + (int64_t)b0 * k * n_knobs, n_knobs);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace rls
