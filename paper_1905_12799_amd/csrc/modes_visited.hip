// The last loop of Algorithm 1 of the paper: samples that were visited before are replaced by mode(s_Theta),
// the configuration made of the mode of each dimension of the trajectory (Sec. 4.2).
//
// knob_hist_kernel   every workgroup keeps the domain values and a histogram over all domain entries in LDS;
//                    a thread takes whole rows of the trajectory, finds for every knob the nearest domain entry
//                    (|x - v| in fp64, first minimum wins, as in the snap kernel; a bisection when the knob's
//                    entries are sorted, of eight knobs side by side where there are few rows) and counts it with an integer LDS atomic, or per entry with a wave
//                    ballot when the knob has only a few; the workgroup then adds its counts to the global
//                    histogram (integer atomics: the result does not depend on the order).
// knob_mode_kernel   one wave per knob: first maximum of its slice of the histogram.
// visited_scan_kernel / visited_apply_kernel  workgroups compare a slice of the visited rows with up to 64 samples and
//                    flag those that are among them; flagged samples are then overwritten with the mode.
//
// A trajectory of ordinary size is a chain of dependent reads: with one bisection after the other and four rows per thread 100,003 x 16
// (domains of up to 165 values) took 30 us, and the maximum, found by a thread per knob, 17; now 15 and 4.  A large one is work instead: see kHistSideRows.
#include <algorithm>

#include "rls_internal.h"

namespace rls {

namespace {

constexpr int kMaxKnobs = RLS_MAX_D;

__global__ void fill_zero_kernel(int32_t *p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// nearest entry of vals[lo, hi) to x: |x - v| in fp64, the first minimum wins.  Any slice, by a scan.
__device__ inline int scanned_entry(const float *vals, int lo, int hi, float xf)
{
    const double x = (double)xf;
    double best = INFINITY;
    int arg = lo;
    for (int v = lo; v < hi; ++v) {
        const double gap = fabs(x - (double)vals[v]);
        if (gap < best) { best = gap; arg = v; }
    }
    return arg;
}

// The same of a slice that does not descend, by a bisection; where entries repeat, any of those that equal it.
__device__ inline int bisected_entry(const float *vals, int lo, int hi, float xf)
{
    int a = lo, b = hi;                       // first entry >= x
    while (a < b) {
        const int m = (a + b) >> 1;
        if (vals[m] < xf) a = m + 1; else b = m;
    }
    if (a == hi) return hi - 1;
    // entry below against entry at or above: the lower index wins a tie
    return a > lo && fabs((double)xf - (double)vals[a - 1]) <= fabs((double)xf - (double)vals[a]) ? a - 1 : a;
}

// what is known of a knob's entries
constexpr int kUnsorted = 1, kRepeats = 2;

// SIDE: the bisections of eight knobs side by side, a few large workgroups; else one after the other
template <bool SIDE>
__global__ void __launch_bounds__(SIDE ? 1024 : 256) knob_hist_kernel(const float *__restrict__ X, int64_t N, int64_t ldx,
                                                                      DomainArgs dm, int n_total, int32_t *__restrict__ hist)
{
    constexpr int kHistThreads = SIDE ? 1024 : 256;
    extern __shared__ __align__(16) unsigned char smem[];
    float *vals = reinterpret_cast<float *>(smem);                 // [n_total]
    int *cnt = reinterpret_cast<int *>(vals + n_total);            // [n_total]
    __shared__ int offs[kMaxKnobs + 1];
    __shared__ int traits[kMaxKnobs];
    __shared__ int begin[kMaxKnobs], span[kMaxKnobs];      // what a bisection begins with: the knob's slice; empty past the last knob and where entries descend
    const int tid = threadIdx.x, lane = tid & 63;
    for (int e = tid; e < n_total; e += kHistThreads) { vals[e] = dm.values[e]; cnt[e] = 0; }
    if (tid <= dm.n_knobs) offs[tid] = dm.offsets[tid];
    if (tid < kMaxKnobs) {
        const int j = min(tid, dm.n_knobs - 1), lo = dm.offsets[j], hi = dm.offsets[j + 1];
        traits[tid] = 0;
        begin[tid] = lo;
        span[tid] = tid < dm.n_knobs ? hi - lo : 0;
    }
    __syncthreads();
    for (int e = tid; e + 1 < n_total; e += kHistThreads) {
        if (!(vals[e] < vals[e + 1])) {
            // a descent or a repetition inside one knob's slice (not across a boundary) marks that knob
            const bool descends = vals[e + 1] < vals[e];
            for (int j = 0; j < dm.n_knobs; ++j) {
                if (e < offs[j] || e + 1 >= offs[j + 1]) continue;
                atomicOr(&traits[j], descends ? kUnsorted : kRepeats);
                if (descends) span[j] = 0;
            }
        }
    }
    __syncthreads();

    // whole waves enter the loop together (the ballots below need every lane of a wave)
    const int64_t stride = (int64_t)gridDim.x * kHistThreads;
    const int64_t rounds = (N + stride - 1) / stride;
    for (int64_t r = 0; r < rounds; ++r) {
        const int64_t i = r * stride + (int64_t)blockIdx.x * kHistThreads + tid;
        const bool valid = i < N;
        const float *row = X + (valid ? i : 0) * ldx;
        // the knob columns of the row eight at a time: all eight loads are out before the first search starts
        for (int j0 = 0; j0 < dm.n_knobs; j0 += 8) {
            float xv[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) xv[u] = row[min(j0 + u, dm.n_knobs - 1)];
            int at[8];
            if constexpr (SIDE) {
                // the first entry that is not below the value, of all eight knobs
                int left[8], most = 0;
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    at[u] = begin[j0 + u];
                    left[u] = span[j0 + u];
                    most = max(most, left[u]);
                }
                for (; most > 0; most >>= 1) {
                    float mid[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) mid[u] = vals[min(at[u] + (left[u] >> 1), n_total - 1)];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int half = left[u] >> 1;
                        const bool above = left[u] > 0 && mid[u] < xv[u];
                        at[u] = above ? at[u] + half + 1 : at[u];
                        left[u] = above ? left[u] - half - 1 : half;
                    }
                }
                // that entry against the one below it: the lower index wins a tie
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int lo = begin[j0 + u], hi = lo + span[j0 + u];
                    const float below = vals[max(at[u] - 1, 0)], here = vals[min(at[u], n_total - 1)];
                    const bool inside = at[u] > lo && at[u] < hi;
                    const bool lower = inside && fabs((double)xv[u] - (double)below) <= fabs((double)xv[u] - (double)here);
                    at[u] = at[u] < hi ? (lower ? at[u] - 1 : at[u]) : hi - 1;
                }
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int j = j0 + u;
                if (j >= dm.n_knobs) break;              // same for every lane
                const int lo = offs[j], hi = offs[j + 1], trait = traits[j];
                int arg = -1;
                if (valid) {
                    if (trait & kUnsorted) arg = scanned_entry(vals, lo, hi, xv[u]);
                    else if constexpr (SIDE) arg = at[u];
                    else arg = bisected_entry(vals, lo, hi, xv[u]);
                    if (trait == kRepeats)
                        while (arg > lo && vals[arg - 1] == vals[arg]) --arg;     // equal entries: the first of them
                }
                if (hi - lo <= 8) {
                    // few entries: most lanes would hit the same counters; count per entry with a ballot instead
                    for (int v = lo; v < hi; ++v) {
                        const int c = __popcll(__ballot(arg == v));
                        if (lane == 0 && c) atomicAdd(&cnt[v], c);
                    }
                } else if (valid) {
                    atomicAdd(&cnt[arg], 1);
                }
            }
        }
    }
    __syncthreads();
    for (int e = tid; e < n_total; e += kHistThreads)
        if (cnt[e] != 0) atomicAdd(&hist[e], cnt[e]);
}

// Up to this many rows the bisections of a row are a chain of dependent reads and go side by side; beyond it they are work, and side by side
// every knob takes as many steps as the largest domain asks for.  Calls, one after the other | side by side, domains of 220, 40, 40, 10, 2, 2, 3, 2 values:
// 100,003 rows 32 | 18 us, 1M 52 | 47, 8M 169 | 267; with a ninth knob of 40 values 1M 55 | 63, 8M 191 | 419; eight of 1000 values 1M 107 | 56; descending
// ones, which are scanned, 100,003 91 | 38, 1M 123 | 122, 8M 696 | 948.
constexpr int64_t kHistSideRows = 1 << 20;

__global__ void knob_mode_kernel(DomainArgs dm, const int32_t *__restrict__ hist, int32_t *__restrict__ mode_cfg)
{
    const int j = blockIdx.x, lane = threadIdx.x;
    const int lo = dm.offsets[j], hi = dm.offsets[j + 1];
    int most = -1, arg = 0;
    constexpr int U = 4;
    for (int v0 = lo; v0 < hi; v0 += 64 * U) {
        int count[U];
#pragma unroll
        for (int u = 0; u < U; ++u) count[u] = hist[min(v0 + 64 * u + lane, hi - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int v = v0 + 64 * u + lane;
            if (v < hi && count[u] > most) { most = count[u]; arg = v - lo; }      // (the lane's entries ascend)
        }
    }
    for (int off = 32; off >= 1; off >>= 1) {
        const int other = __shfl_xor(most, off, 64), oarg = __shfl_xor(arg, off, 64);
        if (other > most || (other == most && oarg < arg)) { most = other; arg = oarg; }
    }
    if (lane == 0) mode_cfg[j] = arg;
}

// grid (visited rows, samples): a workgroup compares its rows with up to kScanSamples samples, each row read once; most rows differ in
// the first knobs already.  What it has found it notes in LDS and hands on at the end, one word per sample: rows that repeat are
// compared no further, and no queue forms at the samples' flags.  (Rows of 8 knobs, the call with its three launches.  Flags in memory set by every
// wave that found a sample: 1M rows that all equal the 64 samples 6.0 ms, 0.17 now; where none does 36 us, 35 now.  A workgroup per sample and slice of the
// rows, which read them once for every sample: 0.09 ms and 73 us; 65,536 rows, 32 samples 8.7 us, 7.3 now.)
constexpr int kScanThreads = 256, kScanSamples = 64;

__global__ void __launch_bounds__(kScanThreads) visited_scan_kernel(const int32_t *__restrict__ cfg, int k, int n_knobs,
                                                                    const int32_t *__restrict__ visited, int64_t n_visited, int samples,
                                                                    int32_t *__restrict__ replaced)
{
    __shared__ int mine[kScanSamples * kMaxKnobs];
    __shared__ int found[kScanSamples];
    const int i0 = blockIdx.y * samples, n = min(samples, k - i0), tid = threadIdx.x;
    for (int e = tid; e < n * n_knobs; e += kScanThreads) mine[e] = cfg[(int64_t)i0 * n_knobs + e];
    if (tid < kScanSamples) found[tid] = 0;
    __syncthreads();
    volatile int *const known = found;       // (set by any wave, to the same value; seen late it costs a comparison)
    for (int64_t v = (int64_t)blockIdx.x * kScanThreads + tid; v < n_visited; v += (int64_t)gridDim.x * kScanThreads) {
        const int32_t *row = visited + v * n_knobs;
        const int last = n_knobs - 1;
        const int r0 = row[0], r1 = row[min(1, last)], r2 = row[min(2, last)], r3 = row[min(3, last)];
#pragma unroll 4       // (with two, as the compiler takes, 1M rows, 64 samples 36.2 us, 35.1 so)
        for (int i = 0; i < n; ++i) {
            const int *const m = mine + i * n_knobs;
            bool same = r0 == m[0] && r1 == m[min(1, last)] && r2 == m[min(2, last)] && r3 == m[min(3, last)];
            if (!same) continue;
            if (known[i] != 0) continue;
            for (int j = 4; j < n_knobs; ++j) same &= row[j] == m[j];
            if (same) known[i] = 1;
        }
    }
    __syncthreads();
    if (tid < n && found[tid] != 0) replaced[i0 + tid] = 1;
}

// one thread per (sample, knob): visited samples take the mode
__global__ void visited_apply_kernel(int32_t *__restrict__ cfg, int k, int n_knobs, const int32_t *__restrict__ mode_cfg,
                                     const int32_t *__restrict__ replaced)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= k * n_knobs) return;
    if (replaced[e / n_knobs]) cfg[e] = mode_cfg[e % n_knobs];
}

// Configuration updater of the search agent (Sec. 4.1 of the paper): one thread per (configuration, knob) adds the
// direction to the domain index and holds it at the domain's borders; optionally writes the knob's value as feature.
// (cfg and cfg_out may be the same array: neither is declared restrict; a thread reads its element before it writes it)
__global__ void apply_actions_kernel(const int32_t *cfg, const signed char *__restrict__ action, int64_t m,
                                     DomainArgs dm, int32_t *cfg_out, float *__restrict__ features, int64_t ldf)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= m * dm.n_knobs) return;
    const int64_t i = e / dm.n_knobs;
    const int j = (int)(e % dm.n_knobs);
    const int lo = dm.offsets[j], size = dm.offsets[j + 1] - lo;
    int a = action[e];
    a = a < -1 ? -1 : (a > 1 ? 1 : a);                 // directions only
    int v = cfg[e];
    v = v < 0 ? 0 : (v > size - 1 ? size - 1 : v);     // a configuration outside its domain is brought inside first
    v += a;
    v = v < 0 ? 0 : (v > size - 1 ? size - 1 : v);
    cfg_out[e] = v;
    if (features) features[i * ldf + j] = dm.values[lo + v];
}

}  // namespace

hipError_t launch_knob_modes(const float *X, int64_t N, int64_t ldx, const DomainArgs &dm, int32_t n_total,
                             int32_t *mode_cfg, int32_t *hist, hipStream_t s)
{
    hipLaunchKernelGGL(fill_zero_kernel, dim3((n_total + 255) / 256), dim3(256), 0, s, hist, (int)n_total);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t lds = (size_t)n_total * 8;
    if (N <= kHistSideRows) {
        // a row per thread as long as the chip has room for that, then four, then enough to fill it twice.  (Large workgroups: all add
        // their counts to the same few entries, one after the other.)
        const int64_t one = (N + 1023) / 1024;
        const int64_t blocks = std::min<int64_t>(std::max<int64_t>(std::min<int64_t>(one, 256), (one + 3) / 4), 512);
        hipLaunchKernelGGL(knob_hist_kernel<true>, dim3((unsigned)blocks), dim3(1024), lds, s, X, N, ldx, dm, (int)n_total, hist);
    } else {
        const int64_t blocks = std::min<int64_t>((N + 1023) / 1024, 2048);       // (to fill the chip a few times)
        hipLaunchKernelGGL(knob_hist_kernel<false>, dim3((unsigned)blocks), dim3(256), lds, s, X, N, ldx, dm, (int)n_total, hist);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(knob_mode_kernel, dim3((unsigned)dm.n_knobs), dim3(64), 0, s, dm, hist, mode_cfg);
    return hipGetLastError();
}

hipError_t launch_replace_visited(int32_t *cfg, int32_t k, int32_t n_knobs, const int32_t *visited, int64_t n_visited,
                                  const int32_t *mode_cfg, int32_t *replaced, hipStream_t s)
{
    hipLaunchKernelGGL(fill_zero_kernel, dim3((k + 255) / 256), dim3(256), 0, s, replaced, (int)k);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || n_visited == 0) return e;
    // a row per thread up to some 1024 workgroups in all (k is at most 65535); where there are fewer than 512, each with fewer samples
    // (1000 rows, 64 samples: four workgroups 11.1 us, 5.5 so)
    const int64_t most = std::min<int64_t>((n_visited + kScanThreads - 1) / kScanThreads, 1024);
    int samples = kScanSamples;
    while (samples > 4 && most * ((k + samples - 1) / samples) < 512) samples /= 2;
    const unsigned batches = (unsigned)((k + samples - 1) / samples);
    const unsigned rows = (unsigned)std::min<int64_t>(most, std::max(1024u / batches, 4u));
    hipLaunchKernelGGL(visited_scan_kernel, dim3(rows, batches), dim3(kScanThreads), 0, s, cfg, (int)k, (int)n_knobs, visited, n_visited,
                       samples, replaced);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(visited_apply_kernel, dim3((k * n_knobs + 255) / 256), dim3(256), 0, s, cfg, (int)k, (int)n_knobs,
                       mode_cfg, replaced);
    return hipGetLastError();
}

hipError_t launch_apply_actions(const int32_t *cfg, const signed char *action, int64_t m, const DomainArgs &dm,
                                int32_t *cfg_out, float *features, int64_t ldf, hipStream_t s)
{
    const int64_t total = m * dm.n_knobs;
    hipLaunchKernelGGL(apply_actions_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, cfg, action, m, dm, cfg_out,
                       features, ldf);
    return hipGetLastError();
}

}  // namespace rls
