// k-means++ seeding chain (D^2 sampling) for the k-means runs of Algorithm 1 (Sec. 4.2 of the paper;
// the paper leaves the initialisation open, the chain is this library's choice).
//
// Step j keeps, per point, the fp64 squared distance D_i to the nearest of the j centres chosen so
// far, draws r = u_j * sum(D) with u_j from SplitMix64, and takes the first point whose running
// prefix of D exceeds r.  Distances use the direct form sum_l (x_l - c_l)^2 in fp64, ascending l,
// with separately rounded multiply and add.  Sums are hierarchical (thread -> wave -> block ->
// blocks) in a fixed order, so a chain is reproducible run to run.
//
// Two forms.  Up to about a million points the whole chain is one launch with the points in registers
// (seed_chain_kernel); a batch that does not fit together goes in parts of as many spaces as fit, where that pays
// (chain_in_parts_pays).  More points, and the other batches, are walked in memory, one update and one draw launch per centre:
// Most rows are never read after the first steps: with each point the position a_i of its nearest centre is kept, and
// when centre c is added a point with D_i <= |c_{a_i} - c|^2 / 4 cannot come closer to c than it is to c_{a_i}
// (triangle inequality: |x_i - c| >= |c_{a_i} - c| - |x_i - c_{a_i}| >= sqrt(D_i)), so D_i stays and the row is not
// fetched.  The bound carries a margin of 2^-30, far above the rounding of the fp64 sums, so every skipped point is one
// whose computed distance would not have been smaller: D, the block sums and the chain are the same with and without it.
#include <algorithm>
#include <atomic>
#include <mutex>
#include <type_traits>

#include "rls_internal.h"

namespace rls {

namespace {

__device__ inline uint64_t splitmix64(uint64_t seed, uint64_t j)
{
    uint64_t z = seed + (j + 1) * 0x9E3779B97F4A7C15ULL;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
    return z ^ (z >> 31);
}

__device__ inline double uniform01(uint64_t seed, uint64_t j)
{
    return (double)(splitmix64(seed, j) >> 11) * 0x1.0p-53;
}

// How long a workgroup of seed_chain_kernel waits for the others before it gives up, in ticks of the 100 MHz clock: 2 ms in
// its first exchange, which some workgroups may never reach while other streams hold compute units (beside a tree scoring of 1M x 16
// that fills the chip the last one arrives after 0.7 to 0.9 ms; giving up costs the chain again, 0.9 ms at 65,536 x 16 and 3.4 at
// 1M x 16 with 64 centres), then 50 ms, since from there on all are running.  Of a batch in parts each could wait that long, one after the
// other, and 64 x (262,144 x 16) has 16: once one has given up, the chip is known to be held, and those behind it wait 0.1 ms for the first exchange
// (workgroups that find the chip free are all there within 20 us).  A test may change these limits for the launches of its own host thread.
constexpr long long kArriveTicks = 200000;
constexpr long long kArriveTicksHeld = 10000;
constexpr long long kWaitTicks = 5000000;
thread_local long long t_wait_ticks = -1;          // negative: the limits above
thread_local int t_wait_from = 0;                  // first workgroup of a space that the thread's limit holds for

struct SeedList {
    uint64_t seed[64];
};

// the first centre: uniform over the points
__device__ inline int64_t first_centre(uint64_t seed, int64_t N)
{
    const int64_t first = (int64_t)(uniform01(seed, 0) * (double)N);
    return min(first, N - 1);
}

__global__ void seed_first_kernel(SeedList seeds, int b0, int64_t N, int64_t *chain, int64_t chain_batch_stride)
{
    const int b = b0 + blockIdx.x;
    if (threadIdx.x == 0) chain[(int64_t)b * chain_batch_stride] = first_centre(seeds.seed[blockIdx.x], N);
}

// inclusive scan / sum over a 1024-thread block in fixed order; `tmp` holds 17 doubles
__device__ inline double wave_inclusive_scan(double v)
{
    const int lane = threadIdx.x & 63;
    for (int off = 1; off < 64; off <<= 1) {
        const double o = __shfl_up(v, off, 64);
        if (lane >= off) v = __dadd_rn(v, o);
    }
    return v;
}

// D_i <- min(D_i, |x_i - c|^2) for the newest centre, plus one sum per block of kSeedBlock points.
// A thread owns points base + tid + 256 i; which thread sums which point, and in which order, never changes, so the
// block sums are the same in every run.  A point whose D_i is at most thr[a_i] (a quarter of the squared distance of its
// nearest centre to the newest one, written by the pick kernel) keeps D_i without a look at its row.  When rows can be
// read 16 bytes at a time, the rows still wanted of 256 points at a time travel through LDS: consecutive lanes read
// consecutive 16 bytes of the row block (every cache line is fetched by one instruction), and each thread then reads its
// row back from LDS (rows of d + 4 floats: conflict free).  D_i and a_i of the next 256 points, then the rows wanted
// among them, are requested before the arithmetic on the current ones.
// Q: 16-byte units per row when rows can be read that way (d = 4 Q, aligned), 0: rows are read element by element.
struct SeedState {
    double *mind;            // fp64 [N] squared distance to the nearest centre so far
    double *bsum;            // fp64 [seed blocks] block sums of mind
    unsigned char *near;     // [N] chain position of that nearest centre
    double *thr;             // fp64 [k_max] per earlier centre: (1 - 2^-30) / 4 of its squared distance to the newest centre
    int64_t mind_bs, bsum_bs, near_bs, thr_bs;   // batch strides, in elements
};

template <int Q>
__global__ void __launch_bounds__(256) seed_update_kernel(const float *__restrict__ X, int64_t N, int d, int64_t ldx,
                                                         int64_t x_batch_stride, const int64_t *__restrict__ chain,
                                                         int64_t chain_batch_stride, int j, SeedState st)
{
    __shared__ __align__(16) float tile[Q > 0 ? 256 * (4 * Q + 4) : 4];
    __shared__ float cs[RLS_MAX_D];
    __shared__ double thr_s[RLS_MAX_K];
    __shared__ unsigned long long need_s[2][4];
    __shared__ double wsum[4];
    const int b = blockIdx.y;
    const float *Xb = X + (int64_t)b * x_batch_stride;
    double *D = st.mind + (int64_t)b * st.mind_bs;
    unsigned char *NR = st.near + (int64_t)b * st.near_bs;
    const int newest = j - 1;                        // chain position of the centre this step adds
    const int64_t centre = chain[(int64_t)b * chain_batch_stride + newest];
    if (threadIdx.x < d) cs[threadIdx.x] = Xb[centre * ldx + threadIdx.x];
    if ((int)threadIdx.x < newest) thr_s[threadIdx.x] = st.thr[(int64_t)b * st.thr_bs + threadIdx.x];
    double local = 0.0;
    const int64_t base = (int64_t)blockIdx.x * kSeedBlock;
    constexpr int kIter = kSeedBlock / 256;
    const bool first = j == 1;                       // no distances yet: every row is read
    if constexpr (Q > 0) {
        constexpr int q = Q;                         // 16-byte units per row
        constexpr int rs = 4 * Q + 4;                // row stride of the tile, in floats
        constexpr int kMaxQ = Q;
        float stage[kMaxQ][4];
        // unit u = tid + 256 e of a row block is 16 bytes of row u / q at feature 4 (u % q)
        int urow[kMaxQ], ucol[kMaxQ];
#pragma unroll
        for (int e = 0; e < kMaxQ; ++e) {
            const int u = (int)threadIdx.x + 256 * e;
            urow[e] = u / q;
            ucol[e] = 4 * (u % q);
        }
        const int wave = (int)threadIdx.x >> 6;
        double old[kIter];
        int nr[kIter];
        bool need[kIter];
        // state of this thread's point of row block I (points past the end: never wanted)
#define RLS_SEED_STATE(I)                                                                                                \
    do {                                                                                                                 \
        const int64_t p_ = base + threadIdx.x + 256 * (I);                                                               \
        old[I] = 0.0; nr[I] = 0;                                                                                         \
        if (p_ < N && !first) { old[I] = D[p_]; nr[I] = NR[p_]; }                                                        \
    } while (0)
        // which rows of block I are wanted: one bit per point, one word per wave
#define RLS_SEED_WANT(I)                                                                                                 \
    do {                                                                                                                 \
        const int64_t p_ = base + threadIdx.x + 256 * (I);                                                               \
        need[I] = p_ < N && (first || !(old[I] <= thr_s[nr[I] & (RLS_MAX_K - 1)]));                                                        \
        const unsigned long long m_ = __ballot(need[I]);                                                                 \
        if ((threadIdx.x & 63) == 0) need_s[(I) & 1][wave] = m_;                                                         \
    } while (0)
        // (written out with constant indices: the staged rows stay in registers)
#define RLS_SEED_REQUEST(I)                                                                                              \
    do {                                                                                                                 \
        const int64_t row0_ = base + 256 * (I);                                                                          \
        _Pragma("unroll") for (int e = 0; e < kMaxQ; ++e) {                                                              \
            if ((need_s[(I) & 1][urow[e] >> 6] >> (urow[e] & 63)) & 1ull) {                                              \
                const float4 v_ = *reinterpret_cast<const float4 *>(Xb + min(row0_ + urow[e], N - 1) * ldx + ucol[e]);   \
                stage[e][0] = v_.x; stage[e][1] = v_.y; stage[e][2] = v_.z; stage[e][3] = v_.w;                          \
            }                                                                                                            \
        }                                                                                                                \
    } while (0)
#pragma unroll
        for (int e = 0; e < kMaxQ; ++e) stage[e][0] = stage[e][1] = stage[e][2] = stage[e][3] = 0.0f;
        RLS_SEED_STATE(0);
        __syncthreads();                             // cs and thr_s are there
        RLS_SEED_WANT(0);
        __syncthreads();
        RLS_SEED_REQUEST(0);
        if (kIter > 1 && base + 256 < N) RLS_SEED_STATE(1);
#pragma unroll
        for (int i = 0; i < kIter; ++i) {
            if (base + 256 * i >= N) break;          // same for the whole workgroup
            __syncthreads();                         // the tile is free
#pragma unroll
            for (int e = 0; e < kMaxQ; ++e) {
                *reinterpret_cast<float4 *>(tile + urow[e] * rs + ucol[e]) = make_float4(stage[e][0], stage[e][1], stage[e][2], stage[e][3]);
            }
            const bool more = i + 1 < kIter && base + 256 * (i + 1) < N;
            if (more) RLS_SEED_WANT(i + 1 < kIter ? i + 1 : i);
            __syncthreads();                         // the tile, and which rows of the next block are wanted
            if (more) {
                RLS_SEED_REQUEST(i + 1 < kIter ? i + 1 : i);
                if (i + 2 < kIter && base + 256 * (i + 2) < N) RLS_SEED_STATE(i + 2 < kIter ? i + 2 : i);
            }
            const int64_t p = base + threadIdx.x + 256 * i;
            if (p < N) {
                double cur = old[i];
                if (need[i]) {
                    const float *x = tile + threadIdx.x * rs;
                    double acc = 0.0;
#pragma unroll
                    for (int l = 0; l < 4 * Q; l += 4) {
                        const float4 xv = *reinterpret_cast<const float4 *>(x + l);
                        double diff = __dsub_rn((double)xv.x, (double)cs[l]);
                        acc = __dadd_rn(acc, __dmul_rn(diff, diff));
                        diff = __dsub_rn((double)xv.y, (double)cs[l + 1]);
                        acc = __dadd_rn(acc, __dmul_rn(diff, diff));
                        diff = __dsub_rn((double)xv.z, (double)cs[l + 2]);
                        acc = __dadd_rn(acc, __dmul_rn(diff, diff));
                        diff = __dsub_rn((double)xv.w, (double)cs[l + 3]);
                        acc = __dadd_rn(acc, __dmul_rn(diff, diff));
                    }
                    if (first || acc < cur) {
                        cur = acc;
                        D[p] = acc;
                        NR[p] = (unsigned char)newest;
                    }
                }
                local = __dadd_rn(local, cur);
            }
        }
#undef RLS_SEED_REQUEST
#undef RLS_SEED_WANT
#undef RLS_SEED_STATE
    } else {
        __syncthreads();
        for (int i = 0; i < kIter; ++i) {
            const int64_t p = base + threadIdx.x + 256 * i;
            if (p < N) {
                double cur = 0.0;
                bool want = true;
                if (!first) {
                    cur = D[p];
                    want = !(cur <= thr_s[NR[p] & (RLS_MAX_K - 1)]);
                }
                if (want) {
                    const float *x = Xb + p * ldx;
                    double acc = 0.0;
                    for (int l = 0; l < d; ++l) {
                        const double diff = __dsub_rn((double)x[l], (double)cs[l]);
                        acc = __dadd_rn(acc, __dmul_rn(diff, diff));
                    }
                    if (first || acc < cur) {
                        cur = acc;
                        D[p] = acc;
                        NR[p] = (unsigned char)newest;
                    }
                }
                local = __dadd_rn(local, cur);
            }
        }
    }
    // block sum in fixed order: wave butterfly-free reduction via scan's last lane, then 4 waves in order
    const double incl = wave_inclusive_scan(local);
    if ((threadIdx.x & 63) == 63) wsum[threadIdx.x >> 6] = incl;
    __syncthreads();
    if (threadIdx.x == 0)
        st.bsum[(int64_t)b * st.bsum_bs + blockIdx.x] = __dadd_rn(__dadd_rn(wsum[0], wsum[1]), __dadd_rn(wsum[2], wsum[3]));
}

// one workgroup per space: total, draw, locate the block, locate the point; then, for the update that follows, the
// bound of every earlier centre: a quarter of its squared distance to the centre just drawn, less a margin
__global__ void __launch_bounds__(1024) seed_pick_kernel(SeedList seeds, int b0, const float *__restrict__ X, int64_t N, int d,
                                                        int64_t ldx, int64_t x_batch_stride, int j, int seed_blocks,
                                                        SeedState st, int64_t *chain, int64_t chain_batch_stride)
{
    static_assert(RLS_MAX_K * 8 <= 1024 && RLS_MAX_D <= 32, "eight threads fetch one earlier centre, four features each");
    __shared__ double wtot[16];
    __shared__ double s_prefix_before;   // prefix of all blocks before the chosen block
    __shared__ int s_block;
    __shared__ int s_pick;
    __shared__ double s_total;
    __shared__ long long s_final;
    __shared__ float crow_s[RLS_MAX_K][RLS_MAX_D + 1];   // the earlier centres
    __shared__ float cnew_s[RLS_MAX_D];
    const int b = b0 + blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const double *BS = st.bsum + (int64_t)b * st.bsum_bs;
    const double *D = st.mind + (int64_t)b * st.mind_bs;
    int64_t *ch = chain + (int64_t)b * chain_batch_stride;
    const float *Xb = X + (int64_t)b * x_batch_stride;

    // rows of the centres chosen so far (positions 0 .. j-1): requested now, used at the end
    {
        const int m = tid >> 3, l0 = 4 * (tid & 7);
        if (m < j) {
            const float *row = Xb + ch[m] * ldx;
            for (int l = l0; l < l0 + 4 && l < d; ++l) crow_s[m][l] = row[l];
        }
    }

    // segment of blocks per thread
    const int per = (seed_blocks + 1023) / 1024;
    const int s0 = min(tid * per, seed_blocks), s1 = min(s0 + per, seed_blocks);
    double local = 0.0;
    for (int s = s0; s < s1; ++s) local = __dadd_rn(local, BS[s]);
    double incl = wave_inclusive_scan(local);
    if (lane == 63) wtot[wave] = incl;
    if (tid == 0) { s_block = 0x7fffffff; s_pick = 0x7fffffff; }
    __syncthreads();
    double wbase = 0.0;
    for (int w = 0; w < wave; ++w) wbase = __dadd_rn(wbase, wtot[w]);
    if (tid == 1023) s_total = __dadd_rn(wbase, incl);
    __syncthreads();
    const double S = s_total;
    if (!(S > 0.0)) {
        // every point coincides with a chosen centre: smallest index not chosen yet
        if (tid == 0) {
            int64_t pick = -1;
            for (int64_t i = 0; i < N && pick < 0; ++i) {
                bool taken = false;
                for (int m = 0; m < j; ++m) taken |= (ch[m] == i);
                if (!taken) pick = i;
            }
            s_final = pick;
        }
    } else {
        const double r = __dmul_rn(uniform01(seeds.seed[blockIdx.x], (uint64_t)j), S);
        // first block whose inclusive prefix exceeds r
        {
            double run = __dadd_rn(wbase, __dadd_rn(incl, -local));   // exclusive prefix of this thread's segment
            for (int s = s0; s < s1; ++s) {
                const double nxt = __dadd_rn(run, BS[s]);
                if (nxt > r && BS[s] > 0.0) { atomicMin(&s_block, s); break; }
                run = nxt;
            }
        }
        __syncthreads();
        int blk = s_block;
        const bool overflow = (blk == 0x7fffffff);   // r rounded up to S: take the last point with D > 0
        if (overflow) {
            __syncthreads();
            if (tid == 0) s_block = -1;
            __syncthreads();
            for (int s = s0; s < s1; ++s)
                if (BS[s] > 0.0) atomicMax(&s_block, s);
            __syncthreads();
            blk = s_block;
        }
        // exclusive prefix of the chosen block, recomputed in the same order by the thread that owns it
        if (blk >= s0 && blk < s1) {
            double run = __dadd_rn(wbase, __dadd_rn(incl, -local));
            for (int s = s0; s < blk; ++s) run = __dadd_rn(run, BS[s]);
            s_prefix_before = run;
        }
        __syncthreads();
        const double before = s_prefix_before;
        const int64_t p = (int64_t)blk * kSeedBlock + tid;
        const double v = p < N ? D[p] : 0.0;
        const double in_wave = wave_inclusive_scan(v);
        __syncthreads();
        if (lane == 63) wtot[wave] = in_wave;
        __syncthreads();
        double wb = before;
        for (int w = 0; w < wave; ++w) wb = __dadd_rn(wb, wtot[w]);
        const double prefix = __dadd_rn(wb, in_wave);
        if (!overflow) {
            if (v > 0.0 && prefix > r) atomicMin(&s_pick, tid);
            __syncthreads();
            if (s_pick == 0x7fffffff) {   // block-level and point-level rounding disagree: last positive point of the block
                __syncthreads();
                if (tid == 0) s_pick = -1;
                __syncthreads();
                if (v > 0.0) atomicMax(&s_pick, tid);
            }
        } else {
            __syncthreads();
            if (tid == 0) s_pick = -1;
            __syncthreads();
            if (v > 0.0) atomicMax(&s_pick, tid);
        }
        __syncthreads();
        if (tid == 0) s_final = (long long)blk * kSeedBlock + s_pick;
    }
    __syncthreads();
    const long long pick = s_final;
    if (tid == 0) ch[j] = pick;
    // bounds for the update with this centre (a pick outside the data, which valid arguments never give: no skipping)
    const bool inside = pick >= 0 && pick < N;
    if (tid < d) cnew_s[tid] = inside ? Xb[pick * ldx + tid] : 0.0f;
    __syncthreads();
    if (tid < j) {
        double dcc = 0.0;
        for (int l = 0; l < d; ++l) {
            const double diff = (double)crow_s[tid][l] - (double)cnew_s[l];
            dcc += diff * diff;
        }
        const double bound = dcc * (0.25 * (1.0 - 0x1.0p-30));
        st.thr[(int64_t)b * st.thr_bs + tid] = inside ? bound : -1.0;
    }
}

// ---- the chain in one launch --------------------------------------------------------------------------------------
// Up to one point per register slot of the chip (1M points at 16 features) the whole chain runs in one launch: a thread
// keeps the rows and distances of its P points in registers for all steps, and per step the G workgroups of a space
// exchange two messages through memory - every workgroup the sum of its D, then the workgroup that holds the drawn point
// that point's row and index.  What bounds a step is the latency of these two exchanges and of the scans between them:
// two launches per centre (an update of 7 to 12 us, a draw of 9 to 11 us and the ramp of each) took 17 to 23 us.
// (One launch, chains of 128: 1.4 us per centre at 2000 x 8 - a single workgroup skips the scan over the others -, 4.5 at 65,536 x 16,
// 7.2 at 1M x 16, against 13.6, 16.6 and 22.4.)
//
// A message is a word of 8 bytes that carries its own validity - the area is filled with kSlotEmpty before the launch,
// every word is written once, and a row travels as words of (step, value) - so no flags, fences or counters are needed:
// words are stored and polled with agent-scope atomics, which reach past the L2 of an XCD.
//
// No wait is unbounded: the workgroups need not be resident together (two chains on two streams may each hold half of the
// chip, a stream may be confined to a few compute units), so a workgroup that has waited too long gives up, tells the others,
// and leaves its finished word unset.  Any of them may do so in the last step, when the others already have all they need
// from it, and its distances are then missing: so seed_chain_rest_kernel, always launched behind, does the chain again
// unless every workgroup has finished.
constexpr unsigned long long kSlotEmpty = ~0ull;
constexpr int kChainWgs = 256;                                 // workgroups per space at most
constexpr int kRowWords = RLS_MAX_D + 1;                       // row, then the index
constexpr int kExRows = RLS_MAX_K * kChainWgs;                 // word offsets within the exchange area of a space
constexpr int kExDone = kExRows + RLS_MAX_K * kRowWords;        // one per workgroup: 1 when it has finished
constexpr int kExQuit = kExDone + kChainWgs;                   // kGaveUp when a workgroup has given up, kHeld when one of the part before had
constexpr int kExTicket = kExQuit + 1;                         // seed_chain_rest_kernel: the next block of points to be worked on
constexpr int kExSums = kExTicket + 1;                         //   sums of a step, one per block
constexpr int kExCount = kExSums + kChainWgs;                  //   blocks of a step that are done, one per step
constexpr int kExPick = kExCount + RLS_MAX_K;                  //   drawn index, one per step
constexpr int kExWords = kExPick + RLS_MAX_K;
constexpr unsigned long long kGaveUp = 1, kHeld = 2;
static_assert(kExWords * 8 <= kSeedExchangeBytes, "the exchange area must fit its place in the workspace");

struct ChainArgs {
    const float *X;
    int64_t N;
    int32_t d;
    int64_t ldx, x_bs;
    int32_t j_begin, k_max, groups;       // positions j_begin .. k_max - 1 are drawn by `groups` workgroups per space
    double *mind;                         // [N]: read when j_begin > 1, written at the end (a later call may go on from here)
    int64_t mind_bs;
    int64_t *chain;
    int64_t chain_bs;
    unsigned long long *ex;               // exchange area
    int64_t ex_bs;
    const unsigned long long *ex_before;  // a batch in parts: that of the part before (null: none), ...
    int32_t spaces_before;                // ... which has so many spaces
    long long wait_ticks;                 // limit of every wait in workgroups from wait_from on; negative: the default limits
    int32_t wait_from;
};

__global__ void __launch_bounds__(256) seed_begin_kernel(SeedList seeds, ChainArgs a)
{
    const int b = blockIdx.y;
    unsigned long long *ex = a.ex + (int64_t)b * a.ex_bs;
    const int t0 = blockIdx.x * 256 + threadIdx.x, step = gridDim.x * 256;
    for (int e = t0; e < a.k_max * kChainWgs; e += step)
        if (e % kChainWgs < a.groups) ex[e] = kSlotEmpty;
    for (int e = t0; e < a.k_max * kRowWords; e += step) ex[kExRows + e] = kSlotEmpty;
    int64_t *chain = a.chain + (int64_t)b * a.chain_bs;
    if (t0 < a.groups) ex[kExDone + t0] = 0ull;
    if (t0 < a.k_max) {
        ex[kExCount + t0] = 0ull;
        ex[kExPick + t0] = kSlotEmpty;
        if (t0 >= max(a.j_begin, 1)) chain[t0] = 0;
    }
    if (t0 < 64) {
        const bool held = a.ex_before != nullptr && t0 < a.spaces_before && a.ex_before[(int64_t)t0 * a.ex_bs + kExQuit] != 0ull;
        const unsigned long long any = __ballot(held);
        if (t0 == 0) {
            ex[kExQuit] = any != 0ull ? kHeld : 0ull;
            ex[kExTicket] = 0ull;
            if (a.j_begin == 0) chain[0] = first_centre(seeds.seed[b], a.N);
        }
    }
}

// lane exchanges inside rows of 16 (shift right by 1, 2, 4, 8) and across them (broadcast of lanes 15 and 31): a lane
// without a source, or in a row that is masked out, receives zero
template <int CTRL, int ROWS>
__device__ inline double dpp_or_zero(double v)
{
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, false),
                            __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, false));
}
// inclusive prefix sums over the wave; lane 63 holds the total
__device__ inline double wave_scan_dpp(double v)
{
    v = __dadd_rn(v, dpp_or_zero<0x111, 0xf>(v));
    v = __dadd_rn(v, dpp_or_zero<0x112, 0xf>(v));
    v = __dadd_rn(v, dpp_or_zero<0x114, 0xf>(v));
    v = __dadd_rn(v, dpp_or_zero<0x118, 0xf>(v));
    v = __dadd_rn(v, dpp_or_zero<0x142, 0xa>(v));
    v = __dadd_rn(v, dpp_or_zero<0x143, 0xc>(v));
    return v;
}
__device__ inline double lane_value(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane), __builtin_amdgcn_readlane(__double2loint(v), lane));
}
// one after the other
template <int P>
__device__ inline double sum_of(const double (&v)[P])
{
    double s = v[0];
#pragma unroll
    for (int i = 1; i < P; ++i) s = __dadd_rn(s, v[i]);
    return s;
}
__device__ inline double lane_before(double v) { return dpp_or_zero<0x138, 0xf>(v); }     // the value of the lane below; 0 in lane 0

// Of E values per lane, numbered lane * E + e, with exclusive prefixes that start at `before` (`incl`: inclusive prefix
// sums over the lanes): the first whose inclusive
// prefix exceeds r (a value of zero is never taken), and the prefix before it; none (r rounded up to the sum): the last
// positive one.  Same answer in every lane; -1 when no value is positive.
template <int E>
__device__ inline int wave_locate(const double (&v)[E], double incl, double before, double r, double &prefix)
{
    double run = __dadd_rn(before, lane_before(incl)), at = 0.0;
    int hit = -1, last = -1;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const double nxt = __dadd_rn(run, v[e]);
        if (v[e] > 0.0) {
            if (hit < 0 && nxt > r) { hit = e; at = run; }
            last = e;
        }
        run = nxt;
    }
    const unsigned long long hits = __ballot(hit >= 0);
    if (hits) {
        const int ln = __ffsll((long long)hits) - 1;
        prefix = lane_value(at, ln);
        return ln * E + __builtin_amdgcn_readlane(hit, ln);
    }
    const unsigned long long pos = __ballot(last >= 0);
    prefix = r;                                    // nothing below exceeds it either: the last positive value again
    if (!pos) return -1;
    const int ln = 63 - __clzll((long long)pos);
    return ln * E + __builtin_amdgcn_readlane(last, ln);
}

__device__ inline void post(unsigned long long *p, unsigned long long v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline unsigned long long peek(const unsigned long long *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Looks again and again until everything is there (`look`: the same answer in every lane); false after `limit` ticks, or
// soon after another workgroup has given up.  The clock is read before a look, so what is missing in the end is missing after the limit.
template <class Look>
__device__ inline bool wait_for(long long limit, const unsigned long long *quit, Look look)
{
    constexpr long long kUndisturbed = 2000;       // 20 us: no exchange lasts that long when all workgroups are running
    // (most waits are over within a few looks, and reading the clock takes as long as one of them)
    if (limit > kUndisturbed) {
        for (int i = 0; i < 8; ++i)
            if (look()) return true;
    }
    const long long t0 = wall_clock64();
    for (;;) {
        const long long waited = wall_clock64() - t0;
        if (look()) return true;
        if (waited > limit || (quit && waited > kUndisturbed && (peek(quit) & kGaveUp) != 0ull)) return false;
    }
}

// smallest index that is not among the j chosen ones (N >= k_max: it exists)
__device__ inline int64_t first_not_chosen(const int64_t *chosen, int j)
{
    for (int64_t i = 0;; ++i) {
        bool taken = false;
        for (int m = 0; m < j; ++m) taken |= chosen[m] == i;
        if (!taken) return i;
    }
}

// DP: padded features (a padded feature is zero on both sides and adds +0), P: points per thread.
// Where they fit, the rows are in LDS as well, as are the distances, and wave 0 alone draws: it finds the point
// among the 64 P of an entry, a wave's, reads its row and hands it out, with one barrier before and one behind.  Beyond that the wave that
// holds the entry does (and a third barrier, of the drawing workgroup only).  (64 points of a wave's per scan, rows converted to fp64
// in every step and three barriers, chains of 128: 2000 x 8 1.9 us per centre, 1.5 so, 65,536 x 16 5.0 and 4.5, 65,536 x 32 5.9 and 5.0,
// 1M x 16 8.0 and 7.4.)
__host__ __device__ constexpr bool chain_rows_in_lds(int dp, int p) { return 1024 * p * (8 + 4 * dp) <= 152 * 1024; }
// The rows come by way of LDS in either case, a wave's 64 P all at once or, where that is more than 8 KB, one half of the features
// after the other.  (A lane that reads its own rows asks for a line per row with every instruction, and with a branch around every
// feature that may not be there each load waited for the one before.  A chain of two centres at 500,009 x 16 44 -> 17 us, at
// 1,000,003 x 13 52 -> 29, at 262,144 x 32 42 -> 15; of 128 713 -> 683, 942 -> 919, 700 -> 690.)
__host__ __device__ constexpr int stage_width(int dp, int p) { return 64 * p * dp * 4 > 8192 ? dp / 2 : dp; }      // features at a time
__host__ __device__ constexpr int stage_bytes(int dp, int p) { return 1024 * p * stage_width(dp, p) * 4; }          // all waves
__host__ __device__ constexpr int chain_lds_bytes(int dp, int p) { return stage_bytes(dp, p) + (chain_rows_in_lds(dp, p) ? 1024 * p * 8 : 0); }
// where a quad of features of a staged row lies: turned from row to row, so that lanes whose rows begin at the same banks read different ones
template <int W>
__device__ inline int row_quad(int row, int q) { return row * W + 4 * (q ^ ((row * W / 64) & (W / 4 - 1))); }

// whether rows can be read 16 bytes at a time
__device__ inline bool rows_in_quads(const float *X, int d, int64_t ldx) { return (d & 3) == 0 && (ldx & 3) == 0 && (reinterpret_cast<uintptr_t>(X) & 15) == 0; }
// Features f0 .. f0 + W - 1 of 64 P rows from `first` on, zero past the last feature (past the last row its values: nobody uses them),
// read side by side by the lanes of a wave and put down in its `area`.
template <int P, int W>
__device__ inline void stage_rows(const float *X, int64_t N, int d, int64_t ldx, bool quads, int64_t first, int f0, float *area)
{
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));       // (addresses are worked out by every call: kept between two they take the registers that rows need)
    if (quads) {
        constexpr int U = P * W / 4, RU = 256 / W;             // quads per lane, rows per step
        const int q = lane % (W / 4), r0 = lane / (W / 4), f = f0 + 4 * q;
        float4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const float4 *>(X + min(first + r0 + RU * u, N - 1) * ldx + min(f, d - 4));
#pragma unroll
        for (int u = 0; u < U; ++u) *reinterpret_cast<float4 *>(area + row_quad<W>(r0 + RU * u, q)) = f < d ? v[u] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    } else {
        constexpr int U = P * W, RU = 64 / W;
        const int l = lane % W, r0 = lane / W, f = f0 + l;
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = X[min(first + r0 + RU * u, N - 1) * ldx + min(f, d - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) area[row_quad<W>(r0 + RU * u, l >> 2) + (l & 3)] = f < d ? v[u] : 0.0f;
    }
    // (what the wave's lanes have put down is read by its lanes alone, and the LDS keeps their order)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int DP, int P>
__global__ void __launch_bounds__(1024) seed_chain_kernel(SeedList seeds, ChainArgs a)
{
    constexpr bool ROWS = chain_rows_in_lds(DP, P);
    extern __shared__ __align__(16) unsigned char smem[];
    double *const D_s = reinterpret_cast<double *>(smem);                       // ROWS: distances [1024 P], then rows [1024 P][DP]
    float *const rows_s = reinterpret_cast<float *>(smem + (ROWS ? 1024 * P * 8 : 0));
    __shared__ __align__(16) double cs[DP];
    __shared__ double wsum[64];                     // sums of the 16 waves, then zeros
    __shared__ int64_t chosen[RLS_MAX_K];
    __shared__ double s_before, s_r;
    __shared__ int s_entry;                         // not ROWS: the wave to draw from, or -1 where another workgroup draws
    __shared__ int s_quit;                          // a wait of this workgroup ran out
    __shared__ int s_held;                          // a workgroup of the part before gave up
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int w = blockIdx.x, G = a.groups, b = blockIdx.y, d = a.d;
    const float *Xb = a.X + (int64_t)b * a.x_bs;
    double *mind = a.mind + (int64_t)b * a.mind_bs;
    int64_t *chain = a.chain + (int64_t)b * a.chain_bs;
    unsigned long long *ex = a.ex + (int64_t)b * a.ex_bs;
    const uint64_t seed = seeds.seed[b];
    const int j0 = a.j_begin > 1 ? a.j_begin : 1;
    const bool own_limit = w >= a.wait_from && a.wait_ticks >= 0;

    // this workgroup's points are base .. base + 1024 P - 1, P in a row belong to a thread: one scan per wave
    const int64_t base = (int64_t)w * (1024 * P);
    const bool has_points = base + 64 * P * __builtin_amdgcn_readfirstlane(wave) < a.N;     // (of this wave; the sums of the others stay zero)
    using Coord = std::conditional_t<ROWS, double, float>;      // (in fp64 where the registers hold it)
    Coord x[P][DP];
    double D[P];                                    // 0 for a point past the end: it is never drawn
    constexpr int W = stage_width(DP, P);
    float *const area = rows_s + wave * (64 * P) * W;
    const bool quads = rows_in_quads(Xb, d, a.ldx);
#pragma unroll
    for (int f0 = 0; f0 < DP; f0 += W) {
        stage_rows<P, W>(Xb, a.N, d, a.ldx, quads, base + 64 * P * wave, f0, area);
#pragma unroll
        for (int i = 0; i < P; ++i)
#pragma unroll
            for (int q = 0; q < W / 4; ++q) {
                const float4 v = *reinterpret_cast<const float4 *>(area + row_quad<W>(P * lane + i, q));
                x[i][f0 + 4 * q + 0] = v.x; x[i][f0 + 4 * q + 1] = v.y; x[i][f0 + 4 * q + 2] = v.z; x[i][f0 + 4 * q + 3] = v.w;
            }
        __builtin_amdgcn_wave_barrier();
    }
#pragma unroll
    for (int i = 0; i < P; ++i) {
        const int64_t p = base + P * tid + i;
        D[i] = a.j_begin > 1 && p < a.N ? mind[p] : 0.0;
    }
    // (a single workgroup has no seed_begin_kernel before it: the first centre is its own to draw, and nobody gives up; sweeps of
    // 100 x 8 45.6 -> 44.0 us, 2000 x 8 153.2 -> 151.3.  Asked by the size of the grid: with a.groups d_pad 32 spilled more scalars, 1.6%)
    if (gridDim.x == 1 && a.j_begin == 0) {
        if (tid == 0) chosen[0] = chain[0] = first_centre(seed, a.N);
    } else if (tid < j0) {
        chosen[tid] = chain[tid];
    }
    if (tid < 64) wsum[tid] = 0.0;
    if (tid == 0) {
        const unsigned long long quit = gridDim.x > 1 ? peek(ex + kExQuit) : 0ull;
        s_quit = (quit & kGaveUp) != 0ull;          // started when another had already given up
        s_held = (quit & kHeld) != 0ull;
    }
    __syncthreads();
    if (s_quit) return;
    if (tid < DP) cs[tid] = tid < d ? (double)Xb[chosen[j0 - 1] * a.ldx + tid] : 0.0;
    __syncthreads();

    for (int j = j0; j < a.k_max; ++j) {
        // ---- the newest centre
        if (has_points) {
            double acc[P] = {};
            constexpr int AT_ONCE = !ROWS && DP == 32 ? 8 : DP;      // features (with all 32 of both points mixed, 27 registers were spilled)
#pragma unroll
            for (int l0 = 0; l0 < DP; l0 += AT_ONCE) {
                if constexpr (AT_ONCE < DP) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < P; ++i) {
#pragma unroll
                    for (int l = l0; l < l0 + AT_ONCE; ++l) {
                        const double diff = __dsub_rn((double)x[i][l], cs[l]);
                        acc[i] = __dadd_rn(acc[i], __dmul_rn(diff, diff));
                    }
                    if (l0 + AT_ONCE < DP) continue;
                    if (base + P * tid + i < a.N && (j == 1 || acc[i] < D[i])) D[i] = acc[i];
                    if constexpr (ROWS) D_s[P * tid + i] = D[i];
                }
            }
            const double incl = wave_scan_dpp(sum_of(D));
            if (lane == 63) wsum[wave] = incl;
        }
        __syncthreads();
        // ---- total, draw, and whose point it is: wave 0 of every workgroup finds the same answer
        if (wave == 0) {
            const double u01 = uniform01(seed, (uint64_t)j);
            const double own[1] = {wsum[lane]}, own_incl = wave_scan_dpp(own[0]), total = lane_value(own_incl, 63);
            double v[4] = {0.0, 0.0, 0.0, 0.0};
            bool there = true;
            if (G > 1) {
                unsigned long long *slot = ex + j * kChainWgs;
                if (lane == 0) {
                    unsigned long long bits = (unsigned long long)__double_as_longlong(total);
                    if (bits == kSlotEmpty) bits = 0x7ff8000000000000ull;
                    post(slot + w, bits);
                }
                there = wait_for(own_limit ? a.wait_ticks : (j != j0 ? kWaitTicks : (s_held ? kArriveTicksHeld : kArriveTicks)), ex + kExQuit, [&] {
                    bool miss = false;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if (4 * lane + q < G) {
                            const unsigned long long bits = peek(slot + 4 * lane + q);
                            miss = miss || bits == kSlotEmpty;
                            v[q] = __longlong_as_double((long long)bits);
                        }
                    }
                    return __ballot(miss) == 0ull;
                });
            }
            int owner = -1, entry = 0;              // (owner -1: every point coincides with a chosen centre)
            double before = 0.0, r = 0.0;
            if (G == 1) {
                // nothing to exchange: the same draw without the scan over the workgroups
                if (total > 0.0) {
                    r = __dmul_rn(u01, total);
                    owner = w;
                    entry = max(wave_locate<1>(own, own_incl, total > r ? 0.0 : r, r, before), 0);
                }
            } else if (there) {
                const double incl = wave_scan_dpp(__dadd_rn(__dadd_rn(__dadd_rn(v[0], v[1]), v[2]), v[3])), S = lane_value(incl, 63);
                if (S > 0.0) {
                    r = __dmul_rn(u01, S);
                    owner = wave_locate<4>(v, incl, 0.0, r, before);
                    if (owner == w) {
                        double at;
                        entry = max(wave_locate<1>(own, own_incl, before, r, at), 0);
                        before = at;
                    }
                }
            }
            // ---- the drawn point: its workgroup hands out row and index
            float mine = 0.0f;
            int64_t pick = 0;
            bool have_row = true;
            if (!there) {
                have_row = false;
            } else if (owner < 0) {
                pick = first_not_chosen(chosen, j);
                if (lane < DP) mine = lane < d ? Xb[pick * a.ldx + lane] : 0.0f;
            } else if (owner == w) {
                if constexpr (ROWS) {
                    double dv[P], at;
#pragma unroll
                    for (int i = 0; i < P; ++i) dv[i] = D_s[P * (64 * entry + lane) + i];
                    const int pt = 64 * P * entry + max(wave_locate<P>(dv, wave_scan_dpp(sum_of(dv)), before, r, at), 0);
                    if (lane < DP) mine = rows_s[row_quad<W>(pt, lane >> 2) + (lane & 3)];
                    pick = min(base + pt, a.N - 1);
                    if (G > 1 && (lane < DP || lane == RLS_MAX_D))
                        post(ex + kExRows + j * kRowWords + lane, ((unsigned long long)j << 32) | (lane < DP ? __float_as_uint(mine) : (unsigned)pick));
                } else {
                    have_row = false;               // (below)
                    if (lane == 0) { s_before = before; s_r = r; }
                }
            } else {
                const bool reads = lane < DP || lane == RLS_MAX_D;
                unsigned long long bits = 0ull;
                there = wait_for(own_limit ? a.wait_ticks : kWaitTicks, ex + kExQuit, [&] {
                    if (reads) bits = peek(ex + kExRows + j * kRowWords + lane);
                    return __ballot(reads && bits == kSlotEmpty) == 0ull;
                });
                mine = __uint_as_float((unsigned)bits);
                pick = (int64_t)(unsigned)__builtin_amdgcn_readlane((int)(unsigned)bits, RLS_MAX_D);
            }
            if (have_row && lane < DP) cs[lane] = (double)mine;
            if (lane == 0) {
                chosen[j] = pick;
                if (w == 0 && have_row) chain[j] = pick;
                if constexpr (!ROWS) s_entry = there && owner == w ? entry : -1;
                if (!there) {
                    s_quit = 1;
                    post(ex + kExQuit, s_held ? kGaveUp | kHeld : kGaveUp);
                }
            }
        }
        __syncthreads();
        if (s_quit) return;                         // same for the whole workgroup
        if constexpr (!ROWS) {
            const int entry = s_entry;
            if (entry >= 0) {
                if (wave == entry) {
                    double at;
                    const int pt = __builtin_amdgcn_readfirstlane(max(wave_locate<P>(D, wave_scan_dpp(sum_of(D)), s_before, s_r, at), 0));
                    const int ln = pt / P, ii = pt % P;
                    float mine = 0.0f;
#pragma unroll
                    for (int l = 0; l < DP; ++l) {
                        float val = x[0][l];
#pragma unroll
                        for (int i = 1; i < P; ++i)
                            if (ii == i) val = x[i][l];
                        const int got = __builtin_amdgcn_readlane(__float_as_int(val), ln);
                        if (lane == l) mine = __int_as_float(got);
                    }
                    const int64_t pick = min(base + 64 * P * wave + pt, a.N - 1);
                    if (G > 1 && (lane < DP || lane == RLS_MAX_D))
                        post(ex + kExRows + j * kRowWords + lane, ((unsigned long long)j << 32) | (lane < DP ? __float_as_uint(mine) : (unsigned)pick));
                    if (lane < DP) cs[lane] = (double)mine;
                    if (lane == 0) {
                        chosen[j] = pick;
                        if (w == 0) chain[j] = pick;
                    }
                }
                __syncthreads();
            }
        }
    }
#pragma unroll
    for (int i = 0; i < P; ++i) {
        const int64_t p = base + P * tid + i;
        if (p < a.N) mind[p] = D[i];
    }
    if (tid == 0) ex[kExDone + w] = 1ull;
}

// The chain again, where a workgroup of seed_chain_kernel gave up.  It must not need its workgroups to be resident together,
// so they own no points: a step is `groups` blocks of 1024 P points, and whoever is free takes the next block by a ticket.
// A block waits for the draw of the step before, that is for blocks with smaller tickets, which workgroups hold that are
// running and wait for smaller tickets still - so whatever number of workgroups is running, every wait ends.  Who finishes
// the last block of a step draws.  The distances to the centres drawn by earlier calls are worked out again (some of them may be
// half updated).  Distances, block sums and the draw are those of seed_chain_kernel, and so is the way in which rows are read.  Rows and
// distances come from memory in every step, and between two steps lie a ticket, a count and a message: chains of 128 take 7.6 us per
// centre at 65,536 x 16, 34 at 1M x 16, 30 at 524,288 x 32, against 4.5, 7.2 and 7.5 undisturbed.  (Every lane reading its own rows, feature
// by feature: 14, 178 and 163.  One workgroup that walked all points: 631, 9970 and 8790.  All waves fencing in all three places
// instead of one wave, acquire or release: 45, 175 and 313, where 14, 55 and 167 were reached.)
constexpr int kRestWgs = 256;                      // workgroups per space at most: launched for nothing almost always
constexpr long long kRestTicks = 1000000000;       // 10 s.  Only another call that uses the same workspace at the same time can make a
                                                   // wait last that long; its results are undefined then, but it ends
template <int DP, int P>
__global__ void __launch_bounds__(1024) seed_chain_rest_kernel(SeedList seeds, ChainArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];       // staged rows
    constexpr int W = stage_width(DP, P);
    __shared__ float cs[DP];
    __shared__ double wsum[64];                    // sums of the 16 waves, then zeros
    __shared__ int64_t chosen[RLS_MAX_K];
    __shared__ int64_t s_pick;
    __shared__ double s_before, s_r;
    __shared__ int s_ticket, s_last, s_owner, s_entry;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int G = a.groups, b = blockIdx.y, d = a.d;
    unsigned long long *ex = a.ex + (int64_t)b * a.ex_bs;
    if (!__syncthreads_or(tid < G && ex[kExDone + tid] == 0ull)) return;
    const float *Xb = a.X + (int64_t)b * a.x_bs;
    double *D = a.mind + (int64_t)b * a.mind_bs;
    int64_t *chain = a.chain + (int64_t)b * a.chain_bs;
    const int j0 = a.j_begin > 1 ? a.j_begin : 1;
    if (tid < j0) chosen[tid] = chain[tid];
    if (tid < 64) wsum[tid] = 0.0;
    for (;;) {
        if (tid == 0) s_ticket = (int)__hip_atomic_fetch_add(ex + kExTicket, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        const int j = j0 + s_ticket / G, blk = s_ticket % G;
        if (j >= a.k_max) return;
        if (j > j0) {
            if (wave == 0) {
                const bool there = wait_for(kRestTicks, nullptr, [&] { return peek(ex + kExPick + j - 1) != kSlotEmpty; });
                if (lane == 0) s_last = there;
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");     // what others have written counts from the barrier on
            }
            __syncthreads();
            if (!s_last) return;
            if (tid >= j0 && tid < j) chosen[tid] = (int64_t)peek(ex + kExPick + tid);
        }
        // ---- the newest centre (the first time: all that are known)
        const int64_t base = (int64_t)blk * 1024 * P;
        for (int m = j == j0 ? 0 : j - 1; m < j; ++m) {
            __syncthreads();
            if (tid < DP) cs[tid] = tid < d ? Xb[chosen[m] * a.ldx + tid] : 0.0f;
            __syncthreads();
            double acc[P] = {};
            float *const area = reinterpret_cast<float *>(smem) + wave * (64 * P) * W;
#pragma unroll
            for (int f0 = 0; f0 < DP; f0 += W) {
                stage_rows<P, W>(Xb, a.N, d, a.ldx, rows_in_quads(Xb, d, a.ldx), base + 64 * P * wave, f0, area);
#pragma nounroll
                for (int q = 0; q < W / 4; ++q)
#pragma unroll
                    for (int i = 0; i < P; ++i) {
                        const float4 v = *reinterpret_cast<const float4 *>(area + row_quad<W>(P * lane + i, q));
                        const float x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const double diff = __dsub_rn((double)x[e], (double)cs[f0 + 4 * q + e]);
                            acc[i] = __dadd_rn(acc[i], __dmul_rn(diff, diff));
                        }
                    }
                __builtin_amdgcn_wave_barrier();
            }
            double loc = 0.0;
#pragma unroll
            for (int i = 0; i < P; ++i) {
                const int64_t p = base + P * tid + i;
                double cur = 0.0;
                if (p < a.N) {
                    cur = acc[i];
                    if (m > 0) {
                        const double old = D[p];
                        if (!(cur < old)) cur = old;
                    }
                    D[p] = cur;
                }
                loc = i == 0 ? cur : __dadd_rn(loc, cur);
            }
            const double incl = wave_scan_dpp(loc);
            if (lane == 63) wsum[wave] = incl;
        }
        __builtin_amdgcn_s_waitcnt(0x0f70);        // vmcnt(0): this wave's distances have left the compute unit ...
        __syncthreads();
        if (wave == 0) {
            const double total = lane_value(wave_scan_dpp(wsum[lane]), 63);
            if (lane == 0) {
                post(ex + kExSums + blk, (unsigned long long)__double_as_longlong(total));
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");     // ... and are there for all, with the sum, before the block counts as done
                s_last = __hip_atomic_fetch_add(ex + kExCount + j, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned long long)(G - 1);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        __syncthreads();
        if (!s_last) continue;
        // ---- the draw
        if (wave == 0) {
            double v[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (4 * lane + q < G) v[q] = __longlong_as_double((long long)peek(ex + kExSums + 4 * lane + q));
            const double incl = wave_scan_dpp(__dadd_rn(__dadd_rn(__dadd_rn(v[0], v[1]), v[2]), v[3])), S = lane_value(incl, 63);
            int owner = -1;
            double before = 0.0, r = 0.0;
            if (S > 0.0) {
                r = __dmul_rn(uniform01(seeds.seed[b], (uint64_t)j), S);
                owner = wave_locate<4>(v, incl, 0.0, r, before);
            }
            if (lane == 0) { s_owner = owner; s_before = before; s_r = r; }
        }
        __syncthreads();
        if (s_owner < 0) {
            if (tid == 0) s_pick = first_not_chosen(chosen, j);
        } else {
            const int64_t from = (int64_t)s_owner * 1024 * P;
            double loc = 0.0;
            for (int i = 0; i < P; ++i) {
                const int64_t p = from + P * tid + i;
                const double cur = p < a.N ? D[p] : 0.0;
                loc = i == 0 ? cur : __dadd_rn(loc, cur);
            }
            const double incl = wave_scan_dpp(loc);
            if (lane == 63) wsum[wave] = incl;
            __syncthreads();
            if (wave == 0) {
                const double own[1] = {wsum[lane]};
                double at;
                const int entry = max(wave_locate<1>(own, wave_scan_dpp(own[0]), s_before, s_r, at), 0);
                if (lane == 0) { s_entry = entry; s_before = at; }
            }
            __syncthreads();
            if (wave == s_entry) {
                const int64_t first = from + (int64_t)64 * P * wave;
                double v[P], at;                   // (what is not there is zero and never drawn)
#pragma unroll
                for (int i = 0; i < P; ++i) v[i] = first + P * lane + i < a.N ? D[first + P * lane + i] : 0.0;
                const int e = max(wave_locate<P>(v, wave_scan_dpp(sum_of(v)), s_before, s_r, at), 0);
                if (lane == 0) s_pick = min(first + e, a.N - 1);
            }
        }
        __syncthreads();
        if (tid == 0) {
            chain[j] = s_pick;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            post(ex + kExPick + j, (unsigned long long)s_pick);
        }
    }
}

}  // namespace

void set_seed_wait_ticks(int32_t first_workgroup, long long ticks)
{
    t_wait_ticks = ticks;
    t_wait_from = first_workgroup;
}

// compute units of the current device, asked for once per device
static int compute_units()
{
    constexpr int kMaxDevices = 64;
    static std::atomic<int> known[kMaxDevices];
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 0;
    int n = known[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        known[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

// Points per thread of seed_chain_kernel: the fewest with which the workgroups of all spaces fit the compute units one
// each (a workgroup of 1024 threads with up to 64 row registers fills one); 0: they do not fit, the points are walked in
// memory, one update and one draw per centre.  Up to 4096 points of a space stay in one workgroup, which has nothing to exchange.
static int chain_points_per_thread(int64_t N, int dp, int spaces, int cus, int *groups)
{
    const int most = 64 / dp;
    for (int p = 1; p <= most; p *= 2) {
        const int64_t g = (N + 1024 * p - 1) / (1024 * p);
        if (g > 1 && N <= 4096 && 2 * p <= most && p < 4) continue;
        if (g * spaces > cus || g > kChainWgs) continue;
        *groups = (int)g;
        return p;
    }
    return 0;
}

// Whether a chain whose spaces do not fit the chip together is faster in parts, one launch for as many spaces as do, than walked
// in memory, all spaces side by side.  A part costs 17.5 us of launches and first reads of its rows and 6.8 us a centre (the two exchanges,
// not the points); the walk 15 us a centre for its two launches and what it moves: state of nine bytes a point and the rows
// that the bounds leave, 5, 8.5 and 12.5 us a million points at 8, 16 and 32 features (a third more where rows cannot be read 16 bytes at a
// time).  The walk's figures are those of rows with structure, where most rows are left out; of others it takes up to twice as long.  Chain
// and one round of a batched sweep, walked and in parts: 64 x (262,144 x 16) knob rows, k = 32 6481 and 4721 us, k = 4 1671 and 1632, k = 2
// 1216 and 1430; 64 x (20,000 x 16), k = 32 902 and 536, k = 2 184 and 203; 16 x (1,048,576 x 16) 6269 and 4895; 64 x (131,072 x 32) 5023 and
// 4715; 6 x (300,000 x 32) 1474 and 1682; 8 x (524,288 x 32) 2725 and 2481; 2 x (2M x 8) 1309 and 754; rows without structure 64 x (262,144 x 16)
// 9137 and 4698, 64 x (262,144 x 8) 5885 and 2590, 64 x (131,072 x 32) 8348 and 4728.
// A part needs its workgroups resident together, the walk does not.  Beside another stream of tree scorings that fill the chip (256 trees x 1M, 512 x 8M,
// 2048 x 8M rows a launch) 64 x (262,144 x 16), k = 32 takes 14.5, 18.6 and 31.2 ms walked and 10.4, 15.4 and 30.1 in parts.  At the worst, with other
// streams holding the chip throughout, the first part gives up after 2 ms, each later one after 0.1, and each is drawn by tickets instead (10 to 30 us a centre).
static bool chain_in_parts_pays(int64_t points, int dp, bool quads, int parts, int centres)
{
    if (centres < 1) return false;
    const double million = (double)points * 1e-6 * (quads ? 1.0 : 4.0 / 3.0);
    const double walked = 15.0 + million * (dp == 8 ? 5.0 : (dp == 16 ? 8.5 : 12.5));
    return parts * (17.5 / centres + 6.8) < walked;
}

// How a chain is drawn: all spaces side by side, or as many at a time as the chip holds, or (0) walked in memory.
static int chain_spaces_at_once(int64_t N, int32_t d, int spaces, bool quads, int j_begin, int k_max, int cus, int *points, int *groups)
{
    const int dp = padded_d(d);
    int at_once = spaces, p = 0;
    while (at_once > 0 && (p = chain_points_per_thread(N, dp, at_once, cus, groups)) == 0) --at_once;
    if (at_once > 0 && at_once < spaces && !chain_in_parts_pays(N * spaces, dp, quads, (spaces + at_once - 1) / at_once, k_max - std::max(j_begin, 1)))
        at_once = 0;
    *points = p;
    return at_once;
}

int seed_spaces_at_once(int64_t N, int32_t d, int spaces, bool quads, int k_max, int cus)
{
    int points = 0, groups = 0;
    return chain_spaces_at_once(N, d, spaces, quads, 0, k_max, cus, &points, &groups);
}

static hipError_t launch_chain_in_one(int dp, int p, int spaces, const SeedList &sl, const ChainArgs &a, hipStream_t s)
{
    if (a.groups > 1) hipLaunchKernelGGL(seed_begin_kernel, dim3(16, spaces), dim3(256), 0, s, sl, a);
    const dim3 grid(a.groups, spaces), block(1024);
    const dim3 rest(std::min(a.groups, kRestWgs), spaces);
#define RLS_SEED_CHAIN(DPV, PV)                                                                                          \
    case DPV * 16 + PV: {                                                                                                \
        static std::once_flag once;                                                                                      \
        static hipError_t attr = hipSuccess;                                                                             \
        std::call_once(once, [] {                                                                                        \
            attr = hipFuncSetAttribute(reinterpret_cast<const void *>(seed_chain_kernel<DPV, PV>),                       \
                                       hipFuncAttributeMaxDynamicSharedMemorySize, chain_lds_bytes(DPV, PV));            \
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(seed_chain_rest_kernel<DPV, PV>),    \
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, stage_bytes(DPV, PV));  \
            if (attr == hipSuccess) attr = e;                                                                            \
        });                                                                                                              \
        if (attr != hipSuccess) return attr;                                                                             \
        hipLaunchKernelGGL((seed_chain_kernel<DPV, PV>), grid, block, chain_lds_bytes(DPV, PV), s, sl, a);               \
        if (a.groups > 1) hipLaunchKernelGGL((seed_chain_rest_kernel<DPV, PV>), rest, block, stage_bytes(DPV, PV), s, sl, a); \
    } break
    switch (dp * 16 + p) {
    RLS_SEED_CHAIN(8, 1);
    RLS_SEED_CHAIN(8, 2);
    RLS_SEED_CHAIN(8, 4);
    RLS_SEED_CHAIN(8, 8);
    RLS_SEED_CHAIN(16, 1);
    RLS_SEED_CHAIN(16, 2);
    RLS_SEED_CHAIN(16, 4);
    RLS_SEED_CHAIN(32, 1);
    RLS_SEED_CHAIN(32, 2);
    default: return hipErrorInvalidValue;
    }
#undef RLS_SEED_CHAIN
    return hipGetLastError();
}

hipError_t launch_seed_chain(const float *X, int64_t N, int32_t d, int64_t ldx, int64_t x_batch_stride, int32_t batch,
                             int32_t k_max, const uint64_t *seeds_host, int64_t *chain, int64_t chain_batch_stride,
                             char *ws, const SweepLayout &L, hipStream_t s, int32_t j_begin)
{
    // positions j_begin .. k_max-1 of the chain are produced; the distance state of an earlier call for the same
    // chain (positions 0 .. j_begin-1) must still be in the workspace
    const int32_t seed_blocks = L.seed_blocks;
    const unsigned long long *ex_before = nullptr;
    int32_t spaces_before = 0;
    for (int b0 = 0; b0 < batch; b0 += 64) {
        const int nb = batch - b0 < 64 ? batch - b0 : 64;
        SeedList sl;
        for (int i = 0; i < 64; ++i) sl.seed[i] = seeds_host[b0 + (i < nb ? i : 0)];
        char *wsb = ws + (int64_t)b0 * L.per_batch;
        if (k_max <= 1) {
            if (j_begin == 0) hipLaunchKernelGGL(seed_first_kernel, dim3(nb), dim3(64), 0, s, sl, b0, N, chain, chain_batch_stride);
            continue;
        }
        const int dp = padded_d(d);
        const bool quads = d % 4 == 0 && ldx % 4 == 0 && (nb == 1 || x_batch_stride % 4 == 0) && (reinterpret_cast<uintptr_t>(X) & 15) == 0;
        int groups = 0, p = 0;
        const int at_once = chain_spaces_at_once(N, d, nb, quads, j_begin, k_max, compute_units(), &p, &groups);
        if (at_once > 0) {
            for (int i0 = 0; i0 < nb; i0 += at_once) {
                const int64_t first = b0 + i0;
                const int spaces = std::min(at_once, nb - i0);
                SeedList part = sl;
                for (int i = 0; i < spaces; ++i) part.seed[i] = sl.seed[i0 + i];
                ChainArgs ca;
                ca.X = X + first * x_batch_stride; ca.N = N; ca.d = d; ca.ldx = ldx; ca.x_bs = x_batch_stride;
                ca.j_begin = j_begin; ca.k_max = k_max; ca.groups = groups;
                ca.mind = reinterpret_cast<double *>(ws + first * L.per_batch + L.mind); ca.mind_bs = L.per_batch / 8;
                ca.chain = chain + first * chain_batch_stride; ca.chain_bs = chain_batch_stride;
                ca.ex = reinterpret_cast<unsigned long long *>(ws + first * L.per_batch + L.colstat_part); ca.ex_bs = L.per_batch / 8;
                ca.ex_before = ex_before; ca.spaces_before = spaces_before;
                ca.wait_ticks = t_wait_ticks; ca.wait_from = t_wait_from;
                const hipError_t e = launch_chain_in_one(dp, p, spaces, part, ca, s);
                if (e != hipSuccess) return e;
                ex_before = groups > 1 ? ca.ex : nullptr;
                spaces_before = spaces;
            }
            continue;
        }
        SeedState st;
        st.mind = reinterpret_cast<double *>(wsb + L.mind); st.mind_bs = L.per_batch / 8;
        st.bsum = reinterpret_cast<double *>(wsb + L.bsum); st.bsum_bs = L.per_batch / 8;
        st.near = reinterpret_cast<unsigned char *>(wsb + L.near); st.near_bs = L.per_batch;
        st.thr = reinterpret_cast<double *>(wsb + L.seedthr); st.thr_bs = L.per_batch / 8;
        if (j_begin == 0) hipLaunchKernelGGL(seed_first_kernel, dim3(nb), dim3(64), 0, s, sl, b0, N, chain, chain_batch_stride);
        for (int j = j_begin > 1 ? j_begin : 1; j < k_max; ++j) {
            const float *Xg = X + (int64_t)b0 * x_batch_stride;
            // rows 16 bytes at a time when every space's rows allow it
            const bool vec = (d % 4 == 0) && (ldx % 4 == 0) && (x_batch_stride % 4 == 0 || nb == 1) &&
                             ((reinterpret_cast<uintptr_t>(Xg) & 15) == 0);
#define RLS_SEED_UPDATE(QV)                                                                                              \
    hipLaunchKernelGGL(seed_update_kernel<QV>, dim3(seed_blocks, nb), dim3(256), 0, s, Xg, N, (int)d, ldx,                \
                       x_batch_stride, chain + (int64_t)b0 * chain_batch_stride, chain_batch_stride, j, st)
            switch (vec ? d / 4 : 0) {
            case 1: RLS_SEED_UPDATE(1); break;
            case 2: RLS_SEED_UPDATE(2); break;
            case 3: RLS_SEED_UPDATE(3); break;
            case 4: RLS_SEED_UPDATE(4); break;
            case 5: RLS_SEED_UPDATE(5); break;
            case 6: RLS_SEED_UPDATE(6); break;
            case 7: RLS_SEED_UPDATE(7); break;
            case 8: RLS_SEED_UPDATE(8); break;
            default: RLS_SEED_UPDATE(0); break;
            }
#undef RLS_SEED_UPDATE
            hipLaunchKernelGGL(seed_pick_kernel, dim3(nb), dim3(1024), 0, s, sl, 0, Xg, N, (int)d, ldx, x_batch_stride, j,
                               (int)seed_blocks, st, chain + (int64_t)b0 * chain_batch_stride, chain_batch_stride);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace rls
