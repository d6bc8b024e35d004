// Sweeps over a few thousand points: one workgroup takes a whole run, all rounds and the final pass, in one launch.
//
// With a step and a centroid launch per round such a sweep waits for launches (2000 x 8, k 1..16: 17 us a round for some 3 us
// of work in a few dozen workgroups).  Here a workgroup keeps the run's centroids, their operand rows, the exact sums, the
// labels and - if they fit - the rows in LDS and needs two barriers per round; its waves read the points' operands from the
// prepared copy, which the second-level cache holds.  The arithmetic is that of kmeans_lloyd.hip: distances on the matrix
// pipeline, close calls settled with the exact form, integer sums, means rounded once, losses added in the same order.
//
// 2000 x 8, k 1..16, 20 rounds: 96 us instead of 390, 4.6 a round.  Of a round's 11,000 cycles (with the clock read between the phases,
// which takes some 1500 of them) the waves spend 2600 on the distances of their four blocks (two blocks ahead did not help, the
// second copy of the loop's code cost as much), 1300 on close calls, 1200 on labels and moves, 1700 waiting for the wave that takes
// longest and 2000 on the new centroids.  One block per wave at a time: with two the 128 registers that 16 waves leave spilled (116 us
// against 102, as the rest was then); eight waves of 256 registers each hide less (126).
#include <algorithm>
#include <mutex>

#include "lloyd_device.h"

namespace rls {

namespace {

// (at d_pad 32 a wave takes 200 registers)
__host__ __device__ constexpr int small_threads_of(int dp) { return dp <= 16 ? 1024 : 512; }

struct SmallCarve {
    int opA, cs, sums, cnts, lows, labels, misc, jpart, rows, total;
};
__host__ __device__ inline SmallCarve small_carve(int dp, int k, int copies, int n, int parts)
{
    SmallCarve c;
    int off = 0;
    c.opA = off;  off += (k + 31) / 32 * tile_bytes_of(dp);                     // operand rows of the centroids
    c.cs = off;   off += (k * (dp + 4) * 4 + 15) / 16 * 16;                     // centroids, rows of dp + 4 floats
    c.sums = off; off += (copies * k * (dp + 1) * 8 + 15) / 16 * 16;            // fixed-point sums of the members (biased rows), all rounds
    c.cnts = off; off += (copies * k * 4 + 15) / 16 * 16;                       // members
    c.lows = off; off += k * dp * 8;                                            // low-order sums of wide columns
    c.labels = off; off += (n + 15) / 16 * 16;                                  // one byte per point
    c.misc = off; off += 1024;
    c.jpart = off; off += parts * 8;                                            // partial losses
    c.rows = (off + 15) / 16 * 16;                                              // the rows, dp floats each, if they fit
    c.total = off;
    return c;
}
__host__ __device__ inline int rows_end(const SmallCarve &c, int dp, int64_t n) { return (int)std::min<int64_t>(c.rows + n * dp * 4, 1 << 30); }
// copies of the sums: lanes that meet at one cluster are spread over them
__host__ __device__ inline int small_copies(int dp, int k)
{
    int copies = 8;
    while (copies > 1 && copies * k * (dp + 1) * 8 > 24 * 1024) copies >>= 1;
    return copies;
}

struct SmallArgs {
    const float *X;
    int64_t N, ldx, x_bs;
    int32_t d, k_min, n_runs, iters;
    const int64_t *init_idx;
    int64_t init_bs;
    float *C;
    int64_t c_bs;
    int32_t *labels;
    int64_t lab_bs;
    double *inertia;
    const int32_t *status;
    const char *colinfo;          // mean, shift, wide columns, scale (as the step kernel reads them)
    const char *xp;               // prepared copy of the points
    int64_t ws_bs;
};

// VEC: rows may be read 16 bytes at a time.  ROWS: they are kept in LDS.
template <int DP, bool VEC, bool ROWS>
__global__ void __launch_bounds__(small_threads_of(DP)) lloyd_small_kernel(SweepPlan plan, SmallArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int kSmallThreads = small_threads_of(DP), kSmallWaves = kSmallThreads / 64, NP = prep_slots_of(DP);
    constexpr int H = DP / 2, NK = ksteps_of(DP), HP = 8 * NK, NS = tile_slots_of(DP), CS = DP + 4;
    const int b = blockIdx.y;
    if (a.status[b] != 0) return;
    const int run = a.n_runs - 1 - (int)blockIdx.x, k = a.k_min + run, d = a.d;     // large runs first
    const int copies = small_copies(DP, k), n_tiles = (k + 31) / 32;
    // the group that the run has with a launch per round: its chunks give the order in which the losses are added
    int gi = 0;
    while (gi + 1 < plan.n_groups && plan.g[gi + 1].run0 <= run) ++gi;
    const int n_chunks = plan.g[gi].n_chunks, chunk_len = plan.g[gi].chunk_len, slab = 32 * slab_blocks_of(DP, plan.g[gi].S);
    constexpr int WV = step_threads_of(DP) / 64;
    const SmallCarve cv = small_carve(DP, k, copies, (int)a.N, n_chunks * WV);
    uint4 *opA_s = reinterpret_cast<uint4 *>(smem + cv.opA);
    float *cs_s = reinterpret_cast<float *>(smem + cv.cs);
    unsigned long long *sums_s = reinterpret_cast<unsigned long long *>(smem + cv.sums), *lows_s = reinterpret_cast<unsigned long long *>(smem + cv.lows);
    int *cnts_s = reinterpret_cast<int *>(smem + cv.cnts);
    unsigned char *labels_s = smem + cv.labels;
    float *mu_s = reinterpret_cast<float *>(smem + cv.misc);                  // [32]
    int *shift_s = reinterpret_cast<int *>(smem + cv.misc + 128);             // [32]
    int *pow2hi_s = reinterpret_cast<int *>(smem + cv.misc + 256);            // [32]
    int *wide_s = reinterpret_cast<int *>(smem + cv.misc + 384);              // [33]
    unsigned *cnmax_s = reinterpret_cast<unsigned *>(smem + cv.misc + 520);   // [2] largest norm of the centroids, of even and odd rounds
    double *jpart_s = reinterpret_cast<double *>(smem + cv.jpart);             // [n_chunks][WV]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, hl = lane >> 5, f0 = hl * H;
    const char *info = a.colinfo + (int64_t)b * a.ws_bs;
    const float *const Xb = a.X + (int64_t)b * a.x_bs;
    const int row0 = rows_before(a.k_min, run);
    float *const Cb = a.C + (int64_t)b * a.c_bs + (int64_t)row0 * d;
    const float scale = *reinterpret_cast<const float *>(info + kColScaleOff);
    const int kbits = key_bits(32 * n_tiles);
    int mask = key_mask(kbits);
    asm volatile("" : "+v"(mask));                  // keep the mask in a VGPR

    // ---- column information, padding rows, empty sums, the initial centroids
    if (tid < 32) {
        const int shift = reinterpret_cast<const int *>(info + 128)[tid];
        mu_s[tid] = tid < DP ? reinterpret_cast<const float *>(info)[tid] : 0.0f;
        shift_s[tid] = shift;
        pow2hi_s[tid] = (1023 + shift) << 20;
    }
    if (tid < 2) cnmax_s[tid] = 0u;
    if (tid < 33) wide_s[tid] = reinterpret_cast<const int *>(info + 256)[tid];
    {
        unsigned ph, pm, pl;
        split3(kPadNorm, ph, pm, pl);
        for (int e = tid; e < n_tiles * NS * 64; e += kSmallThreads) {
            const int sl = (e / 64) % NS, ln = e % 64;
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (sl == NS - 1) v = ln < 32 ? make_uint4(ph | (pm << 16), pl, 0u, 0u) : make_uint4(0x3f803f80u, 0x3f80u, 0u, 0u);
            opA_s[e] = v;
        }
    }
    for (int e = tid; e < copies * k * (DP + 1); e += kSmallThreads) sums_s[e] = 0ull;
    for (int e = tid; e < copies * k; e += kSmallThreads) cnts_s[e] = 0;
    for (int e = tid; e < (int)a.N; e += kSmallThreads) labels_s[e] = 0xff;
    for (int e = tid; e < k * DP; e += kSmallThreads) {
        lows_s[e] = 0ull;
        const int j = e / DP, l = e % DP;
        cs_s[j * CS + l] = l < d ? Xb[a.init_idx[(int64_t)b * a.init_bs + j] * a.ldx + l] : 0.0f;
    }
    if (ROWS) {
        float *const rows = reinterpret_cast<float *>(smem + cv.rows);
        if (VEC) {
            for (int e = tid; e < (int)a.N * (DP / 4); e += kSmallThreads) {
                const int p = e / (DP / 4), l = e % (DP / 4) * 4;
                reinterpret_cast<float4 *>(rows)[e] = l < d ? *reinterpret_cast<const float4 *>(Xb + p * a.ldx + l) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            }
        } else {
            for (int e = tid; e < (int)a.N * DP; e += kSmallThreads) rows[e] = e % DP < d ? Xb[e / DP * a.ldx + e % DP] : 0.0f;
        }
    }

    // this lane's half of a point's row, zero past the last feature
    float *const rows_s = reinterpret_cast<float *>(smem + cv.rows);
    auto half_row = [&](int p, float (&x)[H]) {
        if (ROWS) {
#pragma unroll
            for (int c4 = 0; c4 < H / 4; ++c4) {
                const float4 v = *reinterpret_cast<const float4 *>(rows_s + p * DP + f0 + 4 * c4);
                x[4 * c4 + 0] = v.x; x[4 * c4 + 1] = v.y; x[4 * c4 + 2] = v.z; x[4 * c4 + 3] = v.w;
            }
            return;
        }
        const float *row = Xb + p * a.ldx;
        if (VEC) {
#pragma unroll
            for (int c4 = 0; c4 < H / 4; ++c4) {
                float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                if (f0 + 4 * c4 < d) v = *reinterpret_cast<const float4 *>(row + f0 + 4 * c4);
                x[4 * c4 + 0] = v.x; x[4 * c4 + 1] = v.y; x[4 * c4 + 2] = v.z; x[4 * c4 + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int s = 0; s < H; ++s) x[s] = f0 + s < d ? row[f0 + s] : 0.0f;
        }
    };
    auto whole_row = [&](int p, float (&x)[DP]) {
        if (ROWS) {
#pragma unroll
            for (int l = 0; l < DP; l += 4) {
                const float4 v = *reinterpret_cast<const float4 *>(rows_s + p * DP + l);
                x[l] = v.x; x[l + 1] = v.y; x[l + 2] = v.z; x[l + 3] = v.w;
            }
            return;
        }
        const float *row = Xb + p * a.ldx;
        if (VEC) {
#pragma unroll
            for (int l = 0; l < DP; l += 4) {
                float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                if (l < d) v = *reinterpret_cast<const float4 *>(row + l);
                x[l] = v.x; x[l + 1] = v.y; x[l + 2] = v.z; x[l + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int l = 0; l < DP; ++l) x[l] = l < d ? row[l] : 0.0f;
        }
    };
    __syncthreads();                                // column information and centroids are there
    const bool any_wide = wide_s[32] != 0;

    // ---- new centroids (from the sums, unless these are the initial ones), their operand rows and norms: DP lanes that follow
    // each other have one centroid
    auto renew = [&](int t) {
        if (tid == 0) cnmax_s[(t + 1) & 1] = 0u;    // (the next one's; nobody reads it any more)
        for (int e = tid; e < (k * DP + 63) / 64 * 64; e += kSmallThreads) {
            const int j = min(e / DP, k - 1), l = e % DP;
            const bool real = e < k * DP && l < d;
            float c = cs_s[j * CS + l];
            if (t > 0) {
                unsigned long long v = 0ull;
                int cnt = 0;
#pragma unroll
                for (int cp = 0; cp < 8; ++cp) {                       // (all reads under way at once)
                    const int at = min(cp, copies - 1) * k + j;
                    const unsigned long long vs = sums_s[at * (DP + 1) + l];
                    const int cs = cnts_s[at];
                    v += cp < copies ? vs : 0ull;
                    cnt += cp < copies ? cs : 0;
                }
                const long long sum = (long long)(v - kFixBias * (unsigned long long)(long long)cnt);      // below 2^57
                double mean;
                if (!any_wide || wide_s[l] == 0) {
                    mean = ldexp((double)sum, -shift_s[l]);            // (rounded once: to the nearest, ties to even)
                } else {
                    // total = main * 2^kLowBits + low, on the scale 2^-(shift + kLowBits)
                    const long long low = (long long)lows_s[j * DP + l];
                    long long hi = sum >> 63;
                    unsigned long long lo = (unsigned long long)sum;
                    hi = (long long)(((unsigned long long)hi << kLowBits) | (lo >> (64 - kLowBits)));
                    lo = lo << kLowBits;
                    const unsigned long long nlo = lo + (unsigned long long)low;
                    hi += (low >> 63) + (nlo < lo ? 1 : 0);
                    mean = fixed128_to_double(hi, nlo, shift_s[l] + kLowBits);
                }
                if (cnt > 0) c = (float)(mean / (double)cnt);          // (no members: it stays)
            }
            const float cp = real ? fmaf(c, scale, mu_s[l]) : 0.0f;
            float nrm = cp * cp;                                       // summed over the lanes of the centroid
            nrm += __int_as_float(dpp_move<kDppSwap1>(__float_as_int(nrm)));
            nrm += __int_as_float(dpp_move<kDppSwap2>(__float_as_int(nrm)));
            nrm += __int_as_float(dpp_move<kDppHalfMirror>(__float_as_int(nrm)));
            if (DP >= 16) nrm += __int_as_float(dpp_move<kDppMirror>(__float_as_int(nrm)));
            if (DP >= 32) {
                const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(nrm), __float_as_uint(nrm), false, false);
                nrm = __uint_as_float(r[0]) + __uint_as_float(r[1]);
            }
            const float top = -wave_min_f32(-nrm);
            if (lane == 0) atomicMax(&cnmax_s[t & 1], __float_as_uint(top));
            if (!real) continue;
            cs_s[j * CS + l] = c;
            const int m = j & 31, h = l / H, sf = l % H, ks = sf >> 3, el = sf & 7;
            unsigned short ph, pl;
            split2(-2.0f * cp, ph, pl);
            unsigned short *op = reinterpret_cast<unsigned short *>(opA_s) + (j >> 5) * NS * 512;
            op[(ks * 64 + h * 32 + m) * 8 + el] = ph;
            op[((NK + ks) * 64 + h * 32 + m) * 8 + el] = pl;
            if (l == 0) {
                unsigned nh, nm, nl;
                split3(nrm, nh, nm, nl);
                unsigned short *bias = op + (2 * NK * 64 + m) * 8;
                bias[0] = (unsigned short)nh; bias[1] = (unsigned short)nm; bias[2] = (unsigned short)nl;
            }
        }
        __syncthreads();
    };
    renew(0);

    // (the bound on the error of two distances of the matrix pipeline, as in lloyd_step_kernel)
    const float eps_a = pair_error_of(DP), shrink = key_shrink(kbits);
    unsigned long long *const sums_l = sums_s + (lane & (copies - 1)) * k * (DP + 1);
    int *const cnts_l = cnts_s + (lane & (copies - 1)) * k;
    const int n_blocks = (int)((a.N + 31) / 32);
    const uint4 *const xp = reinterpret_cast<const uint4 *>(a.xp + (int64_t)b * a.ws_bs);
    uint4 px[NP];                                   // operands and norms of the block on its way
    uint2 pn;
    auto fetch = [&](int blk) {
        const uint4 *bp = xp + min(blk, n_blocks - 1) * prep_block_u4_of(DP);
#pragma unroll
        for (int sl = 0; sl < NP; ++sl) px[sl] = bp[sl * 64 + lane];
        pn = reinterpret_cast<const uint2 *>(bp + NP * 64)[n];
    };
    fetch(wave);
    for (int t = 0; t <= a.iters; ++t) {
        const bool last = t == a.iters;
        const float tol_run = eps_a * __uint_as_float(cnmax_s[t & 1]) + kTolFloor;
        for (int blk = wave; blk < n_blocks; blk += kSmallWaves) {
            f16x8 bx[2][NK];
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) {
                bx[0][ks] = as_f16x8(px[ks]);
                bx[1][ks] = as_f16x8(px[NK + ks]);
            }
            const uint2 norm = pn;
            const bf16x8 bb = hl ? as_bf16x8(make_uint4(norm.x, norm.y, 0u, 0u)) : as_bf16x8(make_uint4(0x3f803f80u, 0x3f80u, 0u, 0u));
            int k1 = kBigKey, k2 = kBigKey;
            fetch(blk + kSmallWaves < n_blocks ? blk + kSmallWaves : wave);       // (at the end: the next round's first block)
            for (int tile = 0; tile < n_tiles; ++tile) {
                uint4 op[NS];
#pragma unroll
                for (int sl = 0; sl < NS; ++sl) op[sl] = opA_s[(tile * NS + sl) * 64 + lane];
                floatx16 acc = floatx16{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
                for (int ks = 0; ks < NK; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(op[NK + ks]), bx[0][ks], acc, 0, 0, 0);
#pragma unroll
                for (int ks = 0; ks < NK; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(op[ks]), bx[1][ks], acc, 0, 0, 0);
#pragma unroll
                for (int ks = 0; ks < NK; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(op[ks]), bx[0][ks], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(op[2 * NK]), bb, acc, 0, 0, 0);
                // (row 8 q + 4 h + e of a tile is centroid 32 tile + 8 q + 4 h + e: result 4 q + e of half-wave h)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (q > 0 && 32 * tile + 8 * q >= k) continue;                // eight rows of padding
                    int idx[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        idx[e] = 32 * tile + 8 * q + e;
                        asm("" : "+s"(idx[e]));
                    }
#pragma unroll
                    for (int e = 0; e < 4; e += 2)
                        insert2x2(pack_key(acc[4 * q + e], mask, idx[e]), pack_key(acc[4 * q + e + 1], mask, idx[e + 1]), k1, k2);
                }
            }
            const int p = 32 * blk + n, pc = min(p, (int)a.N - 1);
            const bool valid = p < (int)a.N;
            const int was = labels_s[pc];
            // the run spans both half-waves: add the half bit to the index, then merge with the partner lane
            k1 |= hl << 2;
            {
                const int o1 = xchg32(k1), o2 = xchg32(k2);
                insert2(o1, k1, k2);
                insert2(o2, k1, k2);
            }
            const float xn = (__uint_as_float(norm.x << 16) + __uint_as_float(norm.x & 0xffff0000u)) + __uint_as_float(norm.y << 16);
            const bool close = valid && !(fmaf(__int_as_float(k2), shrink, -__int_as_float(k1)) > fmaf(eps_a, xn, tol_run));
            int label = k1 & ~mask;
            unsigned todo = (unsigned)__builtin_amdgcn_ballot_w64(close);         // (both halves hold the same points)
            if (4 * __popc(todo) > k) {
                // many for so few centroids: together, each lane half of the centroids of its own point
                if (close) {
                    float x[DP];
                    whole_row(p, x);
                    double best = INFINITY;
                    int arg = 0x7fffffff;
                    for (int j = hl; j < k; j += 2) {
                        const double dist = exact_distance<DP>(x, cs_s + j * CS);
                        if (dist < best) { best = dist; arg = j; }
                    }
                    const double other = __hiloint2double(xchg32(__double2hiint(best)), xchg32(__double2loint(best)));
                    const int oarg = xchg32(arg);
                    label = other < best || (other == best && oarg < arg) ? oarg : arg;
                }
            } else if (todo != 0u) {
                float x[H];
                half_row(pc, x);
                while (todo) {
                    const int src = __ffs((int)todo) - 1;
                    float xs[DP];
#pragma unroll
                    for (int s = 0; s < H; ++s) {
                        xs[s] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x[s]), src));
                        xs[H + s] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x[s]), src + 32));
                    }
                    const int arg = exact_argmin_wave<DP>(xs, cs_s, CS, k);
                    if (n == src) label = arg;
                    todo &= todo - 1u;
                }
            }
            if (last) {
                if (valid && hl == 0) {
                    labels_s[p] = (unsigned char)label;
                    if (a.labels) a.labels[(int64_t)b * a.lab_bs + (int64_t)run * a.N + p] = label;
                }
                continue;
            }
            if (!valid || was == label) continue;
            unsigned long long *const sn = sums_l + label * (DP + 1) + f0, *const so = sums_l + (was == 0xff ? 0 : was) * (DP + 1) + f0;
            const bool leaves = was != 0xff;
            if (any_wide) {
                for (int s = 0; s < H && f0 + s < d; ++s) {
                    const float x = ROWS ? rows_s[p * DP + f0 + s] : Xb[p * a.ldx + f0 + s];
                    const unsigned long long v = (unsigned long long)to_fixed(x, shift_s[f0 + s]) + kFixBias;
                    atomicAdd(sn + s, v);
                    if (leaves) __hip_atomic_fetch_sub(so + s, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    if (wide_s[f0 + s] == 0) continue;
                    const unsigned long long low = (unsigned long long)fixed_low(x, shift_s[f0 + s]);
                    atomicAdd(lows_s + label * DP + f0 + s, low);
                    if (leaves) __hip_atomic_fetch_sub(lows_s + was * DP + f0 + s, low, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            } else {
                float x[H];
                half_row(p, x);
#pragma unroll
                for (int s = 0; s < H; ++s) {
                    const unsigned long long v = fixed_biased(x[s], pow2hi_s[f0 + s]);
                    atomicAdd(sn + s, v);
                    if (leaves) __hip_atomic_fetch_sub(so + s, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
            if (hl == 0) {
                atomicAdd(cnts_l + label, 1);
                if (leaves) atomicAdd(cnts_l + was, -1);
                labels_s[p] = (unsigned char)label;
            }
        }
        if (!last) {
            __syncthreads();
            renew(t + 1);
        }
    }
    for (int e = tid; e < k * d; e += kSmallThreads) Cb[e] = cs_s[(e / d) * CS + e % d];
    __syncthreads();
    // ---- the loss: the additions of the final pass of lloyd_step_kernel, in the same order (lanes of a wave over its slabs
    // of a chunk, the lanes, the waves, the chunks), so that the sum is the same to the last bit
    for (int q = tid >> 5; q < n_chunks * WV; q += kSmallThreads / 32) {
        const int first = q / WV * chunk_len, end = min(first + chunk_len, (int)a.N);
        double sum = 0.0;
        for (int s0 = first + q % WV * slab; s0 < end; s0 += WV * slab)
            for (int p = s0 + n; p < min(s0 + slab, end); p += 32) {
                float x[DP];
                whole_row(p, x);
                sum = __dadd_rn(sum, exact_distance<DP>(x, cs_s + labels_s[p] * CS));
            }
        sum = half_sum_f64(sum);                       // (partners as there)
        if (n == 0) jpart_s[q] = sum;
    }
    __syncthreads();
    if (tid < n_chunks) {
        double v = 0.0;
        for (int w = 0; w < WV; ++w) v = __dadd_rn(v, jpart_s[tid * WV + w]);
        jpart_s[tid * WV] = v;
    }
    __syncthreads();
    if (tid == 0) {
        double v = 0.0;
        for (int c = 0; c < n_chunks; ++c) v = __dadd_rn(v, jpart_s[c * WV]);
        a.inertia[(int64_t)b * a.n_runs + run] = v;
    }
}

template <int DP>
hipError_t launch_small_dp(const SweepPlan &plan, const SmallArgs &a, int32_t batch, hipStream_t s)
{
    static std::once_flag attr_once;
    static hipError_t attr_status = hipSuccess;
    std::call_once(attr_once, [] {
        const void *fns[] = {reinterpret_cast<const void *>(lloyd_small_kernel<DP, false, false>), reinterpret_cast<const void *>(lloyd_small_kernel<DP, true, false>),
                             reinterpret_cast<const void *>(lloyd_small_kernel<DP, false, true>), reinterpret_cast<const void *>(lloyd_small_kernel<DP, true, true>)};
        for (const void *fn : fns) {
            const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
            if (e != hipSuccess) attr_status = e;
        }
    });
    if (attr_status != hipSuccess) return attr_status;
    int lds = 0, lds_rows = 0;
    for (int gi = 0; gi < plan.n_groups; ++gi)
        for (int r = plan.g[gi].run0; r < plan.g[gi].run0 + plan.g[gi].n_runs; ++r) {
            const int k = a.k_min + r;
            const SmallCarve c = small_carve(DP, k, small_copies(DP, k), (int)a.N, plan.g[gi].n_chunks * (step_threads_of(DP) / 64));
            lds = std::max(lds, c.total);
            lds_rows = std::max(lds_rows, rows_end(c, DP, a.N));
        }
    const bool vec = a.d % 4 == 0 && a.ldx % 4 == 0 && (a.x_bs % 4 == 0 || batch == 1) && (reinterpret_cast<uintptr_t>(a.X) & 15) == 0;
    const bool rows = lds_rows <= 160 * 1024;
    const dim3 grid(a.n_runs, batch), block(small_threads_of(DP));
    if (rows && vec) hipLaunchKernelGGL((lloyd_small_kernel<DP, true, true>), grid, block, lds_rows, s, plan, a);
    else if (rows) hipLaunchKernelGGL((lloyd_small_kernel<DP, false, true>), grid, block, lds_rows, s, plan, a);
    else if (vec) hipLaunchKernelGGL((lloyd_small_kernel<DP, true, false>), grid, block, lds, s, plan, a);
    else hipLaunchKernelGGL((lloyd_small_kernel<DP, false, false>), grid, block, lds, s, plan, a);
    return hipGetLastError();
}

}  // namespace

// One workgroup per run and space, at most one per compute unit.  A run's time grows with the points and its tiles, that of the
// launches hardly before they fill the chip; it grows with the number of runs instead.  Measured against the launches:
// 2048 x 8: k 2 2.26x, 64 1.39x, 128 1.09x, 1..16 2.42x, 97..128 1.57x, 1..128 1.98x; 4096 x 8: k 64 1.01x, 128 0.84x, 1..16 1.71x,
// 97..128 1.15x; 4096 x 16: 64 1.01x, 1..16 1.48x, 97..128 1.12x; 6144 x 16: 1..16 1.16x, 49..64 1.15x;
// 1024 x 32: 64 1.23x, 128 1.05x; 2048 x 32: 64 0.96x, 1..16 1.29x, 97..128 1.10x; 3072 x 32: 1..16 0.98x, 17..32 1.10x.
bool sweep_is_small(const SweepPlan &plan, int64_t N, int32_t batch, int32_t iters, bool trace)
{
    if (trace || iters < 1 || (int64_t)plan.n_runs * batch > 256) return false;
    int64_t limit = plan.dp == 32 ? 1280 : 3072;
    if (plan.n_runs >= 16) limit *= 2;
    if (plan.k_min + plan.n_runs - 1 > 64) limit = limit * 2 / 3;
    return N <= limit;
}

hipError_t launch_small_sweep(const SweepPlan &plan, const SweepLayout &L, const SweepArgs &sa, hipStream_t s)
{
    SmallArgs a;
    a.X = sa.X; a.N = sa.N; a.ldx = sa.ldx; a.x_bs = sa.x_batch_stride;
    a.d = sa.d; a.k_min = plan.k_min; a.n_runs = plan.n_runs; a.iters = sa.iters;
    a.init_idx = sa.init_idx; a.init_bs = sa.init_batch_stride;
    a.C = sa.centroids; a.c_bs = (int64_t)plan.total_rows * sa.d;
    a.labels = sa.labels; a.lab_bs = (int64_t)plan.n_runs * sa.N;
    a.inertia = sa.inertia; a.status = sa.status;
    a.colinfo = sa.ws + L.colinfo; a.ws_bs = L.per_batch;
    a.xp = sa.ws + L.xp;
    switch (plan.dp) {
    case 8: return launch_small_dp<8>(plan, a, sa.batch, s);
    case 16: return launch_small_dp<16>(plan, a, sa.batch, s);
    default: return launch_small_dp<32>(plan, a, sa.batch, s);
    }
}

}  // namespace rls
