// Device code that the Lloyd kernels share: matrix operands, exact assignment, fixed-point rows, exact sums to fp64.
#pragma once

#include "rls_internal.h"

namespace rls {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

namespace {

constexpr float kPadNorm = 1.0e30f;           // squared norm given to padding rows: never the minimum
constexpr int kBigKey = 0x7f000000;           // larger than any key of a finite distance below 1.7e38
constexpr int kGridBits = 44;                 // bits of |x * 2^shift| kept by the main accumulator
constexpr int kLowBits = 36;                  // further bits kept by the low accumulator (wide columns)
// The centred data is scaled by a power of two so that |x'| < 2^13 and |2 c'| < 2^14 sit well inside fp16; an fp16
// piece below 2^-14 (subnormal) may be lost, which costs a distance at most 0.078 d + S 2^-24 in scaled units (see pair_error_of)
constexpr int kScaledMsb = 14;
constexpr float kTolFloor = 8.0f;             // twice that loss at d = 32, in scaled squared units

// Bound on the summed error of two matrix-pipeline distances, relative to S = |x'|^2 + max |c'|^2 (centred and scaled), in units of
// 2^-23 S.  Per distance:
//   6    what the two pieces per operand leave out: the product of the two low pieces and the two remainders, each below 2^-22
//        |x'| |2c'|, and |x'| |2c'| <= S
//   5.5  (7.5 at d_pad = 32) the MFMA of the high pieces (two of them).  What an instruction leaves out, on gfx950 (tests/matrix_model.py
//        has it as a model, tests/test_gpu_bound.py holds the instruction to it): the halves of K follow each other; the eight
//        products of a half, and the accumulator where it is smaller, are cut off below 2^-24 of the largest product's power of
//        two, so at most eight times that is lost (4 units over all halves, whose largest products are no more than S together),
//        and the sum is rounded to the nearest, now and then the other way (one unit at most in the last place of its largest term; half of
//        that, and of up to S, is 1 and 2 units).  The MFMAs of the low pieces, a 2^-10 of the magnitude, lose nothing that counts
//   5    the MFMA of the norms: products by one, whose pieces lose nothing, and two additions of up to 2 S
//   2.5  (3) the norm of the centroid: five (six) roundings.  (That of the point is the same in both distances.)
//   2    centring
//   0.5  pieces below 2^-14 (fp16 subnormals) counted as lost altogether: at most 2^-14 sqrt(d) (|x'| + |2c'|)
//        <= 2^-24 S + 0.078 d, hence the absolute term kTolFloor next to the relative one
// 21.5 (24): twice that is 43 (48), the bound used is 48 (56).  The largest error seen of a distance, over operands made to be hard, is
// 3.3 units besides the centring.  (The pieces were rounded toward zero and every MFMA charged five units per distance before, 120 and
// 200: 2.5 and 3.6 times as many close calls.)
__host__ __device__ constexpr float pair_error_of(int dp) { return (dp == 32 ? 56.0f : 48.0f) * 1.1920928955078125e-07f; }
constexpr int kColScaleOff = 400;             // byte offset of the scale factor in the column info block

// MFMA operands: a lane holds 8 fp16 values of its half of the features per K-step (v_mfma_f32_32x32x16_f16);
// a 32-row tile stores, per K-step, the two pieces (high, low) of -2c', and then one bias slot (bf16).
__host__ __device__ constexpr int ksteps_of(int dp) { return dp == 32 ? 2 : 1; }
__host__ __device__ constexpr int tile_slots_of(int dp) { return 2 * ksteps_of(dp) + 1; }          // 16-byte slots per lane
__host__ __device__ constexpr int tile_bytes_of(int dp) { return tile_slots_of(dp) * 64 * 16; }    // per 32-row tile

// 32-point blocks a wave takes per slab.  Up to d_pad = 16: one, which keeps a wave under 168 registers so that three
// waves fit a SIMD (measured: 6% shorter launches than two waves with two blocks each).  At d_pad = 32 three waves do
// not fit; there a wave takes two blocks, except with eight runs side by side, where the best keys of 4 runs x 2 blocks
// would not fit the registers next to the operands.
__host__ __device__ constexpr int slab_blocks_of(int dp, int s) { return dp <= 16 ? 1 : (s < 2 ? 1 : 2); }
// threads of a step workgroup: up to d_pad = 16 one block per slab leaves room for three waves per SIMD
__host__ __device__ constexpr int step_threads_of(int dp) { return dp <= 16 ? 768 : 512; }

// Prepared copy of the points (written once per sweep by lloyd_prepare_kernel): per block of 32 points the B operands
// of the distance tiles in the lane order of the step kernel - 2 * ksteps slots (high pieces, then low pieces, per
// K-step) of 64 lanes x 16 bytes - followed by 32 entries of 8 bytes with the point's squared norm as the three bf16
// pieces the bias slot wants (their sum, which is the norm cut off below 2^-24 of itself, serves the error bound - in the step kernel the
// highest of them alone, see eps_x there).
__host__ __device__ constexpr int prep_slots_of(int dp) { return 2 * ksteps_of(dp); }
__host__ __device__ constexpr int prep_block_u4_of(int dp) { return prep_slots_of(dp) * 64 + 16; }   // 16-byte units per block
// x * 2^shift truncated toward zero, |x * 2^shift| < 2^kGridBits; exact whenever x is a multiple of 2^-shift.
// The scaling is exact in fp64; adding 2^52 + 2^51 leaves the integer in the low bits of the significand.
__device__ inline long long to_fixed(float x, int shift)
{
    const double t = trunc(ldexp((double)x, shift));
    return __double_as_longlong(__dadd_rn(t, 6755399441055744.0)) - 0x4338000000000000ll;
}

// The accumulators hold "biased" fixed-point rows: the bit pattern of the double 2^52 + 2^51 + x * 2^shift, which is
// kFixBias plus the two's complement integer x * 2^shift.  A row that enters a cluster adds its patterns, a row that
// leaves subtracts them, so an accumulator is off by kFixBias times the net number of rows - the member count delta,
// which is tracked anyway - and the bias is taken out once per chunk.  For a column whose values are all multiples of
// 2^-shift the product is an exact integer and one fused multiply-add (by the power of two 2^shift, whose high word
// comes from LDS) yields the pattern: two vector instructions per feature.
constexpr unsigned long long kFixBias = 0x4338000000000000ull;
__device__ inline unsigned long long fixed_biased(float x, int pow2_hi)
{
    return (unsigned long long)__double_as_longlong(fma((double)x, __hiloint2double(pow2_hi, 0), 6755399441055744.0));
}

// The part of x below the column grid 2^-shift, scaled by 2^(shift + kLowBits): the bits that to_fixed drops.
// Non-zero only in columns whose values span more than kGridBits binary digits.
__device__ inline long long fixed_low(float x, int shift)
{
    const unsigned u = __float_as_uint(x);
    int e = (int)((u >> 23) & 0xffu);
    unsigned m = u & 0x7fffffu;
    if (e == 0) {
        if (m == 0) return 0;
        e = 1;
    } else {
        m |= 0x800000u;
    }
    const int sh = e - 150 + shift;
    if (sh >= 0) return 0;
    const int drop = -sh > 24 ? 24 : -sh;                     // dropped bits of the 24-bit significand
    const unsigned long long low = (unsigned long long)(m & ((1u << drop) - 1u));
    // value of the dropped bits is low * 2^sh on the grid scale; on the low scale it is low * 2^(sh + kLowBits)
    const int up = sh + kLowBits;
    const long long q = up >= 0 ? (long long)(low << up) : (long long)(low >> (-up > 63 ? 63 : -up));
    return (u >> 31) ? -q : q;
}

// value of the lane 32 places away (the other half-wave), by a register swap: no trip through LDS
__device__ inline int xchg32(int v)
{
    const auto r = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    return (int)((threadIdx.x & 32) ? r[0] : r[1]);
}
__device__ inline unsigned xchg32(unsigned v) { return (unsigned)xchg32((int)v); }
__device__ inline float xchg32(float v) { return __int_as_float(xchg32(__float_as_int(v))); }

// Minimum over the wave, in every lane, without a trip through LDS: lane exchanges inside rows of 16 by DPP (swap
// neighbours, swap pairs, mirror halves of 8, mirror the row: after each step twice as many lanes agree), then
// between rows with the two row-swap instructions.
template <int CTRL>
__device__ inline int dpp_move(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true); }   // every lane has a source
template <int CTRL>
__device__ inline double dpp_move(double v)
{
    return __hiloint2double(dpp_move<CTRL>(__double2hiint(v)), dpp_move<CTRL>(__double2loint(v)));
}
constexpr int kDppSwap1 = 0xB1, kDppSwap2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;
__device__ inline double wave_min_f64(double v)
{
    v = fmin(v, dpp_move<kDppSwap1>(v));
    v = fmin(v, dpp_move<kDppSwap2>(v));
    v = fmin(v, dpp_move<kDppHalfMirror>(v));
    v = fmin(v, dpp_move<kDppMirror>(v));
    {
        const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
        const auto rl = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto rh = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        v = fmin(__hiloint2double((int)rh[0], (int)rl[0]), __hiloint2double((int)rh[1], (int)rl[1]));   // own row, other row
    }
    {
        const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
        const auto rl = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto rh = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        v = fmin(__hiloint2double((int)rh[0], (int)rl[0]), __hiloint2double((int)rh[1], (int)rl[1]));
    }
    return v;
}
__device__ inline int wave_min_i32(int v)
{
    v = min(v, dpp_move<kDppSwap1>(v));
    v = min(v, dpp_move<kDppSwap2>(v));
    v = min(v, dpp_move<kDppHalfMirror>(v));
    v = min(v, dpp_move<kDppMirror>(v));
    {
        const auto r = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
        v = min((int)r[0], (int)r[1]);
    }
    {
        const auto r = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
        v = min((int)r[0], (int)r[1]);
    }
    return v;
}

__device__ inline float wave_min_f32(float v)
{
    v = fminf(v, __int_as_float(dpp_move<kDppSwap1>(__float_as_int(v))));
    v = fminf(v, __int_as_float(dpp_move<kDppSwap2>(__float_as_int(v))));
    v = fminf(v, __int_as_float(dpp_move<kDppHalfMirror>(__float_as_int(v))));
    v = fminf(v, __int_as_float(dpp_move<kDppMirror>(__float_as_int(v))));
    {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = fminf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    }
    {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = fminf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    }
    return v;
}

// sum and largest value over each half-wave, in all of its lanes
__device__ inline float half_sum_f32(float v)
{
    v += __int_as_float(dpp_move<kDppSwap1>(__float_as_int(v)));
    v += __int_as_float(dpp_move<kDppSwap2>(__float_as_int(v)));
    v += __int_as_float(dpp_move<kDppHalfMirror>(__float_as_int(v)));
    v += __int_as_float(dpp_move<kDppMirror>(__float_as_int(v)));
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ inline float half_max_f32(float v)
{
    v = fmaxf(v, __int_as_float(dpp_move<kDppSwap1>(__float_as_int(v))));
    v = fmaxf(v, __int_as_float(dpp_move<kDppSwap2>(__float_as_int(v))));
    v = fmaxf(v, __int_as_float(dpp_move<kDppHalfMirror>(__float_as_int(v))));
    v = fmaxf(v, __int_as_float(dpp_move<kDppMirror>(__float_as_int(v))));
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// sum over each half-wave, in all of its lanes: partners 16, 8, 4, 2, 1 lanes apart
__device__ inline double half_sum_f64(double v)
{
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    const auto rl = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto rh = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    v = __dadd_rn(__hiloint2double((int)rh[0], (int)rl[0]), __hiloint2double((int)rh[1], (int)rl[1]));
    v = __dadd_rn(v, dpp_move<0x128>(v));          // turned by 8, 4, 2, 1 lanes of 16
    v = __dadd_rn(v, dpp_move<0x124>(v));
    v = __dadd_rn(v, dpp_move<0x122>(v));
    v = __dadd_rn(v, dpp_move<0x121>(v));
    return v;
}

// the exact squared distance: fp64, features in rising order, products and sums rounded one by one
template <int DP>
__device__ inline double exact_distance(const float (&x)[DP], const float *crow)
{
    double dist = 0.0;
#pragma unroll
    for (int l = 0; l < DP; l += 4) {
        const float4 c = *reinterpret_cast<const float4 *>(crow + l);
        double diff = __dsub_rn((double)x[l], (double)c.x);
        dist = __dadd_rn(dist, __dmul_rn(diff, diff));
        diff = __dsub_rn((double)x[l + 1], (double)c.y);
        dist = __dadd_rn(dist, __dmul_rn(diff, diff));
        diff = __dsub_rn((double)x[l + 2], (double)c.z);
        dist = __dadd_rn(dist, __dmul_rn(diff, diff));
        diff = __dsub_rn((double)x[l + 3], (double)c.w);
        dist = __dadd_rn(dist, __dmul_rn(diff, diff));
    }
    return dist;
}

// The assignment as it is defined, by one whole wave: fp64 direct-form distances sum_l (x_l - c_l)^2, features in
// rising order, of one point to the k centroids of a run (one or two per lane), then the lexicographic minimum of
// (distance, index) over the wave.  Every lane returns the winner.  The point arrives as wave-uniform values (read
// out of the registers of the two lanes that hold its halves); the centroid rows come from the LDS copy, which is
// zero beyond the last feature, as is the register copy of the point: padded terms add +0.
//
// Almost every call is settled by a first stage in fp32: the same direct form (difference, square, sum; all terms
// are non-negative, so nothing cancels) is within (DP + 2) 2^-24 of the real-number distance, relatively, and the
// fp64 form within (DP + 2) 2^-53.  A centroid whose fp32 distance exceeds the smallest one by more than 8 (DP + 2)
// 2^-24 of it (more than twice the two errors and the rounding of the threshold itself) cannot have the smallest
// fp64 distance; when a single centroid is left it is the winner.  Several left (true ties, duplicated centroids),
// or a smallest distance so small or large that fp32 may have lost it (below 1e-30, infinite): fp64 over the whole run.
template <int DP>
__device__ inline int exact_argmin_wave(const float (&x)[DP], const float *crun, int cstride, int k)
{
    const int lane = threadIdx.x & 63;
    {
        float d32[2] = {INFINITY, INFINITY};        // this lane's centroids: lane and lane + 64 (k <= 128)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int j = lane + 64 * u;
            if (u == 1 && k <= 64) break;           // wave-uniform
            const float *crow = crun + min(j, k - 1) * cstride;
            float acc = 0.0f;
#pragma unroll
            for (int l = 0; l < DP; l += 4) {
                const float4 cv = *reinterpret_cast<const float4 *>(crow + l);
                float diff = x[l] - cv.x;
                acc = fmaf(diff, diff, acc);
                diff = x[l + 1] - cv.y;
                acc = fmaf(diff, diff, acc);
                diff = x[l + 2] - cv.z;
                acc = fmaf(diff, diff, acc);
                diff = x[l + 3] - cv.w;
                acc = fmaf(diff, diff, acc);
            }
            if (j < k) d32[u] = acc;
        }
        const float wmin = wave_min_f32(fminf(d32[0], d32[1]));
        const float thr = fmaf(wmin, (float)(8 * (DP + 2)) * 5.9604644775390625e-08f, wmin);
        const unsigned long long c0 = __ballot(d32[0] <= thr), c1 = __ballot(d32[1] <= thr);
        if (__popcll(c0) + __popcll(c1) == 1 && wmin >= 1.0e-30f && wmin < INFINITY)
            return c0 ? __ffsll((long long)c0) - 1 : 63 + __ffsll((long long)c1);
    }
    double best = INFINITY;
    int arg = 0x7fffffff;
    for (int j = lane; j < k; j += 64) {
        const double dist = exact_distance<DP>(x, crun + j * cstride);
        if (dist < best) { best = dist; arg = j; }
    }
    // smallest distance of the wave, then the smallest index among the lanes that hold it
    const double wbest = wave_min_f64(best);
    const unsigned long long tied = __ballot(best == wbest);
    // up to 64 centroids a lane's index is its number: the first lane that holds the minimum has the smallest index
    if (k <= 64) return __ffsll((long long)tied) - 1;
    return wave_min_i32(best == wbest ? arg : 0x7fffffff);
}

// v = h + m + l exactly, each piece a bf16 (8 significant bits): h and m by truncation, l is what is left
__device__ inline void split3(float v, unsigned &h, unsigned &m, unsigned &l)
{
    const unsigned b = __float_as_uint(v);
    h = b >> 16;
    const float r = v - __uint_as_float(b & 0xffff0000u);
    const unsigned rb = __float_as_uint(r);
    m = rb >> 16;
    const float r2 = r - __uint_as_float(rb & 0xffff0000u);
    l = __float_as_uint(r2) >> 16;
}

__device__ inline bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }
__device__ inline f16x8 as_f16x8(uint4 v) { return __builtin_bit_cast(f16x8, v); }

// Two fp16 pieces of a value, rounded to the nearest: v = h + l + r with |l| <= 2^-11 |v| and |r| <= 2^-22 |v| while the
// pieces are normal fp16 numbers (11 significant bits each; v - h is exact in fp32).  The pair form packs a's pieces into the
// low halves and b's into the high halves, as two neighbouring operand elements.
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef _Float16 fp16x2 __attribute__((ext_vector_type(2)));
__device__ inline void split2_pair(float a, float b, unsigned &h, unsigned &l)
{
    const fp16x2 hh = __builtin_convertvector((floatx2{a, b}), fp16x2);
    h = __builtin_bit_cast(unsigned, hh);
    const floatx2 rest = {a - (float)hh[0], b - (float)hh[1]};
    l = __builtin_bit_cast(unsigned, __builtin_convertvector(rest, fp16x2));
}
__device__ inline void split2(float v, unsigned short &h, unsigned short &l)
{
    unsigned ph, pl;
    split2_pair(v, 0.0f, ph, pl);
    h = (unsigned short)(ph & 0xffffu);
    l = (unsigned short)(pl & 0xffffu);
}

// The index that phase A packs into the low bits of a key (7 at most) is the centroid index within the run:
// centroid j lives in tile (j/4)/S, slot (j/4)%S of its run, row j%4 (see GroupDesc).
template <int S>
__device__ inline int key_index(int t, int a, int i)
{
    if (S == 1) return 4 * t + i;
    if (S == 2) return 8 * t + 4 * (a & 1) + i;
    if (S == 4) return 16 * t + 4 * a + i;
    return 32 * t + 4 * a + i;   // S == 8: bit 4 (the half-wave) is added after the tile loop
}
// quads of a lane's four that differ in their indices (the others repeat them in another run)
__host__ __device__ constexpr int index_quads_of(int s) { return s == 1 ? 1 : (s == 2 ? 2 : 4); }
template <int S>
__device__ inline int state_of(int a) { return S == 1 ? a : (S == 2 ? (a >> 1) : 0); }

// Keys: the low bits of a distance give way to the index, as many as the indices of a slab take (kidx < 2^bits).
__device__ inline int key_mask(int bits) { return (int)(0xffffffffu << bits); }
__device__ inline int key_bits(int indices) { return indices > 1 ? 32 - __builtin_clz((unsigned)(indices - 1)) : 0; }
// 1 - 2^(bits - 22): read as a float a key g lies within 2^(bits - 23) |v| of the value v it was packed from, so
// v2 - v1 >= g2 (1 - 2^(bits - 22)) - g1 whenever g2 >= |g1|
__device__ inline float key_shrink(int bits) { return __uint_as_float(0x3f800000u - (4u << bits)); }

// (bits & mask) | idx.  The mask is kept opaque to the compiler (a VGPR) so that this selects one and-or
// instruction with the index as its scalar operand.  It must stay a compiler-visible operation (not inline
// assembly): it reads MFMA results, and the wait states between an MFMA and the first read of its result
// are inserted by the compiler.
__device__ inline int pack_key(float v, int mask, int idx)
{
    return (__float_as_int(v) & mask) | idx;
}

// median of three; the compiler selects the single med3 instruction for this shape
__device__ inline int med3i(int a, int b, int c) { return max(min(a, b), min(max(a, b), c)); }

// insert a key into the ascending pair (m1, m2) of the smallest keys seen so far
__device__ inline void insert2(int key, int &m1, int &m2)
{
    m2 = med3i(m1, m2, key);      // second smallest of {m1, m2, key} given m1 <= m2
    m1 = min(m1, key);
}

// insert two keys at once: the new smallest is the smallest of {m1, a, b} (one min3); the second smallest of
// {m1, m2, a, b} is the smaller of m2 and the second smallest of {m1, a, b} (one med3, one min), because m2 >= m1
__device__ inline void insert2x2(int a, int b, int &m1, int &m2)
{
    const int second = med3i(m1, a, b);
    // (written as one instruction: left to itself the compiler takes two minima here; the operands are packed keys,
    // results of vector instructions, so no wait states of the matrix pipeline are involved)
    asm("v_min3_i32 %0, %1, %2, %3" : "=v"(m1) : "v"(m1), "v"(a), "v"(b));
    m2 = min(m2, second);
}

// fold the 16 results of one 32x32 tile (4 quads of 4 rows) into the per-run states: the two smallest keys
// (five vector instructions per two distances: two and-or, min3, med3, min).  The second key shows whether the
// first is a clear winner.
template <int S, int ST, int NKI>
__device__ inline void fold_tile(const floatx16 &acc, const int (&kidx)[NKI], int mask, int (&m1)[ST], int (&m2)[ST])
{
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int st = state_of<S>(q);
#pragma unroll
        for (int i = 0; i < 4; i += 2)
            insert2x2(pack_key(acc[4 * q + i], mask, kidx[(4 * q + i) % NKI]), pack_key(acc[4 * q + i + 1], mask, kidx[(4 * q + i + 1) % NKI]),
                      m1[st], m2[st]);
    }
}

// 128-bit two's complement sum (hi, lo) -> fp64 with one round-to-nearest-even, scaled by 2^-shift
__device__ inline double fixed128_to_double(long long hi, unsigned long long lo, int shift)
{
    const bool neg = hi < 0;
    unsigned long long mh = (unsigned long long)hi, ml = lo;
    if (neg) {
        ml = ~ml + 1ull;
        mh = ~mh + (ml == 0ull ? 1ull : 0ull);
    }
    double mag;
    if (mh == 0ull && (ml >> 53) == 0ull) {
        mag = (double)ml;                       // exact
        mag = ldexp(mag, -shift);
    } else {
        const int nbits = mh ? 128 - __clzll((long long)mh) : 64 - __clzll((long long)ml);
        const int sh = nbits - 53;              // >= 1
        // top = mag >> sh (53 bits), rem = mag & (2^sh - 1)
        unsigned long long top, rem_hi, rem_lo;
        if (sh >= 64) {
            top = mh >> (sh - 64);
            rem_hi = sh == 64 ? 0ull : (mh & ((1ull << (sh - 64)) - 1ull));
            rem_lo = ml;
        } else {
            top = (ml >> sh) | (mh ? (mh << (64 - sh)) : 0ull);
            rem_hi = 0ull;
            rem_lo = ml & ((1ull << sh) - 1ull);
        }
        // compare remainder with half = 2^(sh-1)
        int cmp;   // -1 below half, 0 equal, 1 above
        if (sh > 64) {
            const unsigned long long half_hi = 1ull << (sh - 65);
            cmp = rem_hi > half_hi ? 1 : (rem_hi < half_hi ? -1 : (rem_lo ? 1 : 0));
        } else if (sh == 64) {
            const unsigned long long half_lo = 1ull << 63;
            cmp = rem_lo > half_lo ? 1 : (rem_lo < half_lo ? -1 : 0);
        } else {
            const unsigned long long half_lo = 1ull << (sh - 1);
            cmp = rem_lo > half_lo ? 1 : (rem_lo < half_lo ? -1 : 0);
        }
        if (cmp > 0 || (cmp == 0 && (top & 1ull))) top += 1ull;
        mag = ldexp((double)top, sh - shift);   // top <= 2^53: exact
    }
    return neg ? -mag : mag;
}

}  // namespace
}  // namespace rls
