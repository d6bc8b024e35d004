// Lloyd's k-means for every k of a range at once: the "k-means(s_Theta, k)" call inside the loop of
// Algorithm 1 (Sec. 4.2 of the paper), all k side by side, iterations in lock step.
//
// Per iteration one launch of lloyd_step_kernel covers every (group of runs, chunk of points).  A workgroup
// stages its group's operand rows, a copy of its centroids and integer accumulators in LDS once; then each of
// its waves (twelve up to d_pad = 16, eight at 32) works through its own points without any barrier:
//   load     each lane loads its half of the features of its points straight into registers, one step ahead; from
//            the second round on the lanes load the matrix operands themselves, which lloyd_prepare_kernel derives
//            once per sweep from the rows (centred, scaled, split into fp16 pieces, squared norm), and a raw row
//            is read again only for a point that needs it: a close call or a changed label
//   assign   distances in the expansion |c'|^2 + |x'|^2 - 2 x'.c' on data centred by the column means and scaled
//            by one power of two into fp16 range, on the 16-bit matrix pipeline: every fp32 operand is split
//            into two fp16 pieces (22 significant bits) and the three leading cross products are accumulated
//            in fp32 (fp32-class accuracy; the 16-bit pipeline runs beside the vector ALU, the fp32 one does
//            not); per point and run the two smallest packed (value, index) keys are kept.  When they are
//            closer than the error bound of these distances the pair is decided again with the direct
//            form sum_l (x_l - c_l)^2 - the arithmetic that defines the assignment - by a scan of the whole
//            run: in fp32 first, whose relative error bound leaves a single candidate almost always, then in
//            fp64 among several; labels never depend on the rounding of the matrix-pipeline distances
//   update   exact centroid sums, kept as running totals: only points whose label differs from the one
//            of the previous round (kept as one byte per point and run, the runs of a group side by side, so
//            that a lane compares all its runs in one instruction) move their fixed-point row from the old cluster's int64 accumulators
//            to the new one's (integer LDS atomics; integer adds commute and cancel exactly, so the totals
//            equal a fresh sum in any order); per-chunk deltas go to global memory and lloyd_centroids_kernel
//            adds them to the 128-bit totals, rounds once to fp64, divides by the count and rounds to fp32
// The final pass replaces the update by the fp64 loss of every point and the label output.
//
// Two other forms share this file's plan and arithmetic, and give the same labels, centroids and losses: sweeps with much distance
// work run on a copy of the points in spatial order (kmeans_order.hip), where a unit of neighbouring points meets only the
// tiles of centroids that can win there (ORD, make_lists); sweeps of a few thousand points are one launch (kmeans_small.hip).
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "lloyd_device.h"

namespace rls {

namespace {

constexpr int kThreads = 512;                // workgroup of the helper kernels (the step kernel: step_threads_of)
constexpr int kPartRows = 8;                 // centroids of a run that one workgroup of the centroid kernel renews
constexpr int kMaxParts = RLS_MAX_K / kPartRows;
// parts of the runs k' = 1 .. k together: the sum of ceil(k' / kPartRows)
__host__ __device__ inline int parts_upto(int k)
{
    const int q = k / kPartRows;
    return kPartRows * q * (q + 1) / 2 + (k - kPartRows * q) * (q + 1);
}
__host__ __device__ constexpr int tile_points_of(int dp) { return dp == 32 ? 256 : 512; }
// Tile lists of an ordered sweep.  A unit is 32 points (64 at d_pad = 32) that follow each other in the order; for every
// unit, and each of the eight quad slots of a group's tiles, a list names the tiles whose quad in that slot may hold the
// nearest centroid of one of the unit's points.  16 words per unit and group, four bits per tile: eight of first words (one per
// slot: entries 0 to 6, and above them the length of the longest of the eight lists, less one), eight of second words (entries 7
// to 14, read by the few units that have so many).  A list that ends before the longest one goes on with tiles that are not on it:
// their centroids are farther away, and nothing else is wrong with them.  A list as long as the group has tiles is all of them in
// their order (of sixteen, entry 15 is what the length says).  Long ones of that kind need no second words and no way back from
// steps to tiles, and a long list that would leave out a single tile is made one of them.  (All long lists worked off alike:
// 1,000,003 x 12 integers 0..8, k 1..64, 10 rounds 6.67 ms, 6.51 now, 6.51 before long lists were followed.)
__host__ __device__ constexpr int unit_blocks_of(int dp) { return dp == 32 ? 2 : 1; }
constexpr int kListWords = 16, kListHead = 7;
constexpr unsigned kAllMore = 0xedcba987u;    // the second word of all tiles in their order
__device__ inline unsigned list_entry(unsigned head, unsigned more, int e) { return ((e < kListHead || e == 15 ? head : more) >> (4 * (e < kListHead ? e : (e == 15 ? 7 : e - kListHead)))) & 15u; }
constexpr int kListMinTiles = 3;              // groups of fewer tiles meet them all: there is little to leave out
constexpr int kListMaxTiles = 16;             // groups of an ordered sweep have no more

// ---- LDS carve of lloyd_step_kernel (bytes), shared by the planner and the kernel ------------
struct Carve {
    int opA, cs, sums, cnts, rowpos, rowidx, misc, total;
};
__host__ __device__ inline Carve carve_lds(int dp, int d, int n_tiles, int real_rows, int copies, bool ordered)
{
    Carve c;
    int off = 0;
    c.opA = off;     off += n_tiles * tile_bytes_of(dp);                // MFMA operand rows of the group (fp16 pieces + bias slot)
    c.cs = off;      off += real_rows * (dp + 4) * 4;                   // centroids as given, rows of dp + 4 floats, zero-padded
    // accumulators: `copies` of them side by side (a lane adds to copy lane % copies, which spreads the lanes that
    // hit one cluster of a run with few clusters over several addresses; the copies are summed at the end)
    c.sums = off;    off += (copies * real_rows * (dp + 1) * 8 + 15) / 16 * 16;   // fixed-point sum deltas
    c.cnts = off;    off += (copies * real_rows * 4 + 15) / 16 * 16;    // member count deltas
    c.rowpos = off;  off += ordered ? (real_rows * 2 + 15) / 16 * 16 : 0;   // places of the centroids among the group's rows
    c.rowidx = off;  off += ordered ? (real_rows + 15) / 16 * 16 : 0;       // which centroid of its run has a place
    c.misc = off;    off += 2048;
    c.total = off;
    return c;
}

struct StepArgs {
    const float *X;
    int64_t N;
    int32_t d;
    int64_t ldx;
    int64_t x_bs;            // elements between spaces of a batch
    const float *C;          // current centroids, packed [total_rows][d]
    int64_t c_bs;
    int32_t *labels;         // [n_runs][N] or null (final pass only)
    int64_t lab_bs;
    const int32_t *status;   // [batch]
    char *ws;                // workspace base
    int64_t ws_bs;           // bytes per batch element
    int64_t off_colinfo, off_opA, off_cnmax, off_psum, off_pcnt, off_pj, off_losum, off_prev, off_xp;
    int64_t off_xs, off_centres, off_radius, off_rowpos, off_rowidx, off_lists;      // (ordered copy)
    int32_t first_round;     // 1: no point has a label yet (every pair enters a cluster, nothing leaves one)
    int32_t batch;           // spaces swept by the launch
};

// Everything a wave needs to run its share of a chunk.  The waves of a workgroup share the group's
// operand rows, centroid copy and integer accumulators (LDS), but each wave owns its points from the global
// load to the accumulator update, so there is no barrier inside the tile loop and waves in different phases
// (matrix pipeline / vector ALU / LDS atomics) overlap on a SIMD.
struct WaveCtx {
    const uint4 *opA_s;           // LDS: operand slots of the group's tiles
    const float *cs;              // LDS: the group's centroids as given, rows of DP + 4 floats, zero past feature d
    unsigned long long *sums;     // LDS: fixed-point sum deltas [copy][row][DP + 1]
    int *cnts;                    // LDS: member count deltas [copy][row]
    int copies, real_rows;        // accumulator copies (a power of two) and rows per copy
    const float *mu_s;            // LDS: -(column mean * scale) [32]
    float scale;                  // power of two that brings the centred data into fp16 range
    const int *shift_s;           // LDS: fixed-point shifts [32]
    const int *pow2hi_s;          // LDS: high words of the doubles 2^shift [32]
    const int *wide_s;            // LDS: wide-column flags [32], any at [32]
    const float *cnmax_s;         // LDS: per-run maximum squared norm of the centred centroids [8]
    const float *X;               // this space's rows (on the prepared copy of an ordered sweep: the rows in that order)
    const uint4 *xp;              // global: prepared copy of this space's points (see prep_block_u4_of)
    const unsigned short *rowpos; // LDS: place of each of the group's centroids among its rows (ordered copy; else places are indices)
    const unsigned char *rowidx;  // LDS: the centroid of its run that has a place
    const unsigned *lists;        // global: the tile lists of the group's units, or null
    int64_t ldx, N;
    int d, k0, n_runs, n_tiles, grow0;
    unsigned char *prev;          // global: labels of the last round for the group's run slots, [point][8 / S]
    int32_t *labels_out;          // global: labels of the group's runs [run][N] (final pass) or null
    long long *losum;             // global: low-order sums of wide columns [row][d]
    int64_t chunk_begin, chunk_end;
    int *next_slab;               // LDS: next slab of the chunk to hand out
    bool vec_x;                   // rows of X may be read 16 bytes at a time
    bool first_round;             // no point has a label yet
    float eps_a;
};

// VEC: rows of X may be read 16 bytes at a time.  A template parameter and not a run-time branch: with both load
// paths in one function the compiler merges them into 4-byte loads, and a wave's rows then cost four times the
// cache look-ups (which bounds sweeps over few k).
// PRE: the operands come from the prepared copy; the raw rows are read on demand (not in a pass that sums the loss,
// which needs every row, and not in the first round, where every row enters a cluster).
// ORD: a round on the ordered copy; FIRST: its first one, when no point has a label yet (other sweeps take the points as they come
// in their first round).
template <int DP, int S, bool FINAL, bool TRACE, bool VEC, bool PRE, bool ORD, bool FIRST>
__device__ inline void wave_loop(const WaveCtx &c, double (&jloc)[8])
{
    static_assert(!PRE || (!FINAL && !TRACE), "the prepared copy serves the plain assign + update pass only");
    static_assert(!ORD || (PRE && VEC), "the ordered copy is a prepared one, with rows of DP floats");
    static_assert(!FIRST || ORD, "a first round on the prepared copy is one of an ordered sweep");
    const int64_t ldx = ORD ? DP : c.ldx;
    constexpr int NB = slab_blocks_of(DP, S);       // blocks of 32 points per wave and slab
    // with 2 blocks at d_pad = 32 the rows of the next slab are requested after the tile loop, when the operand
    // registers are free again, instead of before it
    constexpr bool LATE_FETCH = DP == 32 && NB == 2;
    constexpr int H = DP / 2;                       // features per half-wave
    constexpr int CS = DP + 4;                      // row stride of the LDS copy of the centroids
    constexpr int NK = ksteps_of(DP);               // K-steps of 16 per cross term
    constexpr int NS = tile_slots_of(DP);           // operand slots per tile and lane
    constexpr int HP = 8 * NK;                      // feature slots per half-wave (H padded to whole K-steps)
    constexpr int ST = S == 1 ? 4 : (S == 2 ? 2 : 1);   // runs owned by a lane
    constexpr int SLAB_ = 32 * NB;                  // points a wave takes at a time
    constexpr int NM = 3 * NK + 1;                  // MFMAs per tile block
    constexpr int VPER = (40 + 16 + NM - 1) / NM;   // vector ops to slot in after each MFMA of a chain
    constexpr bool LOSS = FINAL || TRACE;
    constexpr int NKI = 4 * index_quads_of(S);      // indices of a tile's rows that differ for this lane
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 31, hl = lane >> 5;
    const int d = c.d;
    const int f0 = hl * H;                          // first feature of this lane's half
    const int nf = min(max(d - f0, 0), H);          // real features of this lane's half
    const uint4 *opA_s = c.opA_s;
    // the index bits of a key: what the tiles that a slab meets take
    // (eight slots: always 7, the steps become tiles while the halves of a run are still to be compared)
    int kbits = S == 8 ? 7 : key_bits(4 * S * c.n_tiles);
    int mask = key_mask(kbits);
    asm volatile("" : "+v"(mask));                  // keep the mask in a VGPR

    // this lane's copy of the accumulators
    unsigned long long *const sums_l = c.sums + (lane & (c.copies - 1)) * c.real_rows * (DP + 1);
    int *const cnts_l = c.cnts + (lane & (c.copies - 1)) * c.real_rows;

    // Raw features of this lane's half of its points.  The rows of the next step are loaded while this step
    // runs: the loads are unconditional (addresses clamped into the chunk and the row, masking happens when the
    // values are used) and nothing touches their registers before settle(), so no wait is placed early.
    // Addresses are a wave-uniform base (the slab's first row) plus a 32-bit lane offset: the row index inside
    // the slab is clamped to the chunk's last row, the feature offset to the row's last 16 bytes.
    float xnext[PRE ? 1 : NB][PRE ? 1 : HP];
    constexpr int NP = prep_slots_of(DP);            // operand slots per lane and block in the prepared copy
    uint4 pnext[PRE ? NB : 1][PRE ? NP : 1];          // PRE: the operand slots of the slab being fetched
    uint2 nnext[PRE ? NB : 1];                        // PRE: its norm entries
    const unsigned ldx32 = (unsigned)ldx;          // checked on the host: 64 rows of ldx floats fit 32 bits
    // this lane's clamped feature offsets (fixed for the launch; with the prepared copy they are worked out where
    // a row is read, which is rare, instead of being kept in registers)
    auto feat_off = [&](int s) { return (unsigned)(ORD ? f0 + s : (VEC ? min(f0 + (s & ~3), d - 4) + (s & 3) : min(f0 + s, d - 1))); };
    unsigned foff[PRE ? 1 : H];
    if constexpr (!PRE) {
#pragma unroll
        for (int s = 0; s < H; ++s) foff[s] = feat_off(s);
    }
    // The labels of the last round are kept per group as one byte per (point, run slot of the group), the R = 8 / S
    // slots of a point side by side: a lane reads and writes the labels of its ST runs as one word.
    constexpr int R = 8 / S;                         // run slots of the group
    using LabWord = std::conditional_t<ST == 4, unsigned, std::conditional_t<ST == 2, unsigned short, unsigned char>>;
    const unsigned lab_off = S == 8 ? 0u : (unsigned)(hl * ST);     // this lane's first byte within a point's R bytes
    unsigned oldn[NB];                               // previous labels of the slab being fetched (byte st: run st of this lane)
    unsigned run_off[ST];                            // offset of this lane's runs in the label output (runs are N apart)
    unsigned actmask = 0u;                           // bytes of a label word that belong to real runs of this lane
#pragma unroll
    for (int st = 0; st < ST; ++st) {
        const unsigned rl = S == 8 ? 0u : (unsigned)(hl * ST + st);
        run_off[st] = min(rl, (unsigned)(c.n_runs - 1)) * (unsigned)c.N;
        if (((S == 8) ? (hl == 0) : true) && (int)rl < c.n_runs) actmask |= 0xffu << (8 * st);
    }
    for (int pb = 0; pb < NB; ++pb) oldn[pb] = 0xffffffffu;
    unsigned char *const prev_chunk = c.prev + c.chunk_begin * R;          // the chunk's first label byte
    const unsigned chunk_pts = (unsigned)(c.chunk_end - c.chunk_begin);   // points of the chunk (at most 2^17)
    // tile lists: a lane feeds row lane % 32 of the tiles, which belongs to this slot of theirs
    const unsigned a_slot = (unsigned)(((lane >> 3) & 3) + (lane & 4));
    constexpr int kUnitShift = unit_blocks_of(DP) == 2 ? 6 : 5;
    const unsigned *const lists = ORD && c.lists ? c.lists + (c.chunk_begin >> kUnitShift) * kListWords : nullptr;
    const uint4 *const xp_chunk = PRE ? c.xp + (c.chunk_begin >> 5) * prep_block_u4_of(DP) : nullptr;    // chunks start on a block boundary
    unsigned listn = 0x76543210u;                    // the list of the slab being fetched (groups without lists: all tiles, fewer than eight)
    static_assert(kListMinTiles <= 8, "groups without lists");
    // the word of this lane's row slot, of the unit that holds a point of the chunk (a scalar base and a lane offset of 32 bits)
    auto list_word = [&](unsigned pt, unsigned second) -> unsigned {
        const char *const at = reinterpret_cast<const char *>(lists + (pt >> kUnitShift) * kListWords + second);
        unsigned slot = 4u * a_slot;
        asm volatile("" : "+v"(slot));
        return *reinterpret_cast<const unsigned *>(at + slot);
    };
    auto load_labels = [&](unsigned pt) -> unsigned {                    // of a point within the chunk
        return (unsigned)*reinterpret_cast<const LabWord *>(prev_chunk + (pt * (unsigned)R + lab_off));
    };
    auto fetch = [&](int slab) {
        const unsigned first = (unsigned)slab * SLAB_;                   // the slab's first point within the chunk
        const unsigned last = min((unsigned)(SLAB_ - 1), chunk_pts - 1u - first);
        if constexpr (PRE) {
            const unsigned blk_last = (chunk_pts - 1u) >> 5;
#pragma unroll
            for (int pb = 0; pb < NB; ++pb) {
                const uint4 *bp = xp_chunk + min((first >> 5) + pb, blk_last) * (unsigned)prep_block_u4_of(DP);
#pragma unroll
                for (int sl = 0; sl < NP; ++sl) pnext[pb][sl] = bp[sl * 64 + lane];
                nnext[pb] = reinterpret_cast<const uint2 *>(bp + NP * 64)[n];
                const unsigned li = min((unsigned)(pb * 32 + n), last);
                if constexpr (!FIRST) oldn[pb] = load_labels(first + li);
            }
            if constexpr (ORD) {
                if (lists) listn = list_word(first, 0u);
            }
            return;
        }
        const int64_t slab_base = c.chunk_begin + first;
        const float *Xs = c.X + slab_base * ldx;
#pragma unroll
        for (int pb = 0; pb < NB; ++pb) {
            const unsigned li = min((unsigned)(pb * 32 + n), last);
            const unsigned ro = li * ldx32;
            if (VEC) {
#pragma unroll
                for (int c4 = 0; c4 < H / 4; ++c4) {
                    const float4 v = *reinterpret_cast<const float4 *>(Xs + (ro + foff[4 * c4]));
                    xnext[pb][4 * c4 + 0] = v.x; xnext[pb][4 * c4 + 1] = v.y; xnext[pb][4 * c4 + 2] = v.z; xnext[pb][4 * c4 + 3] = v.w;
                }
            } else {
#pragma unroll
                for (int s = 0; s < H; ++s) xnext[pb][s] = Xs[ro + foff[s]];
            }
            // labels these (point, run) pairs had in the previous round, 0xff before the first one
            if (!FINAL) oldn[pb] = load_labels(first + li);
        }
    };
    // the outstanding loads of fetch() have to be complete here
    auto settle = [&]() {
        if constexpr (PRE) {
#pragma unroll
            for (int pb = 0; pb < NB; ++pb) {
#pragma unroll
                for (int sl = 0; sl < NP; ++sl)
                    asm volatile("" : "+v"(pnext[pb][sl].x), "+v"(pnext[pb][sl].y), "+v"(pnext[pb][sl].z), "+v"(pnext[pb][sl].w));
                asm volatile("" : "+v"(nnext[pb].x), "+v"(nnext[pb].y));
            }
            if constexpr (ORD) asm volatile("" : "+v"(listn));
        } else {
#pragma unroll
            for (int pb = 0; pb < NB; ++pb)
#pragma unroll
                for (int s = 0; s < H; ++s) asm volatile("" : "+v"(xnext[pb][s]));
        }
        if constexpr (!FINAL && !FIRST) {
#pragma unroll
            for (int pb = 0; pb < NB; ++pb) asm volatile("" : "+v"(oldn[pb]));
        }
    };
    // The chunk is handed out in slabs of SLAB points: one per wave statically, the rest from a counter in
    // LDS, so the waves of the workgroup finish together however their close calls and updates are spread.
    constexpr int SLAB = SLAB_;
    const int n_slabs = (int)((c.chunk_end - c.chunk_begin + SLAB - 1) / SLAB);
    // (a pass that sums the loss hands its slabs out in a fixed order instead - wave w takes slabs w, w + waves, ... -
    // so that the fp64 partial sums of a wave, and with them the reported loss, are the same in every run)
    int fixed_next = wave;
    const int n_waves = (int)(blockDim.x >> 6);
    auto grab = [&]() -> int {
        if (LOSS) {
            fixed_next += n_waves;
            return fixed_next;
        }
        int v = 0;
        // (an address known to be the same in every lane would make it a count of lanes and a scan)
        typedef __attribute__((address_space(3))) int lds_int;
        unsigned at = (unsigned)(uintptr_t)(lds_int *)c.next_slab;
        asm volatile("" : "+v"(at));
        if (lane == 0) v = __hip_atomic_fetch_add((lds_int *)(uintptr_t)at, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        return __builtin_amdgcn_readfirstlane(v);
    };
    int cur = wave;
    fetch(min(cur, n_slabs - 1));
    const bool any_wide = c.wide_s[32] != 0;
    // part of the error bound that belongs to a run (the centroids' largest squared norm), of the runs this lane owns
    float tol_runs = 0.0f;                           // (the largest over them)
#pragma unroll
    for (int st = 0; st < ST; ++st) tol_runs = fmaxf(tol_runs, c.eps_a * c.cnmax_s[S == 8 ? 0 : hl * ST + st] + kTolFloor);
    // |x'|^2 for the error bound: on the prepared copy its upper piece, which is at most 2^-7 of it below
    const float eps_x = PRE ? c.eps_a * 1.0078125f : c.eps_a;
    // accumulator rows of this lane's runs: run rl of the group begins at row rl k0 + rl (rl - 1) / 2
    const unsigned rl0 = S == 8 ? 0u : (unsigned)(hl * ST);
    const unsigned row0 = rl0 * (unsigned)c.k0 + rl0 * (rl0 - 1u) / 2u, row_step = (unsigned)c.k0 + rl0;
    double jown[ST];                                 // loss sums of the runs this lane owns
#pragma unroll
    for (int st = 0; st < ST; ++st) jown[st] = 0.0;
    // ---- moved pairs (PRE).  A pair's record names the point within the chunk and the two accumulator rows (within the group)
    // outright: point | row of the new label << 17, and the row of the old one (FIRST: 0xffff for a point that comes from nowhere).
    // A wave gathers them one per lane, in registers, and works them off 64 at a time.  (A ring in global memory, as before, drained
    // the wave's stores and waited for them to come back before the rows could be asked for: 8M x 32 8.41 -> 8.29 ms a round,
    // 64 x (262,144 x 16) 1286 -> 1256 us)
    unsigned rec_lo = 0u, rec_hi = 0u;
    int rec_n = 0;                                   // lanes 0 .. rec_n - 1 hold one
    auto log_flush = [&](int nrec) {
        // Works off `nrec` <= 64 records: a few lanes per record, eight features each (four at d_pad = 8) - the row is
        // read (16 bytes per load where rows can be read that way), put on the fixed-point grid and moved from the old
        // cluster's accumulators to the new one's.  Integer adds: the order in which records are worked off does not
        // matter.  What is the same for all lanes of a record (its fields, the row address, the accumulator rows) is
        // worked out by 4 (2, 2) lanes instead of one per feature, and a flush is 4 (2, 2) steps of 16 (32, 32) records.
        constexpr int FPL = DP >= 16 ? 8 : 4;   // features per lane
        constexpr int LPR = DP / FPL, RPS = 64 / LPR, STEPS = 64 / RPS, BATCH = STEPS < 4 ? STEPS : 4;   // steps whose rows are in flight together
        // (made opaque: what follows from the lane is worked out here, not kept in registers through the tile loop)
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const int fq = FPL * (ln % LPR), g = ln / LPR;     // this lane's first feature, its record within a step
        // this lane's feature columns in its copy of the accumulators (the lane group picks the copy)
        // (other bits of the record's number than those that order its features)
        const int cp = ((g >> 3) | (g << 2)) & (c.copies - 1);
        unsigned long long *const scol = c.sums + (int64_t)cp * c.real_rows * (DP + 1) + fq;
        const float *const xcol = c.X + c.chunk_begin * ldx + fq;
        // member counts: the lane that holds a record moves its one member, once per flush
        if (lane < nrec) {
            int *const ccol = c.cnts + (ln & (c.copies - 1)) * c.real_rows;
            const int nrow = (int)((rec_lo >> 17) & 0xfffu), orow = (int)rec_hi;
            atomicAdd(ccol + nrow, 1);
            if (!FIRST || orow != 0xffff) atomicAdd(ccol + orow, -1);
        }
        if (!any_wide) {
            // Every lane takes its features in an order of its own, feature j ^ (g mod FPL) in step j: neighbouring records move
            // between the same clusters more often than not (always where the points lie in spatial order), and the lanes of one
            // instruction would queue up at one address.  The quads are swapped by their addresses, the features inside a quad in
            // registers.  All d_pad features are moved: past the last one they are zeros, and nobody reads those sums.
            const int swz = g & (FPL - 1);
            auto order4 = [&](auto &v0, auto &v1, auto &v2, auto &v3) {
                const bool s1 = swz & 1, s2 = swz & 2;
                auto a0 = s1 ? v1 : v0, a1 = s1 ? v0 : v1, a2 = s1 ? v3 : v2, a3 = s1 ? v2 : v3;
                v0 = s2 ? a2 : a0; v1 = s2 ? a3 : a1; v2 = s2 ? a0 : a2; v3 = s2 ? a1 : a3;
            };
            const int q0 = FPL == 8 ? (swz & 4) : 0;             // first float of the quad that is taken first
            int pow2hi[FPL];
#pragma unroll
            for (int h = 0; h < FPL / 4; ++h) {
                const int4 v = *reinterpret_cast<const int4 *>(c.pow2hi_s + fq + ((4 * h) ^ q0));
                pow2hi[4 * h + 0] = v.x; pow2hi[4 * h + 1] = v.y; pow2hi[4 * h + 2] = v.z; pow2hi[4 * h + 3] = v.w;
                order4(pow2hi[4 * h], pow2hi[4 * h + 1], pow2hi[4 * h + 2], pow2hi[4 * h + 3]);
            }
            for (int s0 = 0; s0 < STEPS && s0 * RPS < nrec; s0 += BATCH) {
                unsigned lo[BATCH], hi[BATCH];
                float xv[BATCH][FPL];
#pragma unroll
                for (int u = 0; u < BATCH; ++u) {
                    const int src = (s0 + u) * RPS + g;
                    lo[u] = (unsigned)__shfl((int)rec_lo, src, 64);
                    hi[u] = (unsigned)__shfl((int)rec_hi, src, 64);
                    const bool ok = src < nrec;
                    const float *const row = xcol + (int64_t)(lo[u] & 0x1ffffu) * ldx;
#pragma unroll
                    for (int h = 0; h < FPL / 4; ++h) {
                        const int f = (4 * h) ^ q0;
                        float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                        if (VEC) {
                            if (ok && (ORD || fq + f < d)) v = *reinterpret_cast<const float4 *>(row + f);     // d is a multiple of four here
                        } else if (ok) {
                            if (fq + f + 0 < d) v.x = row[f + 0];
                            if (fq + f + 1 < d) v.y = row[f + 1];
                            if (fq + f + 2 < d) v.z = row[f + 2];
                            if (fq + f + 3 < d) v.w = row[f + 3];
                        }
                        xv[u][4 * h + 0] = v.x; xv[u][4 * h + 1] = v.y; xv[u][4 * h + 2] = v.z; xv[u][4 * h + 3] = v.w;
                    }
                }
#pragma unroll
                for (int u = 0; u < BATCH; ++u) {
                    const int src = (s0 + u) * RPS + g;
                    if (src < nrec) {
                        unsigned long long *const srow_n = scol + ((lo[u] >> 17) & 0xfffu) * (DP + 1);
                        unsigned long long *const srow_o = scol + (hi[u] & 0xffffu) * (DP + 1);
                        const int enters = FIRST && (hi[u] & 0xffffu) == 0xffffu;         // nothing to take back
#pragma unroll
                        for (int h = 0; h < FPL / 4; ++h) order4(xv[u][4 * h], xv[u][4 * h + 1], xv[u][4 * h + 2], xv[u][4 * h + 3]);
#pragma unroll
                        for (int j = 0; j < FPL; ++j) {
                            const unsigned long long v = fixed_biased(xv[u][j], pow2hi[j]);
                            const int at = j ^ swz;
                            atomicAdd(srow_n + at, v);
                            if (!FIRST || enters == 0) __hip_atomic_fetch_sub(srow_o + at, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        }
                    }
                }
            }
            return;
        }
        // some column has bits below its grid
        for (int s0 = 0; s0 < STEPS && s0 * RPS < nrec; s0 += BATCH) {
            unsigned lo[BATCH], hi[BATCH];
            float xv[BATCH][FPL];
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const int src = (s0 + u) * RPS + g;
                lo[u] = (unsigned)__shfl((int)rec_lo, src, 64);
                hi[u] = (unsigned)__shfl((int)rec_hi, src, 64);
                const bool ok = src < nrec;
                const float *const row = xcol + (int64_t)(lo[u] & 0x1ffffu) * ldx;
                if (VEC) {
#pragma unroll
                    for (int h = 0; h < FPL / 4; ++h) {
                        float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                        if (ok && fq + 4 * h < d) v = *reinterpret_cast<const float4 *>(row + 4 * h);     // d is a multiple of four here
                        xv[u][4 * h + 0] = v.x; xv[u][4 * h + 1] = v.y; xv[u][4 * h + 2] = v.z; xv[u][4 * h + 3] = v.w;
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < FPL; ++j) xv[u][j] = (ok && fq + j < d) ? row[j] : 0.0f;
                }
            }
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const int src = (s0 + u) * RPS + g;
                if (src < nrec) {
                    const int nrow = (int)((lo[u] >> 17) & 0xfffu), orow = (int)(hi[u] & 0xffffu);
                    unsigned long long *const srow_n = scol + nrow * (DP + 1);
                    unsigned long long *const srow_o = scol + orow * (DP + 1);
#pragma unroll
                    for (int j = 0; j < FPL; ++j) {
                        if (fq + j >= d) continue;
                        const unsigned long long v = (unsigned long long)to_fixed(xv[u][j], c.shift_s[fq + j]) + kFixBias;
                        atomicAdd(srow_n + j, v);
                        if (!FIRST || orow != 0xffff) __hip_atomic_fetch_sub(srow_o + j, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        if (c.wide_s[fq + j] != 0) {
                            // bits below the grid of a wide column go to a global integer accumulator (rare)
                            const long long low = fixed_low(xv[u][j], c.shift_s[fq + j]);
                            if (low != 0) {
                                if (!FIRST || orow != 0xffff) atomicAdd(reinterpret_cast<unsigned long long *>(&c.losum[(int64_t)(c.grow0 + orow) * d + fq + j]), (unsigned long long)(-low));
                                atomicAdd(reinterpret_cast<unsigned long long *>(&c.losum[(int64_t)(c.grow0 + nrow) * d + fq + j]), (unsigned long long)low);
                            }
                        }
                    }
                }
            }
        }
    };
    // puts the records of the lanes in `bal` behind those that wait; 64 of them are worked off
    auto gather = [&](bool has, unsigned long long bal, unsigned lo, unsigned hi) {
        const int n_new = (int)__popcll(bal);
        const int rank = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(bal >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0u));
        // (the lanes without a record take the places that are left: every lane sends to another one)
        const int to = (rec_n + (has ? rank : n_new + lane - rank)) & 63;
        const unsigned new_lo = (unsigned)__builtin_amdgcn_ds_permute(4 * to, (int)lo), new_hi = (unsigned)__builtin_amdgcn_ds_permute(4 * to, (int)hi);
        rec_lo = lane < rec_n ? rec_lo : new_lo;
        rec_hi = lane < rec_n ? rec_hi : new_hi;
        rec_n += n_new;
        if (rec_n >= 64) {
            log_flush(64);
            rec_n -= 64;
            rec_lo = new_lo;                         // (what came round to the first lanes)
            rec_hi = new_hi;
        }
    };
    // the words of this lane's slots 4 hl .. 4 hl + 3, from lanes that feed them
    auto slot_words = [&](unsigned w, unsigned (&out)[4]) {
#pragma unroll
        for (int a = 0; a < 4; ++a) out[a] = (unsigned)__builtin_amdgcn_ds_bpermute(16 * hl + 32 * a, (int)w);
    };
    settle();
    if (cur >= n_slabs) return;
    int nxt = grab();

    while (cur < n_slabs) {
        const int64_t base = c.chunk_begin + (int64_t)cur * SLAB;     // first point of this wave's slab
        // (a lane past the end of the chunk holds a copy of the chunk's last row: its pairs are never active)
        // (PRE: the raw rows are not there yet; the lanes that need theirs load them after the fold)
        float xraw[NB][HP];
        if constexpr (!PRE) {
#pragma unroll
            for (int pb = 0; pb < NB; ++pb) {
#pragma unroll
                for (int s = 0; s < HP; ++s) xraw[pb][s] = s < H ? xnext[pb][s] : 0.0f;
            }
        }
        if (!PRE && d < DP) {
            // padded features: the clamped loads brought real values of other features, they count as zero
#pragma unroll
            for (int pb = 0; pb < NB; ++pb)
#pragma unroll
                for (int s = 0; s < H; ++s)
                    if (s >= nf) xraw[pb][s] = 0.0f;
        }
        const int nxt2 = grab();

        // ---- B operands of this lane's points: two fp16 pieces of the centred, scaled x' per K-step, and the bias
        // slot in bf16 (|x'|^2 in three pieces on the upper half-wave, ones on the lower: it meets (1,1,1 | pieces of |c'|^2))
        f16x8 bx[NB][2][NK];
        bf16x8 bb[NB];
        float xn[NB];
        int m1[NB][ST], m2[NB][ST];
        unsigned oldl[NB];                // labels in the previous round, one byte per run of this lane
        // the tiles this slab meets: all of them in order, or those of its unit's list - this lane's slot meets its own ones
        const unsigned list = listn;
        unsigned list_more = kAllMore;
        unsigned own[4] = {list, list, list, list};    // the first words of this lane's slots 4 hl .. 4 hl + 3, from lanes that feed them
        int n_it = c.n_tiles;
        if constexpr (ORD) {
            if (lists) {
                n_it = (int)((unsigned)__builtin_amdgcn_readfirstlane((int)list) >> 28) + 1;
                if (n_it > kListHead && n_it < c.n_tiles) list_more = list_word((unsigned)cur * SLAB, 8u);
                slot_words(list, own);
                if constexpr (S < 8) {
                    kbits = key_bits(4 * S * n_it);
                    mask = key_mask(kbits);
                    asm volatile("" : "+v"(mask));
                }
            }
        }
        auto old_of = [&](int pb, int st) -> int { return (int)((oldl[pb] >> (8 * st)) & 0xffu); };
        if constexpr (PRE) {
#pragma unroll
            for (int pb = 0; pb < NB; ++pb) {
#pragma unroll
                for (int ks = 0; ks < NK; ++ks) {
                    bx[pb][0][ks] = as_f16x8(pnext[pb][0 * NK + ks]);
                    bx[pb][1][ks] = as_f16x8(pnext[pb][1 * NK + ks]);
                }
                xn[pb] = __uint_as_float(nnext[pb].x << 16);            // (the upper piece: see eps_x)
                bb[pb] = hl ? as_bf16x8(make_uint4(nnext[pb].x, nnext[pb].y, 0u, 0u)) : as_bf16x8(make_uint4(0x3f803f80u, 0x3f80u, 0u, 0u));
#pragma unroll
                for (int st = 0; st < ST; ++st) { m1[pb][st] = kBigKey; m2[pb][st] = kBigKey; }
                oldl[pb] = oldn[pb];
            }
        } else {
#pragma unroll
        for (int pb = 0; pb < NB; ++pb) {
            float xc[HP];
            float part = 0.0f;
#pragma unroll
            for (int s = 0; s < HP; ++s) {
                xc[s] = s < H ? fmaf(xraw[pb][s], c.scale, c.mu_s[f0 + s]) : 0.0f;   // (x - mean) * scale, one rounding
                part = fmaf(xc[s], xc[s], part);
            }
            xn[pb] = part + xchg32(part);
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) {
                unsigned ph[4], pl[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) split2_pair(xc[8 * ks + 2 * i], xc[8 * ks + 2 * i + 1], ph[i], pl[i]);
                bx[pb][0][ks] = as_f16x8(make_uint4(ph[0], ph[1], ph[2], ph[3]));
                bx[pb][1][ks] = as_f16x8(make_uint4(pl[0], pl[1], pl[2], pl[3]));
            }
            unsigned nh, nm, nl;
            split3(xn[pb], nh, nm, nl);
            bb[pb] = hl ? as_bf16x8(make_uint4(nh | (nm << 16), nl, 0u, 0u)) : as_bf16x8(make_uint4(0x3f803f80u, 0x3f80u, 0u, 0u));
#pragma unroll
            for (int st = 0; st < ST; ++st) { m1[pb][st] = kBigKey; m2[pb][st] = kBigKey; }
            oldl[pb] = oldn[pb];                    // fetched with the rows, a slab ago
        }
        }

        // The rows and previous labels of the next slab are asked for now and only needed when that slab starts, a
        // whole slab of work away.  Always issued - for the last slab it re-reads that slab - so that the number
        // of requests in flight is the same on every path.
        if (!LATE_FETCH) fetch(min(nxt, n_slabs - 1));

        // ---- distances tile by tile; the results of one block are folded while the matrix pipeline runs the next
        // (the tile loop is written out twice so that the operand buffers and accumulators alternate by name
        // instead of being copied)
        uint4 a_even[NS], a_odd[NS];
        // operands of step t: tile t, or the tile that is next in the list of this lane's slot
        auto load_a = [&](uint4 (&dst)[NS], int t) {
            const uint4 *at = opA_s + t * (NS * 64) + lane;
            if constexpr (ORD) at = reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(opA_s + lane) + __umul24(list_entry(list, list_more, t), NS * 1024));
#pragma unroll
            for (int sl = 0; sl < NS; ++sl) dst[sl] = at[sl * 64];
        };
        load_a(a_even, 0);
        if constexpr (NB == 1) {
            // One block per slab: the four (d_pad = 32: seven) MFMAs of a tile form one dependent chain, so the wave interleaves them in
            // program order with the fold of the tile before - a quarter of the fold (one quad of rows) behind each MFMA -
            // and the two accumulators alternate by name.  The order is pinned: left to itself the compiler folds first
            // and then issues the chain into the same registers, and nothing of the wave overlaps.
            floatx16 acc_a, acc_b = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};     // (acc_b: never read before the second tile writes it)
            int kidx_prev[NKI];
            // `init`: the first tile of a slab - the first two keys of a run start its pair of smallest keys outright
            // (no sentinel values to set up and compare against)
            auto fold_quad = [&](const floatx16 &acc, const int (&kidx)[NKI], int q, auto init) {
                const int st = state_of<S>(q);
                const bool starts = decltype(init)::value && (S == 1 || (S == 2 && (q & 1) == 0) || (S >= 4 && q == 0));
                const int ka = pack_key(acc[4 * q], mask, kidx[(4 * q) % NKI]), kb = pack_key(acc[4 * q + 1], mask, kidx[(4 * q + 1) % NKI]);
                if (starts) {
                    m1[0][st] = min(ka, kb);
                    m2[0][st] = max(ka, kb);
                } else {
                    insert2x2(ka, kb, m1[0][st], m2[0][st]);
                }
                insert2x2(pack_key(acc[4 * q + 2], mask, kidx[(4 * q + 2) % NKI]), pack_key(acc[4 * q + 3], mask, kidx[(4 * q + 3) % NKI]),
                          m1[0][st], m2[0][st]);
            };
            // `fold`: 0 nothing to fold (first tile), 1 the tile before is the slab's first, 2 any later tile
            auto tile_step = [&](const uint4 (&a_cur)[NS], uint4 (&a_nxt)[NS], int t, auto fold, floatx16 &acc_new, const floatx16 &acc_old) {
                load_a(a_nxt, t + 1 < n_it ? t + 1 : t);
                int kidx[NKI];
#pragma unroll
                for (int e = 0; e < NKI; ++e) {
                    kidx[e] = key_index<S>(t, e >> 2, e & 3);
                    asm("" : "+s"(kidx[e]));
                }
                constexpr int kFold = decltype(fold)::value;
                using Init = std::integral_constant<bool, kFold == 1>;
                const floatx16 zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
                // small cross terms first, then the leading one, then the bias slot: all in one fp32 accumulator; a quad of
                // the other accumulator is folded behind the last MFMA of each of the four parts
                acc_new = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(a_cur[1 * NK]), bx[0][0][0], zero, 0, 0, 0);               // l.h
                if constexpr (NK == 2) acc_new = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(a_cur[1 * NK + 1]), bx[0][0][1], acc_new, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (kFold) fold_quad(acc_old, kidx_prev, 0, Init{});
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int ks = 0; ks < NK; ++ks) acc_new = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(a_cur[ks]), bx[0][1][ks], acc_new, 0, 0, 0);   // h.l
                __builtin_amdgcn_sched_barrier(0);
                if (kFold) fold_quad(acc_old, kidx_prev, 1, Init{});
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int ks = 0; ks < NK; ++ks) acc_new = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(a_cur[ks]), bx[0][0][ks], acc_new, 0, 0, 0);   // h.h
                __builtin_amdgcn_sched_barrier(0);
                if (kFold) fold_quad(acc_old, kidx_prev, 2, Init{});
                __builtin_amdgcn_sched_barrier(0);
                acc_new = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a_cur[2 * NK]), bb[0], acc_new, 0, 0, 0);                 // norms
                __builtin_amdgcn_sched_barrier(0);
                if (kFold) fold_quad(acc_old, kidx_prev, 3, Init{});
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int e = 0; e < NKI; ++e) kidx_prev[e] = kidx[e];
            };
            using NoFold = std::integral_constant<int, 0>;
            using FoldFirst = std::integral_constant<int, 1>;
            using FoldLater = std::integral_constant<int, 2>;
            tile_step(a_even, a_odd, 0, NoFold{}, acc_a, acc_b);
            if (n_it == 1) {
#pragma unroll
                for (int q = 0; q < 4; ++q) fold_quad(acc_a, kidx_prev, q, std::true_type{});
            } else {
                tile_step(a_odd, a_even, 1, FoldFirst{}, acc_b, acc_a);
                int t = 2;
                for (; t + 2 <= n_it; t += 2) {
                    tile_step(a_even, a_odd, t, FoldLater{}, acc_a, acc_b);
                    tile_step(a_odd, a_even, t + 1, FoldLater{}, acc_b, acc_a);
                }
                if (t < n_it) {
                    tile_step(a_even, a_odd, t, FoldLater{}, acc_a, acc_b);
                    fold_tile<S, ST>(acc_a, kidx_prev, mask, m1[0], m2[0]);
                } else {
                    fold_tile<S, ST>(acc_b, kidx_prev, mask, m1[0], m2[0]);
                }
            }
        } else {
        floatx16 acc_prev;                 // results of the block before the current one, folded one block late
            int kidx_old[NKI];
            // `first`: the very first block of the slab has no block before it to fold
            auto tile_step = [&](const uint4 (&a_cur)[NS], uint4 (&a_nxt)[NS], int t, auto first) {
                load_a(a_nxt, t + 1 < n_it ? t + 1 : t);
                // per-row key indices of this tile as opaque scalars (one scalar operand per and-or)
                int kidx[NKI];
#pragma unroll
                for (int e = 0; e < NKI; ++e) {
                    kidx[e] = key_index<S>(t, e >> 2, e & 3);
                    asm("" : "+s"(kidx[e]));
                }
#pragma unroll
                for (int pb = 0; pb < NB; ++pb) {
                    // small cross terms first, then the leading one, then the bias slot: all in one fp32 accumulator
                    floatx16 acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
                    for (int ks = 0; ks < NK; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(a_cur[1 * NK + ks]), bx[pb][0][ks], acc, 0, 0, 0);   // l.h
#pragma unroll
                    for (int ks = 0; ks < NK; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(a_cur[0 * NK + ks]), bx[pb][1][ks], acc, 0, 0, 0);   // h.l
#pragma unroll
                    for (int ks = 0; ks < NK; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(a_cur[0 * NK + ks]), bx[pb][0][ks], acc, 0, 0, 0);   // h.h
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a_cur[2 * NK]), bb[pb], acc, 0, 0, 0);                                         // norms
                    if (pb == 0) {
                        if (!decltype(first)::value) fold_tile<S, ST>(acc_prev, kidx_old, mask, m1[NB - 1], m2[NB - 1]);
                    } else {
                        fold_tile<S, ST>(acc_prev, kidx, mask, m1[pb - 1], m2[pb - 1]);
                    }
#pragma unroll
                    for (int s = 0; s < NM; ++s) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // one MFMA
                        __builtin_amdgcn_sched_group_barrier(0x002, VPER, 0);   // then a share of the fold
                    }
                    acc_prev = acc;
                }
#pragma unroll
                for (int e = 0; e < NKI; ++e) kidx_old[e] = kidx[e];
            };
            {
                tile_step(a_even, a_odd, 0, std::true_type{});
                int t = 1;
                for (; t + 2 <= n_it; t += 2) {
                    tile_step(a_odd, a_even, t, std::false_type{});
                    tile_step(a_even, a_odd, t + 1, std::false_type{});
                }
                if (t < n_it) tile_step(a_odd, a_even, t, std::false_type{});
            }
            fold_tile<S, ST>(acc_prev, kidx_old, mask, m1[NB - 1], m2[NB - 1]);
        }
        // The keys hold steps of the lists: the step becomes the tile that the winner's slot met there.  The index is then in the
        // lowest seven bits (six where runs have one slot), whatever else the key holds.  (The second key's index is not used.)
        auto steps_to_tiles = [&]() {
            constexpr int kStepShift = S == 1 ? 2 : (S == 2 ? 3 : (S == 4 ? 4 : 5));
            constexpr unsigned kTileMask = (15u << kStepShift) & 127u;       // (16, 16, 8, 4 tiles at most)
            // four times the step: it is a list's entry, of four bits
            const unsigned step_mask = (unsigned)~mask >> kStepShift << 2;
            auto shift_of = [&](int key) -> unsigned { return (S == 1 ? (unsigned)key : (unsigned)key >> (kStepShift - 2)) & step_mask; };
            // the word of the slot that a run's key came from (selects by bit masks: an index would put the words in memory)
            auto either = [](unsigned w0, unsigned w1, int key, int bit) { return w0 ^ ((w0 ^ w1) & (0u - (((unsigned)key >> bit) & 1u))); };
            auto pick = [&](const unsigned (&w)[4], int st, int key) -> unsigned {
                if (S == 1) return w[st];
                if (S == 2) return st == 0 ? either(w[0], w[1], key, 2) : either(w[2], w[3], key, 2);
                return either(either(w[0], w[1], key, 2), either(w[2], w[3], key, 2), key, 3);
            };
            auto put = [&](int &key, unsigned tile) { key = (int)(((tile << kStepShift) & kTileMask) | ((unsigned)key & ~kTileMask)); };
            if (n_it <= kListHead) {
#pragma unroll
                for (int pb = 0; pb < NB; ++pb)
#pragma unroll
                    for (int st = 0; st < ST; ++st) put(m1[pb][st], pick(own, st, m1[pb][st]) >> shift_of(m1[pb][st]));
            } else if (S < 8 && n_it == c.n_tiles) {
                // (all tiles in their order: a step is its tile.  Eight slots have four tiles at most, and their keys are still wanted)
#pragma unroll
                for (int pb = 0; pb < NB; ++pb)
#pragma unroll
                    for (int st = 0; st < ST; ++st) m1[pb][st] &= ~mask;
            } else {
                unsigned more[4];
                slot_words(list_more, more);
#pragma unroll
                for (int pb = 0; pb < NB; ++pb)
#pragma unroll
                    for (int st = 0; st < ST; ++st) {
                        const int key = m1[pb][st];
                        put(m1[pb][st], list_entry(pick(own, st, key), pick(more, st, key), (int)(shift_of(key) >> 2)));
                    }
            }
        };
        if (ORD && S == 8 && lists) steps_to_tiles();
        if (LATE_FETCH) fetch(min(nxt, n_slabs - 1));

        // ---- labels, close calls, sums
        constexpr int NBST = NB * ST;               // (block, run) pairs a lane owns
        // this lane's points within the chunk, and whether they exist (the last slab of a chunk may be ragged)
        const unsigned pt0 = (unsigned)cur * SLAB;
        unsigned ptl[NB];
        bool pvalid[NB];
#pragma unroll
        for (int pb = 0; pb < NB; ++pb) {
            ptl[pb] = pt0 + (unsigned)(pb * 32 + n);
            pvalid[pb] = ptl[pb] < chunk_pts;
        }
        // Keys: which pairs does the exact arithmetic have to confirm?  Bit pb * ST + st of a lane's mask, put together
        // only when the wave has such a pair at all.
        unsigned pend = 0;
        float clear[NB][ST];                        // by how much the second key is above the first
        bool any_close = false;
        const float shrink = key_shrink(kbits);
#pragma unroll
        for (int pb = 0; pb < NB; ++pb) {
            if (S == 8) {
                // the run spans both half-waves: add the half bit to the index, then merge with the partner lane
                int k1 = m1[pb][0], k2 = m2[pb][0];
                if (k1 < kBigKey) k1 |= hl << 4;
                if (k2 < kBigKey) k2 |= hl << 4;
                const int o1 = xchg32(k1), o2 = xchg32(k2);
                insert2(o1, k1, k2);
                insert2(o2, k1, k2);
                m1[pb][0] = k1; m2[pb][0] = k2;
            }
            // Error bound of the two expansions (rounding of norms, products and the centring) plus the mantissa bits given up to
            // the index.  The keys are compared as they are, index bits included (see key_shrink; a negative first key - a distance
            // of zero within the bound - is smaller than the bound's own slack).
#pragma unroll
            for (int st = 0; st < ST; ++st) clear[pb][st] = fmaf(__int_as_float(m2[pb][st]), shrink, -__int_as_float(m1[pb][st]));
            if (c.n_runs < R) {
                asm volatile("");                   // (a branch: few groups have slots without a run, which hold padding rows only)
#pragma unroll
                for (int st = 0; st < ST; ++st) clear[pb][st] = ((actmask >> (8 * st)) & 0xffu) != 0u ? clear[pb][st] : INFINITY;
            }
            float least = clear[pb][0];
#pragma unroll
            for (int st = 1; st < ST; ++st) least = fminf(least, clear[pb][st]);
            any_close = any_close || !(least > fmaf(eps_x, xn[pb], tol_runs));
        }
        // from here on m1 holds indices
        if (ORD && lists) {
            if constexpr (S < 8) steps_to_tiles();
        } else {
#pragma unroll
            for (int pb = 0; pb < NB; ++pb)
#pragma unroll
                for (int st = 0; st < ST; ++st) m1[pb][st] &= ~mask;
        }
        if (__builtin_amdgcn_ballot_w64(any_close) != 0ull) {
#pragma unroll
            for (int pb = 0; pb < NB; ++pb)
#pragma unroll
                for (int st = 0; st < ST; ++st) {
                    const bool close = pvalid[pb] && (S < 8 || hl == 0) && !(clear[pb][st] > fmaf(eps_x, xn[pb], tol_runs));
                    pend |= (unsigned)close << (pb * ST + st);
                }
            if constexpr (ORD && S <= 2) {
                // Where points lie close together their close calls come together as well (on knob data whole blocks of points tie
                // exactly), and a wave that settles 256 of them one by one holds up its launch.  Many at a time are settled by the
                // lanes that own them, each its own pair: the exact arithmetic over the centroids that the unit's lists name.
                // One by one they take 100 to 350 instructions each, together 75 per listed centroid, of which there are 4 S n_it: with a
                // short list eight pairs are enough, with more than kListHead tiles on it 1.5 pairs per slot and tile.  (Eight whatever the
                // length: 200,003 x 16 integers 0..3, k 1..64, 10 rounds 2.97 ms, 2.46 now; the same of 0..1 3.26 and 3.15.  Long lists
                // one by one always: 2.46 and 4.02.)
                const int kMany = n_it <= kListHead ? 8 : 3 * S * n_it / 2;
                if (lists && __popcll(__builtin_amdgcn_ballot_w64(pend != 0u)) >= kMany) {
                int half = hl;                           // (opaque: nothing of this is worked out ahead of the branch)
                asm volatile("" : "+v"(half));
#pragma unroll
                for (int i = 0; i < NBST; ++i) {
                    const int pb = i / ST, st = i % ST;
                    const bool mine = (pend >> i) & 1u;
                    if (__popcll(__builtin_amdgcn_ballot_w64(mine)) < kMany) continue;
                    if (mine) {
                        float x[DP];
                        const float *const row = c.X + c.chunk_begin * DP + ptl[pb] * (unsigned)DP;
#pragma unroll
                        for (int l = 0; l < DP; l += 4) {
                            const float4 v = *reinterpret_cast<const float4 *>(row + l);
                            x[l] = v.x; x[l + 1] = v.y; x[l + 2] = v.z; x[l + 3] = v.w;
                        }
                        const int rl = half * ST + st, k = c.k0 + rl, rowbase = rl * c.k0 + rl * (rl - 1) / 2;
                        double best = INFINITY;
                        int arg = 0, at = 0;             // the nearest so far: its index, its place
                        for (int a = 0; a < S; ++a) {
                            const unsigned slot = (unsigned)(half * 4 + st * S + a);
                            const unsigned head = lists[(pt0 >> kUnitShift) * kListWords + slot], more = lists[(pt0 >> kUnitShift) * kListWords + 8 + slot];
                            for (int q = 0; q < 4 * n_it; ++q) {
                                const int tile = (int)list_entry(head, more, q >> 2);
                                const int place = 4 * (S * tile + a) + (q & 3);
                                if (place >= k) continue;                        // padding
                                const int j = (int)c.rowidx[rowbase + place];
                                const double dist = exact_distance<DP>(x, c.cs + (rowbase + j) * CS);
                                if (dist < best || (dist == best && j < arg)) { best = dist; arg = j; at = place; }
                            }
                        }
                        m1[pb][st] = at;
                        pend &= ~(1u << i);
                    }
                }
                }
            }
        }

        // A close call (about one pair in a thousand on knob data; every pair where centroids coincide or integer
        // data ties exactly) is settled by the whole wave with the exact arithmetic over the run.  The point's row is
        // read out of the registers of the two lanes that hold its halves.
        auto settle_close_calls = [&](const float (&xr)[NB][HP]) {
            unsigned long long todo = __builtin_amdgcn_ballot_w64(pend != 0u);
            while (todo) {
                const int src = __ffsll((long long)todo) - 1;
                const unsigned sbits = (unsigned)__builtin_amdgcn_readlane((int)pend, src);
                const int idx = __ffs(sbits) - 1, pb = idx / ST, st = idx % ST;
                const int srl = S == 8 ? 0 : (src >> 5) * ST + st;
                const float *crun = c.cs + (srl * c.k0 + srl * (srl - 1) / 2) * CS;
                float xs[DP];
#pragma unroll
                for (int s = 0; s < H; ++s) {
                    float v = xr[0][s];
#pragma unroll
                    for (int q = 1; q < NB; ++q)
                        if (pb == q) v = xr[q][s];
                    xs[s] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), src & 31));
                    xs[H + s] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), (src & 31) + 32));
                }
                int arg = exact_argmin_wave<DP>(xs, crun, CS, c.k0 + srl);
                if constexpr (ORD) {
                    const int rowbase = srl * c.k0 + srl * (srl - 1) / 2;
                    arg = (int)c.rowpos[rowbase + arg] - rowbase;
                }
                if (lane == src) {
                    pend &= pend - 1u;
#pragma unroll
                    for (int i = 0; i < NBST; ++i)
                        if (i == idx) m1[i / ST][i % ST] = arg;
                }
                todo = __builtin_amdgcn_ballot_w64(pend != 0u);
            }
        };
        if constexpr (PRE) {
            // Raw rows on demand: the exact arithmetic of a close call needs the point's row; both lanes of such a
            // point (each holds half of the features) load their half.  (The exact sums need the rows of the points
            // whose label changed: those are read when the wave works off the moved pairs it has gathered.)  Loads, wait and
            // scans sit in one branch, so that a slab without close calls never waits on the memory counter here: what
            // is in flight then are the operands of the next slab, wanted a whole slab later.
            if (__builtin_amdgcn_ballot_w64(pend != 0u) != 0ull) {
                unsigned need = pend;
                need |= xchg32(need);
                float xr[NB][HP];
#pragma unroll
                for (int pb = 0; pb < NB; ++pb)
#pragma unroll
                    for (int s = 0; s < HP; ++s) xr[pb][s] = 0.0f;
                const float *Xs = c.X + base * ldx;
                // (the row index is made opaque here so that the offsets below are worked out on the spot: hoisted out
                // of the slab loop they would sit in registers, or in spill slots, through the tile loop)
                unsigned nrow = (unsigned)n;
                asm volatile("" : "+v"(nrow));
#pragma unroll
                for (int pb = 0; pb < NB; ++pb) {
                    if ((need >> (pb * ST)) & ((1u << ST) - 1u)) {       // an active pair: the point lies inside the chunk
                        const unsigned ro = ((unsigned)(pb * 32) + nrow) * ldx32;
                        if (VEC) {
#pragma unroll
                            for (int c4 = 0; c4 < H / 4; ++c4) {
                                const float4 v = *reinterpret_cast<const float4 *>(Xs + (ro + feat_off(4 * c4)));
                                xr[pb][4 * c4 + 0] = v.x; xr[pb][4 * c4 + 1] = v.y; xr[pb][4 * c4 + 2] = v.z; xr[pb][4 * c4 + 3] = v.w;
                            }
                        } else {
#pragma unroll
                            for (int s = 0; s < H; ++s) xr[pb][s] = Xs[ro + feat_off(s)];
                        }
                        if (!ORD && d < DP) {                    // (the ordered copy's rows are padded with zeros)
#pragma unroll
                            for (int s = 0; s < H; ++s)
                                if (s >= nf) xr[pb][s] = 0.0f;
                        }
                    }
                }
                // the rows have to be there before the branch ends (the wait belongs to this path alone)
#pragma unroll
                for (int pb = 0; pb < NB; ++pb)
#pragma unroll
                    for (int s = 0; s < H; ++s) asm volatile("" : "+v"(xr[pb][s]));
                settle_close_calls(xr);
            }
        } else {
            settle_close_calls(xraw);
        }

        // labels are final: the new label word of every block, and which of its bytes differ from the last round's
        // (the stores wait until the end of the slab)
        unsigned neww[NB], diffw[NB];
        unsigned mv = 0;                            // bit pb * ST + st: that pair moved
#pragma unroll
        for (int pb = 0; pb < NB; ++pb) {
            // the indices side by side (byte permutes)
            unsigned w;
            if constexpr (ST == 4) {
                w = (__builtin_amdgcn_perm((unsigned)m1[pb][1], (unsigned)m1[pb][0], 0x0c0c0400u) |
                     __builtin_amdgcn_perm((unsigned)m1[pb][3], (unsigned)m1[pb][2], 0x04000c0cu));
            } else if constexpr (ST == 2) {
                w = __builtin_amdgcn_perm((unsigned)m1[pb][1], (unsigned)m1[pb][0], 0x0c0c0400u);
            } else {
                w = (unsigned)m1[pb][0];
            }
            if constexpr (ORD) w &= S == 1 ? 0x3f3f3f3fu : 0x7f7f7f7fu;          // (all else that the keys hold)
            neww[pb] = w;
            diffw[pb] = 0u;
            if constexpr (!FINAL && !FIRST) diffw[pb] = pvalid[pb] ? ((w ^ oldl[pb]) & actmask) : 0u;
        }
        if constexpr (!FINAL && !PRE) {
            bool any = false;
#pragma unroll
            for (int pb = 0; pb < NB; ++pb) any = any || diffw[pb] != 0u;
            if (__builtin_amdgcn_ballot_w64(any) != 0ull) {
#pragma unroll
                for (int pb = 0; pb < NB; ++pb)
#pragma unroll
                    for (int st = 0; st < ST; ++st) mv |= (unsigned)(((diffw[pb] >> (8 * st)) & 0xffu) != 0u) << (pb * ST + st);
            }
        }

        auto new_of = [&](int pb, int st) -> int { return (int)((neww[pb] >> (8 * st)) & 0xffu); };
        if constexpr (PRE) {
            // Exact sums, later: the moved pairs are gathered, and worked off 64 at a time.
            unsigned fromw[NB];                                 // the labels before: where the point comes from, 0xff: from nowhere
#pragma unroll
            for (int pb = 0; pb < NB; ++pb) fromw[pb] = FIRST ? 0u : oldl[pb];
            if constexpr (FIRST) {
                // No point has a label yet, so every one enters a cluster of every run - but the centroids of a run are those of
                // the run before and one more, and most points keep the nearest one they had there.  Only the group's first
                // run is filled point by point; a later run logs the points whose centroid is another one than in the run
                // before it, as moves, and its sums are those of the run before plus what its own moves change (put together
                // when the workgroup is done).  (Wide columns: their low-order sums are global, every run is filled.)
#pragma unroll
                for (int pb = 0; pb < NB; ++pb) {
                    int idx[ST];                                // the labels as indices
#pragma unroll
                    for (int st = 0; st < ST; ++st) {
                        const unsigned rb = row0 + (unsigned)st * row_step + (unsigned)(st * (st - 1) / 2);
                        const bool real = ((actmask >> (8 * st)) & 0xffu) != 0u && pvalid[pb];
                        idx[st] = real ? (int)c.rowidx[rb + (unsigned)new_of(pb, st)] : 0;
                    }
                    const int below = xchg32(idx[ST - 1]);      // the last run of the lower half-wave
#pragma unroll
                    for (int st = 0; st < ST; ++st) {
                        const unsigned rb = row0 + (unsigned)st * row_step + (unsigned)(st * (st - 1) / 2);
                        const bool real = ((actmask >> (8 * st)) & 0xffu) != 0u && pvalid[pb];
                        const bool fills = any_wide || (hl == 0 && st == 0);
                        const int before = st == 0 ? below : idx[st > 0 ? st - 1 : 0];
                        const bool logs = real && (fills || before != idx[st]);
                        const unsigned from = fills ? 0xffu : (unsigned)c.rowpos[logs ? rb + (unsigned)before : 0u] - rb;
                        const unsigned to = (unsigned)new_of(pb, st);
                        fromw[pb] |= (logs ? from : to) << (8 * st);
                        diffw[pb] |= logs ? (from ^ to) << (8 * st) : 0u;
                    }
                }
            }
            unsigned any_diff = 0u;
#pragma unroll
            for (int pb = 0; pb < NB; ++pb) any_diff |= diffw[pb];
            if (__builtin_amdgcn_ballot_w64(any_diff != 0u) != 0ull) {
                // (one run slot after the other, not unrolled: working off is a thousand instructions)
                unsigned moved = diffw[0], now = fromw[0] ^ diffw[0], was = fromw[0], pt = ptl[0];
                unsigned rowbase = row0, step = row_step;
#pragma nounroll
                for (int i = 0; i < NBST; ++i) {
                    const bool has = (moved & 0xffu) != 0u;
                    const unsigned long long bal = __builtin_amdgcn_ballot_w64(has);
                    if (bal != 0ull) {
                        const unsigned o = was & 0xffu;
                        gather(has, bal, pt | ((rowbase + (now & 0xffu)) << 17), FIRST && o == 0xffu ? 0xffffu : rowbase + o);   // rows: below 2^12
                    }
                    moved >>= 8;
                    now >>= 8;
                    was >>= 8;
                    rowbase += step;
                    ++step;
                    if (NB > 1 && i == ST - 1) {
                        moved = diffw[NB - 1]; now = fromw[NB - 1] ^ diffw[NB - 1]; was = fromw[NB - 1]; pt = ptl[NB - 1];
                        rowbase = row0; step = row_step;
                    }
                }
            }
        }
        if (!FINAL && !PRE) {
            // Exact sums: a point whose label changed moves its fixed-point row from the old cluster to the new
            // one.  Both lanes of the point's pair take part (each holds half of the features); one pair per pass.
            const unsigned mvo = xchg32(mv);
            unsigned both = hl ? (mvo | (mv << NBST)) : (mv | (mvo << NBST));
            // bits below the grid of a wide column go to a global integer accumulator (rare)
            auto add_low = [&](int64_t p, int rowbase, int ol, int nl) {
                const int64_t crow = c.grow0 + rowbase;
                for (int s = 0; s < nf; ++s) {
                    if (c.wide_s[f0 + s] == 0) continue;
                    const long long lo = fixed_low(c.X[p * c.ldx + f0 + s], c.shift_s[f0 + s]);
                    if (lo == 0) continue;
                    if (ol != 0xff) atomicAdd(reinterpret_cast<unsigned long long *>(&c.losum[(crow + ol) * d + f0 + s]), (unsigned long long)(-lo));
                    atomicAdd(reinterpret_cast<unsigned long long *>(&c.losum[(crow + nl) * d + f0 + s]), (unsigned long long)lo);
                }
            };
            if (__ballot(both != 0u) != 0ull) {
                // this lane's half of its points' rows on the fixed-point grid (zero beyond the last feature)
                unsigned long long fx[NB][H];
                if (any_wide) {
                    // some column has bits below its grid: those are cut off here (and summed apart, see add_low)
#pragma unroll
                    for (int pb = 0; pb < NB; ++pb)
#pragma unroll
                        for (int s = 0; s < H; ++s) fx[pb][s] = (unsigned long long)to_fixed(xraw[pb][s], c.shift_s[f0 + s]) + kFixBias;
                } else {
#pragma unroll
                    for (int pb = 0; pb < NB; ++pb)
#pragma unroll
                        for (int s = 0; s < H; ++s) fx[pb][s] = fixed_biased(xraw[pb][s], c.pow2hi_s[f0 + s]);   // xraw is 0 past the last feature
                }
                if (c.first_round) {
                    // no point has a label yet: every pair of the slab enters its cluster, run by run
#pragma unroll
                    for (int pb = 0; pb < NB; ++pb) {
                        const int64_t p = base + pb * 32 + n;
                        for (int r = 0; r < c.n_runs; ++r) {
                            const int oh = S == 8 ? 0 : r / ST, ost = S == 8 ? 0 : r % ST;
                            int nl = 0;
#pragma unroll
                            for (int st = 0; st < ST; ++st)
                                if (st == ost) nl = m1[pb][st];
                            const int nlo = xchg32(nl);
                            if (hl != oh) nl = nlo;
                            const int rowbase = r * c.k0 + r * (r - 1) / 2;
                            if (pvalid[pb]) {
                                unsigned long long *sn = sums_l + (rowbase + nl) * (DP + 1) + f0;
#pragma unroll
                                for (int s = 0; s < H; ++s) atomicAdd(sn + s, fx[pb][s]);
                                if (hl == 0) atomicAdd(&cnts_l[rowbase + nl], 1);
                                if (any_wide) add_low(p, rowbase, 0xff, nl);
                            }
                        }
                    }
                } else do {
                    const bool act = both != 0u;
                    const int bit = act ? __ffs(both) - 1 : 0;
                    both &= both - 1u;
                    const int oh = bit / NBST, idx = bit % NBST, pb = idx / ST, st = idx % ST;
                    int kk = 0;                         // the owner's (old << 8) | new
#pragma unroll
                    for (int i = 0; i < NBST; ++i)
                        if (i == idx) kk = m1[i / ST][i % ST] | (old_of(i / ST, i % ST) << 8);
                    const int kko = xchg32(kk);
                    if (hl != oh) kk = kko;
                    const int nl = kk & 0xff, ol = kk >> 8;
                    const int r = S == 8 ? 0 : oh * ST + st;
                    const int rowbase = r * c.k0 + r * (r - 1) / 2;
                    if (act) {
                        unsigned long long *sn = sums_l + (rowbase + nl) * (DP + 1) + f0;
                        unsigned long long v[H];
#pragma unroll
                        for (int s = 0; s < H; ++s) {
                            v[s] = fx[0][s];
#pragma unroll
                            for (int q = 1; q < NB; ++q)
                                if (pb == q) v[s] = fx[q][s];
                            atomicAdd(sn + s, v[s]);
                        }
                        if (hl == 0) atomicAdd(&cnts_l[rowbase + nl], 1);
                        if (ol != 0xff) {   // 0xff: no label yet, nothing to take back
                            unsigned long long *so = sums_l + (rowbase + ol) * (DP + 1) + f0;
#pragma unroll
                            for (int s = 0; s < H; ++s)
                                __hip_atomic_fetch_sub(so + s, v[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                            if (hl == 0) atomicAdd(&cnts_l[rowbase + ol], -1);
                        }
                        if (any_wide) add_low(base + pb * 32 + n, rowbase, ol, nl);
                    }
                } while (__ballot(both != 0u) != 0ull);
            }
        }
        if (LOSS) {
            // Loss of this assignment: every lane sums, for each (point, run) pair it owns, the exact squared distance
            // to the assigned centroid over all features in rising order; the other half of the row comes from the
            // partner lane by register swap.  Padded features are zero on both sides and add +0.
#pragma unroll
            for (int pb = 0; pb < NB; ++pb) {
                float xf[DP];
#pragma unroll
                for (int s = 0; s < H; ++s) {
                    const float other = xchg32(xraw[pb][s]);
                    xf[s] = hl ? other : xraw[pb][s];
                    xf[H + s] = hl ? xraw[pb][s] : other;
                }
#pragma unroll
                for (int st = 0; st < ST; ++st) {
                    const int rl = S == 8 ? 0 : hl * ST + st;
                    const bool active = ((S == 8) ? (hl == 0) : true) && rl < c.n_runs && pvalid[pb];
                    const int row = active ? rl * c.k0 + rl * (rl - 1) / 2 + m1[pb][st] : 0;
                    const double dist = exact_distance<DP>(xf, c.cs + row * CS);
                    if (active) jown[st] = __dadd_rn(jown[st], dist);
                }
            }
        }
        // The rows of the next slab have to be there now.  Asking here, before this slab's stores are issued, keeps
        // the in-order memory counter from tying the next slab to those stores.
        settle();
#pragma unroll
        for (int pb = 0; pb < NB; ++pb) {
            const int64_t p = base + pb * 32 + n;
            if (FINAL) {
#pragma unroll
                for (int st = 0; st < ST; ++st) {
                    const int rl = S == 8 ? 0 : hl * ST + st;
                    const bool active = ((S == 8) ? (hl == 0) : true) && rl < c.n_runs && p < c.chunk_end;
                    const unsigned off = run_off[st] + (unsigned)(pb * 32 + n);      // used for active pairs only: inside the chunk
                    if (active && c.labels_out) (c.labels_out + base)[off] = m1[pb][st];
                }
            } else {
                // a word with a changed byte is written back whole (bytes of run slots without a run are never looked at)
                if (FIRST ? pvalid[pb] && actmask != 0u : diffw[pb] != 0u)
                    *reinterpret_cast<LabWord *>(prev_chunk + (ptl[pb] * (unsigned)R + lab_off)) = (LabWord)neww[pb];
            }
        }
        cur = nxt;
        nxt = nxt2;
    }
    if constexpr (PRE) {
        if (rec_n > 0) log_flush(rec_n);
    }
    if (LOSS) {
        // hand the sums over by run: run r of the group is owned by half-wave r / ST (by the lower one when S = 8)
#pragma unroll
        for (int r = 0; r < 8 / S; ++r) {
            const int oh = S == 8 ? 0 : r / ST, ost = S == 8 ? 0 : r % ST;
            jloc[r] = hl == oh ? jown[ost] : 0.0;
        }
    }
}

// The tile lists of the workgroup's units, 32 units per wave at a time: their centres take the place of 32 points.
//
// For a unit with centre b and radius r, and a run whose centroid nearest to b is m, every point x of the unit has
// |x - c_m| <= |b - c_m| + r and |x - c_j| >= |b - c_j| - r: a centroid with |b - c_j| > |b - c_m| + 2 r is not the nearest of
// any of them.  A quad of centroids stays when its smallest distance to b is within that bound; the distances are the
// matrix pipeline's, so they enter with twice their error bound (which leaves a margin between the winner and what is left
// out that no rounding of the exact arithmetic reaches).  The quads' distances stay in registers until the bound is known.
// Cost: some 25 instructions per tile and 150 more for 32 units, where a tile left out saves a unit 50.
template <int DP, int S>
__device__ __forceinline__ void make_lists(const WaveCtx &c, const uint4 *centres, const float *radius, unsigned *lists)
{
    constexpr int NK = ksteps_of(DP), NS = tile_slots_of(DP), NP = prep_slots_of(DP), UP = 32 * unit_blocks_of(DP);
    constexpr int ST = S == 1 ? 4 : (S == 2 ? 2 : 1);
    const int lane = threadIdx.x & 63, n = lane & 31, hl = lane >> 5;
    const int u0 = (int)(c.chunk_begin / UP), u1 = (int)((c.chunk_end + UP - 1) / UP);
    const floatx16 zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (int blk = (u0 >> 5) + (int)(threadIdx.x >> 6); blk * 32 < u1; blk += (int)(blockDim.x >> 6)) {
        const uint4 *bp = centres + (int64_t)blk * prep_block_u4_of(DP);
        f16x8 bh[NK], bl[NK];
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) {
            bh[ks] = as_f16x8(bp[ks * 64 + lane]);
            bl[ks] = as_f16x8(bp[(NK + ks) * 64 + lane]);
        }
        const uint2 nn = reinterpret_cast<const uint2 *>(bp + NP * 64)[n];
        const float rad = radius[blk * 32 + n];
        const float bn = (__uint_as_float(nn.x << 16) + __uint_as_float(nn.x & 0xffff0000u)) + __uint_as_float(nn.y << 16);
        const bf16x8 bb = hl ? as_bf16x8(make_uint4(nn.x, nn.y, 0u, 0u)) : as_bf16x8(make_uint4(0x3f803f80u, 0x3f80u, 0u, 0u));
        // the smallest distance of each quad of this lane's slots, and of each run
        float quad[kListMaxTiles][4], lim[ST];
#pragma unroll
        for (int st = 0; st < ST; ++st) lim[st] = 2.0f * kPadNorm;
#pragma unroll
        for (int t = 0; t < kListMaxTiles; ++t) {
            if (t >= c.n_tiles) continue;
            const uint4 *at = c.opA_s + t * NS * 64 + lane;
            floatx16 acc = zero;
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(at[(NK + ks) * 64]), bh[ks], acc, 0, 0, 0);
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(at[ks * 64]), bl[ks], acc, 0, 0, 0);
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(at[ks * 64]), bh[ks], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(at[2 * NK * 64]), bb, acc, 0, 0, 0);
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                quad[t][a] = fminf(fminf(acc[4 * a], acc[4 * a + 1]), fminf(acc[4 * a + 2], acc[4 * a + 3]));
                lim[state_of<S>(a)] = fminf(lim[state_of<S>(a)], quad[t][a]);
            }
        }
#pragma unroll
        for (int st = 0; st < ST; ++st) {
            if (S == 8) lim[st] = fminf(lim[st], xchg32(lim[st]));
            const float err = fmaf(c.eps_a, bn + c.cnmax_s[S == 8 ? 0 : hl * ST + st], kTolFloor);
            const float reach = sqrtf(fmaxf(lim[st], 0.0f) + err) + 2.0f * rad;
            lim[st] = lim[st] < 0.5f * kPadNorm ? fmaf(reach, reach * 1.00001f, 2.0f * err) : -1.0f;     // (-1: a slot without a run)
        }
        unsigned in[4] = {0u, 0u, 0u, 0u};                   // bit t: tile t is on the slot's list
#pragma unroll
        for (int t = 0; t < kListMaxTiles; ++t) {
            if (t >= c.n_tiles) continue;
#pragma unroll
            for (int a = 0; a < 4; ++a) in[a] |= quad[t][a] <= lim[state_of<S>(a)] ? 1u << t : 0u;
        }
        int longest = max(max(__popc(in[0]), __popc(in[1])), max(__popc(in[2]), __popc(in[3])));
        longest = max(max(longest, xchg32(longest)), 1);
        const unsigned all = (1u << c.n_tiles) - 1u;
        if (longest > kListHead && longest == c.n_tiles - 1) longest = c.n_tiles;
        unsigned head[4], more[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            head[a] = (unsigned)(longest - 1) << 28;
            more[a] = 0u;
            if (longest == c.n_tiles) in[a] = all;
            in[a] |= (all & ~in[a]) << 16;                   // behind the tiles on the list the others
        }
        // (as many entries as the longest list of these units has)
        auto next = [&](int a) -> unsigned {
            const unsigned e = (unsigned)(__ffs(in[a]) - 1) & 15u;
            in[a] &= in[a] - 1u;
            return e;
        };
        for (int i = 0; i < kListHead && __builtin_amdgcn_ballot_w64(i < longest) != 0ull; ++i)
#pragma unroll
            for (int a = 0; a < 4; ++a) head[a] |= next(a) << (4 * i);
        const bool any_more = __builtin_amdgcn_ballot_w64(longest > kListHead) != 0ull;
        if (any_more)
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int a = 0; a < 4; ++a) more[a] |= next(a) << (4 * i);
        const int u = blk * 32 + n;
        if (u >= u0 && u < u1) {
            uint4 *out = reinterpret_cast<uint4 *>(lists + (int64_t)u * kListWords) + hl;
            out[0] = make_uint4(head[0], head[1], head[2], head[3]);
            if (any_more) out[2] = make_uint4(more[0], more[1], more[2], more[3]);
        }
    }
}

template <int DP, bool FINAL, bool TRACE, bool VEC, bool PRE, bool ORD, bool FIRST>
__device__ inline void wave_loop_of(int S, const WaveCtx &c, double (&jloc)[8])
{
    switch (S) {
    case 1: wave_loop<DP, 1, FINAL, TRACE, VEC, PRE, ORD, FIRST>(c, jloc); break;
    case 2: wave_loop<DP, 2, FINAL, TRACE, VEC, PRE, ORD, FIRST>(c, jloc); break;
    case 4: wave_loop<DP, 4, FINAL, TRACE, VEC, PRE, ORD, FIRST>(c, jloc); break;
    default: wave_loop<DP, 8, FINAL, TRACE, VEC, PRE, ORD, FIRST>(c, jloc); break;
    }
}

// The groups, one per lane: all are asked for together, and the one that a workgroup belongs to is found and taken from the
// lane that has it.  (Walked one by one every group was a trip to the kernel's arguments, which no cache holds when a launch
// begins: step and centroid launches 0.3 to 0.8 us longer.)
static_assert(kMaxGroups <= 64, "one group per lane");
static_assert(sizeof(GroupDesc) % 4 == 0, "taken over word by word");
__device__ inline GroupDesc group_of_lane(const SweepPlan &plan) { return plan.g[min((int)(threadIdx.x & 63), kMaxGroups - 1)]; }
// the number of groups in the front that satisfy `holds` in their lanes, less one
__device__ inline int last_group(const SweepPlan &plan, bool holds)
{
    return __popcll(__builtin_amdgcn_ballot_w64((int)(threadIdx.x & 63) < plan.n_groups && holds)) - 1;
}
__device__ inline GroupDesc take_group(const GroupDesc &mine, int gi)
{
    int w[sizeof(GroupDesc) / 4];
    __builtin_memcpy(w, &mine, sizeof(w));
#pragma unroll
    for (unsigned i = 0; i < sizeof(GroupDesc) / 4; ++i) w[i] = __builtin_amdgcn_readlane(w[i], gi);
    GroupDesc g;
    __builtin_memcpy(&g, w, sizeof(w));
    return g;
}

template <int DP, bool FINAL, bool TRACE, bool PRE, bool ORD, bool FIRST>
__global__ void __launch_bounds__(step_threads_of(DP)) lloyd_step_kernel(SweepPlan plan, StepArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int TH = step_threads_of(DP), WV = TH / 64;

    // Workgroup order.  Large inputs: the chunks of all spaces of the batch, numbered space by space, are taken in blocks of
    // plan.chunk_block; within a block the groups go heaviest first (the dispatcher hands workgroups out in index order,
    // light ones fill the end), and the workgroups of all groups for one chunk sit a multiple of eight apart - they run
    // at about the same time on the same XCD, so that what one of them reads of the chunk (its rows or its part of the
    // prepared copy) the others find in that XCD's L2.
    // Small inputs (chunk_block 0): every group has chunks of its own, of about equal cost over all groups, one per compute
    // unit; the chunks of a group that land on one XCD (every eighth workgroup) follow each other in the points.
    int gi, chunk, b;
    const GroupDesc mine = group_of_lane(plan);
    if (plan.chunk_block > 0) {
        const int B = plan.chunk_block;
        const int n_chunks = plan.g[0].n_chunks;
        const int n_all = n_chunks * a.batch;               // chunks of the whole batch
        const int per_block = B * plan.n_groups;
        const int blk = blockIdx.x / per_block, rem = blockIdx.x % per_block;
        const int c0 = blk * B;
        const int bw = min(B, n_all - c0);                  // chunks of this block (the last one may be short)
        gi = plan.sched[rem / bw];
        const int vc = c0 + rem % bw;
        b = vc / n_chunks;
        chunk = vc - b * n_chunks;
    } else {
        b = blockIdx.x / plan.n_wgs;
        const int v = blockIdx.x - b * plan.n_wgs;
        gi = last_group(plan, mine.wg0 <= v);
        const GroupDesc g = take_group(mine, gi);
        const int r = v - g.wg0, nc = g.n_chunks;
        const int first = blockIdx.x - r;                   // launch index of the group's first workgroup
        chunk = r >> 3;
        for (int q = 0; q < (int)(blockIdx.x & 7); ++q) chunk += (nc - ((q - first) & 7) + 7) >> 3;   // chunks of the XCDs before this one
    }
    // The division leaves these in vector registers although they are the same in every lane.  At d_pad 32 the
    // kernel sits at the limit of 256 vector registers and spilled 35 of them over it (3% longer launches); as
    // scalars they cost none.
    b = __builtin_amdgcn_readfirstlane(b);
    chunk = __builtin_amdgcn_readfirstlane(chunk);
    gi = __builtin_amdgcn_readfirstlane(gi);
    const int bad = a.status[b];                    // (looked at below, when it has come with everything else)
    const GroupDesc g = take_group(mine, gi);
    const int d = a.d;
    const int k0 = plan.k_min + g.run0;                                   // k of the group's first run
    const int grow0 = rows_before(plan.k_min, g.run0);                    // first centroid row of the group
    const int real_rows = rows_before(plan.k_min, g.run0 + g.n_runs) - grow0;
    const int copies = g.copies;
    const Carve cv = carve_lds(DP, d, g.n_tiles, real_rows, copies, ORD);

    uint4 *opA_s = reinterpret_cast<uint4 *>(smem + cv.opA);
    float *cs_lds = reinterpret_cast<float *>(smem + cv.cs);
    unsigned long long *sums = reinterpret_cast<unsigned long long *>(smem + cv.sums);
    int *cnts = reinterpret_cast<int *>(smem + cv.cnts);
    unsigned short *rowpos_s = reinterpret_cast<unsigned short *>(smem + cv.rowpos);
    unsigned char *rowidx_s = smem + cv.rowidx;
    float *mu_s = reinterpret_cast<float *>(smem + cv.misc);              // [32]
    int *shift_s = reinterpret_cast<int *>(smem + cv.misc + 128);         // [32]
    int *wide_s = reinterpret_cast<int *>(smem + cv.misc + 256);          // [32] + any at [32]
    float *cnmax_s = reinterpret_cast<float *>(smem + cv.misc + 400);     // [8]
    int *next_slab = reinterpret_cast<int *>(smem + cv.misc + 448);
    int *pow2hi_s = reinterpret_cast<int *>(smem + cv.misc + 1536);       // [32]
    double *jpart = reinterpret_cast<double *>(smem + cv.misc + 512);     // [8][WV]

    const int tid = threadIdx.x;
    char *wsb = a.ws + (int64_t)b * a.ws_bs;
    const float *Xb = a.X + (int64_t)b * a.x_bs;
    const float *Cb = a.C + (int64_t)b * a.c_bs;

    // group operands, centroids and column info into LDS; accumulators to zero.  Everything is requested in batches
    // before anything is put down (ten trips to memory for the centroids, four for the operands and one per part of a run
    // for the largest norms took 8 us of a launch of 42 at 65,536 x 16, k 1..64; now 6).
    {
        const float *colmean = reinterpret_cast<const float *>(wsb + a.off_colinfo);
        const int *colshift = reinterpret_cast<const int *>(wsb + a.off_colinfo + 128);
        const int *colwide = reinterpret_cast<const int *>(wsb + a.off_colinfo + 256);
        const float mean_v = colmean[tid & (DP - 1)];
        const int shift_v = colshift[tid & 31], wide_v = colwide[min(tid, 32)];
        // the largest squared norm of a run's centroids: the centroid kernel leaves one maximum per part of the run
        static_assert(kMaxParts == 16 && TH >= 128, "sixteen lanes per run");
        float pmax = 0.0f;
        {
            const int r = (tid >> 4) & 7, part = tid & 15;
            if (r < g.n_runs && part < (k0 + r + kPartRows - 1) / kPartRows)
                pmax = reinterpret_cast<const float *>(wsb + a.off_cnmax)[(g.run0 + r) * kMaxParts + part];
        }
        const uint4 *src = reinterpret_cast<const uint4 *>(wsb + a.off_opA + (int64_t)g.tile0 * tile_bytes_of(DP));
        const float *csrc = Cb + (int64_t)grow0 * d;
        const int n_op = g.n_tiles * (tile_bytes_of(DP) / 16), n_cs = real_rows * DP;
        auto stage = [&](auto op_batch, auto cs_batch) {
            constexpr int UO = decltype(op_batch)::value, UC = decltype(cs_batch)::value;
            for (int i0 = 0; i0 * TH * UO < n_op || i0 * TH * UC < n_cs; ++i0) {
                uint4 v[UO];
#pragma unroll
                for (int u = 0; u < UO; ++u) v[u] = src[min(tid + (i0 * UO + u) * TH, n_op - 1)];
                float w[UC];
#pragma unroll
                for (int u = 0; u < UC; ++u) {
                    const int e = min(tid + (i0 * UC + u) * TH, n_cs - 1);
                    w[u] = csrc[(e / DP) * d + min(e % DP, d - 1)];
                }
                if (!FINAL && i0 == 0) {                 // (while the loads are on their way)
                    for (int e = tid; e < copies * real_rows * (DP + 1); e += TH) sums[e] = 0ull;
                    for (int e = tid; e < copies * real_rows; e += TH) cnts[e] = 0;
                }
#pragma unroll
                for (int u = 0; u < UO; ++u) {
                    const int e = tid + (i0 * UO + u) * TH;
                    if (e < n_op) opA_s[e] = v[u];
                }
#pragma unroll
                for (int u = 0; u < UC; ++u) {
                    const int e = tid + (i0 * UC + u) * TH;
                    if (e < n_cs) cs_lds[(e / DP) * (DP + 4) + e % DP] = e % DP < d ? w[u] : 0.0f;
                }
            }
        };
        // A batch takes the loads it is made for, whatever there is to load: small groups take one of their own (2003 x 8, k = 8: 9.8 -> 8.1 us
        // a launch; sweeps of one group below 20,000 points 4% shorter), and skipping loads one by one made the compiler wait between
        // them (65,536 x 16, k 1..64: 4% longer sweeps).
        if (n_op <= TH && n_cs <= 2 * TH) stage(std::integral_constant<int, 1>{}, std::integral_constant<int, 2>{});
        else stage(std::integral_constant<int, 6>{}, std::integral_constant<int, 12>{});
        if (tid < 32) {
            mu_s[tid] = tid < DP ? mean_v : 0.0f;                          // colmean: already negated and scaled
            shift_s[tid] = shift_v;
            pow2hi_s[tid] = (1023 + shift_v) << 20;                        // 2^shift as a double: the high word
        }
        if (tid < 33) wide_s[tid] = wide_v;
        if constexpr (ORD) {
            const unsigned short *rowpos = reinterpret_cast<const unsigned short *>(wsb + a.off_rowpos) + grow0;
            const unsigned char *rowidx = reinterpret_cast<const unsigned char *>(wsb + a.off_rowidx) + grow0;
            for (int e = tid; e < real_rows; e += TH) {
                rowpos_s[e] = rowpos[e];
                rowidx_s[e] = rowidx[e];
            }
        }
        if (tid == 0) *next_slab = WV;
        if (bad != 0) return;
        if (tid < 128) {
#pragma unroll
            for (int off = 8; off >= 1; off >>= 1) pmax = fmaxf(pmax, __shfl_xor(pmax, off, 64));
            if ((tid & 15) == 0) cnmax_s[tid >> 4] = pmax;
        }
    }
    __syncthreads();

    WaveCtx c;
    c.opA_s = opA_s;
    c.cs = cs_lds;            // the group's centroids as given, rows padded to d + 4 floats
    c.next_slab = next_slab;
    c.sums = sums; c.cnts = cnts; c.copies = copies; c.real_rows = real_rows; c.mu_s = mu_s; c.shift_s = shift_s; c.pow2hi_s = pow2hi_s; c.wide_s = wide_s; c.cnmax_s = cnmax_s;
    c.scale = *reinterpret_cast<const float *>(wsb + a.off_colinfo + kColScaleOff);
    c.xp = reinterpret_cast<const uint4 *>(wsb + a.off_xp);
    c.rowpos = rowpos_s;
    c.rowidx = rowidx_s;
    c.lists = nullptr;
    c.X = Xb; c.ldx = a.ldx; c.N = a.N; c.d = d; c.k0 = k0; c.n_runs = g.n_runs; c.n_tiles = g.n_tiles; c.grow0 = grow0;
    c.prev = reinterpret_cast<unsigned char *>(wsb + a.off_prev) + (int64_t)g.lab0 * ((a.N + 15) / 16 * 16);
    c.labels_out = (FINAL && a.labels) ? a.labels + (int64_t)b * a.lab_bs + (int64_t)g.run0 * a.N : nullptr;
    c.losum = reinterpret_cast<long long *>(wsb + a.off_losum);
    c.chunk_begin = (int64_t)chunk * g.chunk_len;
    c.chunk_end = min(a.N, c.chunk_begin + g.chunk_len);
    // 16-byte loads need whole quads of features and aligned rows
    c.first_round = a.first_round != 0;
    c.vec_x = (d % 4 == 0) && (a.ldx % 4 == 0) && ((reinterpret_cast<uintptr_t>(Xb) & 15) == 0);
    if constexpr (ORD) {
        c.X = reinterpret_cast<const float *>(wsb + a.off_xs);
        c.ldx = DP;
    }
    c.eps_a = pair_error_of(DP);

    if constexpr (ORD) {
        if (g.list0 >= 0) {
            const int64_t n_units = (a.N + 32 * unit_blocks_of(DP) - 1) / (32 * unit_blocks_of(DP));
            unsigned *lists = reinterpret_cast<unsigned *>(wsb + a.off_lists) + g.list0 * n_units * kListWords;
            const uint4 *centres = reinterpret_cast<const uint4 *>(wsb + a.off_centres);
            const float *radius = reinterpret_cast<const float *>(wsb + a.off_radius);
            switch (g.S) {
            case 1: make_lists<DP, 1>(c, centres, radius, lists); break;
            case 2: make_lists<DP, 2>(c, centres, radius, lists); break;
            case 4: make_lists<DP, 4>(c, centres, radius, lists); break;
            default: make_lists<DP, 8>(c, centres, radius, lists); break;
            }
            c.lists = lists;
            __syncthreads();
        }
    }

    double jloc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) jloc[i] = 0.0;

    // (a chunk is never empty)
    if constexpr (ORD) {
        wave_loop_of<DP, FINAL, TRACE, true, PRE, ORD, FIRST>(g.S, c, jloc);
    } else {
        if (c.vec_x) wave_loop_of<DP, FINAL, TRACE, true, PRE, ORD, FIRST>(g.S, c, jloc);
        else wave_loop_of<DP, FINAL, TRACE, false, PRE, ORD, FIRST>(g.S, c, jloc);
    }

    if (FINAL || TRACE) {
        const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            double v = jloc[i];
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) v = __dadd_rn(v, __shfl_xor(v, off, 64));
            if (lane == 0) jpart[i * WV + wave] = v;
        }
    }
    __syncthreads();   // every wave has finished its points: accumulators and partial losses are complete

    if (!FINAL) {
        unsigned long long *psum = reinterpret_cast<unsigned long long *>(wsb + a.off_psum) +
                                   ((int64_t)g.part0 + (int64_t)chunk * real_rows) * d;
        int *pcnt = reinterpret_cast<int *>(wsb + a.off_pcnt) + (int64_t)g.part0 + (int64_t)chunk * real_rows;
        if constexpr (FIRST) {
            // the accumulator rows that make up a centroid after a first round on the ordered copy: its own and, unless a column is
            // wide, those of the same centroid in the group's earlier runs (see FIRST above)
            const bool adds_up = c.wide_s[32] == 0;
            auto each_row = [&](int e, auto &&use) {
                use((int)rowpos_s[e]);
                if (adds_up) {
                    int r = 0;
                    while (r + 1 < g.n_runs && (r + 1) * k0 + (r + 1) * r / 2 <= e) ++r;
                    const int j = e - (r * k0 + r * (r - 1) / 2);
                    for (int q = r - 1; q >= 0 && j < k0 + q; --q) use((int)rowpos_s[q * k0 + q * (q - 1) / 2 + j]);
                }
            };
            for (int e = tid; e < real_rows * d; e += TH) {
                unsigned long long v = 0ull;
                long long rows_in = 0;     // rows that entered minus rows that left: each carried the bias once
                each_row(e / d, [&](int row) {
                    for (int cp = 0; cp < copies; ++cp) {
                        v += sums[(cp * real_rows + row) * (DP + 1) + e % d];
                        rows_in += cnts[cp * real_rows + row];
                    }
                });
                psum[e] = v - kFixBias * (unsigned long long)rows_in;
            }
            for (int e = tid; e < real_rows; e += TH) {
                int v = 0;
                each_row(e, [&](int row) {
                    for (int cp = 0; cp < copies; ++cp) v += cnts[cp * real_rows + row];
                });
                pcnt[e] = v;
            }
        } else {
            // Several elements or copies at a time, whose reads are under way together (one by one, the flush of 484 rows of 16
            // took 6200 cycles, now 1500).  The count of a row's members is read with each of its features.
            static_assert(TH % DP == 0, "a thread keeps its feature");
            const int l = tid % DP;
            auto flush = [&](auto elements, auto copies_at_once) {
                constexpr int U = decltype(elements)::value, Q = decltype(copies_at_once)::value;
                for (int row0 = tid / DP; row0 < real_rows; row0 += U * (TH / DP)) {
                    unsigned long long v[U];
                    int rows_in[U], at[U];     // rows that entered minus rows that left: each carried the bias once
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int row = min(row0 + u * (TH / DP), real_rows - 1);
                        at[u] = ORD ? (int)rowpos_s[row] : row;
                        v[u] = 0ull;
                        rows_in[u] = 0;
                    }
                    for (int cp = 0; cp < copies; cp += Q) {           // (both are powers of two: Q copies are there)
#pragma unroll
                        for (int q = 0; q < Q; ++q)
#pragma unroll
                            for (int u = 0; u < U; ++u) {
                                const int row = (cp + q) * real_rows + at[u];
                                v[u] += sums[row * (DP + 1) + l];
                                rows_in[u] += cnts[row];
                            }
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int row = row0 + u * (TH / DP);
                        if (row < real_rows && l < d) {
                            psum[row * d + l] = v[u] - kFixBias * (unsigned long long)(long long)rows_in[u];
                            if (l == 0) pcnt[row] = rows_in[u];
                        }
                    }
                }
            };
            if (copies == 1) flush(std::integral_constant<int, 4>{}, std::integral_constant<int, 1>{});
            else if (copies == 2) flush(std::integral_constant<int, 2>{}, std::integral_constant<int, 2>{});
            else flush(std::integral_constant<int, 1>{}, std::integral_constant<int, 4>{});
        }
    }
    if (FINAL || TRACE) {
        if (tid < g.n_runs) {
            double v = 0.0;
            for (int w = 0; w < WV; ++w) v = __dadd_rn(v, jpart[tid * WV + w]);
            reinterpret_cast<double *>(wsb + a.off_pj)[(int64_t)(g.wg0 + chunk) * 8 + tid] = v;
        }
    }
}

// ---- column statistics: mean (for centring), fixed-point shift and range check ----------------
struct ColPart {
    double sum;
    int min_lsb, max_msb, bad, pad;
    float vmin, vmax;     // smallest and largest value (of a column that is not bad)
    double sumsq;         // (for the order of the points only)
};

static_assert(kStatBlocks * 32 * sizeof(ColPart) >= kSeedExchangeBytes, "the seeding chain's exchange area lies in this block");

__device__ inline void add_part(ColPart &t, const ColPart &o)
{
    t.sum = __dadd_rn(t.sum, o.sum);
    t.sumsq += o.sumsq;
    t.min_lsb = min(t.min_lsb, o.min_lsb);
    t.max_msb = max(t.max_msb, o.max_msb);
    t.bad |= o.bad;
    t.vmin = fminf(t.vmin, o.vmin);
    t.vmax = fmaxf(t.vmax, o.vmax);
}

// A thread takes one column of every T / dp-th row.  What bounds it is the work per value and the waves that hide its loads: without a
// branch per value, the highest bit taken once from the extremes, and where one space has to fill the chip, or has long columns, 16 waves per workgroup
// instead of 8 (us, 512 | 1024 threads: 1M x 16 28 | 22, 300,007 x 13 10.4 | 9.6, 4 x (1M x 16) 71 | 67).  With many spaces the chip is full as it is, and with
// few values per thread putting them together is what is left (64 x (262,144 x 16) 265 | 293, 64 x (262,144 x 8) 142 | 180, 64 x (20,000 x 16)
// 27 | 43, 64 x (2000 x 8) 5.4 | 7.2, 16 x (1M x 16) 251 | 256, 2000 x 8 4.8 | 5.4).  (512 threads with a branch per value: 32, 11.7, 72, 260, 148, 28, 6.5, 248, 5.4.)
constexpr int kStatFew = 512;
inline int stat_threads(int64_t N, int dp, int stat_blocks, int batch)
{
    const int64_t rows = (N + stat_blocks - 1) / stat_blocks, workgroups = (int64_t)stat_blocks * batch;
    return (workgroups <= 256 && rows * dp > 4096) || (workgroups <= 1024 && rows >= 4096) ? 1024 : kStatFew;
}
template <int T>
__global__ void __launch_bounds__(T) colstats_kernel(const float *__restrict__ X, int64_t N, int d, int dp, int64_t ldx,
                                                    int64_t x_bs, char *ws, int64_t ws_bs, int64_t off_part)
{
    __shared__ ColPart sh[T];
    const int b = blockIdx.y;
    const float *Xb = X + (int64_t)b * x_bs;
    const int tid = threadIdx.x;
    const int l = tid % dp, pg = tid / dp, ppp = T / dp;
    const int64_t per = (N + gridDim.x - 1) / gridDim.x;
    const int64_t r0 = (int64_t)blockIdx.x * per, r1 = min(N, r0 + per);
    ColPart c = {0.0, 1 << 20, -(1 << 20), 0, 0, INFINITY, -INFINITY, 0.0};
    if (l < d) {
        // eight rows of this thread's column in flight at a time (the walk is bound by their latency); the values
        // are taken in row order, so the sum does not depend on the depth
        constexpr int U = 8;
        for (int64_t rb = r0 + pg; rb < r1; rb += (int64_t)U * ppp) {
            float xs[U];
#pragma unroll
            for (int u = 0; u < U; ++u) xs[u] = Xb[min(rb + (int64_t)u * ppp, r1 - 1) * ldx + l];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (rb + (int64_t)u * ppp >= r1) continue;
                const float x = xs[u];
                const unsigned bits = __float_as_uint(x);
                const int e = (int)((bits >> 23) & 0xffu);
                c.bad |= e == 255 ? 1 : 0;                   // (nothing else of such a column is used)
                c.sum = __dadd_rn(c.sum, (double)x);
                c.sumsq = fma((double)x, (double)x, c.sumsq);
                c.vmin = fminf(c.vmin, x);
                c.vmax = fmaxf(c.vmax, x);
                const unsigned m = (bits & 0x7fffffu) | (e != 0 ? 0x800000u : 0u);
                const int lsb = max(e, 1) - 151 + __ffs((int)m);
                c.min_lsb = min(c.min_lsb, m != 0u ? lsb : 1 << 20);
            }
        }
        const unsigned far = max(__float_as_uint(fabsf(c.vmin)), __float_as_uint(fabsf(c.vmax)));      // (of no values: infinity, and a column of them is bad)
        if (r0 + pg < r1 && (far & 0x7fffffffu) != 0u) {
            const int e = (int)(far >> 23);
            c.max_msb = e != 0 ? e - 127 : (31 - __clz((int)far)) - 149;
        }
    }
    sh[tid] = c;
    __syncthreads();
    // eight threads per column add up an eighth each, then one of them the eight (in a fixed order)
    if (tid < 8 * dp) {
        for (int g = tid + 8 * dp; g < T; g += 8 * dp) add_part(c, sh[g]);
        sh[tid] = c;
    }
    __syncthreads();
    if (tid < dp) {
        for (int g = 1; g < 8; ++g) add_part(c, sh[g * dp + tid]);
        reinterpret_cast<ColPart *>(ws + (int64_t)b * ws_bs + off_part)[blockIdx.x * 32 + tid] = c;
    }
}

__global__ void __launch_bounds__(256) colstats_final_kernel(int64_t N, int d, int n_blocks, char *ws, int64_t ws_bs, int64_t off_part,
                                                            int64_t off_colinfo, int64_t off_keyinfo, int32_t *status)
{
    // 256 threads: eight walk the partial results of one column, every eighth block each, eight loads in flight (the
    // walk is bound by their latency); the eight are then combined in a fixed order, so the mean is the same in every run
    constexpr int G = 8, U = 8;
    __shared__ int flags;
    __shared__ ColPart comb[G][32];
    __shared__ unsigned char place_s[32][12];
    static_assert(kKeyColBits <= 12, "places of a column's bits");
    const int b = blockIdx.x, l = threadIdx.x & 31, g = threadIdx.x >> 5;
    if (threadIdx.x == 0) flags = 0;
    const ColPart *part = reinterpret_cast<const ColPart *>(ws + (int64_t)b * ws_bs + off_part);
    ColPart t = {0.0, 1 << 20, -(1 << 20), 0, 0, INFINITY, -INFINITY, 0.0};
    if (l < d) {
        for (int g0 = g; g0 < n_blocks; g0 += G * U) {
            ColPart o[U];
#pragma unroll
            for (int u = 0; u < U; ++u) o[u] = part[min(g0 + u * G, n_blocks - 1) * 32 + l];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (g0 + u * G >= n_blocks) continue;
                t.sum = __dadd_rn(t.sum, o[u].sum);
                t.sumsq += o[u].sumsq;
                t.min_lsb = min(t.min_lsb, o[u].min_lsb);
                t.max_msb = max(t.max_msb, o[u].max_msb);
                t.bad |= o[u].bad;
                t.vmin = fminf(t.vmin, o[u].vmin);
                t.vmax = fmaxf(t.vmax, o[u].vmax);
            }
        }
    }
    comb[g][l] = t;
    __syncthreads();
    float mean = 0.0f;
    int shift = 0, wide = 0, msb = -(1 << 20);
    if (g == 0) {
        if (l < d) {
            for (int q = 1; q < G; ++q) {
                const ColPart o = comb[q][l];
                t.sum = __dadd_rn(t.sum, o.sum);
                t.sumsq += o.sumsq;
                t.min_lsb = min(t.min_lsb, o.min_lsb);
                t.max_msb = max(t.max_msb, o.max_msb);
                t.bad |= o.bad;
                t.vmin = fminf(t.vmin, o.vmin);
                t.vmax = fmaxf(t.vmax, o.vmax);
            }
            if (t.bad) atomicOr(&flags, RLS_STATUS_NONFINITE);
            else {
                mean = (float)(t.sum / (double)N);
                // largest distance of a value (or of a centroid, which lies between the extremes) from the mean; the
                // exponent of the next power of two above it, with the rounding of the two differences allowed for
                const float reach = fmaxf(t.vmax - mean, mean - t.vmin) * 1.000001f;
                if (reach > 0.0f) msb = ilogbf(reach);
                if (t.max_msb >= t.min_lsb) {
                    // grid: the finest bit kept by the main accumulator. |x * 2^shift| < 2^kGridBits, and a chunk moves
                    // at most 2^17 rows in and out of a cluster within 63 bits. Bits below the grid (wide columns) go to
                    // the low accumulator, which keeps kLowBits more; anything finer cannot be summed exactly.
                    int grid = t.max_msb - (kGridBits - 1);
                    if (grid < t.min_lsb) grid = t.min_lsb;
                    shift = -grid;
                    if (t.min_lsb < grid) wide = 1;
                    if (t.min_lsb < grid - kLowBits) atomicOr(&flags, RLS_STATUS_RANGE);
                }
            }
        }
        float *colmean = reinterpret_cast<float *>(ws + (int64_t)b * ws_bs + off_colinfo);
        int *colshift = reinterpret_cast<int *>(ws + (int64_t)b * ws_bs + off_colinfo + 128);
        int *colwide = reinterpret_cast<int *>(ws + (int64_t)b * ws_bs + off_colinfo + 256);
        // One power of two for all columns (distances keep their order): with |x - mean| < 2^(M+1) in every column the
        // centred values obey |x - mean| * 2^(kScaledMsb - M - 2) < 2^(kScaledMsb - 1), one bit inside what fp16 holds for
        // 2 c'.  The exponent is kept inside the fp32 range: no distance from the mean reaches 2^129 (an infinite one, rounded up, counts
        // as that), and data that asks for more than 2^100 is so small that every comparison is a close call.
        // (the 32 threads of the columns are the lower half of one wave: the exchange stays among them)
        for (int off = 16; off >= 1; off >>= 1) msb = max(msb, __shfl_xor(msb, off, 64));
        int e = kScaledMsb - 2 - (msb > -(1 << 20) ? msb : 0);
        e = min(max(e, kScaledMsb - 2 - 128), 100);
        const float scale = ldexpf(1.0f, e);
        colmean[l] = -(mean * scale);      // what the kernels add after multiplying by the scale
        colshift[l] = shift;
        colwide[l] = wide;
        if (l == 0) *reinterpret_cast<float *>(ws + (int64_t)b * ws_bs + off_colinfo + kColScaleOff) = scale;
        if (wide) atomicOr(&flags, 1 << 16);
        if (off_keyinfo >= 0) {
            // bits of the ordering key: each goes to the column whose cells are the widest, against the column's spread
            KeyInfo *ki = reinterpret_cast<KeyInfo *>(ws + (int64_t)b * ws_bs + off_keyinfo);
            const double mu = t.sum / (double)N;
            float width = l < d && !t.bad ? sqrtf((float)fmax(t.sumsq / (double)N - mu * mu, 0.0)) : 0.0f;
            if (!(width < INFINITY)) width = 0.0f;
            int nb = 0;
            for (int s = 0; s < kKeyBits; ++s) {
                const float top = half_max_f32(width);
                const unsigned long long who = __ballot(width == top);
                if (top > 0.0f && l == __ffsll((long long)who) - 1) {
                    place_s[l][nb++] = (unsigned char)(kKeyBits - 1 - s);
                    width = nb < kKeyColBits ? width * 0.5f : 0.0f;
                }
            }
            const unsigned long long with = __ballot(nb > 0);
            const float range = t.vmax - t.vmin;
            int first = nb > 0 ? 1 << nb : 0;                     // inclusive, then exclusive sums over the columns
            for (int off = 1; off < 32; off <<= 1) {
                const int o = __shfl_up(first, off, 64);
                if (l >= off) first += o;
            }
            if (nb > 0) {
                const int at = __popcll(with & ((1ull << l) - 1ull));
                ki->col[at] = l;
                ki->bits[at] = nb;
                ki->first[at] = first - (1 << nb);
                ki->lo[at] = t.vmin;
                ki->mul[at] = range > 0.0f && range < INFINITY ? (float)(1 << nb) / range : 0.0f;
                for (int i = 0; i < nb; ++i) ki->place[at][i] = place_s[l][i];
            }
            if (l == 0) ki->n_cols = __popcll(with);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int *colwide = reinterpret_cast<int *>(ws + (int64_t)b * ws_bs + off_colinfo + 256);
        colwide[32] = (flags >> 16) & 1;
        status[b] = flags & 0xffff;
    }
}

// ---- the prepared copy of the points (see prep_block_u4_of): what the step kernel would derive from a row in every
//      launch and for every group of runs - centring, scaling, the two fp16 pieces, the squared norm - done once per sweep.
//      One thread per (point, half of the features), in the lane order of the step kernel; the arithmetic is the
//      step kernel's own, instruction for instruction.
template <int DP>
__global__ void __launch_bounds__(256) lloyd_prepare_kernel(const float *__restrict__ X, int64_t N, int d, int64_t ldx, int64_t x_bs,
                                                            const int32_t *__restrict__ status, char *ws, int64_t ws_bs,
                                                            int64_t off_colinfo, int64_t off_xp)
{
    constexpr int H = DP / 2, NK = ksteps_of(DP), HP = 8 * NK;
    const int b = blockIdx.y;
    if (status[b] != 0) return;
    char *wsb = ws + (int64_t)b * ws_bs;
    const float *Xb = X + (int64_t)b * x_bs;
    const float *colmean = reinterpret_cast<const float *>(wsb + off_colinfo);      // -(mean * scale)
    const float scale = *reinterpret_cast<const float *>(wsb + off_colinfo + kColScaleOff);
    uint4 *xp = reinterpret_cast<uint4 *>(wsb + off_xp);
    const int64_t n_blocks = (N + 31) / 32;
    const int lane = threadIdx.x & 63, n = lane & 31, hl = lane >> 5;
    const int f0 = hl * H;
    for (int64_t blk = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); blk < n_blocks;
         blk += (int64_t)gridDim.x * (blockDim.x >> 6)) {
        const int64_t p = blk * 32 + n;
        float xc[HP];
        float part = 0.0f;
#pragma unroll
        for (int s = 0; s < HP; ++s) {
            const int f = f0 + s;
            const float x = (s < H && f < d && p < N) ? Xb[p * ldx + f] : 0.0f;
            // a point past the end and a padded feature count as a zero of the centred data
            xc[s] = (s < H && f < d && p < N) ? fmaf(x, scale, colmean[f]) : 0.0f;
            part = fmaf(xc[s], xc[s], part);
        }
        const float xn = part + xchg32(part);
        uint4 *bp = xp + blk * prep_block_u4_of(DP);
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) {
            unsigned ph[4], pl[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) split2_pair(xc[8 * ks + 2 * i], xc[8 * ks + 2 * i + 1], ph[i], pl[i]);
            bp[(0 * NK + ks) * 64 + lane] = make_uint4(ph[0], ph[1], ph[2], ph[3]);
            bp[(1 * NK + ks) * 64 + lane] = make_uint4(pl[0], pl[1], pl[2], pl[3]);
        }
        if (hl == 0) {
            unsigned nh, nm, nl;
            split3(xn, nh, nm, nl);
            reinterpret_cast<uint2 *>(bp + prep_slots_of(DP) * 64)[n] = make_uint2(nh | (nm << 16), nl);
        }
    }
}

// ---- the same for an ordered sweep: the copy is in the order of the places, the rows go along (padded with zeros to DP
//      floats, so that rows of any length are read 16 bytes at a time later on), and every unit leaves its centre - the mean
//      of its points as the operand pieces hold it - and an upper bound of the distance from there to its points.
template <int DP>
__global__ void __launch_bounds__(256) lloyd_prepare_ordered_kernel(const float *__restrict__ X, int64_t N, int d, int64_t ldx, int64_t x_bs,
                                                                    const int32_t *__restrict__ status, char *ws, int64_t ws_bs,
                                                                    int64_t off_colinfo, int64_t off_perm, int64_t off_xp, int64_t off_xs,
                                                                    int64_t off_centres, int64_t off_radius)
{
    constexpr int H = DP / 2, NK = ksteps_of(DP), HP = 8 * NK, UB = unit_blocks_of(DP);
    const int b = blockIdx.y;
    if (status[b] != 0) return;
    char *wsb = ws + (int64_t)b * ws_bs;
    const float *Xb = X + (int64_t)b * x_bs;
    const bool vec = (d % 4 == 0) && (ldx % 4 == 0) && ((reinterpret_cast<uintptr_t>(Xb) & 15) == 0);
    const float *colmean = reinterpret_cast<const float *>(wsb + off_colinfo);      // -(mean * scale)
    const float scale = *reinterpret_cast<const float *>(wsb + off_colinfo + kColScaleOff);
    const int32_t *perm = reinterpret_cast<const int32_t *>(wsb + off_perm);
    uint4 *xp = reinterpret_cast<uint4 *>(wsb + off_xp), *centres = reinterpret_cast<uint4 *>(wsb + off_centres);
    float *xs = reinterpret_cast<float *>(wsb + off_xs), *radius = reinterpret_cast<float *>(wsb + off_radius);
    const int64_t n_blocks = (N + 31) / 32, n_units = (n_blocks + UB - 1) / UB;
    const int lane = threadIdx.x & 63, n = lane & 31, hl = lane >> 5;
    const int f0 = hl * H;
    float mean_h[H];
#pragma unroll
    for (int s = 0; s < H; ++s) mean_h[s] = f0 + s < d ? colmean[f0 + s] : 0.0f;
    // operand pieces of one lane's half of a row, and the norm of the row
    auto pieces = [&](const float (&xc)[HP], float norm, uint4 *bp, int at, bool store) {
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) {
            unsigned ph[4], pl[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) split2_pair(xc[8 * ks + 2 * i], xc[8 * ks + 2 * i + 1], ph[i], pl[i]);
            if (store) {
                bp[(0 * NK + ks) * 64 + 32 * hl + at] = make_uint4(ph[0], ph[1], ph[2], ph[3]);
                bp[(1 * NK + ks) * 64 + 32 * hl + at] = make_uint4(pl[0], pl[1], pl[2], pl[3]);
            }
        }
        unsigned nh, nm, nl;
        split3(norm, nh, nm, nl);
        if (store && hl == 0) reinterpret_cast<uint2 *>(bp + prep_slots_of(DP) * 64)[at] = make_uint2(nh | (nm << 16), nl);
    };
    for (int64_t unit = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); unit < n_units;
         unit += (int64_t)gridDim.x * (blockDim.x >> 6)) {
        float xc[UB][HP];
        float sum[H];
#pragma unroll
        for (int s = 0; s < H; ++s) sum[s] = 0.0f;
#pragma unroll
        for (int ub = 0; ub < UB; ++ub) {
            const int64_t blk = unit * UB + ub, p = blk * 32 + n;
            const bool valid = p < N;
            float xr[H];
            const float *row = Xb + (int64_t)(valid ? perm[p] : 0) * ldx;
            if (vec) {
#pragma unroll
                for (int c4 = 0; c4 < H / 4; ++c4) {
                    float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    if (valid && f0 + 4 * c4 < d) v = *reinterpret_cast<const float4 *>(row + f0 + 4 * c4);
                    xr[4 * c4 + 0] = v.x; xr[4 * c4 + 1] = v.y; xr[4 * c4 + 2] = v.z; xr[4 * c4 + 3] = v.w;
                }
            } else {
#pragma unroll
                for (int s = 0; s < H; ++s) xr[s] = valid && f0 + s < d ? row[f0 + s] : 0.0f;
            }
            float part = 0.0f;
#pragma unroll
            for (int s = 0; s < HP; ++s) {
                // a point past the end and a padded feature count as a zero of the centred data
                xc[ub][s] = s < H && valid && f0 + s < d ? fmaf(xr[s < H ? s : 0], scale, mean_h[s < H ? s : 0]) : 0.0f;
                part = fmaf(xc[ub][s], xc[ub][s], part);
            }
            const float xn = part + xchg32(part);
            if (blk < n_blocks) {
#pragma unroll
                for (int c4 = 0; c4 < H / 4; ++c4)
                    *reinterpret_cast<float4 *>(xs + p * DP + f0 + 4 * c4) = make_float4(xr[4 * c4], xr[4 * c4 + 1], xr[4 * c4 + 2], xr[4 * c4 + 3]);
            }
            pieces(xc[ub], xn, xp + blk * prep_block_u4_of(DP), n, blk < n_blocks);
#pragma unroll
            for (int s = 0; s < H; ++s) sum[s] += xc[ub][s];
        }
        const float inv_n = 1.0f / (float)min(N - unit * (32 * UB), (int64_t)(32 * UB));
        float bc[HP];
        float norm = 0.0f;
#pragma unroll
        for (int s = 0; s < HP; ++s) bc[s] = s < H ? half_sum_f32(sum[s < H ? s : 0]) * inv_n : 0.0f;
#pragma unroll
        for (int s = 0; s < HP; s += 2) {                     // what the pieces hold of it, exactly
            unsigned h, l;
            split2_pair(bc[s], bc[s + 1], h, l);
            const fp16x2 hh = __builtin_bit_cast(fp16x2, h), ll = __builtin_bit_cast(fp16x2, l);
            bc[s] = (float)hh[0] + (float)ll[0];
            bc[s + 1] = (float)hh[1] + (float)ll[1];
            norm = fmaf(bc[s], bc[s], fmaf(bc[s + 1], bc[s + 1], norm));
        }
        norm += xchg32(norm);
        float far = 0.0f;
#pragma unroll
        for (int ub = 0; ub < UB; ++ub) {
            float r2 = 0.0f;
#pragma unroll
            for (int s = 0; s < H; ++s) {
                const float diff = xc[ub][s] - bc[s];
                r2 = fmaf(diff, diff, r2);
            }
            r2 += xchg32(r2);
            if ((unit * UB + ub) * 32 + n < N) far = fmaxf(far, r2);
        }
        far = half_max_f32(far);
        pieces(bc, norm, centres + (unit >> 5) * prep_block_u4_of(DP), (int)(unit & 31), n == 0);
        if (lane == 0) radius[unit] = sqrtf(far) * 1.00001f + 1.0e-6f;     // (rounding of the differences: below d 2^-24 of it)
    }
}

// workgroups of lloyd_prepare_ordered_kernel: 4 waves each, about 4 units per wave
constexpr int kPrepareGrid = 4096;
inline int64_t ordered_prepare_grid(int64_t n_units) { return std::min<int64_t>((n_units + 4 * 4 - 1) / (4 * 4), kPrepareGrid); }

// Places of the centroids of every run, in the order of the points they start from: centroids that lie close together share
// quads, and a unit meets fewer of them (1M x 16, k = 64: 3.3 tiles instead of 5.7).  The places stay for the whole sweep.
__global__ void __launch_bounds__(RLS_MAX_K) lloyd_rowpos_kernel(SweepPlan plan, const int64_t *__restrict__ init_idx, int64_t init_bs,
                                                                 const int32_t *__restrict__ status, char *ws, int64_t ws_bs,
                                                                 int64_t off_inv, int64_t off_rowpos, int64_t off_rowidx, OrderSpread sp)
{
    __shared__ int at[RLS_MAX_K];
    const int b = blockIdx.y, run = blockIdx.x, k = plan.k_min + run, j = threadIdx.x;
    if (status[b] != 0) return;
    char *wsb = ws + (int64_t)b * ws_bs;
    if (j < k) {
        const uint32_t place = (uint32_t)reinterpret_cast<const int32_t *>(wsb + off_inv)[init_idx[(int64_t)b * init_bs + j]];
        const uint32_t unit = place >> sp.unit_shift;                     // its place before the units were dealt out
        const uint32_t sorted = unit < sp.n_full ? (uint32_t)((uint64_t)unit * sp.back % sp.n_full) : unit;
        at[j] = (int)(sorted << sp.unit_shift | (place & ((1u << sp.unit_shift) - 1u)));
    }
    __syncthreads();
    if (j >= k) return;
    int pos = 0;
    for (int i = 0; i < k; ++i) pos += at[i] < at[j] || (at[i] == at[j] && i < j) ? 1 : 0;
    int gi = 0;
    while (gi + 1 < plan.n_groups && plan.g[gi + 1].run0 <= run) ++gi;
    const int row0 = rows_before(plan.k_min, run);
    reinterpret_cast<unsigned short *>(wsb + off_rowpos)[row0 + j] = (unsigned short)(row0 - rows_before(plan.k_min, plan.g[gi].run0) + pos);
    reinterpret_cast<unsigned char *>(wsb + off_rowidx)[row0 + pos] = (unsigned char)j;
}

// ---- start of a sweep: padding operand rows are zero vectors with a huge norm; running totals are zero;
//      no point has a label yet
struct InitArgs {
    char *ws;
    int64_t ws_bs;
    int64_t off_opA, off_losum, off_tot, off_totcnt, off_prev;
    int64_t n_tiles, n_losum, n_tot, n_totcnt, n_prev16;   // element counts (prev in 16-byte units)
    int32_t dp;
};
__global__ void sweep_init_kernel(InitArgs a)
{
    char *wsb = a.ws + (int64_t)blockIdx.y * a.ws_bs;
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    uint4 *opA = reinterpret_cast<uint4 *>(wsb + a.off_opA);
    long long *losum = reinterpret_cast<long long *>(wsb + a.off_losum);
    long long *tot = reinterpret_cast<long long *>(wsb + a.off_tot);
    long long *totcnt = reinterpret_cast<long long *>(wsb + a.off_totcnt);
    uint4 *prev = reinterpret_cast<uint4 *>(wsb + a.off_prev);
    {
        // a row without a centroid: zero pieces and, in the bias slot, the pieces of a huge squared norm
        // (lower half-wave) next to the ones that meet the pieces of |x'|^2 (upper half-wave)
        const int ns = tile_slots_of(a.dp);
        unsigned ph, pm, pl;
        split3(kPadNorm, ph, pm, pl);
        for (int64_t e = t0; e < a.n_tiles * ns * 64; e += step) {
            const int sl = (int)((e / 64) % ns), ln = (int)(e % 64);
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (sl == ns - 1) v = ln < 32 ? make_uint4(ph | (pm << 16), pl, 0u, 0u) : make_uint4(0x3f803f80u, 0x3f80u, 0u, 0u);
            opA[e] = v;
        }
    }
    for (int64_t e = t0; e < a.n_losum; e += step) losum[e] = 0;
    for (int64_t e = t0; e < a.n_tot; e += step) tot[e] = 0;
    for (int64_t e = t0; e < a.n_totcnt; e += step) totcnt[e] = 0;
    const uint4 none = make_uint4(0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu);
    for (int64_t e = t0; e < a.n_prev16; e += step) prev[e] = none;
}

// Adds the per-chunk deltas of one (centroid, feature) element for chunks [c_begin, c_end) to a 128-bit sum and the
// member count deltas to cnt.  The values sit a whole chunk block apart in memory: eight loads are kept in flight,
// the walk is bound by their latency (integer sums: any order gives the same result).
__device__ inline void sum_chunks(const long long *pe, const int *pc, int64_t estride, int64_t cstride, int c_begin, int c_end,
                                  long long &hi, unsigned long long &lo, long long &cnt)
{
    constexpr int U = 8;
    if (c_end - c_begin <= 2) {                    // (eight loads for one or two: 44 instead of 37 us for 64 x (262,144 x 16), k 1..32)
        for (int c = c_begin; c < c_end; ++c) {
            const long long v = pe[c * estride];
            const unsigned long long nlo = lo + (unsigned long long)v;
            hi += (v >> 63) + (nlo < lo ? 1 : 0);
            lo = nlo;
            cnt += pc[c * cstride];
        }
        return;
    }
    for (int c0 = c_begin; c0 < c_end; c0 += U) {
        long long v[U];
        int m[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = min(c0 + u, c_end - 1);
            v[u] = pe[c * estride];
            m[u] = pc[c * cstride];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (c0 + u >= c_end) { v[u] = 0; m[u] = 0; }
            const unsigned long long nlo = lo + (unsigned long long)v[u];
            hi += (v[u] >> 63) + (nlo < lo ? 1 : 0);
            lo = nlo;
            cnt += m[u];
        }
    }
}

struct CentroidArgs {
    const float *X;
    int64_t N;
    int32_t d;
    int64_t ldx, x_bs;
    const int64_t *init_idx;     // [batch][init_bs] (INIT only)
    int64_t init_bs;
    float *C;
    int64_t c_bs;
    const int32_t *status;
    char *ws;
    int64_t ws_bs;
    int64_t off_colinfo, off_opA, off_cnmax, off_psum, off_pcnt, off_losum, off_tot, off_totcnt;
    int64_t off_rowpos;          // places of the centroids among the rows of their group, or -1: by index
};

// One workgroup per run and part of kPartRows of its centroids: new centroids (from the seeding rows, or from the
// running totals after adding this round's per-chunk deltas), then the centred, -2-scaled MFMA operand rows and their
// squared norms.  (One workgroup per run left the large runs to the memory bandwidth of a single compute unit.)
template <int DP, bool INIT>
__global__ void __launch_bounds__(kThreads) lloyd_centroids_kernel(SweepPlan plan, CentroidArgs a)
{
    static_assert(kPartRows * DP <= kThreads, "one thread per (centroid, feature) element of a part");
    __shared__ float norms[kPartRows];       // squared norms of this part's centred centroids
    __shared__ long long part_hi[INIT ? 1 : kThreads], part_cnt[INIT ? 1 : kThreads];
    __shared__ unsigned long long part_lo[INIT ? 1 : kThreads];
    const int b = blockIdx.y, tid = threadIdx.x;
    const int bad = a.status[b];                    // (looked at before the first store, when it has come with everything else)
    if (INIT && bad != 0) return;                   // (the seeding's choices are not there)
    // blockIdx.x counts the parts of all runs in run order: the run is the last one that starts at or before it
    const int parts0 = parts_upto(plan.k_min - 1);
    int run = 0;
    for (int step = 64; step >= 1; step >>= 1)
        if (run + step < plan.n_runs && parts_upto(plan.k_min + run + step - 1) - parts0 <= (int)blockIdx.x) run += step;
    const int d = a.d, k = plan.k_min + run;
    const int part = (int)blockIdx.x - (parts_upto(k - 1) - parts0);
    const int j0 = part * kPartRows, rows = min(kPartRows, k - j0);
    const int row0 = rows_before(plan.k_min, run);
    const GroupDesc mine = group_of_lane(plan);
    const GroupDesc g = take_group(mine, last_group(plan, mine.run0 <= run));
    const int rl = run - g.run0;
    char *wsb = a.ws + (int64_t)b * a.ws_bs;
    const float *colmean = reinterpret_cast<const float *>(wsb + a.off_colinfo);   // -(mean * scale)
    const int *colshift = reinterpret_cast<const int *>(wsb + a.off_colinfo + 128);
    const int *colwide = reinterpret_cast<const int *>(wsb + a.off_colinfo + 256);
    const float scale = *reinterpret_cast<const float *>(wsb + a.off_colinfo + kColScaleOff);
    float *Cb = a.C + (int64_t)b * a.c_bs;
    // operand block of the group: per tile, tile_slots_of(DP) slots of 64 lanes x 8 halves (fp16 pieces, bf16 bias)
    unsigned short *opA = reinterpret_cast<unsigned short *>(wsb + a.off_opA + (int64_t)g.tile0 * tile_bytes_of(DP));
    constexpr int NK = ksteps_of(DP), NS = tile_slots_of(DP);

    // The chunks are split over `nsl` thread slices per (centroid, feature) element, so that the per-chunk deltas are
    // not read one after the other by a handful of threads; integer sums, any order.
    const int E = rows * DP;
    const int nsl = INIT ? 1 : kThreads / E;
    // what the element's owner needs beside the deltas is requested first
    long long tot_hi = 0, tot_lo = 0, tot_cnt = 0;
    int col_shift = 0, col_wide = 0;
    float col_mean = 0.0f, c_old = 0.0f;
    const int run_row = row0 - rows_before(plan.k_min, g.run0);      // the run's first row in its group
    const unsigned short *rowpos = a.off_rowpos >= 0 ? reinterpret_cast<const unsigned short *>(wsb + a.off_rowpos) + row0 + j0 : nullptr;
    int place = j0 + tid / DP;                                       // of the element's centroid
    if (rowpos && tid < E) place = rowpos[tid / DP] - run_row;
    if (tid < E && tid % DP < d) {
        const int l = tid % DP;
        const int64_t at = (int64_t)(row0 + j0 + tid / DP) * d + l;
        col_mean = colmean[l];
        if (!INIT) {
            const long long *tot = reinterpret_cast<const long long *>(wsb + a.off_tot) + at * 2;
            tot_hi = tot[0];
            tot_lo = tot[1];
            tot_cnt = reinterpret_cast<const long long *>(wsb + a.off_totcnt)[at];
            col_shift = colshift[l];
            col_wide = colwide[l];
            c_old = Cb[at];
        }
    }
    if (!INIT) {
        const int e = tid % E, sl = tid / E;
        const int j = j0 + e / DP, l = e % DP;
        long long hi = 0, cnt = 0;
        unsigned long long lo = 0;
        if (sl < nsl && l < d) {
            const int grow0 = rows_before(plan.k_min, g.run0);
            const int grows = rows_before(plan.k_min, g.run0 + g.n_runs) - grow0;      // rows of the group
            const int64_t at = (int64_t)g.part0 + row0 - grow0 + j;
            const long long *psum = reinterpret_cast<const long long *>(wsb + a.off_psum) + at * d + l;
            const int *pcnt = reinterpret_cast<const int *>(wsb + a.off_pcnt) + at;
            const int c_begin = (int)((int64_t)g.n_chunks * sl / nsl), c_end = (int)((int64_t)g.n_chunks * (sl + 1) / nsl);
            sum_chunks(psum, pcnt, (int64_t)grows * d, grows, c_begin, c_end, hi, lo, cnt);
        }
        if (bad != 0) return;
        part_hi[tid] = hi; part_lo[tid] = lo; part_cnt[tid] = cnt;
        __syncthreads();
    }

    if (tid < E) {
        const int e = tid;
        const int jj = e / DP, j = j0 + jj, l = e % DP;
        float cp = 0.0f;
        if (l < d) {
            float c;
            if (INIT) {
                const int64_t src = a.init_idx[(int64_t)b * a.init_bs + j];
                c = a.X[(int64_t)b * a.x_bs + src * a.ldx + l];
                Cb[(int64_t)(row0 + j) * d + l] = c;
            } else {
                long long *tot = reinterpret_cast<long long *>(wsb + a.off_tot) + ((int64_t)(row0 + j) * d + l) * 2;
                long long *totcnt = reinterpret_cast<long long *>(wsb + a.off_totcnt) + (int64_t)(row0 + j) * d + l;
                long long hi = tot_hi;
                unsigned long long lo = (unsigned long long)tot_lo;
                long long cnt = tot_cnt;
                for (int sl = 0; sl < nsl; ++sl) {
                    const unsigned long long nlo = lo + part_lo[sl * E + e];
                    hi += part_hi[sl * E + e] + (nlo < lo ? 1 : 0);
                    lo = nlo;
                    cnt += part_cnt[sl * E + e];
                }
                tot[0] = hi;
                tot[1] = (long long)lo;
                *totcnt = cnt;
                int shift = col_shift;
                if (col_wide) {
                    // total = main * 2^kLowBits + low, on the scale 2^-(shift + kLowBits)
                    const long long low = reinterpret_cast<const long long *>(wsb + a.off_losum)[(int64_t)(row0 + place) * d + l];
                    hi = (long long)(((unsigned long long)hi << kLowBits) | (lo >> (64 - kLowBits)));
                    lo = lo << kLowBits;
                    const unsigned long long nlo = lo + (unsigned long long)low;
                    hi += (low >> 63) + (nlo < lo ? 1 : 0);
                    lo = nlo;
                    shift += kLowBits;
                }
                if (cnt > 0) {
                    c = (float)(fixed128_to_double(hi, lo, shift) / (double)cnt);
                    Cb[(int64_t)(row0 + j) * d + l] = c;
                } else {
                    c = c_old;                               // a cluster without members keeps its centroid
                }
            }
            cp = fmaf(c, scale, col_mean);       // (c - mean) * scale, one rounding, as for the points
        }
        // squared norm, summed over the DP lanes of the centroid
        float nrm = cp * cp;
        nrm += __int_as_float(dpp_move<kDppSwap1>(__float_as_int(nrm)));
        nrm += __int_as_float(dpp_move<kDppSwap2>(__float_as_int(nrm)));
        nrm += __int_as_float(dpp_move<kDppHalfMirror>(__float_as_int(nrm)));
        if (DP >= 16) nrm += __int_as_float(dpp_move<kDppMirror>(__float_as_int(nrm)));
        if (DP >= 32) {
            const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(nrm), __float_as_uint(nrm), false, false);
            nrm = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        }
        // operand position of (centroid j, feature l)
        const int qd = place >> 2, i = place & 3;
        const int t = qd / g.S, slot = rl * g.S + qd % g.S;
        const int m = 8 * (slot & 3) + 4 * (slot >> 2) + i;
        const int h = l / (DP / 2), sf = l % (DP / 2);
        unsigned short ph, pl;
        split2(-2.0f * cp, ph, pl);
        const int ks = sf >> 3, el = sf & 7, ln = h * 32 + m;
        opA[((int64_t)(t * NS + 0 * NK + ks) * 64 + ln) * 8 + el] = ph;
        opA[((int64_t)(t * NS + 1 * NK + ks) * 64 + ln) * 8 + el] = pl;
        if (l == 0) {
            // bias slot, lower half-wave lane of this row: pieces of the squared norm
            unsigned nh, nm, nl;
            split3(nrm, nh, nm, nl);
            unsigned short *bias = opA + ((int64_t)(t * NS + 2 * NK) * 64 + m) * 8;
            bias[0] = (unsigned short)nh; bias[1] = (unsigned short)nm; bias[2] = (unsigned short)nl;
            norms[jj] = nrm;
        }
    }
    __syncthreads();
    // the run's maximum is taken over its parts by the reader
    if (tid < 64) {
        static_assert(kPartRows <= 64, "the first wave holds them all");
        float mx = tid < rows ? norms[tid] : 0.0f;
        for (int off = kPartRows / 2; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
        if (tid == 0) reinterpret_cast<float *>(wsb + a.off_cnmax)[run * kMaxParts + part] = mx;
    }
}

// ---- the end of an ordered sweep: the labels go back to the points' own order, and every point's exact distance to its centroid
//      is added up.  The additions are those of the final pass over the points as they come (lloyd_step_kernel), one by one and
//      in the same order - lanes over their slabs of a chunk, the lanes of a wave, the waves, the chunks (lloyd_loss_kernel) -, so
//      that a sweep has the same losses to the last bit whichever form it takes.  (Losses from the exact sums of the clusters and
//      the squares of all points cost next to nothing, but where a column spans many binary digits next to nothing is left of them:
//      their terms agree in more digits than two doubles hold.)
//      `plan` is the plan of that other form.  A workgroup takes one of its chunks and the runs of a span: runs whose chunks are
//      the same there and whose label bytes lie side by side here.  Where a wave of the step takes 32 points at a time, 32 lanes do
//      so here: up to d_pad 16 in two half-waves, each every other run of the span (1M x 16, k 1..64: 230 us, one half-wave for all
//      runs 250); at d_pad 32, where spans have down to two runs, one for all of them, which converts the row to fp64 once (4M x 32,
//      k 1..128: 5.0 ms, two 5.8).  Bound by vector issue: per point, run and feature a conversion (8 cycles a wave) and three fp64
//      operations (4 each), three quarters of the time at 1M x 16; the labels alone took 94 us there.
struct RunSpan {
    int16_t run0, lab0;                    // first run; the label bytes' place (see GroupDesc::lab0)
    uint8_t n_runs, group;                 // runs; the group of `plan`
    uint8_t slots, first;                  // label bytes of a point, and which of them is that of the first run
};
struct RunSpans {
    int32_t n;
    RunSpan s[RLS_MAX_K];
};
static_assert(sizeof(SweepPlan) + sizeof(RunSpans) + 256 <= 4096, "kernel arguments");
struct EndArgs {
    const float *X;
    int64_t N, ldx, x_bs;
    int32_t d;
    const float *C;
    int64_t c_bs;
    int32_t *labels;                       // or null
    int64_t lab_bs;
    const int32_t *status;
    char *ws;
    int64_t ws_bs;
    int64_t off_inv, off_rowidx, off_prev, off_pj;
    int32_t batch, wgs;                    // spaces; chunks of all spans
};
constexpr int end_lds_bytes(int dp, int rows) { return rows * (dp + 4) * 4 + (step_threads_of(dp) / 64) * 8 * 8 + rows; }

constexpr int end_halves_of(int dp) { return dp <= 16 ? 2 : 1; }
constexpr int end_threads_of(int dp) { return step_threads_of(dp) / 2 * end_halves_of(dp); }

template <int DP, bool VEC>
__global__ void __launch_bounds__(end_threads_of(DP)) lloyd_ordered_end_kernel(SweepPlan plan, RunSpans spans, EndArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int HS = end_halves_of(DP), TH = end_threads_of(DP), WV = step_threads_of(DP) / 64, CS = DP + 4, NR = 8 / HS;
    const int tid = threadIdx.x, n = tid & 31, hl = (tid >> 5) & (HS - 1), w = tid / (32 * HS);
    int b, chunk, span;
    if (plan.chunk_block > 0) {
        // the same chunks for every span: the spans of a chunk follow each other on one XCD, they read the same rows
        const int turn = (int)(blockIdx.x >> 3), at = turn / spans.n * 8 + (int)(blockIdx.x & 7);
        span = turn % spans.n;
        b = at / plan.g[0].n_chunks;
        chunk = at - b * plan.g[0].n_chunks;
        if (b >= a.batch) return;
    } else {
        // chunks of their own, hardly more than compute units: no workgroup without one, which would leave another compute unit
        // two of them (1,000,003 x 16, k 8..23: 106 us with such, 75 without).  Two spans per lane find where theirs begin.
        b = blockIdx.x / a.wgs;
        const int v = blockIdx.x - b * a.wgs, lane = tid & 63;
        const int c0 = 2 * lane < spans.n ? plan.g[spans.s[2 * lane].group].n_chunks : 0;
        const int c1 = 2 * lane + 1 < spans.n ? plan.g[spans.s[2 * lane + 1].group].n_chunks : 0;
        int before = c0 + c1;                            // inclusive, then exclusive sums
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(before, off, 64);
            if (lane >= off) before += o;
        }
        before -= c0 + c1;
        const int from = __popcll(__builtin_amdgcn_ballot_w64(before <= v)) - 1;        // (behind the last span: the sum of all, above v)
        chunk = v - __shfl(before, from, 64);
        const int first = __shfl(c0, from, 64);
        span = 2 * from + (chunk >= first ? 1 : 0);
        if (chunk >= first) chunk -= first;
        b = __builtin_amdgcn_readfirstlane(b); chunk = __builtin_amdgcn_readfirstlane(chunk); span = __builtin_amdgcn_readfirstlane(span);
    }
    const RunSpan sp = spans.s[span];
    const GroupDesc g = plan.g[sp.group];
    if (a.status[b] != 0) return;
    const int d = a.d, k0 = plan.k_min + sp.run0;
    const int grow0 = rows_before(plan.k_min, sp.run0), rows = rows_before(plan.k_min, sp.run0 + sp.n_runs) - grow0;
    float *cs_s = reinterpret_cast<float *>(smem);
    double *jpart_s = reinterpret_cast<double *>(smem + rows * CS * 4);          // [WV][8]
    unsigned char *rowidx_s = smem + rows * CS * 4 + WV * 8 * 8;
    const char *wsb = a.ws + (int64_t)b * a.ws_bs;
    const float *Xb = a.X + (int64_t)b * a.x_bs, *Cb = a.C + (int64_t)b * a.c_bs + (int64_t)grow0 * d;
    const int32_t *inv = reinterpret_cast<const int32_t *>(wsb + a.off_inv);
    const unsigned char *prev = reinterpret_cast<const unsigned char *>(wsb + a.off_prev) + (int64_t)sp.lab0 * ((a.N + 15) / 16 * 16);
    static_assert(TH % DP == 0, "a thread keeps its feature");
    for (int r0 = tid / DP; r0 < rows; r0 += 8 * (TH / DP)) {            // (eight on their way at a time)
        const int l = tid % DP;
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = Cb[min(r0 + u * (TH / DP), rows - 1) * d + min(l, d - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (r0 + u * (TH / DP) < rows) cs_s[(r0 + u * (TH / DP)) * CS + l] = l < d ? v[u] : 0.0f;
    }
    for (int e = tid; e < rows; e += TH) rowidx_s[e] = reinterpret_cast<const unsigned char *>(wsb + a.off_rowidx)[grow0 + e];
    __syncthreads();

    const int begin = chunk * g.chunk_len, end = (int)min(a.N, (int64_t)begin + g.chunk_len);
    const int twice = slab_blocks_of(DP, g.S) - 1;                     // a slab is one block of 32 points, or two
    const int n_slabs = (end - begin + (32 << twice) - 1) / (32 << twice);
    const int steps = n_slabs > w ? ((n_slabs - w + WV - 1) / WV) << twice : 0;
    auto point = [&](int t) { return begin + ((((t >> twice) * WV + w) << twice) + (t & twice)) * 32 + n; };
    // (past the end: the chunk's last point)
    auto place_of = [&](int t) { return inv[min(point(t), end - 1)]; };
    auto fetch = [&](int t, int place, float (&x)[DP], uint2 &word) {
        const unsigned char *at = prev + (int64_t)place * sp.slots;
        word = make_uint2(0u, 0u);
        if (sp.slots == 8) word = *reinterpret_cast<const uint2 *>(at);
        else if (sp.slots == 4) word.x = *reinterpret_cast<const unsigned *>(at);
        else if (sp.slots == 2) word.x = *reinterpret_cast<const unsigned short *>(at);
        else word.x = *at;
        const float *row = Xb + (int64_t)min(point(t), end - 1) * a.ldx;
#pragma unroll
        for (int l = 0; l < DP; l += 4) {
            float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (VEC) {
                if (l < d) v = *reinterpret_cast<const float4 *>(row + l);
            } else {
                if (l + 0 < d) v.x = row[l + 0];
                if (l + 1 < d) v.y = row[l + 1];
                if (l + 2 < d) v.z = row[l + 2];
                if (l + 3 < d) v.w = row[l + 3];
            }
            x[l] = v.x; x[l + 1] = v.y; x[l + 2] = v.z; x[l + 3] = v.w;
        }
    };
    // runs hl, hl + HS, ... of the span: their first rows and label bytes (one of the last runs twice, rather than one that is not there)
    double sum[NR];
    int row[NR], byte[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const int r = min(HS * i + hl, sp.n_runs - 1);
        sum[i] = 0.0;
        row[i] = r * k0 + r * (r - 1) / 2;
        byte[i] = sp.first + r;
    }
    // (requested ahead: a point's place by two steps, its row and label bytes by one; further ahead measured the same)
    float xn[DP];
    uint2 wordn;
    fetch(0, place_of(0), xn, wordn);
    int placen = place_of(1);
    for (int t = 0; t < steps; ++t) {
        const int p = point(t);
        const bool valid = p < end;
        const uint2 word = wordn;
        int label[NR];
#pragma unroll
        for (int i = 0; i < NR; ++i) label[i] = rowidx_s[row[i] + (int)(((byte[i] < 4 ? word.x : word.y) >> (8 * (byte[i] & 3))) & 127u)];
        if (valid && a.labels) {
            int32_t *const out = a.labels + (int64_t)b * a.lab_bs + (int64_t)sp.run0 * a.N + p;
#pragma unroll
            for (int i = 0; i < NR; ++i)
                if (HS * i + hl < sp.n_runs) out[(HS * i + hl) * a.N] = label[i];
        }
        float x[DP];
#pragma unroll
        for (int l = 0; l < DP; ++l) x[l] = xn[l];
        fetch(t + 1, placen, xn, wordn);
        placen = place_of(t + 2);
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            if (HS * i >= sp.n_runs) continue;
            const double dist = exact_distance<DP>(x, cs_s + (row[i] + label[i]) * CS);
            sum[i] = __dadd_rn(sum[i], valid ? dist : 0.0);
        }
    }
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const double v = half_sum_f64(sum[i]);
        if (n == 0) jpart_s[w * 8 + HS * i + hl] = v;
    }
    __syncthreads();
    if (tid < sp.n_runs) {
        double v = 0.0;
        for (int q = 0; q < WV; ++q) v = __dadd_rn(v, jpart_s[q * 8 + tid]);
        reinterpret_cast<double *>(const_cast<char *>(wsb) + a.off_pj)[(int64_t)(g.wg0 + chunk) * 8 + (sp.run0 - g.run0) + tid] = v;
    }
}

// the spans of an ordered sweep: every run lies in one
inline RunSpans run_spans(const SweepPlan &plan, const SweepPlan &plain)
{
    RunSpans r;
    r.n = 0;
    int gi = 0, pi = 0;
    for (int run = 0; run < plan.n_runs;) {
        while (gi + 1 < plan.n_groups && plan.g[gi + 1].run0 <= run) ++gi;
        while (pi + 1 < plain.n_groups && plain.g[pi + 1].run0 <= run) ++pi;
        const GroupDesc &g = plan.g[gi], &p = plain.g[pi];
        const int end = std::min(g.run0 + g.n_runs, p.run0 + p.n_runs);
        r.s[r.n++] = RunSpan{(int16_t)run, g.lab0, (uint8_t)(end - run), (uint8_t)pi, (uint8_t)(8 / g.S), (uint8_t)(run - g.run0)};
        run = end;
    }
    return r;
}

// sum of the per-chunk partial losses of every run, in chunk order
__global__ void lloyd_loss_kernel(SweepPlan plan, const int32_t *status, const char *ws, int64_t ws_bs,
                                  int64_t off_pj, double *out, int64_t out_bs, int64_t out_stride, int64_t out_off)
{
    const int b = blockIdx.x, r = threadIdx.x;
    if (r >= plan.n_runs || status[b] != 0) return;
    int gi = 0;
    while (gi + 1 < plan.n_groups && plan.g[gi + 1].run0 <= r) ++gi;
    const int n_chunks = plan.g[gi].n_chunks;
    const double *pj = reinterpret_cast<const double *>(ws + (int64_t)b * ws_bs + off_pj) + (int64_t)plan.g[gi].wg0 * 8 + (r - plan.g[gi].run0);
    double v = 0.0;
    // eight loads in flight at a time (the walk is bound by their latency); the additions keep the chunk order
    constexpr int U = 8;
    for (int c0 = 0; c0 < n_chunks; c0 += U) {
        double t[U];
#pragma unroll
        for (int u = 0; u < U; ++u) t[u] = pj[(int64_t)min(c0 + u, n_chunks - 1) * 8];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (c0 + u < n_chunks) v = __dadd_rn(v, t[u]);
    }
    out[(int64_t)b * out_bs + (int64_t)r * out_stride + out_off] = v;
}

template <int DP>
hipError_t launch_sweep_dp(const SweepPlan &plan, const SweepLayout &L, const SweepArgs &a, hipStream_t s)
{
    // the kernels' LDS limit is raised once per process, whichever host thread comes first
    static std::once_flag attr_once;
    static hipError_t attr_status = hipSuccess;
    std::call_once(attr_once, [] {
        const void *fns[] = {
            reinterpret_cast<const void *>(lloyd_step_kernel<DP, false, false, false, false, false>),
            reinterpret_cast<const void *>(lloyd_step_kernel<DP, false, false, true, false, false>),
            reinterpret_cast<const void *>(lloyd_step_kernel<DP, false, false, true, true, true>),
            reinterpret_cast<const void *>(lloyd_step_kernel<DP, false, false, true, true, false>),
            reinterpret_cast<const void *>(lloyd_step_kernel<DP, false, true, false, false, false>),
            reinterpret_cast<const void *>(lloyd_step_kernel<DP, true, false, false, false, false>),
            reinterpret_cast<const void *>(lloyd_ordered_end_kernel<DP, false>),
            reinterpret_cast<const void *>(lloyd_ordered_end_kernel<DP, true>),
        };
        for (const void *fn : fns) {
            const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
            if (e != hipSuccess) attr_status = e;
        }
    });
    if (attr_status != hipSuccess) return attr_status;
    const int batch = a.batch;
    // Rounds after the first run on the prepared copy of the points - unless the loss of every round is wanted (that
    // pass needs every row), or the sweep is so light in distance work (a single k up to 32: one tile of centroids per
    // group) that reading the rows is what it costs: the prepared copy is 6 to 12% larger than the rows.
    const bool trace = a.trace != nullptr;
    const bool use_pre = sweep_uses_prepared(plan, a.iters, trace);
    const bool ordered = plan.ordered != 0, small = sweep_is_small(plan, a.N, batch, a.iters, trace);
    const int64_t n_units = (a.N + 32 * unit_blocks_of(DP) - 1) / (32 * unit_blocks_of(DP));
    // column statistics
    if (!a.reuse_colstats) {
        const int threads = stat_threads(a.N, DP, L.stat_blocks, batch);
        hipLaunchKernelGGL(threads == 1024 ? colstats_kernel<1024> : colstats_kernel<kStatFew>, dim3(L.stat_blocks, batch), dim3(threads), 0, s, a.X, a.N,
                           (int)a.d, DP, a.ldx, a.x_batch_stride, a.ws, L.per_batch, L.colstat_part);
        hipLaunchKernelGGL(colstats_final_kernel, dim3(batch), dim3(256), 0, s, a.N, (int)a.d, (int)L.stat_blocks, a.ws,
                           L.per_batch, L.colstat_part, L.colinfo, plan.ordered ? L.keyinfo : (int64_t)-1, a.status);
    }
    if (ordered && !a.reuse_prepared) {
        const hipError_t e = launch_order(a.X, a.N, a.d, a.ldx, a.x_batch_stride, batch, a.status, a.ws, L.per_batch, L.keyinfo, L.perm, L.inv, L.xs,
                                          unit_blocks_of(DP) == 2 ? 6 : 5, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((lloyd_prepare_ordered_kernel<DP>), dim3((unsigned)ordered_prepare_grid(n_units), batch), dim3(256), 0, s, a.X, a.N,
                           (int)a.d, a.ldx, a.x_batch_stride, a.status, a.ws, L.per_batch, L.colinfo, L.perm, L.xp, L.xs, L.centres, L.radius);
    } else if (small || (use_pre && !a.reuse_prepared)) {
        // the prepared copy: a wave takes a block of 32 points at a time, 4 waves per workgroup; one block as long as the chip has
        // room for all of them, then about 8 (8 throughout: 2000 x 8 7.0 instead of 4.8 us, 65,536 x 16 13.1 instead of 5.6)
        const int64_t n_blocks = (a.N + 31) / 32;
        const int64_t room = std::max<int64_t>(2048 / batch, 1);
        const int64_t grid_x = std::max(std::min((n_blocks + 3) / 4, room), std::min<int64_t>((n_blocks + 4 * 8 - 1) / (4 * 8), 4096));
        hipLaunchKernelGGL((lloyd_prepare_kernel<DP>), dim3((unsigned)grid_x, batch), dim3(256), 0, s, a.X, a.N, (int)a.d, a.ldx,
                           a.x_batch_stride, a.status, a.ws, L.per_batch, L.colinfo, L.xp);
    }
    if (small) return launch_small_sweep(plan, L, a, s);
    InitArgs ia;
    ia.ws = a.ws; ia.ws_bs = L.per_batch;
    ia.off_opA = L.opA; ia.off_losum = L.losum; ia.off_tot = L.tot; ia.off_totcnt = L.totcnt; ia.off_prev = L.prev;
    ia.n_tiles = plan.total_tiles; ia.dp = DP;
    ia.n_losum = (int64_t)plan.total_rows * a.d; ia.n_tot = ia.n_losum * 2; ia.n_totcnt = ia.n_losum;
    ia.n_prev16 = ordered ? 0 : (int64_t)plan.lab_slots * align_up(a.N, 16) / 16;      // (an ordered first round writes them all)
    hipLaunchKernelGGL(sweep_init_kernel, dim3(512, batch), dim3(256), 0, s, ia);
    if (ordered)
        hipLaunchKernelGGL(lloyd_rowpos_kernel, dim3(plan.n_runs, batch), dim3(RLS_MAX_K), 0, s, plan, a.init_idx, a.init_batch_stride, a.status,
                           a.ws, L.per_batch, L.inv, L.rowpos, L.rowidx, order_spread(a.N, unit_blocks_of(DP) == 2 ? 6 : 5));

    CentroidArgs ca;
    ca.X = a.X; ca.N = a.N; ca.d = a.d; ca.ldx = a.ldx; ca.x_bs = a.x_batch_stride;
    ca.init_idx = a.init_idx; ca.init_bs = a.init_batch_stride;
    ca.C = a.centroids; ca.c_bs = (int64_t)plan.total_rows * a.d;
    ca.status = a.status; ca.ws = a.ws; ca.ws_bs = L.per_batch;
    ca.off_colinfo = L.colinfo; ca.off_opA = L.opA; ca.off_cnmax = L.cnmax;
    ca.off_psum = L.psum; ca.off_pcnt = L.pcnt; ca.off_losum = L.losum; ca.off_tot = L.tot; ca.off_totcnt = L.totcnt;
    ca.off_rowpos = ordered ? L.rowpos : -1;
    const dim3 centroid_grid(parts_upto(plan.k_min + plan.n_runs - 1) - parts_upto(plan.k_min - 1), batch);
    hipLaunchKernelGGL((lloyd_centroids_kernel<DP, true>), centroid_grid, dim3(kThreads), 0, s, plan, ca);

    StepArgs sa;
    sa.X = a.X; sa.N = a.N; sa.d = a.d; sa.ldx = a.ldx; sa.x_bs = a.x_batch_stride;
    sa.C = a.centroids; sa.c_bs = ca.c_bs;
    sa.labels = a.labels; sa.lab_bs = (int64_t)plan.n_runs * a.N;
    sa.status = a.status; sa.ws = a.ws; sa.ws_bs = L.per_batch;
    sa.off_colinfo = L.colinfo; sa.off_opA = L.opA; sa.off_cnmax = L.cnmax;
    sa.off_psum = L.psum; sa.off_pcnt = L.pcnt; sa.off_pj = L.pj; sa.off_losum = L.losum; sa.off_prev = L.prev;
    sa.off_xp = L.xp;
    sa.off_xs = L.xs; sa.off_centres = L.centres; sa.off_radius = L.radius; sa.off_rowpos = L.rowpos; sa.off_rowidx = L.rowidx; sa.off_lists = L.lists;

    size_t lds = 0;
    for (int gi = 0; gi < plan.n_groups; ++gi) {
        const GroupDesc &g = plan.g[gi];
        const int rr = rows_before(plan.k_min, g.run0 + g.n_runs) - rows_before(plan.k_min, g.run0);
        const size_t need = (size_t)carve_lds(DP, a.d, g.n_tiles, rr, g.copies, ordered).total;
        if (need > lds) lds = need;
    }
    const dim3 grid((unsigned)((int64_t)plan.n_wgs * batch), 1);
    sa.batch = batch;
    const bool prof = profile_enabled();
    for (int t = 0; t < a.iters; ++t) {
        sa.first_round = t == 0 ? 1 : 0;
        if (prof) { hipError_t e = profile_mark(s, true); if (e != hipSuccess) return e; }
        if (trace) {
            hipLaunchKernelGGL((lloyd_step_kernel<DP, false, true, false, false, false>), grid, dim3(step_threads_of(DP)), lds, s, plan, sa);
            if (prof) { hipError_t e = profile_mark(s, false); if (e != hipSuccess) return e; }
            hipLaunchKernelGGL(lloyd_loss_kernel, dim3(batch), dim3(128), 0, s, plan, a.status, a.ws,
                               L.per_batch, L.pj, a.trace, (int64_t)plan.n_runs * (a.iters + 1), (int64_t)(a.iters + 1), (int64_t)t);
        } else {
            // the first round brings every row into a cluster and reads the rows themselves; later rounds take the
            // operands from the prepared copy and read a row only where a label is in doubt or has changed
            if (ordered && t == 0) hipLaunchKernelGGL((lloyd_step_kernel<DP, false, false, true, true, true>), grid, dim3(step_threads_of(DP)), lds, s, plan, sa);
            else if (t == 0 || !use_pre) hipLaunchKernelGGL((lloyd_step_kernel<DP, false, false, false, false, false>), grid, dim3(step_threads_of(DP)), lds, s, plan, sa);
            else if (ordered) hipLaunchKernelGGL((lloyd_step_kernel<DP, false, false, true, true, false>), grid, dim3(step_threads_of(DP)), lds, s, plan, sa);
            else hipLaunchKernelGGL((lloyd_step_kernel<DP, false, false, true, false, false>), grid, dim3(step_threads_of(DP)), lds, s, plan, sa);
            if (prof) { hipError_t e = profile_mark(s, false); if (e != hipSuccess) return e; }
        }
        hipLaunchKernelGGL((lloyd_centroids_kernel<DP, false>), centroid_grid, dim3(kThreads), 0, s, plan, ca);
    }
    if (ordered) {
        // the final assignment is a round like the others; its labels go back to the points, and with them come the losses
        hipLaunchKernelGGL((lloyd_step_kernel<DP, false, false, true, true, false>), grid, dim3(step_threads_of(DP)), lds, s, plan, sa);
        SweepPlan plain;
        if (make_sweep_plan(a.N, a.d, plan.k_min, plan.k_min + plan.n_runs - 1, batch, false, &plain) != RLS_OK) return hipErrorInvalidValue;
        int rows = 0;
        const RunSpans spans = run_spans(plan, plain);
        for (int i = 0; i < spans.n; ++i)
            rows = std::max(rows, rows_before(plan.k_min, spans.s[i].run0 + spans.s[i].n_runs) - rows_before(plan.k_min, spans.s[i].run0));
        EndArgs ea;
        ea.X = a.X; ea.N = a.N; ea.ldx = a.ldx; ea.x_bs = a.x_batch_stride; ea.d = a.d;
        ea.C = a.centroids; ea.c_bs = ca.c_bs; ea.labels = a.labels; ea.lab_bs = sa.lab_bs;
        ea.status = a.status; ea.ws = a.ws; ea.ws_bs = L.per_batch;
        ea.off_inv = L.inv; ea.off_rowidx = L.rowidx; ea.off_prev = L.prev; ea.off_pj = L.pj;
        ea.batch = batch; ea.wgs = 0;
        const bool vec = a.d % 4 == 0 && a.ldx % 4 == 0 && (a.x_batch_stride % 4 == 0 || batch == 1) && (reinterpret_cast<uintptr_t>(a.X) & 15) == 0;
        for (int i = 0; i < spans.n; ++i) ea.wgs += plain.g[spans.s[i].group].n_chunks;
        const int64_t end_wgs = plain.chunk_block > 0 ? ((int64_t)plain.g[0].n_chunks * batch + 7) / 8 * 8 * spans.n : (int64_t)ea.wgs * batch;
        const dim3 end_grid((unsigned)end_wgs), end_block(end_threads_of(DP));
        const size_t end_lds = (size_t)end_lds_bytes(DP, rows);
        if (vec) hipLaunchKernelGGL((lloyd_ordered_end_kernel<DP, true>), end_grid, end_block, end_lds, s, plain, spans, ea);
        else hipLaunchKernelGGL((lloyd_ordered_end_kernel<DP, false>), end_grid, end_block, end_lds, s, plain, spans, ea);
        hipLaunchKernelGGL(lloyd_loss_kernel, dim3(batch), dim3(128), 0, s, plain, a.status, a.ws, L.per_batch,
                           L.pj, a.inertia, (int64_t)plan.n_runs, (int64_t)1, (int64_t)0);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((lloyd_step_kernel<DP, true, false, false, false, false>), grid, dim3(step_threads_of(DP)), lds, s, plan, sa);
    hipLaunchKernelGGL(lloyd_loss_kernel, dim3(batch), dim3(128), 0, s, plan, a.status, a.ws, L.per_batch,
                       L.pj, a.inertia, (int64_t)plan.n_runs, (int64_t)1, (int64_t)0);
    if (trace)
        hipLaunchKernelGGL(lloyd_loss_kernel, dim3(batch), dim3(128), 0, s, plan, a.status, a.ws,
                           L.per_batch, L.pj, a.trace, (int64_t)plan.n_runs * (a.iters + 1), (int64_t)(a.iters + 1),
                           (int64_t)a.iters);
    return hipGetLastError();
}

}  // namespace

// The kernels take minutes to compile: the file is compiled once for each padded number of features, 16 and 32 with
// RLS_LLOYD_DPAD set to it (nothing but that launch), 8 together with everything else.
hipError_t launch_sweep_dpad16(const SweepPlan &plan, const SweepLayout &L, const SweepArgs &a, hipStream_t s);
hipError_t launch_sweep_dpad32(const SweepPlan &plan, const SweepLayout &L, const SweepArgs &a, hipStream_t s);
#if defined(RLS_LLOYD_DPAD) && RLS_LLOYD_DPAD == 16
hipError_t launch_sweep_dpad16(const SweepPlan &plan, const SweepLayout &L, const SweepArgs &a, hipStream_t s) { return launch_sweep_dp<16>(plan, L, a, s); }
#elif defined(RLS_LLOYD_DPAD) && RLS_LLOYD_DPAD == 32
hipError_t launch_sweep_dpad32(const SweepPlan &plan, const SweepLayout &L, const SweepArgs &a, hipStream_t s) { return launch_sweep_dp<32>(plan, L, a, s); }
#else


int padded_d(int d) { return d <= 8 ? 8 : (d <= 16 ? 16 : 32); }

bool sweep_uses_prepared(const SweepPlan &plan, int32_t iters, bool trace)
{
    return !trace && iters >= 2 && plan.total_tiles >= 2 * plan.n_groups;
}

LloydGeometry lloyd_geometry(int dp)
{
    LloydGeometry g;
    g.threads = kThreads;
    g.tile_points = tile_points_of(dp);
    g.lds_budget = 156 * 1024;
    return g;
}

int64_t lloyd_group_lds_bytes(int dp, int d, int n_tiles, int real_rows, int copies, bool ordered)
{
    return carve_lds(dp, d, n_tiles, real_rows, copies, ordered).total;
}

constexpr int kFillWorkgroups = 256;   // one per compute unit
// What a slab of 32 points costs beside the tiles of its group (operand loads, close calls, labels, moved pairs), in tiles.  Sweeps
// at 65 shapes from 20,003 x 8 to 3.2M x 32 with 2, 4, 8 and 12 in its place: 2 up to 27% and 4 up to 12% slower, 8 and 12
// within 5% either way.
constexpr int kSlabCost = 6;
// Workgroups per compute unit when the groups' chunks are cut to equal cost (0: the same chunks for every group), by the work
// `per_cu` that one wave of a compute unit has when all is spread evenly over the chip (tiles of 32 points, about 0.3 us each).
// Equal cost pays where a launch is short or its groups are many; the same chunks let the groups of a chunk share its
// reads.  A workgroup pays some 9 us for its set-up and its last slabs, so a short launch gets one per compute unit; in a long
// one several even out each other's ends.  Sweeps of 8 rounds, time against the same chunks, geometric means over 396 shapes
// of one space (40,003 to 12M points) with up to 4 / 5 to 8 / more than 8 groups:
//   one     per_cu 100 .. 300: 0.86 / 0.87 / 0.87;  650 .. 800: 1.00 / 0.97 / 0.93;  800 .. 1000: 0.99 / 0.97 / 0.98;  1000 .. 2000: 1.02 / 0.99 / 0.98
//   two     per_cu 800 .. 2000: 1.03 / 0.97 / 0.90;  2000 .. 4000: 1.04 / 1.00 / 0.90
//   three   per_cu 2000 .. 4000: 1.05 / 1.00 / 0.89;  4000 .. 10,000: 1.03 / 0.93 / 0.89
//   five    per_cu 4000 .. 10,000: 1.03 / 0.90 / 0.87;  12,000 .. 14,500: - / 1.00 / 0.92;  above: 1.00, chunks of at most 2^16
//           points do not fit five any more
// (5 to 8 groups, 800 .. 2000: 8..63 gains 5%, 1..64 loses 1 to 2%.)
// A batch has at least as many workgroups as groups times spaces, and no freedom to even them out once these fill half of the
// chip.  One per compute unit over 614 batches, per_cu 20 .. 100 / 100 .. 300 / 300 .. 700 / 700 .. 1200: below 64 of them 0.83 /
// 0.91 / 0.98 / 1.03, 64 to 127: 0.88 / 0.95 / 1.00 / 1.08, 128 to 255: 1.02 / 1.11 / 1.13 / 1.18, more: 1.07 / 1.07 / 1.09 / 1.14.
int workgroups_per_cu(int64_t per_cu, int n_groups, int batch)
{
    if (batch > 1) return per_cu < 700 && n_groups * batch < kFillWorkgroups / 2 ? 1 : 0;
    if (per_cu < (n_groups <= 4 ? 1000 : 800)) return 1;
    if (n_groups <= 4 || (n_groups <= 8 && per_cu < 2000)) return 0;
    return (int)std::min<int64_t>(std::max<int64_t>((per_cu + 600) / 1200, 2), 5);
}

// An order of the points costs five launches, the copying of the rows, a dearer last pass and some 6 us a round for the lists, and
// pays by the tiles that the rounds leave out: all but one of a group at most.  The measure: thousands of points times (the tiles
// of the groups with lists, less one for every group, up to 16 features less one more, which the cheaper tiles there take to pay for
// the copying).  Time without against with an order, geometric means over 850 sweeps of one to 64 spaces of knob configurations
// after 10 / 20 / 30 rounds, by that measure:
//   up to 16 features   3000 .. 4000: 0.91 / 0.97 / 0.99;  4000 .. 5000: 0.95 / 1.00 / 1.02;  5000 .. 6000: 0.97 / 1.04 / 1.07;
//                       6000 .. 8000: 1.01 / 1.06 / 1.09;  8000 .. 12,000: 1.07 / 1.13 / 1.16;  12,000 .. 16,000: 1.14 / 1.21 / 1.25
//   17 to 32            1000 .. 3000: 0.92 / 0.95 / 0.97;  3000 .. 4000: 0.96 / 1.00 / 1.02;  4000 .. 5000: 0.99 / 1.03 / 1.05;
//                       5000 .. 6000: 1.03 / 1.06 / 1.07;  6000 .. 8000: 1.04 / 1.08 / 1.10;  8000 .. 12,000: 1.10 / 1.15 / 1.17
// Rows without any structure gain nothing by it, and that cannot be told from the sizes: independent normal deviates take 1.17 times
// as long with an order at 100,003 x 16, k 1..64, 1.18 at 1M, 1.03 at 2M x 32 (20 rounds).  A caller with such rows hands in the
// least workspace.
bool sweep_wants_order(int64_t N, int32_t d, int32_t k_min, int32_t k_max, int32_t batch)
{
    if (N < 16384 || k_max - k_min + 1 < 8) return false;
    SweepPlan plan;
    if (make_sweep_plan(N, d, k_min, k_max, 1, true, &plan) != RLS_OK) return false;
    int64_t tiles = 0;
    for (int gi = 0; gi < plan.n_groups; ++gi) tiles += plan.g[gi].list0 >= 0 ? plan.g[gi].n_tiles : 0;
    const int64_t thousands = N * batch / 1024;
    return plan.dp == 32 ? thousands * (tiles - plan.n_groups) >= 4000 : thousands * (tiles - plan.n_groups - 1) >= 5000;
}

// What a slab of a group costs, in fifths of a tile: its tiles - with lists a fifth of them and one more - and the rest.
static int slab_cost(const GroupDesc &g)
{
    return (g.list0 >= 0 ? 5 + g.n_tiles : 5 * g.n_tiles) + 5 * kSlabCost;
}

int32_t make_sweep_plan(int64_t N, int32_t d, int32_t k_min, int32_t k_max, int32_t batch, bool ordered, SweepPlan *plan)
{
    const int dp = padded_d(d);
    LloydGeometry geo = lloyd_geometry(dp);
    if (ordered) geo.lds_budget = 160 * 1024;      // the places of the centroids have to fit as well
    plan->ordered = ordered ? 1 : 0;
    int n_lists = 0;
    plan->n_runs = k_max - k_min + 1;
    plan->k_min = k_min;
    plan->dp = dp;
    plan->n_groups = 0;
    int tiles = 0;
    int run = 0;
    int lab_slots = 0;       // run slots (8 / S per group) of the groups so far
    while (run < plan->n_runs) {
        // candidates: R runs side by side (8 / R slots each); take the one with the least padding per real
        // row, preferring the larger R - except between candidates that cover the same runs at the same padding
        // (the end of a range, a single k): there the smaller R wins, since a lane keeps state for R runs, used or not
        int best_R = 0, best_tiles = 0, best_nr = 0;
        double best_score = 1e30;
        for (int R = 8; R >= 1; R >>= 1) {
            const int S = 8 / R;
            const int nr = plan->n_runs - run < R ? plan->n_runs - run : R;
            const int kmax_g = k_min + run + nr - 1;
            const int quads = (kmax_g + 3) / 4;
            const int n_tiles = (quads + S - 1) / S;
            const int real_rows = rows_before(k_min, run + nr) - rows_before(k_min, run);
            if (n_tiles > (ordered ? kListMaxTiles : 32)) continue;        // (lists are kept for that many)
            if (lloyd_group_lds_bytes(dp, d, n_tiles, real_rows, 1, ordered) > geo.lds_budget) continue;
            // cost per real row: padded rows and a fixed per-group overhead
            const double score = (n_tiles * 32.0 + 24.0) / real_rows;
            if (score < best_score - 1e-12 || (nr == best_nr && score < best_score + 1e-12)) {
                best_score = score; best_R = R; best_tiles = n_tiles; best_nr = nr;
            }
        }
        if (best_R == 0 || plan->n_groups >= kMaxGroups) return RLS_ERR_INVALID_ARG;
        GroupDesc &g = plan->g[plan->n_groups++];
        g.run0 = (int16_t)run; g.n_runs = (int16_t)best_nr; g.S = (int16_t)(8 / best_R); g.n_tiles = (int16_t)best_tiles;
        g.lab0 = (int16_t)lab_slots; g.tile0 = tiles;
        g.list0 = ordered && best_tiles >= kListMinTiles ? n_lists++ : -1;
        lab_slots += best_R;
        // Runs with few clusters send many lanes of a wave to the same accumulator address (32 / k on average), which
        // the LDS works off one after the other: such groups keep several copies of their accumulators, LDS permitting.
        {
            const int kmax_g = k_min + run + best_nr - 1;
            const int real_rows = rows_before(k_min, run + best_nr) - rows_before(k_min, run);
            int copies = kmax_g <= 8 ? 16 : (kmax_g <= 16 ? 8 : (kmax_g <= 32 ? 4 : (kmax_g <= 64 ? 2 : 1)));
            while (copies > 1 && lloyd_group_lds_bytes(dp, d, best_tiles, real_rows, copies, ordered) > geo.lds_budget) copies >>= 1;
            g.copies = (int16_t)copies;
        }
        tiles += best_tiles;
        run += best_nr;
    }
    plan->total_tiles = tiles;
    plan->lab_slots = lab_slots;
    // launch order: groups by falling cost (tiles per point)
    for (int i = 0; i < plan->n_groups; ++i) plan->sched[i] = (uint8_t)i;
    for (int i = 1; i < plan->n_groups; ++i) {
        const uint8_t v = plan->sched[i];
        int j = i;
        while (j > 0 && plan->g[plan->sched[j - 1]].n_tiles < plan->g[v].n_tiles) { plan->sched[j] = plan->sched[j - 1]; --j; }
        plan->sched[j] = v;
    }
    plan->total_rows = rows_before(k_min, plan->n_runs);
    if (batch < 1) batch = 1;
    const int64_t units = (int64_t)plan->n_groups * batch;
    const int64_t cap = (int64_t)1 << 16;      // points per chunk (the accumulators would allow 2^17)
    plan->chunk_block = -1;
    const int waves = step_threads_of(dp) / 64;
    const int64_t per_round = (int64_t)slab_blocks_of(dp, 1) * 32 * waves;
    int64_t cost = 0;
    for (int gi = 0; gi < plan->n_groups; ++gi) cost += slab_cost(plan->g[gi]);
    const int64_t per_cu = (N + 31) / 32 * cost * batch / (5 * kFillWorkgroups * waves);
    const int per_cu_wgs = workgroups_per_cu(per_cu, plan->n_groups, batch);
    if (per_cu_wgs > 0) {
        // Every group gets chunks of its own length, so that all workgroups take about the same time.  With r rounds of slabs
        // for its waves, a workgroup of group g is busy for r (tiles + kSlabCost): the shortest time is looked for with which
        // the workgroups of all groups fit when every group takes as many whole rounds as that time allows.
        auto chunks_of = [&](const GroupDesc &g, int64_t time) {
            const int64_t rounds = std::max<int64_t>(5 * time / slab_cost(g), 1);
            const int64_t len = std::min(rounds * per_round, cap);
            return (N + len - 1) / len;
        };
        auto fits = [&](int64_t time) {
            int64_t n = 0;
            for (int gi = 0; gi < plan->n_groups; ++gi) n += chunks_of(plan->g[gi], time);
            return n * batch <= (int64_t)per_cu_wgs * kFillWorkgroups;
        };
        int64_t lo = 0, hi = 2 * per_cu + 1000;
        if (fits(hi)) {
            while (lo + 1 < hi) {
                const int64_t mid = (lo + hi) / 2;
                if (fits(mid)) hi = mid; else lo = mid;
            }
            for (int gi = 0; gi < plan->n_groups; ++gi) {
                GroupDesc &g = plan->g[gi];
                const int64_t nc = chunks_of(g, hi);
                g.chunk_len = (int32_t)std::min<int64_t>(((N + nc - 1) / nc + 63) / 64 * 64, cap);     // spread evenly
                g.n_chunks = (int32_t)((N + g.chunk_len - 1) / g.chunk_len);
            }
            plan->chunk_block = 0;
        }
    }
    if (plan->chunk_block < 0) {
        // Large inputs: the same chunks for every group, two workgroups per compute unit over the whole batch (a workgroup
        // stages its group's rows once, so more and shorter chunks only add set-up: 1024 workgroups measured 4% longer
        // launches at 1M x 16, 256 22% longer); a chunk never exceeds 2^16 points (with the groups of a chunk running side
        // by side shorter chunks measured 2% shorter launches at 8M x 32)
        const int tp = geo.tile_points;
        const int64_t tiles_total = (N + tp - 1) / tp;
        int64_t want = 2 * kFillWorkgroups / units;
        // More groups times spaces than compute units: rather a few workgroups too many than half of the chip idle in the last
        // turn, but chunks of 4096 points at least (64 spaces of 65,537 x 16, k 8..63, 448 groups: one chunk of 2^16 points
        // and one of a single point: 34.3 ms for 8 rounds, two halves 19.1).
        if (units > kFillWorkgroups) want = std::min((2 * kFillWorkgroups + units - 1) / units, (N + 4095) / 4096);
        if (want > tiles_total) want = tiles_total;
        int64_t chunk_len = ((tiles_total + want - 1) / want) * tp;
        if (chunk_len > cap) chunk_len = cap / tp * tp;
        const int64_t n_chunks = (N + chunk_len - 1) / chunk_len;
        for (int gi = 0; gi < plan->n_groups; ++gi) {
            plan->g[gi].chunk_len = (int32_t)chunk_len;
            plan->g[gi].n_chunks = (int32_t)n_chunks;
        }
        // chunks per block of the launch order: about one workgroup per compute unit in a block, a multiple of eight chunks
        // (workgroups go to the eight XCDs in turn, so the groups of one chunk meet on one XCD)
        int32_t cb = (kFillWorkgroups + plan->n_groups - 1) / plan->n_groups;
        cb = (cb + 7) / 8 * 8;
        const int64_t n_all = n_chunks * batch;                                  // chunks of all spaces of the batch
        if (cb > n_all) cb = (int32_t)n_all;
        plan->chunk_block = cb;
    }
    int64_t wgs = 0, parts = 0;
    for (int gi = 0; gi < plan->n_groups; ++gi) {
        GroupDesc &g = plan->g[gi];
        g.wg0 = (int32_t)wgs;
        g.part0 = (int32_t)parts;
        wgs += g.n_chunks;
        parts += (int64_t)g.n_chunks * (rows_before(k_min, g.run0 + g.n_runs) - rows_before(k_min, g.run0));
    }
    if (wgs * batch > 0x7fffffffLL || parts > 0x7fffffffLL) return RLS_ERR_INVALID_ARG;
    plan->n_wgs = plan->loss_wgs = (int32_t)wgs;
    if (ordered) {
        SweepPlan plain;                       // (its chunks are those of the losses)
        const int32_t rc = make_sweep_plan(N, d, k_min, k_max, batch, false, &plain);
        if (rc != RLS_OK) return rc;
        plan->loss_wgs = plain.n_wgs;
    }
    plan->n_lists = n_lists;
    plan->n_parts = (int32_t)parts;
    return RLS_OK;
}

int64_t tile_list_words(const SweepPlan &plan, int64_t N)
{
    return (int64_t)plan.n_lists * ((N + 32 * unit_blocks_of(plan.dp) - 1) / (32 * unit_blocks_of(plan.dp))) * kListWords;
}

void sweep_layout(const SweepPlan &plan, int64_t N, int32_t d, int32_t k_max, int32_t batch, SweepLayout *L)
{
    int64_t off = 0;
    auto take = [&](int64_t bytes) { const int64_t o = off; off += align_up(bytes, 256); return o; };
    L->stat_blocks = (int32_t)(N < 65536 ? (N + 255) / 256 : kStatBlocks);
    if (L->stat_blocks > kStatBlocks) L->stat_blocks = kStatBlocks;
    if (L->stat_blocks < 1) L->stat_blocks = 1;
    L->seed_blocks = (int32_t)((N + kSeedBlock - 1) / kSeedBlock);
    // seeding state and partial column statistics: needed until the first round
    L->colstat_part = take((int64_t)kStatBlocks * 32 * sizeof(ColPart));
    L->mind = take(N * 8);
    L->bsum = take((int64_t)L->seed_blocks * 8);
    L->near = take(N);
    L->seedthr = take((int64_t)k_max * 8);
    L->colinfo = take(512);
    L->chain = take((int64_t)k_max * 8);
    L->xp = take((N + 31) / 32 * prep_block_u4_of(plan.dp) * 16);     // (with the blocks above: the same place whatever the range of k)
    const int64_t n_units = (N + 32 * unit_blocks_of(plan.dp) - 1) / (32 * unit_blocks_of(plan.dp));
    L->keyinfo = L->perm = L->inv = L->xs = L->centres = L->radius = L->rowpos = L->rowidx = L->lists = 0;
    if (plan.ordered) {
        L->keyinfo = take(sizeof(KeyInfo));
        L->perm = take(N * 4);
        L->inv = take(N * 4);
        L->xs = take(std::max(align_up(N, 64) * plan.dp * 4, order_scratch_bytes(N)));
        L->centres = take((n_units + 31) / 32 * prep_block_u4_of(plan.dp) * 16);
        L->radius = take(align_up(n_units, 32) * 4);
        // (from here on: a place that depends on the range of k)
        L->rowpos = take((int64_t)plan.total_rows * 2);
        L->rowidx = take((int64_t)plan.total_rows);
        L->lists = take(tile_list_words(plan, N) * 4);
    }
    L->opA = take((int64_t)plan.total_tiles * tile_bytes_of(plan.dp));
    L->cnmax = take((int64_t)plan.n_runs * kMaxParts * 4);
    L->psum = take((int64_t)plan.n_parts * d * 8);
    L->pcnt = take((int64_t)plan.n_parts * 4);
    L->pj = take((int64_t)plan.loss_wgs * 8 * 8);
    L->losum = take((int64_t)plan.total_rows * d * 8);
    L->tot = take((int64_t)plan.total_rows * d * 16);
    L->totcnt = take((int64_t)plan.total_rows * d * 8);
    L->prev = take((int64_t)plan.lab_slots * align_up(N, 16));
    L->per_batch = off;
    L->total = off * batch;
}

hipError_t launch_sweep(const SweepPlan &plan, const SweepLayout &L, const SweepArgs &a, hipStream_t s)
{
    switch (plan.dp) {
    case 8: return launch_sweep_dp<8>(plan, L, a, s);
    case 16: return launch_sweep_dpad16(plan, L, a, s);
    default: return launch_sweep_dpad32(plan, L, a, s);
    }
}
#endif

}  // namespace rls
