// Launch interface between the C-ABI layer (host) and the gfx950 kernels.
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstdint>

#include "star.h"

namespace star {

constexpr int kBlock = 256;          // threads per workgroup: 4 wave64
constexpr int kFewRows = 6;          // up to this many rows the Gram matrix behind the norms stays in vector registers
constexpr int kGridCap = 1024;       // most workgroups a norm-reducing launch uses (sizes the partial buffer)

// Work queue of one launch: the next tile nobody has claimed yet and the number of workgroups that
// have left the kernel.  16 bytes of device memory, all zero between launches: the last workgroup
// to leave clears it, so no fill is needed before the next launch (stream order does the rest).
struct TileQueue {
    unsigned long long next;
    unsigned int done;
    unsigned int pad;
};

// The ticket of gram_finish_kernel and the one of a call's last launch (Finished) lie behind the queue, in the same 256 bytes.
inline unsigned int* finish_ticket(TileQueue* q) { return reinterpret_cast<unsigned int*>(q + 4); }
inline unsigned int* last_ticket(TileQueue* q) { return reinterpret_cast<unsigned int*>(q + 8); }

// How the host learns that a call no longer uses its workspace slot: the last workgroup of the call's last launch writes `seq` to `word`, which
// lies in pinned memory.  (An event recorded behind the call tells the same, but the GPU takes 4.4 us longer to the next call's kernel, and the
// host 2 to 4 us for the record.)
struct Finished {
    uint32_t* word = nullptr;         // as the device addresses it; null: nobody asks
    uint32_t seq = 0;
    unsigned int* ticket = nullptr;   // device, zero between launches
};
// The tile queue as a kernel is handed it: the last workgroup to leave writes `seq`, if there is a word.
struct TileSource {
    TileQueue* queue;
    uint32_t* word;
    uint32_t seq;
};
inline TileSource tile_source(TileQueue* q, const Finished& f) { return TileSource{q, f.word, f.seq}; }

// Tiles an update hands to a workgroup per claim.  Not a power of two: with 2, 4 or 8 tiles every claim starts
// on an 8/16/32 KB boundary of every row, all workgroups then hit the same memory channels at the same
// moments, and the update measured 5-8 % slower than with 3 (only the heaviest tiles, of which 3 are too long a claim, take 2, and
// launches that read take what their bytes ask for, up to 16: see queue_claim).  Light tiles (few rows: a thread moves less
// than 96 bytes per tile, state included) are finished so quickly that claims of 3 come faster than the
// one counter serves them (it sustains about 80 M atomics/s); 5 measured 15-40 % faster there (one fp32
// row and the state: 0.37 against 0.48 ms on 110 M elements), 6, 7 and 9 slower again.
constexpr int kClaim = 3;
constexpr int kClaimLight = 5;
// What a launch does to memory decides how much work a claim should cover.  A claim's round trip to the
// counter is hidden only if the workgroup has several microseconds of tiles left when it asks, and a
// kernel that only reads gets through a tile much faster than one that also writes the state back:
//   Update   reads the rows, reads and writes the state: 3 tiles, 5 when light (see above), 2 when very heavy;
//   ReadOnly the norms alone, the Gram matrix: about 200 KB per claim (16 bf16 rows, 32 KB a tile: 6 or 7
//            tiles run 0.83-0.86 of the HBM peak against 0.68-0.71 with 3; 8 bf16 rows: 13 tiles 0.82
//            against 0.61 with 5; 16 fp32 rows stay at 3);
//   Reduce   reads the rows, writes one output row per group: about 140 KB per claim (16 bf16 rows: 4
//            tiles 0.75 against 0.71 with 3; 16 fp32 rows: 2 tiles 0.74 against 0.72).
enum class Traffic { Update, ReadOnly, Reduce };
inline int queue_claim(int thread_bytes, Traffic traffic = Traffic::Update) {
    const int tile = (thread_bytes < 1 ? 1 : thread_bytes) * kBlock;
    if (traffic == Traffic::ReadOnly) {
        const int c = (200 * 1024 + tile / 2) / tile;
        return c < 3 ? 3 : (c > 16 ? 16 : c);
    }
    if (traffic == Traffic::Reduce) {
        const int c = (140 * 1024 + tile / 2) / tile;
        return c < 2 ? 2 : (c > 9 ? 9 : c);
    }
    // very heavy tiles (20 to 32 fp32 rows: 90-140 KB a tile): two tiles a claim, 2-4 % ahead of three
    if (thread_bytes >= 320) return 2;
    return thread_bytes < 96 ? kClaimLight : kClaim;
}

// Shards shorter than this many elements keep the static mapping (and need no queue): with few tiles
// per workgroup the claims' round trips show (1 Mi elements: 15 against 7.5 us); from 16 Mi on the
// queue order wins (+12 % with 8 fp32 rows).
constexpr int64_t kQueueMinElements = 16 << 20;
// Shards shorter than this take their norms from direct sums whatever the stream (see decide()).
constexpr int64_t kTinyShardElements = 4096;

// First round of claims (see for_each_claimed_tile): workgroup b of G gets 1 + b % claim tiles, laid out
// one after the other from tile 0; the queue's counter hands out the tiles from `base` on.
// A negative `claim` is the short-shard form: first claims that split all `ntile` tiles evenly between
// the workgroups (consecutive tiles each, counts differ by at most one), so that nothing is left for
// the counter and no workgroup waits for it.  With 2 to 8 tiles per workgroup the unequal first claims
// and their granularity would leave some workgroups with twice the work of others, and a kernel of a
// few microseconds would spend one or two of them on the counter's round trips.
struct FirstClaim {
    int64_t t0;                // first tile of the workgroup's first claim
    int n;                     // tiles in it
    unsigned long long base;   // tiles covered by all first claims together
};
__host__ __device__ inline FirstClaim first_claim_of(const int64_t b, const int64_t G, const int claim,
                                                     const int64_t ntile = 0) {
    if (claim < 0) {   // short shard: the tiles split evenly, workgroup b gets [b ntile / G, (b+1) ntile / G)
        FirstClaim e;
        e.t0 = b * ntile / G;
        e.n = (int)((b + 1) * ntile / G - e.t0);
        e.base = (unsigned long long)ntile;
        return e;
    }
    const int64_t per_group = (int64_t)claim * (claim + 1) / 2;   // tiles taken by `claim` consecutive workgroups
    const int64_t r = b % claim, rg = G % claim;
    FirstClaim f;
    f.t0 = (b / claim) * per_group + r * (r + 1) / 2;
    f.n = (int)r + 1;
    f.base = (unsigned long long)((G / claim) * per_group + rg * (rg + 1) / 2);
    return f;
}

struct RowPtrs {
    const void* p[STAR_MAX_WORKERS];
};

// Coefficients of the collapsed map, passed by value in the kernel arguments
// so that they live in scalar registers:
//   p' = p + (dp*p + m01*v + sum_w b0[w] g_w),   v' = m10*p + m11*v + sum_w b1[w] g_w
struct AffCoef {
    float dp, m01, m10, m11;
    float b0[STAR_MAX_WORKERS];
    float b1[STAR_MAX_WORKERS];
};

// Row counts the kernels are instantiated for; a plan with Wc rows runs on
// padded_rows(Wc) >= Wc rows, the extra ones carrying zero coefficients.
int padded_rows(int Wc);

// Small group tables travel in the kernel arguments instead of through a
// host-to-device copy: a call with one or a few updates (the un-queued
// parameter-server case) is then a single enqueue.
constexpr int kInlineUpdates = 32;
constexpr int kInlineCoef = 256;
struct InlineTables {
    float coef[kInlineCoef];        // [U][Wp]
    float lr[kInlineUpdates];
    uint32_t mask[kInlineUpdates];
    void* out[kInlineUpdates];      // output rows (aggregation only)
};
inline bool tables_fit_inline(int U, int Wp) { return U <= kInlineUpdates && U * Wp <= kInlineCoef; }

struct SeqArgs {
    float* params;
    float* momentum;
    RowPtrs rows;
    const float* coef;     // device [U][Wp], or null: the tables are in `inl`
    const float* lr;       // device [U]
    const uint32_t* mask;  // device [U]
    const InlineTables* inl;  // host; used when coef is null
    const AffCoef* cf;     // host, or null; not null: the update is applied once, as this map (17-32 fp32 rows, update + norms)
    int32_t U;             // updates in this launch
    int32_t members;       // their groups' sizes added up
    float mu, wd;
    int64_t P;
    int32_t head;          // elements before the pointers and P (0 to 63), see rest_element
    void* publish;         // device copy of the new params (P elements), or null
    int32_t publish_dtype; // star_dtype of that copy
    double* partials;      // device [U][grid] sums of gbar^2 per block (norms only)
    TileQueue* queue;      // device, zeroed; null: fixed assignment of tiles to workgroups
    Finished done;         // launch_seq without norms: written by a launch that takes tiles from the queue
    bool* told;            // host, or null: set if the launch does
};

// Rows heavy enough for the kernel that writes in bursts (aff_burst_kernel), see burst_claim.
constexpr bool bursts(int Wp, bool f32_rows) { return Wp >= (f32_rows ? 10 : 12); }

// Which launches take their tiles from the queue when the caller hands one in (the matrix-core kernel
// always does): the step-by-step kernel for one or two updates (longer streams are bound by arithmetic
// and keep the fixed assignment with as many waves as fit), the collapsed one unless it carries the
// register-heavy Gram accumulators of more than kFewRows rows.
inline bool seq_takes_queue(int updates_in_launch) { return updates_in_launch <= 2; }
// Collapsed update with direct norms (step-by-step kernel's norm walk): for 17 to 32 fp32 rows, when the
// stream's direct norm sums cost at most this many multiply-adds per element.  Measured against the Gram
// matrix on the matrix cores, 2 Mi and 64 Mi elements, 6 to 16 updates: the walk wins by 5-14 % up to about
// 130 / 145 / 160 / 175 multiply-adds with 20 / 24 / 28 / 32 rows and loses beyond (at twice that by a third);
// the limit grows with the rows because the matrix-core kernel's time does.  (Up to 24 rows that kernel now works by row
// groups of four and is 6-12 % faster: 20 rows, 25.6 M elements, 84 / 115 / 138 multiply-adds 425 / 466 / 486 us against 470; 24
// rows, 108 / 135 / 162: 500 / 549 / 579 against 542.  The limit stays where it was all the same: the few percent below it are
// not worth norms that lose digits where rows are anti-correlated, 1.8e-5 against 2e-8 at kappa = 4e4.)
inline double direct_norm_fma_limit(int Wp) { return 4.0 * Wp + 48.0; }
// Which Gram launches of the collapsed kernel use the few-rows form (double fold slots in LDS after every
// chunk, tiles from the queue on long shards): up to kFewRows rows -- except the Gram matrix alone on exactly
// kFewRows fp32 rows, whose 21 slot updates per chunk are not hidden by 96 bytes of loads (32 to 96 Mi
// elements: 0.57-0.65 of the HBM peak, against 0.82 with 5 rows and 0.85 with 7); that one takes the form
// of the larger row counts (fp32 slots folded every kGramFold tiles, fixed assignment).
constexpr bool gram_few_rows_form(int Wp, bool f32_rows, bool update) {
    return Wp <= kFewRows && !(Wp == kFewRows && f32_rows && !update);
}
inline bool aff_takes_queue(bool gram, int Wp, bool f32_rows, bool update) {
    return gram ? gram_few_rows_form(Wp, f32_rows, update) : !bursts(Wp, f32_rows);
}

// Collapsed updates without norms on P elements: tiles per claim of the kernel that writes in bursts, 0 for aff_kernel.  Sweep over 1 to 150 M
// elements, 3 to 32 fp32 and 5 to 32 bf16 rows, three states in turn, aff_kernel -> aff_burst_kernel:
//   length and rows   fp32: 40 / 100 M elements, 10 rows 355 / 881 -> 347 / 854 us, 12 rows 410 / 1021 -> 397 / 978, 16 rows 525 / 1309 -> 482 /
//                     1195, 24 rows 729 / 1899 -> 677 / 1709, 32 rows 945 / 2483 -> 880 / 2204; at the limits 13 M, 10 rows 130 -> 122, 11 M, 12
//                     rows 122 -> 116, 8 M, 16 rows 114 -> 110, 3.8 M, 24 rows 82 -> 78.  bf16: 60 / 150 M, 12 rows 403 / 1011 -> 390 / 947, 16 rows
//                     488 / 1154 -> 452 / 1105, 24 rows 653 / 1533 -> 596 / 1455, 32 rows 826 / 1930 -> 741 / 1813; 30 M, 12 rows 202 ->
//                     196, 22 M, 16 rows 176 -> 171, 16 M, 24 rows 170 -> 163.
//   not               lighter rows, which fill the LDS with results before a period of reads has paid (40 / 100 M, 5 / 6 / 8 fp32 rows 238 / 253 /
//                     302 and 579 / 624 / 754 against 237 / 259 / 300 and 579 / 635 / 749), and shorter shards (8 M, 12 fp32 rows 91 against 91, 8 /
//                     12 M, 24 bf16 rows 90 / 134 against 91 / 134, 16 M, 18 rows 136 against 137).
//   in the cache      where rows and state have just been written, and the memory-side cache holds the last 256 MB of them, there is less to gain
//                     (25 M, 12 / 16 / 24 fp32 rows 258 / 326 / 464 against 262 / 333 / 471; 100 M 1007 / 1292 / 1897 -> 990 / 1208 / 1727) and lighter
//                     rows lose (40 M, 8 rows 298 against 309).
//   tiles per claim   90 M, 12 / 16 / 24 fp32 rows, 2 / 3 / 4 / 5: 957 / 855 / 913 / 861, 1149 / 1051 / 1166 / 1089, 1596 / 1510 / - / 1529 us; 30 M, 24
//                     rows, 2 / 3 490 / 507; 120 M, 12 / 16 / 24 bf16 rows, 3 / 4 / 5 / 6: 810 / 776 / 736 / 724, 926 / 903 / 858 / 856,
//                     1157 / 1186 / 1156 / 1166.
inline int burst_claim(int Wp, bool f32_rows, int64_t P) {
    constexpr int64_t kMi = 1 << 20;
    if (!bursts(Wp, f32_rows)) return 0;
    if (f32_rows) {
        if (P < (Wp >= 24 ? 7 * kMi / 2 : (Wp >= 16 ? 7 * kMi : (Wp >= 12 ? 10 * kMi : 12 * kMi)))) return 0;
        if (Wp >= 20 && P < 72 * kMi) return 2;
        return Wp >= 11 ? 3 : 5;
    }
    if (P < (Wp >= 24 ? 15 * kMi : (Wp >= 16 ? 20 * kMi : 24 * kMi))) return 0;
    return Wp >= 24 ? 3 : (Wp >= 16 ? 5 : 6);
}

// The same for the update with norms from the matrix cores (aff_mfma_kernel); 0: it writes as it goes.  Three states in turn, without -> with bursts:
//   fp32 rows   40 / 140 M elements, 14 rows 481 / 1643 -> 468 / 1608 us, 16 rows 542 / 1854 -> 515 / 1771, 20 rows 692 / 2342 -> 670 / 2283;
//               17 M, 14 / 16 / 20 rows 215 / 241 / 312 -> 210 / 230 / 296.  Not 12 M (14 / 16 rows 158 / 177 against 164 / 182), not 12 rows (140 M
//               1462 against 1486), and not 24 and more, whose matrix work one wave per SIMD does not hide (25.6 M, 24 / 32 rows
//               540 / 691 against 551 / 718).
//   bf16 rows   40 / 200 M, 12 rows 273 / 1281 -> 267 / 1264, 16 rows 329 / 1560 -> 313 / 1485; 80 M, 24 / 28 / 32 rows 889 / 1004 / 1142 -> 856 /
//               962 / 1068, 17 M 205 / 232 / 263 -> 199 / 226 / 247 (12 M: 150 / 169 / 192 against 155 / 176 / 197); 5 / 8 M, 8 / 12 / 16 rows 41 / 50 /
//               58 and 63 / 76 / 82 -> 40 / 47 / 55 and 53 / 64 / 77 (3 M level; 7 and 8 rows are in vector registers from 8 Mi to 16 Mi); 7 to 11 rows beyond that: level at 17 M, 80 M, 8 / 11 rows 431 /
//               498 against 436 / 498.  20 rows: 25.6 M 253 against 257.
//   tiles per claim   140 M, 16 fp32 rows, 5 / 6: 1771 / 1788; 200 M, 12 / 16 bf16 rows 1285 / 1264, 1492 / 1485; 25.6 M, 16 rows 208 / 208; 150 M,
//                     32 rows, 5 / 7 / 9: 2004 / 1966 / 1941, 25.6 M 363 / 359 / 354.
constexpr bool mfma_bursts(int Wp, bool f32_rows) { return f32_rows ? Wp >= 14 && Wp <= 20 : Wp >= 7 && Wp != 20; }
inline int mfma_burst_claim(int Wp, bool f32_rows, int64_t P) {
    constexpr int64_t kMi = 1 << 20;
    if (!mfma_bursts(Wp, f32_rows)) return 0;
    if (f32_rows) return P >= 16 * kMi ? 5 : 0;
    if (Wp > 16) return P >= 16 * kMi ? (Wp > 28 ? 9 : 7) : 0;
    if (P < 9 * kMi / 2 || (Wp < 12 && P > 12 * kMi)) return 0;
    return P >= 14 * kMi ? 6 : 5;
}

// Largest number of updates one launch of the step-by-step kernel accepts
// (bounded by the LDS tables and, with norms, the per-thread accumulators).
int seq_max_updates(int Wp, bool norms);

// Step-by-step evaluation.  Returns the grid used in *grid_out (needed to
// reduce the partials).  grid_cap bounds it.
hipError_t launch_seq(int Wp, int dtype, bool norms, const SeqArgs& a, int num_cu, int grid_cap, int* grid_out,
                      hipStream_t s);

// Direct norm sums without an update (params, momentum, publish and the update's fields of `a` are not used),
// up to walk_max_updates() updates a launch.
int walk_max_updates();
hipError_t launch_norm_walk(int Wp, int dtype, const SeqArgs& a, int num_cu, int grid_cap, int* grid_out,
                            hipStream_t s);
// Its grid and the updates of a workgroup on the vector ALUs: `tiles` and perhaps a rest, at most `most` workgroups.
void walk_shape(int W, int most, int num_cu, int64_t tiles, bool rest, int U, int* grid, int* share);
// Whether such a launch goes to the matrix cores: U updates whose groups have `members` in all, P elements behind the head.
bool norms_on_matrix_cores(int Wp, bool f32, int U, int members, int64_t P);

// Coefficients of the norms that a launch carries from the host's pinned memory (as the device addresses it) to device memory.
struct CoefCopy {
    const double* src;
    double* dst;
    int n;   // 0: none
};

struct AffArgs {
    float* params;
    float* momentum;
    RowPtrs rows;
    AffCoef cf;
    int32_t rows_used;      // distinct rows (the rest of the padded count repeats the last one)
    int64_t P;
    int32_t head;           // elements before the pointers and P (0 to 63), see rest_element
    void* publish;          // device copy of the new params (P elements), or null
    int32_t publish_dtype;  // star_dtype of that copy
    double* partials;  // device [Wp(Wp+1)/2][grid] pairwise-product sums per block (gram only)
    TileQueue* queue;  // device, zeroed; null: fixed assignment of tiles to workgroups (not for the matrix-core kernel)
    CoefCopy copy;     // launch_affine with `gram`, without a queue
    int32_t burst;     // with `update`: see burst_claim and mfma_burst_claim (with a queue)
    Finished done;     // launch_affine without `gram`: written by a launch that takes tiles from the queue
    bool* told;        // host, or null: set if the launch does
};

// Collapsed evaluation, optionally accumulating the Gram matrix of the rows.
hipError_t launch_affine(int Wp, int dtype, bool update, bool gram, const AffArgs& a, int num_cu, int grid_cap,
                         int* grid_out, hipStream_t s);

// The same with the Gram matrix formed on the matrix cores (any Wp up to 32; `gram` is implied).
hipError_t launch_affine_mfma(int Wp, int dtype, bool update, const AffArgs& a, int num_cu, int grid_cap,
                              int* grid_out, hipStream_t s);

// out[e] = sum_b partials[e*grid + b] in a fixed order; sums_out (double) and
// sqrt_out (float, square root of the sum) are each optional.
hipError_t launch_reduce(const double* partials, int n_out, int grid, double* sums_out, float* sqrt_out,
                         const Finished& done, hipStream_t s);

// norms_out[u] = sqrt( c_u^T Gamma c_u ), Gamma upper-triangular packed [Wp(Wp+1)/2], coef [U][Wp] doubles.
hipError_t launch_gram_norms(const double* gamma, const double* coef, int U, int Wp, float* norms_out,
                             const Finished& done, hipStream_t s);

// launch_reduce and launch_gram_norms in one launch, see norms_finish_at_once.  `gamma` and `coef` are device memory; `ticket` is zero
// before and after.
hipError_t launch_gram_finish(const double* partials, int grid, double* gamma, const double* coef, int U, int W,
                              unsigned int* ticket, float* norms_out, const Finished& done, hipStream_t s);
constexpr int kFinishRows = 8;
inline bool norms_finish_at_once(int W, int U, int64_t P) { return W <= kFinishRows && U <= 128 && P <= 2 << 20; }

// The same for the Gram matrix: partials of the packed upper triangle over Wp rows [Wp(Wp+1)/2][grid] -> full symmetric [W][W],
// W <= Wp (all zero with a grid of 0).
hipError_t launch_reduce_gram(const double* partials, int grid, int Wp, int W, double* out, const Finished& done, hipStream_t s);

hipError_t launch_fill(float* dst, int64_t n, float value, hipStream_t s);

// ---- the fixed device workspace of the entry point that allocates nothing
// One array of kScratchBytes per GPU, part of the library's device code (no hipMalloc behind it):
//   [0, 256)                                   the tile queue and the ticket of gram_finish_kernel
//   [256, 256 + kScratchTableBytes)            group tables
//   [256 + kScratchTableBytes, kScratchBytes)  per-workgroup partial sums and the reduced Gram matrix
constexpr int kScratchMaxUpdates = 256;                       // longest stream that entry point accepts
constexpr size_t kScratchTableBytes = 128 * 1024;             // tables of 256 updates over 32 rows: 100 KB
constexpr size_t kScratchPartialDoubles = 528 * (size_t)kGridCap + 528;   // Gram partials of 32 rows
constexpr size_t kScratchBytes = 4608 * 1024;                 // 4.5 MiB
static_assert(256 + kScratchTableBytes + kScratchPartialDoubles * sizeof(double) <= kScratchBytes,
              "the three parts fit in the array");

// Device address of the array on the current device (resolved once per device, then cached).
hipError_t scratch_address(void** out);

// dst[0..bytes) = src[0..bytes): host data carried to the device in kernel arguments, a few KB per
// launch -- no copy engine, no staging buffer, nothing allocated.  dst 16-byte aligned.  `clear`, if not null, is set to zero as well.
hipError_t launch_upload(void* dst_dev, const void* src_host, size_t bytes, hipStream_t s, unsigned int* clear = nullptr);

// Puts a tile queue back to "no tile claimed, nobody left".
hipError_t launch_queue_clear(TileQueue* q, hipStream_t s);

// ---- aggregation without the optimizer step (star_group_reduce)
struct ReduceArgs {
    RowPtrs rows;
    const float* coef;       // device [U][Wp], or null: the tables are in `inl`
    const uint32_t* mask;    // device [U]
    void* const* out;        // device array of U output row pointers
    const InlineTables* inl; // host; used when coef is null
    int32_t U;               // groups in this launch
    int32_t out_dtype;       // star_dtype of the outputs
    int64_t P;
    int32_t head;            // elements before the pointers and P (0 to 63), see rest_element
    int32_t norms;           // also accumulate sum of squares per group
    double* partials;        // device [U][grid] (norms only)
    TileQueue* queue;        // device, zeroed; null: fixed assignment of tiles to workgroups
    int32_t burst;           // see mean_burst_claim (with a queue, one group, tables in `inl`, no norms)
    Finished done;           // without norms: written by a launch that takes tiles from the queue
    bool* told;              // host, or null: set if the launch does
};

int reduce_max_updates(int Wp, bool norms);

// Tiles per claim of the kernel that writes the aggregate of one group, without norms, in bursts; 0 for reduce_rows_kernel.  Three states in turn,
// reduce_rows_kernel -> mean_burst_kernel:
//   fp32 rows and result   25.6 M elements, 6 / 8 / 12 / 16 / 24 / 32 rows 123 / 161 / 227 / 289 / 423 / 547 -> 115 / 142 / 202 / 261 / 379 / 497 us;
//                          100 M 460 / 596 / 870 / 1133 / 1725 / 2315 -> 424 / 538 / 768 / 1002 / 1499 / 2000; at the limits 14 M, 6 rows 67 -> 65,
//                          10 M, 7 rows 56 -> 54, 7 M, 9 rows 50 -> 48, 3 M, 12 / 16 / 32 rows 31 / 42 / 77 -> 30 / 37 / 68 (2 M: 20 / 26 / 48
//                          against 22 / 27 / 49; 4 M, 8 rows 27.3 against 28.3).  5 rows: 20 M level, 60 M 243 -> 231, left out.
//   bf16 rows, fp32        18 / 150 M, 12 rows 84 / 692 -> 83 / 641 us, 16 rows 105 / 894 -> 101 / 801, 24 rows 150 / 1326 -> 143 / 1156, 32 rows
//                          196 / 1712 -> 192 / 1538; 10 M, 16 / 24 / 32 rows 67 / 91 / 116 -> 61 / 84 / 112.  10 rows: 150 M level.
//   bf16 result            half the writes, less to gain: 25 / 60 M, 12 / 16 / 24 / 32 fp32 rows 210 / 271 / 396 / 510 and 486 / 639 / 937 / 1223 ->
//                          196 / 255 / 370 / 481 and 460 / 603 / 885 / 1179; 32 bf16 rows 271 / 654 -> 267 / 628, 24 rows 199 / 485 against 202 / 475.
//   tiles per claim        25.6 M, 8 / 12 / 16 / 24 fp32 rows, 2 / 3 / 5 / 7 / 9: - / 164 / 146 / 142 / 147, 232 / 209 / 202 / 211 / 214, 279 / 261 / 272 / 276 /
//                          279, 379 / 391 / 399 / 402 / 404; 140 M, 24 rows, 2 / 3: 2180 / 2109.
inline int mean_burst_claim(int Wp, bool f32_rows, bool bf16_out, int64_t P) {
    constexpr int64_t kMi = 1 << 20;
    if (f32_rows) {
        if (Wp < (bf16_out ? 12 : 6)) return 0;
        const int64_t from = bf16_out ? (Wp >= 14 ? 4 : 14) : (Wp >= 12 ? 3 : (Wp >= 9 ? 7 : (Wp >= 7 ? 8 : 14)));
        if (P < from * kMi) return 0;
        if (Wp >= 24) return P < 72 * kMi ? 2 : 3;
        return Wp >= 14 ? 3 : (Wp >= 9 ? 5 : (Wp >= 7 ? 7 : 9));
    }
    if (bf16_out) return Wp >= 28 && P >= 15 * kMi / 2 ? 3 : 0;
    if (Wp < 12 || P < (Wp >= 20 ? 15 * kMi / 2 : (Wp >= 14 ? 8 * kMi : 16 * kMi))) return 0;
    return Wp >= 20 ? 5 : (Wp >= 14 ? 7 : 9);
}

hipError_t launch_group_reduce(int Wp, int dtype, const ReduceArgs& a, int num_cu, int grid_cap, int* grid_out,
                               hipStream_t s);

}  // namespace star
