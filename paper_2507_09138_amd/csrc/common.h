// Shared declarations of the gfx950 IVF search library (internal; the public ABI is hr_ivf.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hr_ivf.h"

namespace hr {

constexpr int kWave = 64;
// internal storage codes next to HR_F32 / HR_F16 / HR_BF16: float32 rows already split into a
// binary16 hi table and a 2^11-scaled binary16 lo table (the centroid table, split at load), rounded to a binary16 table
// (lists with row tables), and float32 rows of which the scan splits every block in LDS
constexpr int HR_F16X2 = 3, HR_F16HI = 4, HR_F32X2 = 5;
constexpr int kMfmaRows = 16;              // rows per MFMA (M of 16x16x32)
constexpr int kAppendMax = 16;             // most candidates one column can gain per group of kMfmaRows rows
constexpr int kMinSegRows = 256;           // smallest rows-per-work-item
constexpr int kItemTarget = 4096;          // aimed number of scan work items per batch
constexpr int kHistBins = 64;              // per-query histogram of candidate keys (one bin per lane)

// Storage of which the scan leaves something out, the low parts (HR_F32, HR_F16HI) or what the two parts leave over (HR_F32X2), and
// keeps every row that may count with it; the merge computes the exact scores of the few that are left (see scan_slack)
__host__ __device__ constexpr bool scan_bounded(int dtype) { return dtype == HR_F32 || dtype == HR_F16HI || dtype == HR_F32X2; }

// Storage of which both parts of rows and query are multiplied, and storage of four bytes an element
__host__ __device__ constexpr bool scan_split(int dtype) { return dtype == HR_F16X2 || dtype == HR_F32X2; }
__host__ __device__ constexpr bool stored_f32(int dtype) { return dtype == HR_F32 || dtype == HR_F32X2; }

// Parts of a query operand that a wave keeps in registers of their own.  Two operands of d elements leave room for the rest in
// 256 registers up to d = 768.  Beyond that they take two MFMA columns per query (8 queries per wave).
__host__ __device__ constexpr int operand_parts(int dtype, int d)
{
    return (dtype == HR_BF16 || scan_split(dtype)) && d <= 768 ? 2 : 1;
}
// columns (queries) per wave
__host__ __device__ constexpr int cols_per_set(int dtype, int d) { return (dtype == HR_BF16 || scan_split(dtype)) && operand_parts(dtype, d) == 1 ? 8 : 16; }

constexpr int kScanWaves = 8;              // waves of a workgroup of the scan, two per SIMD
// queries of a work item
__host__ __device__ constexpr int tile_cols(int dtype, int d) { return kScanWaves * cols_per_set(dtype, d); }

// Groups of 16 rows that are staged, waited for and filtered together: a block of the scan has 16 * block_groups rows, about
// 16 KB.  16 rows of a short vector are a few KB and a few MFMAs, and a barrier, requests that no wave fills and a filter
// with its compare and branch cost more than they do.  Blocks of 64 rows instead of 16, d = 64: 4000 queries over 60 of 200
// binary16 lists of 3000 rows 880 -> 627 us, 500 over 40 of 2000 lists 426 -> 372, 500 over 40 of 1000 lists of 40 rows 113
// -> 106 (128 rows: 626, 380, 109: a list ends in the middle of a longer block); float32 (split on its way into LDS then), d = 64, the first two
// 1578 -> 1304 and 528 -> 454.  Two planes of 16 rows of d = 256 are 16 KB already: 32 rows of row tables were 10 % faster for
// 4000 queries and 2 .. 4 % slower for fewer.
__host__ __device__ constexpr int block_groups(int dtype, int d)
{
    const int most = 4, long_enough = dtype == HR_F32 || scan_split(dtype) ? 256 : 512;
    return d >= long_enough ? 1 : (long_enough / d < most ? long_enough / d : most);
}
__host__ __device__ constexpr int block_rows(int dtype, int d) { return kMfmaRows * block_groups(dtype, d); }

// Most workgroups of eight waves on a compute unit: two where a wave can do with 128 registers (binary16 rows of up to 256
// elements, of which d = 128 spills four registers, 20 bytes a lane; float32 rows of 128 with fragments fetched two steps at a
// time; the other short ones could, with blocks of 32 rows instead of 64, which cost them 3 .. 7 % where two workgroups do not
// pay).  The waves of one wait for each other at every pair of blocks; the other's fill the pipes meanwhile.  Where that pays is
// in make_plan.  The bound on registers holds for all launches of the kernel: without it binary16 searches of d = 128 that put
// one workgroup on a unit took 0.97 .. 1.03 of the time, 1.00 in the mean of 45 (1 .. 500 queries, 46 .. 526 us).
__host__ __device__ constexpr int groups_per_cu(int dtype, int d)
{
    return (dtype == HR_F16 && d <= 256) || (dtype == HR_F32 && d == 128) ? 2 : 1;
}

// k-steps (of 32 elements) whose row fragments a wave fetches from LDS together
__host__ __device__ constexpr int scan_group(int dtype, int ksteps)
{
    // (blocks of several groups of rows: 8 or 16 k-steps in all)
    if (ksteps < 16) return stored_f32(dtype) ? 2 : 4;
    // (what a long operand in two parts leaves: 253 of 256 registers at 24 k-steps, none spilled; HR_F32X2, which selects too, spills
    // three, 16 bytes a lane.  The bounded kernels keep some hundred scalar registers in vector ones, the others sixty.)
    if (operand_parts(dtype, ksteps * 32) == 2)
        return scan_split(dtype) ? (ksteps >= 24 ? 1 : 2) : (ksteps >= 24 ? 2 : 4);
    return (dtype == HR_F32 && ksteps >= 24) || (scan_split(dtype) && ksteps >= 32) ? 2 : 4;   // (256 registers per lane)
}

// selection buffer capacity per column for a given k: room for k kept entries plus a batch of
// new ones between two prunes (a prune costs about the same for any fill up to 64 entries per
// lane slot, so bigger batches make each candidate cheaper), bounded by LDS
// (high parts alone: what is within their slack of the k-th best is kept too, and half of a buffer that has just been cut, or more, is meant to be free)
constexpr int kRoomAfterCut = 4;           // free entries beyond kAppendMax that a cut has to leave
__host__ __device__ constexpr int sel_cap(int dtype, int k)
{
    int c = k <= 24 ? 64 : (k <= 64 ? 128 : 192);
    if (scan_bounded(dtype) && !scan_split(dtype)) c = k <= 12 ? 64 : (k <= 24 ? 96 : (k <= 36 ? 128 : (k <= 64 ? 192 : 256)));
    if (c < k + kAppendMax + kRoomAfterCut) c = k + kAppendMax + kRoomAfterCut;
    return c;
}

// How k_topk_rows bounds the k best of n keys from below: the want-th largest of size keys spread over the row (size 0: no
// bound, the row is collected whole).  How many sampled keys belong to the k best is close to Poisson with mean lambda =
// k size / n, so want lies 5.5 deviations above it: fewer than k keys are at or above the bound for one row in 10^5.  Nor
// may more than kTopkCollect be, so for large k want is at most midway between the two: one row in 10^5 at
// most on either side up to k 200 of 16384 keys, and then more: one in 450 too many for 128 of 32768, one in 500 too few and
// one in 60 too many for 512 of 16384 (a second pass each).
// Rows that fit the buffer are sampled only where that spares the select half of them; a bound that nearly all keys reach
// would leave out some of the best (512 of 512 keys: every second row).
constexpr int kTopkCollect = 1024;
struct TopkSample { int size, want; };
inline TopkSample topk_sample(int n, int k)
{
    const int size = n > 4 * kTopkCollect ? 1024 : (n > kTopkCollect ? 512 : 256);
    const float lambda = (float)k * (float)size / (float)n;
    int want = (int)(lambda + 5.5f * sqrtf(lambda) + 3.0f);
    if (n <= kTopkCollect) return n > 256 && want * 2 <= size ? TopkSample{size, want} : TopkSample{0, 0};
    const int most = (int)((float)size * (float)(k + kTopkCollect) * 0.5f / (float)n) + 1;
    want = want < most ? want : most;
    return TopkSample{size, want < 2 ? 2 : (want < size ? want : size)};
}

// order-preserving map float -> uint32 (larger float = larger unsigned), and back
__host__ __device__ inline uint32_t enc_key(float f)
{
    uint32_t b = __builtin_bit_cast(uint32_t, f);
    return b ^ ((b >> 31) ? 0xffffffffu : 0x80000000u);
}
__host__ __device__ inline float dec_key(uint32_t u)
{
    uint32_t b = (u >> 31) ? (u ^ 0x80000000u) : ~u;
    return __builtin_bit_cast(float, b);
}
constexpr uint32_t kKeyNegInf = 0x007fffffu;   // enc_key(-inf)

// One candidate: key (enc_key of the score, larger is better) and row number.
struct Cand { uint32_t key; uint32_t row; };

// What bounds the scores of a list's rows: the largest squared norm of its rows and the largest squared norm of what rounding a row to
// binary16 leaves over (their bits, which are in order, as squares are not negative)
struct ListBound { uint32_t norm2, left2; };
__host__ __device__ inline float bound_value(uint32_t b) { return __builtin_bit_cast(float, b); }

// Arguments of the scan kernel (both uses: centroid table with all queries as one dense
// bucket, and the inverted lists with the per-list buckets).
struct ScanArgs {
    const void* rows;           // [nrows, d] storage (HR_F16X2: the hi table)
    const void* rows_lo;        // HR_F16X2: the lo table
    const float* row_norm;      // [nrows] squared norms (used when l2 != 0)
    const int64_t* row_ids;     // [nrows] labels, or nullptr: label = row number
    const void* qop;            // query operand rows (layout depends on dtype)
    const float* queries;       // the queries as they are (dense mode: split while they are loaded, or nullptr: qop)
    uint32_t* thr;              // [nq] running per-query lower bound of the k-th key (enc_key)
    int* slot_cnt;              // [slots]: one slot per (list segment, query of the list's bucket)
    Cand* slot_ent;             // [slots * cap] the selection buffers of the items
    // bounded types (scan_slack)
    const float* qnorm;         // [nq] squared norms of the queries
    const float* qlo;           // [nq] norms of their low parts
    const ListBound* list_bound;   // [nlist]
    const float* rows_f32;      // [nrows, d] the rows as they are
    int* work_counter;          // dense mode: items popped beyond the first of every workgroup (zeroed before launch)
    // bucket mode
    const int* bucket_q;        // [pairs] query index per bucket entry
    const int* dyn;             // device scalars: [0] = items, [1] = rows per segment
    const int4* xq_rec;         // [8][xq_stride][2] the items queued per XCD, each a record of two int4:
                                // (first row, rows, first entry of the list's bucket, width of the bucket),
                                // (query tile, first result slot of the item, list, segment)
    const int* xq_count;        // [8] queue lengths
    int* xq_head;               // [8] items popped beyond those that the workgroups start with (zeroed before launch)
    int xq_stride;
    // dense mode (HR_F16X2, and then key_out is not null): one list = all rows, bucket = all queries
    int dense_items, dense_nqt, dense_seg_rows, dense_nrows;
    int dense_groups;           // groups that the tiles are taken in, so that the items of a segment meet in one XCD (0: plain order)
    int dense_cols;             // queries per wave (d < 512: as many as it has columns for)
    int nq, k, cap, l2;
    int tile;                   // lists: queries of a work item
    int nbuf;                   // staging buffers in LDS
    float* key_out;             // dense mode: [nq, dense_nrows] every key is written here and nothing is selected
    int* hist;                  // [nq][kHistBins] keys found so far per query, by key range (or nullptr)
    const float* hpar;          // [nq][2] lower edge of bin 0 and bin width (width 0: query has no histogram)
};

struct SeedArgs {
    const void* rows;           // [nrows, d] storage
    const float* row_norm;      // [nrows]
    const void* qop;            // query operand rows
    const int* probe;           // [nq, nprobe]; the first resident list among the first 64 places is the one used
    const int* list_off;        // [nlist+1]
    const int* resident;        // [nlist] 1 = the list's vectors are in place
    uint32_t* thr;              // [nq]
    float* hpar;                // [nq][2] histogram parameters of the scan (see ScanArgs)
    const int64_t* state_ids;   // [nq, k] labels and scores of a carried result, or nullptr
    const float* state_scores;
    const float* qnorm;         // [nq] squared norms of the query operands
    const ListBound* list_bound;   // [nlist] float32 rows: see scan_slack
    int nq, nprobe, nlist, k, seed_rows, l2;
};

// Device scalars written by the bucketing kernels (ints in workspace)
enum { DYN_ITEMS = 0, DYN_SEG_ROWS = 1, DYN_ROWS_LO = 2, DYN_ROWS_HI = 3, DYN_PAIRS = 4, DYN_SLOTS = 5, DYN_ROUNDS = 6, DYN_COUNT = 8 };
constexpr int kRounds = 64;                // most rounds of a work queue (see the bucketing kernels)

struct MergeArgs {
    const uint32_t* thr;        // [nq] lower bounds of the k-th keys, as the scan left them
    const int* slot_cnt;
    const Cand* slot_ent;
    int slot_stride;
    const int64_t* row_ids;     // nullptr: label = row number
    const float* qnorm;         // [nq] squared norm of the query operand (L2 only)
    const int* probe;           // [nq, nprobe]
    const int* pair_entry;      // [nq, nprobe] position of the pair inside its list's bucket
    const int* list_off;        // [nlist+1]
    const int* bucket_off;      // [nlist+1]
    const int* slot_base;       // [nlist+1] first result slot of every list
    const int* dyn;
    int nq, nprobe, nlist, k, l2;
    int carried;                // out_ids / out_scores hold a previous result on entry: merged in (ids < 0: empty places)
    int64_t* out_ids;           // [nq, k] or nullptr
    float* out_scores;          // [nq, k] or nullptr
    // bounded types: slots hold upper bounds (scan_slack); the exact keys of those that may count are computed here
    const float* queries;       // [nq, d] the queries as they are
    const float* rows_f32;      // [nrows, d] the rows, or nullptr: the slots hold exact keys
    const float* row_norm;      // [nrows]
    const float* qlo;           // [nq]
    const ListBound* list_bound;   // [nlist]
    int d, split;               // split: the scan multiplied both parts (HR_F32X2)
    int32_t* io_rows;           // [nq, k] or nullptr: row numbers of the entries, carried along with them (-1: empty place)
};

// launchers implemented in the .hip files
hipError_t launch_scan(int dtype, int d, const ScanArgs& a, int grid, size_t lds_bytes, hipStream_t s);
size_t scan_lds_bytes(int dtype, int d, int nbuf);
hipError_t launch_merge(const MergeArgs& a, hipStream_t s);
struct PrepArgs {
    const float* q;             // [nq, d]
    _Float16* qop_coarse;       // hi and scaled lo rows, or nullptr
    float* qnorm_coarse;        // or nullptr
    void* qop_scan;             // operand of the list scan, where that is not the coarse step's, or nullptr
    float* qnorm_scan;          // or nullptr
    float* qlo;                 // [nq] norms of the low parts (see scan_slack), or nullptr
    int* zero;                  // [n_zero] set to 0
    int* neg;                   // [n_neg] set to neg_value
    int64_t nq, n_zero, n_neg;
    int d, dtype, neg_value;    // dtype: form of the list scan's operand
};
hipError_t launch_topk_rows(const float* keys, const float* qnorm, int32_t* out_ids, float* out_scores,
                            int64_t nq, int n, int k, int l2, const PrepArgs* prep, hipStream_t s);
hipError_t launch_row_norms(const void* rows, int dtype, int64_t nrows, int d, float* out, hipStream_t s);
hipError_t launch_prep_queries(const PrepArgs& a, hipStream_t s);
hipError_t launch_fill_i32(int* p, int64_t n, int v, hipStream_t s);
hipError_t launch_hot_lists(const unsigned long long* hits, int nlist, int gc, int32_t* out, hipStream_t s);
struct ListArgs {
    const float* rows;          // float32 rows of the index
    int64_t row0, nrows;        // those that are new
    const int* list_off;        // [nlist+1]
    int nlist, d;
    int l0, lists;              // the lists that have some of them
    float* row_norm;            // [N]
    ListBound* bound;           // [nlist]
    void* hi;                   // [N, d] rows rounded to binary16, or nullptr
    float2* spread;             // [nlist] deviations of the scores of a list's rows, by metric (list_spread)
    int* tight;                 // host memory, by metric: set where lists' windows are too wide (see score_window)
    int* told;                  // by metric: that has been done
    int whole0, whole1;         // the lists of which all rows are new
};
hipError_t launch_list_bounds(const ListArgs& a, hipStream_t s);
constexpr int kWindowShare = 64;           // one row in so many in lists with wide windows: see score_window
hipError_t launch_wide_windows(const ListArgs& a, hipStream_t s);
hipError_t launch_read_hits(unsigned long long* hits, int64_t n, int64_t* out, int reset, hipStream_t s);
hipError_t launch_lists_of_rows(const int32_t* rows, int64_t n, const int* list_off, int nlist, int32_t* out, hipStream_t s);
hipError_t launch_reorder_probes(const int32_t* probe, int np, const int32_t* prev, int pp, const int32_t* hot, int nh,
                                 int64_t nq, int32_t* out, hipStream_t s);
hipError_t launch_rescore(const float* q, int64_t nq, int d, int dtype, const void* rows, const float* row_norm,
                          const int64_t* row_ids, int64_t nrows, const int32_t* cand, int m, int k, int l2,
                          int64_t* out_ids, float* out_scores, int32_t* out_rows, hipStream_t s);
hipError_t launch_bf16_to_f16(const void* x, int64_t n, void* out, int* overflow, hipStream_t s);
hipError_t launch_refresh_bf16(const void* rows, int64_t nrows, int d, float* norm, void* table, int* overflow, hipStream_t s);
hipError_t launch_split_f32(const float* x, int64_t n, void* hi, void* lo, hipStream_t s);
hipError_t launch_set_resident(int* resident, int nlist, const int32_t* lists, int64_t n, int value, hipStream_t s);
hipError_t launch_split_probes(const int32_t* probe, int64_t nq, int np, const int* resident, int nlist, unsigned long long* hits,
                               int32_t* out_resident, int32_t* out_missing, hipStream_t s);
hipError_t launch_check_labels(const int64_t* ids, int64_t n, int* negative, hipStream_t s);

struct BucketArgs {
    const int* probe;           // [nq*nprobe]
    int nq, nprobe, nlist, cw;
    int cw_log2;                // (the queries of a tile are a power of two)
    int half_tiles;             // the shortest segments are counted in tiles of cw / 2 queries (see k_bucket_scan)
    const int* list_off;        // [nlist+1]
    int* list_w;                // [nlist]   (zeroed by the first kernel's launch sequence; a batch grouped in one launch has no use for it)
    int* pair_entry;            // [nq*nprobe]
    int* bucket_off;            // [nlist+1]
    int* bucket_q;              // [nq*nprobe]
    int* slot_base;             // [nlist+1] first result slot of every list
    int* dyn;                   // device scalars
    int4* xq_rec;               // [8][item_cap][2] per-XCD queues of item records (see ScanArgs)
    int* xq_count;              // [8] queue lengths
    int* round_cnt;             // [8][64] items per queue and round, then where each round starts (zeroed before launch)
    int* round_cur;             // [8][64] items placed so far per queue and round (zeroed before launch)
    int item_cap;
    int slot_cap;               // result slots the workspace holds
    int item_target;            // aimed number of work items (rows per segment follow from it)
    int base_rows;              // shortest segments
    int few_items;              // work items below which segments become shorter than that
    int min_rows;               // but not shorter than this
    unsigned long long* hits;   // [nlist] probes per list since load or the last reset (index-owned), or nullptr
    const int* resident;        // [nlist] 1 = the list's vectors are in place; probes of the other lists are dropped
};
// grouping of a batch, all of it, or what comes before and behind k_bucket_scan
hipError_t launch_bucketing(const BucketArgs& a, hipStream_t s);
hipError_t launch_bucketing_before(const BucketArgs& a, hipStream_t s);
hipError_t launch_bucketing_behind(const BucketArgs& a, hipStream_t s);
hipError_t launch_seed(int dtype, int d, const SeedArgs& a, const BucketArgs* group, hipStream_t s);

// Largest batch that one workgroup groups by itself: four pairs and four lists per thread stay in its registers and the
// tables of the lists (64 KB) in LDS, which is where the line lies: up to it the one launch is never slower.  Searches of
// given lists, five launches against one: 64 pairs of 64 lists 77.7 and 70.0 us, 1024 of 1024 120.4 and 114.1, 4096 of 64
// 98.3 and 85.3, 4096 of 4096 235.9 and 226.2; with 4.2 M rows in the lists, 4096 of 4096, 506.7 and 506.0.
constexpr int kWholePairs = 4096, kWholeLists = 4096;
inline bool grouped_whole(const BucketArgs& a) { return (int64_t)a.nq * a.nprobe <= kWholePairs && a.nlist <= kWholeLists; }
// Most queries whose seeding the grouping rides on (see k_group_seed): beyond that the workgroups of the seeding, twice as wide and
// with the tables of the grouping in LDS, two on a compute unit, make more rounds than the launch takes.  Two launches and one: 300
// queries over 12 of 512 lists 165 and 154 us (float32, d = 768), 1000 over 4 208 and 198, 2000 over 2 242 and 234; binary16,
// d = 128, 1000 over 4 187 and 182, 2000 over 2 228 and 231, 4096 over 1 274 and 294.
constexpr int kSeedBeside = 1024;

}  // namespace hr
