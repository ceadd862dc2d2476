// Host side of the C ABI declared in hr_ivf.h: argument checks, workspace layout, launch
// sequence.  Nothing here synchronises the caller's stream except hr_ivf_load, hr_ivf_stats, hr_ivf_profile_end and, with a
// binary16 table of bfloat16 rows, hr_ivf_refresh_rows.
#include <algorithm>
#include <atomic>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <thread>

#include "common.h"

// Scratch memory of hr_ivf_search_static, the entry point for callers that cannot allocate: a
// fixed array in the library's device image, one copy per GPU, held until the process ends.  In
// host code the array's name only stands for the symbol; its address on a device is asked for
// once per device (with that device current) and kept, and that pointer is what the kernels get.
static __device__ __align__(256) unsigned char scratch[HR_STATIC_SCRATCH_BYTES];
static constexpr int kMaxDevices = 64;
static void* g_scratch[kMaxDevices];           // device address of `scratch` per device, null until asked for
static std::mutex g_scratch_mu;

// address of the scratch array on device `dev`, which must be the current device.  (Not a static function: the
// compiler gives a file-scope static device variable a symbol that the runtime can look up only when a host
// function with external linkage names it.)
namespace hr {
hipError_t static_scratch_address(int dev, void** out);
}
hipError_t hr::static_scratch_address(int dev, void** out)
{
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch[dev] == nullptr) {
        void* p = nullptr;
        hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (p == nullptr) return hipErrorInvalidSymbol;
        g_scratch[dev] = p;
    }
    *out = g_scratch[dev];
    return hipSuccess;
}

namespace hr {
hipError_t launch_scan_f32(int d, const ScanArgs& a, int grid, size_t lds, hipStream_t s);
hipError_t launch_scan_f16(int d, const ScanArgs& a, int grid, size_t lds, hipStream_t s);
hipError_t launch_scan_bf16(int d, const ScanArgs& a, int grid, size_t lds, hipStream_t s);
hipError_t launch_scan_f16x2(int d, const ScanArgs& a, int grid, size_t lds, hipStream_t s);
hipError_t launch_scan_f16hi(int d, const ScanArgs& a, int grid, size_t lds, hipStream_t s);
hipError_t launch_scan_f32x2(int d, const ScanArgs& a, int grid, size_t lds, hipStream_t s);

hipError_t launch_seed_f32(int d, const SeedArgs& a, const BucketArgs* group, hipStream_t s);
hipError_t launch_seed_f16(int d, const SeedArgs& a, const BucketArgs* group, hipStream_t s);
hipError_t launch_seed_bf16(int d, const SeedArgs& a, const BucketArgs* group, hipStream_t s);

hipError_t launch_seed(int dtype, int d, const SeedArgs& a, const BucketArgs* group, hipStream_t s)
{
    switch (dtype) {
    case HR_F32: return launch_seed_f32(d, a, group, s);
    case HR_F16: return launch_seed_f16(d, a, group, s);
    case HR_BF16: return launch_seed_bf16(d, a, group, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_scan(int dtype, int d, const ScanArgs& a, int grid, size_t lds, hipStream_t s)
{
    switch (dtype) {
    case HR_F32: return launch_scan_f32(d, a, grid, lds, s);
    case HR_F16: return launch_scan_f16(d, a, grid, lds, s);
    case HR_BF16: return launch_scan_bf16(d, a, grid, lds, s);
    case HR_F16X2: return launch_scan_f16x2(d, a, grid, lds, s);
    case HR_F16HI: return launch_scan_f16hi(d, a, grid, lds, s);
    case HR_F32X2: return launch_scan_f32x2(d, a, grid, lds, s);
    default: return hipErrorInvalidValue;
    }
}

// LDS bytes of one workgroup with nbuf staging buffers (must match the carve-up at the top of k_scan and
// ScanShape::buf_bytes)
size_t scan_lds_bytes(int dtype, int d, int nbuf)
{
    const size_t rows = block_rows(dtype, d), threads = kScanWaves * 64;
    const size_t chunks = rows * d * (stored_f32(dtype) ? 4 : 2) / 16;
    const size_t buf = (chunks + threads - 1) / threads * threads * 16 * (dtype == HR_F16X2 ? 2 : 1);
    return nbuf * (buf + rows * sizeof(float)) + 32;
}
}  // namespace hr

static constexpr int kLdsLimit = 160 * 1024;      // LDS per workgroup on gfx950

// Staging buffers of a list scan: as many as fit in LDS, or in half of it where two workgroups share a unit: 6 or 4 (blocks in
// pairs, one barrier per pair), else 3 or 2 (those of 16 float32 rows of d = 1024 are 64 KB).  More rows on their way is what
// counts when few queries share a list and the scan is bound by HBM (measured with the selection buffers in LDS and 4 row
// buffers instead of 6: C4 +2 %, the 38 M x 1024 index +2.5 %, C3 +1 %).
static int pick_buffers(int dtype, int d, int groups)
{
    for (int nbuf : {6, 4, 3})
        if (hr::scan_lds_bytes(dtype, d, nbuf) <= (size_t)kLdsLimit / groups) return nbuf;
    return 2;
}

using namespace hr;

static thread_local char g_err[512] = "";

static int fail(int code, const char* fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return code;
}

#define HR_HIP(call)                                                                      \
    do {                                                                                  \
        hipError_t e_ = (call);                                                           \
        if (e_ != hipSuccess) return fail(HR_ERR_HIP, "%s: %s", #call, hipGetErrorString(e_)); \
    } while (0)

static constexpr uint64_t kMagic = 0x4852495646313031ULL;   // "HRIVF101"

struct hr_ivf_index {
    uint64_t magic;
    const float* centroids;
    const void* vectors;
    const int64_t* ids;
    int64_t nlist, N;
    int64_t longest;       // rows of the longest list
    int d, dtype;
    int* h_list_off;       // [nlist+1] int32, on the host
    int* d_list_off;       // [nlist+1] int32
    float* d_row_norm;     // [N]
    float* d_cent_norm;    // [nlist]
    void* d_cent_hi;       // [nlist, d] binary16: centroids rounded
    void* d_cent_lo;       // [nlist, d] binary16: (centroid - hi) * 2^11
    void* d_vec_hi;        // float32 lists only, when asked for and memory allows: [N, d] the rows rounded to binary16; else null
    void* d_vec16;         // bfloat16 lists only, when memory and the value range allow: [N, d] the rows as binary16
    int* d_flag;           // device ints: [0] a bfloat16 value did not fit binary16, [1] a negative label, [2] [3] h_tight has been set, by metric
    // with d_vec16: report words of hr_ivf_refresh_rows, one for each call under way (host memory that kernels write; bit i of
    // over_used: word i belongs to a call), else null
    int *h_over, *d_over;  // their address on the host and on the device
    std::atomic<uint64_t> over_used;
    ListBound* d_list_bound;      // float32 lists: [nlist] what scan_slack needs to know of the list's rows, else null
    float2* d_spread;      // float32 lists: [nlist] how far the scores of their rows are apart (list_spread), else null
    // float32 lists: host memory that kernels write, its address there and on the device: [metric] lists' bounds tell little
    int *h_tight, *d_tight;
    std::atomic<int64_t> replaced;     // rows of wholly replaced lists since these were last looked over, while they tell little
    unsigned long long* d_hits;   // [nlist] probes per list since load / last reset
    int* d_resident;       // [nlist] 1 = the list's vectors are in place (all lists, until the caller says otherwise)
    int num_cus;
    int lds_limit;
    int device;            // the device the index lives on
    void* scratch;         // address of the library's static scratch array on that device
    // optional kernel timing (hr_ivf_profile_begin/end)
    hipEvent_t* prof_ev;   // 2 * prof_cap events
    int prof_cap, prof_n;
};

// Float32 lists: are both parts of the rows multiplied?  Scores and their order are the same either way, so what a refresh has written
// here or not yet decides nothing but the time.
static bool both_parts(const hr_ivf_index* ix, int metric) { return ix->h_tight && ((volatile const int*)ix->h_tight)[metric == HR_METRIC_L2] != 0; }
// storage type the list scan runs on
static int scan_dtype(const hr_ivf_index* ix, bool both)
{
    if (ix->dtype == HR_F32) return both ? (int)HR_F32X2 : (ix->d_vec_hi ? (int)HR_F16HI : (int)HR_F32);
    return ix->d_vec16 ? (int)HR_F16 : ix->dtype;
}
// form of the query operand the list scan multiplies (what k_prep_queries is asked for)
static int operand_dtype(const hr_ivf_index* ix) { return ix->d_vec16 ? (int)HR_F16 : ix->dtype; }
// rows and their type for the kernels that read single rows (threshold seeding, rescoring)
static int row_dtype(const hr_ivf_index* ix) { return ix->d_vec16 ? (int)HR_F16 : ix->dtype; }
static const void* row_table(const hr_ivf_index* ix) { return ix->d_vec16 ? ix->d_vec16 : ix->vectors; }

static bool dim_supported(int d)
{
    return d == 64 || d == 128 || d == 256 || d == 512 || d == 768 || d == 1024;
}

static size_t align_up(size_t v) { return (v + HR_WORKSPACE_ALIGN - 1) & ~(size_t)(HR_WORKSPACE_ALIGN - 1); }

// Layout of the caller's workspace for one batch shape.  Offsets in bytes.
struct Plan {
    // coarse step: centroid table scanned with all queries as one dense bucket
    int nbuf_c, cw_c, cols_c, nqt_c, seg_c, nseg_c;
    // list scan
    int dtype_s, groups_s, nbuf_s, cap_s, cw_s, item_cap, item_target, few_items, min_rows, base_rows;
    int slot_cap;                   // result slots: one per (list segment, query of the list's bucket)
    size_t o_zero, n_zero;          // ints cleared per call: list_w[nlist], dyn[DYN_COUNT], counters[8], ..., then
    size_t zoff_round, zoff_hist, zoff_hpar;   // (in ints from o_zero) round counters of the queues, per-query key histograms and their parameters
    size_t o_thr;                   // nq floats (qlo), then nq ints set to "-inf"
    size_t o_qop_c, o_qnorm_c, o_qop_s, o_qnorm_s;
    size_t o_probe;
    size_t o_pair_entry, o_bucket_off, o_bucket_q, o_slot_base, o_xq;
    size_t o_ckeys;                 // coarse step: [cchunk, nlist] keys of one chunk of queries
    int64_t cchunk;                 // queries per coarse chunk
    size_t o_slot_cnt, o_slot_ent;
    size_t total;
    // the regions above in order of their offsets (for hr_ivf_workspace_layout); a guard gap of
    // HR_WORKSPACE_ALIGN bytes that nothing writes lies behind every one
    int nreg;
    size_t reg_off[24], reg_len[24];
};

// What bounds the size of a plan: the aimed number of work items of the list scan (segments are sized so that
// about that many items result: fewer, larger items need fewer result slots) and the bytes of the coarse key table
// (queries are scored in chunks that fit it).
// cap: entries of a selection buffer where those lie in the result slots (0: as many as k asks for).  by_length: bound the
// slots by the longest list too.
struct PlanLimits { int item_target; size_t ckeys_bytes; bool by_length; int cap; };
static constexpr PlanLimits kDefaultLimits = {kItemTarget, (size_t)512 << 20, true, 0};

static constexpr int kShortSegK = 24;          // most neighbours of a search that may go in segments shorter than kMinSegRows
static constexpr int kFullTileK = 12;          // most neighbours of float32 rows that always go in full tiles of queries

// both: float32 lists, multiply both parts (see both_parts); the layout of a workspace is the same either way.
static Plan make_plan(const hr_ivf_index* ix, int64_t nq, int nprobe, int k, bool both, const PlanLimits& lim = kDefaultLimits)
{
    Plan p{};
    const int64_t nlist = ix->nlist;
    // Two workgroups per compute unit where the batch is bound by multiplying and filtering: full tiles (a list is probed by 128
    // queries in the mean) and about 1024 work items of 256 rows or a list each.  4000 queries over 60 of 200 lists of 3000 rows, k
    // 24: d = 64 686 -> 466 us, 128 733 -> 502, 256 938 -> 649, float32 of d = 128 1688 -> 1198; 1000 over 30, k 1, 188 -> 161,
    // 205 -> 174, 238 -> 201.  With fewer items, or many neighbours, more of them start from the seeds alone: 500 over 30 of 64
    // lists, 100000 rows, k 10, 131 -> 139; 500 over 40 of 200 lists, k 100, 343 -> 399; and 30 queries over 20 of 200 lists
    // 112 -> 121.  The rule takes lists and probes to be alike, and is off by up to a fifth where they are far from it.  Probes
    // that are empty, half of them: 4000 over 60 of 200 lists of 3000 rows, d = 128, 490 -> 343, nine in ten: 500 over 60, 147 ->
    // 147, 97 in 100: 8000 over 32 of 64 lists, 146 -> 161.  Nine lists in ten out of place: 500 over 60 of 200, float32, 141 ->
    // 151.  Short lists, d = 128, one and two: 4000 over 100 of 200 lists of 50 rows, sizes as 1 / rank^0.8, 280 and 252, 1000 over
    // 100 of 500 of 80 rows 176 and 203, 4000 over 100 of 2000 of 4 float32 rows 482 and 597.
    const int64_t pairs = nq * nprobe;
    const bool full_tiles = k <= 24 && pairs >= 128 * nlist &&
                            (double)(ix->N / kMinSegRows + nlist) * (double)pairs >= 1024.0 * 128.0 * (double)nlist;
    p.dtype_s = scan_dtype(ix, both);
    p.groups_s = full_tiles ? groups_per_cu(p.dtype_s, ix->d) : 1;
    p.nbuf_s = pick_buffers(p.dtype_s, ix->d, p.groups_s);
    p.nbuf_c = scan_lds_bytes(HR_F16X2, ix->d, 3) <= (size_t)kLdsLimit ? 3 : 2;
    // queries per coarse chunk: the [chunk, nlist] key table stays within its limit, 512 MiB by default (the more
    // queries per launch the better both kernels fill the device: 16384 lists, four chunks of 2048 queries 1.88 ms,
    // one of 8192 1.45 ms)
    p.cchunk = (int64_t)lim.ckeys_bytes / (nlist * 4) / 64 * 64;
    if (p.cchunk < 64) p.cchunk = 64;
    if (p.cchunk > nq) p.cchunk = nq > 0 ? nq : 1;
    // Work items of the coarse step: tiles of queries x rows of the centroid table.  The items are alike, so what counts is
    // how many whole rounds over the compute units they make and how long an item is: its blocks, about four more that loading
    // a tile of 128 queries costs (two for 64, with half the columns of every wave empty: a block takes as long), and, for
    // long items, a few percent by which the last ones end apart.  Mostly that is one round (8192 queries, d = 1024, two
    // rounds with at least 32 rows per item or eight beyond 64 tiles: 512 centroids 144 us, one round 82; 4096 381 and 320;
    // 3001 queries, d = 768, 4096 centroids 121 and 108), and tiles of 64 where those fit it as well, if the vectors are long
    // enough for the loading to count and the table so short that reading it twice as often does not (d = 768, 64 centroids:
    // 100 queries 26.3 -> 24.3 us, 300 28.6 -> 24.5, 3001 40.7 -> 37.3; 2048 centroids, 200 queries 36.1 -> 34.3, but 4096,
    // 100 queries 36.1 -> 37.3; then still with a launch of the preparation).  Rows count in sixteens for short vectors too, whose
    // blocks are of 64 (d = 64) or 32 (d = 128): an item of 16 or 48 rows multiplies copies of its last one, but rounding items
    // up to whole blocks takes as many from the device (1 .. 8192 queries, 64 .. 65536 centroids, 172 cases: as fast in the
    // mean, 0.94 .. 1.04; 777 centroids, d = 64, 300 queries 15.3 -> 16.3, 16384, 3001 122.1 -> 117.0).
    const int64_t nblk = (nlist + kMfmaRows - 1) / kMfmaRows, cus = ix->num_cus;
    const int full = tile_cols(HR_F16X2, ix->d);
    int64_t per_item = nblk;                        // blocks
    double least = 0.0;
    p.cw_c = full;
    for (int cw = full; cw >= full / operand_parts(HR_F16X2, ix->d); cw /= 2) {
        const int64_t nqt = (p.cchunk + cw - 1) / cw;
        // (a single half tile would only have twice the waves multiply: 64 queries, 64 centroids 22.0 -> 23.5)
        if (cw < full && (nqt == 1 || ix->d < 512 || nblk > 128)) break;
        for (int r = 1; r <= 8; r++) {
            const int64_t nseg = r * cus / nqt;
            if (nseg < 1) continue;
            const int64_t blocks = (nblk + nseg - 1) / nseg, items = (nblk + blocks - 1) / blocks * nqt;
            const double cost = (double)((items + cus - 1) / cus) * (4.0 * cw / full + (double)blocks) + (double)blocks / 16.0;
            if (least == 0.0 || cost < least) { least = cost; per_item = blocks; p.cw_c = cw; }
        }
    }
    p.cols_c = p.cw_c / kScanWaves;
    p.nqt_c = (int)((p.cchunk + p.cw_c - 1) / p.cw_c);
    const int64_t seg = per_item * kMfmaRows;
    p.seg_c = (int)seg;
    p.nseg_c = (int)((nlist + seg - 1) / seg);
    auto sizes = [&](int dtype) {
        p.cap_s = lim.cap > 0 ? lim.cap : sel_cap(dtype, k);
        p.cw_s = tile_cols(dtype, ix->d);
        // Many neighbours and few queries per list, float32 rows: tiles of half the queries, half the slots.  Up to 32 queries per list
        // they take as long (a tile that is at most half full goes on all waves either way); at 48 tiles of 128 and 64, k 20, 512 lists: d
        // = 64 170 and 149 us, 128 180 and 165, 256 212 and 201, 768 373 and 391, 1024 270 and 264, 4096 lists, d = 64, 638 and 649; at
        // 64 175 and 175, 195 and 196, 223 and 231, 424 and 479, 302 and 306, 747 and 843; at 96 183 and 213, d = 256 242 and 295, 768 495
        // and 620, 1024 366 and 408; k 100 alike.
        const int narrow = stored_f32(dtype) && cols_per_set(dtype, ix->d) == 16 ? p.cw_s / 2 : p.cw_s;
        if (k > kFullTileK && pairs <= 48 * nlist) p.cw_s = narrow;
        // Work items: sum over probed lists of segments x query tiles.  Segments have at least C / item_target rows, C =
        // sum of rows x tiles, so there are at most item_target items plus one per (list, tile) for the ragged ends.
        // Result slots: sum of segments x bucket width <= cw x item_target, plus one per pair for the ragged ends.  (In a
        // workspace items are bounded for the narrower tiles whatever the batch and k: the plan of a larger batch is never the smaller, and
        // what lies before the slots lies at the same place for every k.)
        p.item_target = lim.item_target;
        p.item_cap = (int)(lim.item_target + pairs / (lim.by_length ? narrow : p.cw_s) + (pairs < nlist ? pairs : nlist) + 8);
        int64_t slots_most = (int64_t)p.cw_s * lim.item_target + pairs;
        // Nor has a pair more slots than the longest list has segments, whatever the batch (one query over 16 of 256 lists of
        // 65536 rows in all, k 10: 268 MB of slots without this bound, 1.3 with it).  Segments shorter than kMinSegRows are of
        // min_rows rows at least, and there are at most few_items of those, and one per pair for the ragged ends.
        // Shorter ones pay where an item takes longer to read than to start and to merge: blocks of 128 KB, vectors of 512 and more,
        // few candidates per segment.  One request, nprobe 16, k 10: 256 lists of 256 float32 rows of d = 768 92 -> 74 us, bfloat16 of
        // d = 1024 63 -> 55, over 2000 lists of 300 rows 67 -> 59; but 256 binary16 rows of d = 256, four requests, 54 -> 61, and k 100,
        // 50 lists, d = 1024, 112 -> 132; and with a second round of items (segments of rows x tiles / 256 without regard to the
        // ragged ends) 16 requests over 16 of 256 lists, d = 64, 68 -> 97.
        p.few_items = std::min(ix->num_cus, lim.item_target);
        // Float32 rows of d = 1024 as they are (blocks of 64 KB, two in LDS, so an item moves 30 GB/s at most): half as long.  700
        // queries over 32 of 512 lists, 48828 rows, 232 -> 204 us, 250 over 16 168 -> 152, 8 over 32 104 -> 96, 700 over 32 of 1024, 97656
        // rows, 246 -> 238, 700 over 16 of 512, k 50, 280 -> 247; shorter rows lose by it (d = 768, 64 over 16 of 512 141 -> 161, bfloat16 of d = 1024 116 -> 127).
        p.base_rows = stored_f32(dtype) && ix->d >= 1024 ? kMinSegRows / 2 : kMinSegRows;
        p.min_rows = k <= kShortSegK && ix->d >= 512 ? ((128 << 10) / (ix->d * (ix->dtype == HR_F32 ? 4 : 2)) + 15) & ~15 : kMinSegRows;
        p.min_rows = std::min(p.min_rows, p.base_rows);          // (what is meant to shorten segments never makes them longer)
        if (p.min_rows < 64) p.min_rows = 64;
        const int64_t in_short = std::min((int64_t)p.cw_s * p.few_items + pairs, pairs * ((ix->longest + p.min_rows - 1) / p.min_rows));
        const int64_t by_length = std::max(pairs * ((ix->longest + p.base_rows - 1) / p.base_rows), in_short);
        if (lim.by_length && by_length < slots_most) slots_most = by_length;
        p.slot_cap = (int)slots_most;
    };
    size_t most_items = 0, most_slots = 0, most_entries = 0;
    auto room = [&](int dtype) {
        sizes(dtype);
        most_items = std::max(most_items, (size_t)p.item_cap);
        most_slots = std::max(most_slots, (size_t)p.slot_cap);
        most_entries = std::max(most_entries, (size_t)p.slot_cap * p.cap_s);
    };
    if (ix->dtype == HR_F32 && lim.by_length) room(scan_dtype(ix, !both));
    room(p.dtype_s);

    size_t o = 0;
    auto take = [&](size_t bytes) {
        size_t at = o;
        p.reg_off[p.nreg] = at; p.reg_len[p.nreg] = bytes; p.nreg++;
        o = align_up(o + bytes) + HR_WORKSPACE_ALIGN;
        return at;
    };
    p.zoff_round = (size_t)nlist + DYN_COUNT + 24;  // + 8 counters, 8 queue lengths, 8 queue heads
    p.zoff_hist = p.zoff_round + 2 * 8 * 64;
    p.zoff_hpar = p.zoff_hist + (size_t)nq * kHistBins;
    p.n_zero = p.zoff_hpar + (size_t)nq * 2;
    p.o_zero = take(p.n_zero * 4);
    p.o_thr = take((size_t)nq * 2 * 4);
    p.o_qop_c = take((size_t)nq * 2 * ix->d * 2);
    p.o_qnorm_c = take((size_t)nq * 4);
    p.o_qop_s = operand_dtype(ix) == HR_F32 ? p.o_qop_c
                                            : take((size_t)nq * (operand_dtype(ix) == HR_BF16 ? 2 : 1) * ix->d * 2);
    p.o_qnorm_s = take((size_t)nq * 4);
    p.o_probe = take((size_t)pairs * 4);
    p.o_pair_entry = take((size_t)pairs * 4);
    p.o_bucket_off = take((size_t)(nlist + 1) * 4);
    p.o_bucket_q = take((size_t)pairs * 4);
    p.o_slot_base = take((size_t)(nlist + 1) * 4);
    p.o_xq = take(most_items * 8 * 2 * sizeof(int4));
    p.o_ckeys = take((size_t)p.cchunk * nlist * 4);
    p.o_slot_cnt = take(most_slots * 4);
    p.o_slot_ent = take(most_entries * sizeof(Cand));
    p.total = o;
    return p;
}

static int check_index(const hr_ivf_index* ix)
{
    if (!ix || ix->magic != kMagic) return fail(HR_ERR_HANDLE, "index handle is null, freed or corrupt");
    return HR_OK;
}

static int check_batch(const hr_ivf_index* ix, int64_t nq, int nprobe, int k, int metric, bool need_k)
{
    if (nq < 0 || nq > (1 << 24)) return fail(HR_ERR_ARG, "nq=%lld out of range", (long long)nq);
    if (nprobe < 1 || nprobe > ix->nlist || nprobe > HR_NPROBE_MAX)
        return fail(HR_ERR_ARG, "nprobe=%d must be in 1..min(nlist=%lld, %d)", nprobe, (long long)ix->nlist, HR_NPROBE_MAX);
    if (need_k && (k < 1 || k > HR_K_MAX)) return fail(HR_ERR_ARG, "k=%d must be in 1..%d", k, HR_K_MAX);
    if (metric != HR_METRIC_IP && metric != HR_METRIC_L2) return fail(HR_ERR_ARG, "unknown metric %d", metric);
    if (nq * (int64_t)nprobe >= (1LL << 30)) return fail(HR_ERR_UNSUPPORTED, "nq*nprobe too large");
    return HR_OK;
}

static int check_ws(const Plan& p, const void* ws, size_t bytes)
{
    if (!ws) return fail(HR_ERR_WORKSPACE, "workspace is null");
    if (((uintptr_t)ws) % HR_WORKSPACE_ALIGN) return fail(HR_ERR_WORKSPACE, "workspace not %d-byte aligned", HR_WORKSPACE_ALIGN);
    if (bytes < p.total) return fail(HR_ERR_WORKSPACE, "workspace has %zu bytes, need %zu", bytes, p.total);
    return HR_OK;
}

extern "C" {

const char* hr_last_error(void) { return g_err; }
const char* hr_version(void) { return "hr_ivf 0.1 gfx950"; }

int hr_ivf_load(const float* centroids, const int64_t* list_offsets, const void* list_vectors,
                const int64_t* list_ids, int64_t nlist, int64_t N, int32_t d, int32_t dtype,
                void* stream, hr_ivf_index** out)
{
    if (!out) return fail(HR_ERR_ARG, "out is null");
    *out = nullptr;
    if (!centroids || !list_offsets) return fail(HR_ERR_ARG, "centroids / list_offsets is null");
    if (nlist < 1 || nlist >= (1LL << 24)) return fail(HR_ERR_ARG, "nlist=%lld out of range", (long long)nlist);
    if (N < 0 || N >= (1LL << 31)) return fail(HR_ERR_ARG, "N=%lld out of range (< 2^31)", (long long)N);
    if (N > 0 && (!list_vectors || !list_ids)) return fail(HR_ERR_ARG, "list_vectors / list_ids is null");
    const bool row_tables = (dtype & HR_LOAD_ROW_TABLES) != 0;
    dtype &= ~HR_LOAD_ROW_TABLES;
    if (dtype != HR_F32 && dtype != HR_F16 && dtype != HR_BF16) return fail(HR_ERR_ARG, "unknown dtype %d", dtype);
    if (d < 1) return fail(HR_ERR_ARG, "d=%d", d);
    if (!dim_supported(d)) return fail(HR_ERR_UNSUPPORTED, "d=%d not one of 64,128,256,512,768,1024", d);
    if (list_offsets[0] != 0 || list_offsets[nlist] != N) return fail(HR_ERR_ARG, "list_offsets must start at 0 and end at N");
    for (int64_t l = 0; l < nlist; l++)
        if (list_offsets[l + 1] < list_offsets[l]) return fail(HR_ERR_ARG, "list_offsets decreases at list %lld", (long long)l);

    hipStream_t s = (hipStream_t)stream;
    int dev = 0;
    HR_HIP(hipGetDevice(&dev));
    hr_ivf_index* ix = new (std::nothrow) hr_ivf_index();
    if (!ix) return fail(HR_ERR_HIP, "out of host memory");
    ix->centroids = centroids; ix->vectors = list_vectors; ix->ids = list_ids;
    ix->nlist = nlist; ix->N = N; ix->d = d; ix->dtype = dtype;
    int* const h_off = ix->h_list_off = new (std::nothrow) int[nlist + 1];
    if (!h_off) { delete ix; return fail(HR_ERR_HIP, "out of host memory"); }
    for (int64_t l = 0; l <= nlist; l++) h_off[l] = (int)list_offsets[l];
    for (int64_t l = 0; l < nlist; l++) ix->longest = std::max(ix->longest, list_offsets[l + 1] - list_offsets[l]);
    ix->device = dev;
    hipError_t e = hipDeviceGetAttribute(&ix->num_cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess) e = hr::static_scratch_address(dev, &ix->scratch);
    ix->lds_limit = 160 * 1024;     // LDS per workgroup on gfx950
    if (e == hipSuccess) {
        hipDeviceProp_t prop;
        e = hipGetDeviceProperties(&prop, dev);
        if (e == hipSuccess && strncmp(prop.gcnArchName, "gfx950", 6) != 0) {
            delete[] h_off;
            delete ix;
            return fail(HR_ERR_UNSUPPORTED, "device is %s; this library is built for gfx950 only", prop.gcnArchName);
        }
    }
    if (e == hipSuccess) e = hipMalloc(&ix->d_list_off, (size_t)(nlist + 1) * 4);
    if (e == hipSuccess) e = hipMalloc(&ix->d_row_norm, (size_t)(N > 0 ? N : 1) * 4);
    if (e == hipSuccess && dtype == HR_F32) e = hipMalloc(&ix->d_list_bound, (size_t)nlist * sizeof(ListBound));
    if (e == hipSuccess && dtype == HR_F32) e = hipMalloc(&ix->d_spread, (size_t)nlist * sizeof(float2));
    if (e == hipSuccess && dtype == HR_F32) e = hipHostMalloc((void**)&ix->h_tight, 2 * sizeof(int), hipHostMallocMapped | hipHostMallocCoherent);
    if (e == hipSuccess && dtype == HR_F32) {
        ix->h_tight[0] = ix->h_tight[1] = 0;
        e = hipHostGetDevicePointer((void**)&ix->d_tight, ix->h_tight, 0);
    }
    if (e == hipSuccess) e = hipMalloc(&ix->d_cent_norm, (size_t)nlist * 4);
    if (e == hipSuccess) e = hipMalloc(&ix->d_cent_hi, (size_t)nlist * d * 2);
    if (e == hipSuccess) e = hipMalloc(&ix->d_cent_lo, (size_t)nlist * d * 2);
    if (e == hipSuccess) e = hipMalloc(&ix->d_hits, (size_t)nlist * 8);
    if (e == hipSuccess) e = hipMalloc(&ix->d_flag, 4 * sizeof(int));
    if (e == hipSuccess) e = hipMalloc(&ix->d_resident, (size_t)nlist * sizeof(int));
    if (e == hipSuccess) e = launch_set_resident(ix->d_resident, (int)nlist, nullptr, nlist, 1, s);
    if (e == hipSuccess) e = hipMemsetAsync(ix->d_hits, 0, (size_t)nlist * 8, s);
    if (e == hipSuccess) e = hipMemsetAsync(ix->d_flag, 0, 4 * sizeof(int), s);
    if (e == hipSuccess) e = launch_check_labels(list_ids, N, ix->d_flag + 1, s);
    if (e == hipSuccess) e = hipMemcpyAsync(ix->d_list_off, h_off, (size_t)(nlist + 1) * 4, hipMemcpyHostToDevice, s);
    if (e == hipSuccess && dtype == HR_F32) {
        // float32 lists, when the caller asks for row tables: the scan multiplies the rows rounded to binary16.  Rounded once
        // here (half the bytes again) they go straight from HBM to LDS like 16-bit lists; else the scan moves
        // float32 rows.  Only when that leaves at least half of the free device memory.
        const size_t bytes = (size_t)N * d * 2;
        size_t free_b = 0, total_b = 0;
        if (row_tables && N > 0 && hipMemGetInfo(&free_b, &total_b) == hipSuccess && bytes <= free_b / 2) {
            if (hipMalloc(&ix->d_vec_hi, bytes) != hipSuccess) ix->d_vec_hi = nullptr;
            if (!ix->d_vec_hi) (void)hipGetLastError();          // (not an error of the load: the other path is taken)
        }
        const ListArgs a{(const float*)list_vectors, 0, N, ix->d_list_off, (int)nlist, d, 0, (int)nlist, ix->d_row_norm, ix->d_list_bound,
                         ix->d_vec_hi, ix->d_spread, ix->d_tight, ix->d_flag + 2, 0, 0};
        e = hipMemsetAsync(ix->d_list_bound, 0, (size_t)nlist * sizeof(ListBound), s);
        if (e == hipSuccess) e = hipMemsetAsync(ix->d_spread, 0x7f, (size_t)nlist * sizeof(float2), s);      // (far apart, until they are known)
        if (e == hipSuccess) e = launch_list_bounds(a, s);
        if (e == hipSuccess && N > 0) e = launch_wide_windows(a, s);
    } else if (e == hipSuccess) {
        e = launch_row_norms(list_vectors, dtype, N, d, ix->d_row_norm, s);
    }
    if (e == hipSuccess) e = launch_row_norms(centroids, HR_F32, nlist, d, ix->d_cent_norm, s);
    if (e == hipSuccess) e = launch_split_f32(centroids, nlist * d, ix->d_cent_hi, ix->d_cent_lo, s);
    if (e == hipSuccess && dtype == HR_BF16 && N > 0 && row_tables) {
        // bfloat16 lists, when the caller asks for row tables: as binary16 (same bytes again) every value
        // keeps its 8 significant bits, and the scan can multiply them with the query rounded to binary16
        // in one MFMA column per query instead of two (bfloat16 hi and lo parts): twice the queries per
        // work item.  Only when that leaves at least half of the free device memory and no value overflows.
        const size_t bytes = (size_t)N * d * 2;
        size_t free_b = 0, total_b = 0;
        if (hipMemGetInfo(&free_b, &total_b) == hipSuccess && bytes <= free_b / 2) {
            if (hipMalloc(&ix->d_vec16, bytes) != hipSuccess) ix->d_vec16 = nullptr;
            if (!ix->d_vec16) (void)hipGetLastError();
            else e = launch_bf16_to_f16(list_vectors, N * d, ix->d_vec16, ix->d_flag, s);
        }
    }
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    int flags[2] = {0, 0};                      // (the first of d_flag)
    if (e == hipSuccess) e = hipMemcpy(flags, ix->d_flag, sizeof flags, hipMemcpyDeviceToHost);
    if (e == hipSuccess && ix->d_vec16 && flags[0]) {      // the lists are scanned as bfloat16
        (void)hipFree(ix->d_vec16);
        ix->d_vec16 = nullptr;
    }
    if (e == hipSuccess && ix->d_vec16) {
        e = hipHostMalloc((void**)&ix->h_over, 64 * sizeof(int), hipHostMallocMapped | hipHostMallocCoherent);
        if (e == hipSuccess) e = hipHostGetDevicePointer((void**)&ix->d_over, ix->h_over, 0);
    }
    if (e != hipSuccess || flags[1]) {
        delete[] h_off;
        if (ix->d_list_off) (void)hipFree(ix->d_list_off);
        if (ix->d_row_norm) (void)hipFree(ix->d_row_norm);
        if (ix->d_list_bound) (void)hipFree(ix->d_list_bound);
        if (ix->d_spread) (void)hipFree(ix->d_spread);
        if (ix->h_tight) (void)hipHostFree(ix->h_tight);
        if (ix->d_cent_norm) (void)hipFree(ix->d_cent_norm);
        if (ix->d_cent_hi) (void)hipFree(ix->d_cent_hi);
        if (ix->d_cent_lo) (void)hipFree(ix->d_cent_lo);
        if (ix->d_hits) (void)hipFree(ix->d_hits);
        if (ix->d_resident) (void)hipFree(ix->d_resident);
        if (ix->d_vec_hi) (void)hipFree(ix->d_vec_hi);
        if (ix->d_vec16) (void)hipFree(ix->d_vec16);
        if (ix->d_flag) (void)hipFree(ix->d_flag);
        if (ix->h_over) (void)hipHostFree(ix->h_over);
        delete ix;
        if (e == hipSuccess) return fail(HR_ERR_ARG, "list_ids holds a negative label (labels must be >= 0: -1 marks an empty place in results)");
        return fail(HR_ERR_HIP, "hr_ivf_load: %s", hipGetErrorString(e));
    }
    ix->magic = kMagic;
    *out = ix;
    return HR_OK;
}

static void drop_events(hr_ivf_index* ix)
{
    if (!ix->prof_ev) return;
    for (int i = 0; i < 2 * ix->prof_cap; i++)
        if (ix->prof_ev[i]) (void)hipEventDestroy(ix->prof_ev[i]);
    delete[] ix->prof_ev;
    ix->prof_ev = nullptr;
    ix->prof_cap = ix->prof_n = 0;
}

int hr_ivf_profile_begin(hr_ivf_index* ix, int32_t max_calls)
{
    if (int rc = check_index(ix)) return rc;
    if (max_calls < 1 || max_calls > 65536) return fail(HR_ERR_ARG, "max_calls=%d", max_calls);
    drop_events(ix);
    ix->prof_ev = new (std::nothrow) hipEvent_t[2 * (size_t)max_calls]();
    if (!ix->prof_ev) return fail(HR_ERR_HIP, "out of host memory");
    ix->prof_cap = max_calls;
    for (int i = 0; i < 2 * max_calls; i++) {
        hipError_t e = hipEventCreate(&ix->prof_ev[i]);
        if (e != hipSuccess) { drop_events(ix); return fail(HR_ERR_HIP, "hipEventCreate: %s", hipGetErrorString(e)); }
    }
    return HR_OK;
}

int hr_ivf_profile_end(hr_ivf_index* ix, int32_t* n, double* scan_ms_avg)
{
    if (int rc = check_index(ix)) return rc;
    if (!n || !scan_ms_avg) return fail(HR_ERR_ARG, "n / scan_ms_avg is null");
    double sum = 0.0;
    int cnt = 0;
    for (int i = 0; i < ix->prof_n; i++) {
        float ms = 0.f;
        hipError_t e = hipEventSynchronize(ix->prof_ev[2 * i + 1]);
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, ix->prof_ev[2 * i], ix->prof_ev[2 * i + 1]);
        if (e != hipSuccess) { drop_events(ix); return fail(HR_ERR_HIP, "event timing: %s", hipGetErrorString(e)); }
        sum += ms;
        cnt++;
    }
    *n = cnt;
    *scan_ms_avg = cnt ? sum / cnt : 0.0;
    drop_events(ix);
    return HR_OK;
}

int hr_ivf_free(hr_ivf_index* ix)
{
    if (int rc = check_index(ix)) return rc;
    drop_events(ix);
    ix->magic = 0;
    (void)hipFree(ix->d_list_off);
    (void)hipFree(ix->d_row_norm);
    if (ix->d_list_bound) (void)hipFree(ix->d_list_bound);
    if (ix->d_spread) (void)hipFree(ix->d_spread);
    if (ix->h_tight) (void)hipHostFree(ix->h_tight);
    (void)hipFree(ix->d_cent_norm);
    (void)hipFree(ix->d_cent_hi);
    (void)hipFree(ix->d_cent_lo);
    (void)hipFree(ix->d_hits);
    (void)hipFree(ix->d_resident);
    if (ix->d_vec_hi) (void)hipFree(ix->d_vec_hi);
    if (ix->d_vec16) (void)hipFree(ix->d_vec16);
    if (ix->d_flag) (void)hipFree(ix->d_flag);
    if (ix->h_over) (void)hipHostFree(ix->h_over);
    delete[] ix->h_list_off;
    delete ix;
    return HR_OK;
}

size_t hr_ivf_workspace_bytes(const hr_ivf_index* ix, int64_t nq, int32_t nprobe, int32_t k)
{
    if (check_index(ix)) return 0;
    // (hr_ivf_scan and its step-wise forms take rows of up to HR_NPROBE_MAX places whatever the number of lists)
    if (nprobe < 1 || nprobe > HR_NPROBE_MAX) { fail(HR_ERR_ARG, "nprobe=%d must be in 1..%d", nprobe, HR_NPROBE_MAX); return 0; }
    if (check_batch(ix, nq, nprobe > ix->nlist ? (int)ix->nlist : nprobe, k, HR_METRIC_IP, true)) return 0;
    // what is enough for k is enough for fewer: searches of few neighbours may take more, shorter segments, so more result slots
    // (one request over 16 of 256 lists, the longest of 11000 rows, k 10 1386 KB of slots, k 100 1034), or wider tiles (1024 queries
    // over 32 of 1024 float32 lists of up to 20000 rows, k 12 297 MB, k 13 237).  Between these k the buffers only grow.
    size_t need = 0;
    for (const int at : {(int)k, kShortSegK, kFullTileK})
        if (at <= k) need = std::max(need, make_plan(ix, nq, nprobe, at, false).total);
    return need;
}

}  // extern "C"

// ---------------------------------------------------------------------------------------
// persistent workgroups: one per CU, or `groups` of them where LDS has room for them
static int scan_grid(const hr_ivf_index* ix, size_t lds, int groups = 1)
{
    const int occ = (int)((size_t)kLdsLimit / lds);
    return ix->num_cus * (occ < 1 ? 1 : (occ < groups ? occ : groups));
}

// query operands for the coarse step (coarse) and / or the list scan (scan), and, in the same launch, what the
// call needs cleared in its workspace
static PrepArgs prep_args(const hr_ivf_index* ix, const Plan& p, char* ws, const float* queries, int64_t nq, bool coarse, bool scan)
{
    const int od = operand_dtype(ix);
    const bool f32 = od == HR_F32;             // the scan multiplies the operand of the coarse step
    PrepArgs a{};
    a.q = queries; a.nq = nq; a.d = ix->d; a.dtype = scan ? od : (int)HR_F32;
    a.qop_coarse = (coarse || (scan && f32)) ? (_Float16*)(ws + p.o_qop_c) : nullptr;
    a.qnorm_coarse = coarse ? (float*)(ws + p.o_qnorm_c) : nullptr;
    a.qop_scan = (scan && !f32) ? ws + p.o_qop_s : nullptr;
    a.qnorm_scan = scan ? (float*)(ws + p.o_qnorm_s) : nullptr;
    a.zero = (int*)(ws + p.o_zero); a.n_zero = (int64_t)p.n_zero;
    a.qlo = scan && scan_bounded(p.dtype_s) ? (float*)(ws + p.o_thr) : nullptr;
    a.neg = (int*)(ws + p.o_thr) + nq; a.n_neg = nq; a.neg_value = (int)kKeyNegInf;
    return a;
}

// coarse scoring + top-nprobe: the scan kernel over the centroid table writes every key of a
// chunk of queries, then one wave per query picks the nprobe best.  The queries are prepared here too, for the list scan as
// well if one follows (scan): in a launch of their own before the scoring, or, where the scoring splits them while it
// loads them, with the selection.  One launch less: 64 lists, d = 64, 300 queries 1.09 times as fast in the mean of list and probe
// counts, d = 768 1.12; longer vectors have no registers to split in (d = 1024, 64 queries, 22.4 -> 25.7 us) and a few
// queries of d = 768 wait longer for their rows than the launch takes (0.94 .. 1.2).  The scoring must not need the cleared work
// counter (one item per workgroup), and its loads want 16-byte addresses.
static int enqueue_coarse(const hr_ivf_index* ix, const Plan& p, char* ws, const float* queries, int64_t nq, int nprobe,
                          int metric, bool scan, int32_t* out_probe, float* out_scores, hipStream_t s)
{
    const size_t lds = scan_lds_bytes(HR_F16X2, ix->d, p.nbuf_c);
    const bool one_item_each = nq <= p.cchunk && (int64_t)p.nseg_c * p.nqt_c <= scan_grid(ix, lds);
    const bool ride = (ix->d <= 512 || (ix->d <= 768 && nq > 16)) && one_item_each && (uintptr_t)queries % 16 == 0;
    const PrepArgs prep = prep_args(ix, p, ws, queries, nq, !ride, scan);
    if (!ride) HR_HIP(launch_prep_queries(prep, s));
    int* zero = (int*)(ws + p.o_zero);
    float* ckeys = (float*)(ws + p.o_ckeys);
    for (int64_t q0 = 0; q0 < nq; q0 += p.cchunk) {
        const int64_t n = nq - q0 < p.cchunk ? nq - q0 : p.cchunk;
        const int nqt = (int)((n + p.cw_c - 1) / p.cw_c);
        ScanArgs a{};
        a.rows = ix->d_cent_hi;
        a.rows_lo = ix->d_cent_lo;
        a.row_norm = ix->d_cent_norm;
        a.qop = ws + p.o_qop_c + (size_t)q0 * 2 * ix->d * 2;
        a.queries = ride ? queries : nullptr;
        a.work_counter = zero + ix->nlist + DYN_COUNT;
        a.dense_items = p.nseg_c * nqt;
        a.dense_nqt = nqt;
        // Long items: up to eight tiles that read the same rows go to one XCD, whose L2 then serves all but the first of them.  In
        // plain order the first items, which are the workgroups' places, put neighbouring tiles into different XCDs: 500 queries,
        // d = 1024, 65536 centroids 456 us, 368 in groups (379 with items as the workgroups came for them), 4096 49 .. 59, 46 (53);
        // 1000 queries, d = 512, 16384 centroids 105 .. 125, 104 (110).  Short items load more queries than rows: 500 queries,
        // d = 64, 16384 centroids, 64 KB of rows an item, 49, 53; 1500, d = 1024, 1024 centroids, 12 tiles, 256 KB, 39.6, 41.6.
        if ((int64_t)p.seg_c * ix->d * 4 >= (nqt <= 8 ? 256 << 10 : 512 << 10)) a.dense_groups = (nqt + 7) / 8;
        a.dense_cols = p.cols_c;
        a.dense_seg_rows = p.seg_c;
        a.dense_nrows = (int)ix->nlist;
        a.key_out = ckeys;
        a.nq = (int)n; a.k = nprobe; a.cap = 0; a.l2 = metric == HR_METRIC_L2;
        a.nbuf = p.nbuf_c;
        if (q0 > 0) HR_HIP(launch_fill_i32(a.work_counter, 1, 0, s));
        int grid = scan_grid(ix, lds);
        if (grid > a.dense_items) grid = a.dense_items;
        HR_HIP(launch_scan(HR_F16X2, ix->d, a, grid, lds, s));
        HR_HIP(launch_topk_rows(ckeys, (const float*)(ws + p.o_qnorm_c) + q0, out_probe + q0 * nprobe,
                                out_scores ? out_scores + q0 * nprobe : nullptr, n, (int)ix->nlist, nprobe,
                                a.l2, ride ? &prep : nullptr, s));
    }
    return HR_OK;
}

// grouping by list + cluster-major scan + per-query merge
static int enqueue_scan(const hr_ivf_index* ix, const Plan& p, char* ws, const float* queries, int64_t nq, const int32_t* probe,
                        int nprobe, int k, int metric, int64_t* out_ids, float* out_scores, hipStream_t s,
                        bool carried = false, int32_t* io_rows = nullptr)
{
    const size_t lds = scan_lds_bytes(p.dtype_s, ix->d, p.nbuf_s);
    int* zero = (int*)(ws + p.o_zero);
    BucketArgs b{};
    b.probe = probe; b.nq = (int)nq; b.nprobe = nprobe; b.nlist = (int)ix->nlist; b.cw = p.cw_s;
    b.cw_log2 = __builtin_ctz((unsigned)p.cw_s);
    b.half_tiles = scan_bounded(p.dtype_s) || operand_parts(p.dtype_s, ix->d) == 2;
    b.list_off = ix->d_list_off;
    b.list_w = zero;
    b.hits = ix->d_hits;
    b.resident = ix->d_resident;
    b.pair_entry = (int*)(ws + p.o_pair_entry);
    b.bucket_off = (int*)(ws + p.o_bucket_off);
    b.bucket_q = (int*)(ws + p.o_bucket_q);
    b.slot_base = (int*)(ws + p.o_slot_base);
    b.slot_cap = p.slot_cap;
    b.item_target = p.item_target;
    b.few_items = p.few_items;
    b.min_rows = p.min_rows;
    b.base_rows = p.base_rows;
    b.dyn = zero + ix->nlist;
    b.xq_rec = (int4*)(ws + p.o_xq);
    b.xq_count = zero + ix->nlist + DYN_COUNT + 8;
    b.round_cnt = zero + p.zoff_round;
    b.round_cur = zero + p.zoff_round + 8 * 64;
    b.item_cap = p.item_cap;
    // (the one workgroup of the grouping rides on the seeding)
    const bool whole = grouped_whole(b), together = whole ? nq <= kSeedBeside : ix->nlist <= kWholeLists;
    if (!together) HR_HIP(launch_bucketing(b, s));
    else if (!whole) HR_HIP(launch_bucketing_before(b, s));

    // starting lower bounds: from a carried result, and from the first rows of every query's best-ranked list
    SeedArgs sd{};
    sd.rows = row_table(ix); sd.row_norm = ix->d_row_norm; sd.qop = ws + p.o_qop_s;
    sd.probe = probe; sd.list_off = ix->d_list_off; sd.resident = ix->d_resident;
    sd.thr = (uint32_t*)(ws + p.o_thr) + nq;
    sd.hpar = (float*)(zero + p.zoff_hpar);
    sd.nq = (int)nq; sd.nprobe = nprobe; sd.nlist = (int)ix->nlist; sd.k = k;
    sd.seed_rows = k + 28 < 64 ? 64 : ((k + 28 + 15) & ~15);
    if (sd.seed_rows > 192) sd.seed_rows = 192;
    sd.l2 = metric == HR_METRIC_L2;
    sd.qnorm = (const float*)(ws + p.o_qnorm_s);
    sd.list_bound = ix->d_list_bound;
    if (carried) { sd.state_ids = out_ids; sd.state_scores = out_scores; }
    HR_HIP(launch_seed(row_dtype(ix), ix->d, sd, together ? &b : nullptr, s));
    if (together && !whole) HR_HIP(launch_bucketing_behind(b, s));

    ScanArgs a{};
    a.rows = p.dtype_s == HR_F16HI ? ix->d_vec_hi : row_table(ix);
    a.row_norm = ix->d_row_norm;
    a.row_ids = ix->ids;
    a.qop = ws + p.o_qop_s;
    a.thr = (uint32_t*)(ws + p.o_thr) + nq;
    a.slot_cnt = (int*)(ws + p.o_slot_cnt);
    a.slot_ent = (Cand*)(ws + p.o_slot_ent);
    a.qnorm = (const float*)(ws + p.o_qnorm_s);
    a.qlo = (const float*)(ws + p.o_thr);
    a.list_bound = ix->d_list_bound;
    a.rows_f32 = (const float*)ix->vectors;
    a.queries = queries;
    a.bucket_q = b.bucket_q;
    a.dyn = b.dyn;
    a.xq_rec = b.xq_rec;
    a.xq_count = b.xq_count;
    a.xq_head = zero + ix->nlist + DYN_COUNT + 16;
    a.xq_stride = p.item_cap;
    a.nq = (int)nq; a.k = k; a.cap = p.cap_s; a.l2 = metric == HR_METRIC_L2;
    a.nbuf = p.nbuf_s;
    a.tile = p.cw_s;
    a.hist = zero + p.zoff_hist;
    a.hpar = (const float*)(zero + p.zoff_hpar);
    hr_ivf_index* mix = const_cast<hr_ivf_index*>(ix);
    const bool timed = mix->prof_ev && mix->prof_n < mix->prof_cap;
    if (timed) HR_HIP(hipEventRecord(mix->prof_ev[2 * mix->prof_n], s));
    HR_HIP(launch_scan(p.dtype_s, ix->d, a, scan_grid(ix, lds, p.groups_s), lds, s));
    if (timed) {
        HR_HIP(hipEventRecord(mix->prof_ev[2 * mix->prof_n + 1], s));
        mix->prof_n++;
    }

    MergeArgs m{};
    m.thr = a.thr;
    m.slot_cnt = a.slot_cnt; m.slot_ent = a.slot_ent; m.slot_stride = p.cap_s;
    m.row_ids = ix->ids;
    m.qnorm = (const float*)(ws + p.o_qnorm_s);
    m.probe = probe; m.pair_entry = b.pair_entry;
    m.list_off = ix->d_list_off; m.bucket_off = b.bucket_off; m.slot_base = b.slot_base; m.dyn = b.dyn;
    m.nq = (int)nq; m.nprobe = nprobe; m.nlist = (int)ix->nlist; m.k = k; m.l2 = a.l2;
    m.out_ids = out_ids; m.out_scores = out_scores;
    m.carried = carried ? 1 : 0;
    m.io_rows = io_rows;
    if (scan_bounded(p.dtype_s)) {
        m.rows_f32 = a.rows_f32;
        m.queries = queries; m.row_norm = ix->d_row_norm; m.qlo = a.qlo; m.list_bound = ix->d_list_bound; m.d = ix->d;
        m.split = scan_split(p.dtype_s);
    }
    HR_HIP(launch_merge(m, s));
    return HR_OK;
}

extern "C" {

int hr_ivf_search(const hr_ivf_index* ix, const float* queries, int64_t nq, int32_t nprobe, int32_t k,
                  int32_t metric, int64_t* out_ids, float* out_scores, void* workspace,
                  size_t workspace_bytes, void* stream)
{
    if (int rc = check_index(ix)) return rc;
    if (int rc = check_batch(ix, nq, nprobe, k, metric, true)) return rc;
    if (nq == 0) return HR_OK;
    if (!queries || !out_ids || !out_scores) return fail(HR_ERR_ARG, "queries / out_ids / out_scores is null");
    const Plan p = make_plan(ix, nq, nprobe, k, both_parts(ix, metric));
    if (int rc = check_ws(p, workspace, workspace_bytes)) return rc;
    char* ws = (char*)workspace;
    hipStream_t s = (hipStream_t)stream;
    int32_t* probe = (int32_t*)(ws + p.o_probe);
    if (int rc = enqueue_coarse(ix, p, ws, queries, nq, nprobe, metric, true, probe, nullptr, s)) return rc;
    return enqueue_scan(ix, p, ws, queries, nq, probe, nprobe, k, metric, out_ids, out_scores, s);
}

// Limits of a plan that has to fit the static scratch array: few, large work items (result slots are
// what takes the room) and a small coarse key table.
static constexpr PlanLimits kStaticLimits[] = {{256, (size_t)4 << 20, false, 0}, {128, (size_t)4 << 20, false, 0}, {64, (size_t)4 << 20, false, 0}};

// The plan of a call on the static array; p.total is beyond it if there is none.  Result slots are item_target x queries of
// a tile.  Storage whose tiles have 128 queries since the low parts of the operands wait for the blocks that need them had 64
// before, float32 rows of d = 1024 32, and what fitted then still does: with 128 or 64 items, as many slots.  But those leave
// compute units idle, so as long as they can the 256 items stay and the selection buffers, which lie in the slots,
// become shorter instead: 256 queries over 48 of 64 lists, k 100, half a million bfloat16 rows of d = 768, tiles of 64 queries
// 1282 us a call, of 128 with 128 items 1537, with 256 and buffers of 184 entries instead of 192 1177.
static Plan static_plan(const hr_ivf_index* ix, int64_t nq, int nprobe, int k, bool both)
{
    const size_t most = HR_STATIC_SCRATCH_BYTES;
    const Plan p = make_plan(ix, nq, nprobe, k, both, kStaticLimits[0]);
    if (p.total <= most || p.dtype_s == HR_F16) return p;
    Plan s = p;
    for (const PlanLimits& lim : kStaticLimits) {
        s = make_plan(ix, nq, nprobe, k, both, lim);
        if (s.total <= most) return s;
        const size_t column = (size_t)s.slot_cap * sizeof(Cand);                 // one entry of every slot
        PlanLimits shorter = lim;
        shorter.cap = (s.cap_s - (int)((s.total - most + column - 1) / column)) & ~3;
        if (shorter.cap < k + kAppendMax + kRoomAfterCut) continue;
        s = make_plan(ix, nq, nprobe, k, both, shorter);
        if (s.total <= most) return s;
    }
    return s;
}

int hr_ivf_search_static(const hr_ivf_index* ix, const float* queries, int64_t nq, int32_t nprobe, int32_t k,
                         int32_t metric, int64_t* out_ids, float* out_scores, void* stream)
{
    if (int rc = check_index(ix)) return rc;
    if (int rc = check_batch(ix, nq, nprobe, k, metric, true)) return rc;
    if (nq == 0) return HR_OK;
    if (!queries || !out_ids || !out_scores) return fail(HR_ERR_ARG, "queries / out_ids / out_scores is null");
    int dev = -1;
    HR_HIP(hipGetDevice(&dev));
    if (dev != ix->device) return fail(HR_ERR_ARG, "current device is %d, the index lives on device %d", dev, ix->device);
    const Plan p = static_plan(ix, nq, nprobe, k, both_parts(ix, metric));      // (both parts: tiles and buffers that are no larger)
    if (p.total > (size_t)HR_STATIC_SCRATCH_BYTES)
        return fail(HR_ERR_WORKSPACE, "this batch (nq=%lld, nprobe=%d, k=%d) needs %zu bytes of scratch, the static array has %zu: "
                                      "use hr_ivf_search with a workspace", (long long)nq, nprobe, k, p.total, (size_t)HR_STATIC_SCRATCH_BYTES);
    char* ws = (char*)ix->scratch;
    hipStream_t s = (hipStream_t)stream;
    int32_t* probe = (int32_t*)(ws + p.o_probe);
    if (int rc = enqueue_coarse(ix, p, ws, queries, nq, nprobe, metric, true, probe, nullptr, s)) return rc;
    return enqueue_scan(ix, p, ws, queries, nq, probe, nprobe, k, metric, out_ids, out_scores, s);
}

int hr_ivf_coarse(const hr_ivf_index* ix, const float* queries, int64_t nq, int32_t nprobe, int32_t metric,
                  int32_t* out_probe_ids, float* out_probe_scores, void* workspace, size_t workspace_bytes,
                  void* stream)
{
    if (int rc = check_index(ix)) return rc;
    if (int rc = check_batch(ix, nq, nprobe, 1, metric, false)) return rc;
    if (nq == 0) return HR_OK;
    if (!queries || !out_probe_ids) return fail(HR_ERR_ARG, "queries / out_probe_ids is null");
    const Plan p = make_plan(ix, nq, nprobe, 1, false);
    if (int rc = check_ws(p, workspace, workspace_bytes)) return rc;
    char* ws = (char*)workspace;
    hipStream_t s = (hipStream_t)stream;
    return enqueue_coarse(ix, p, ws, queries, nq, nprobe, metric, false, out_probe_ids, out_probe_scores, s);
}

int hr_ivf_scan(const hr_ivf_index* ix, const float* queries, int64_t nq, const int32_t* probe_ids,
                int32_t nprobe, int32_t k, int32_t metric, int64_t* out_ids, float* out_scores,
                void* workspace, size_t workspace_bytes, void* stream)
{
    if (int rc = check_index(ix)) return rc;
    if (nprobe < 1 || nprobe > HR_NPROBE_MAX) return fail(HR_ERR_ARG, "nprobe=%d must be in 1..%d", nprobe, HR_NPROBE_MAX);
    int np_plan = nprobe > ix->nlist ? (int)ix->nlist : nprobe;
    if (int rc = check_batch(ix, nq, np_plan, k, metric, true)) return rc;
    if (nq == 0) return HR_OK;
    if (!queries || !probe_ids || !out_ids || !out_scores) return fail(HR_ERR_ARG, "queries / probe_ids / outputs null");
    const Plan p = make_plan(ix, nq, nprobe, k, both_parts(ix, metric));
    if (int rc = check_ws(p, workspace, workspace_bytes)) return rc;
    char* ws = (char*)workspace;
    hipStream_t s = (hipStream_t)stream;
    HR_HIP(launch_prep_queries(prep_args(ix, p, ws, queries, nq, false, true), s));
    return enqueue_scan(ix, p, ws, queries, nq, probe_ids, nprobe, k, metric, out_ids, out_scores, s);
}

static int scan_step(const hr_ivf_index* ix, const float* queries, int64_t nq, const int32_t* probe_ids,
                     int32_t nprobe, int32_t k, int32_t metric, int64_t* io_ids, float* io_scores, int32_t* io_rows,
                     void* workspace, size_t workspace_bytes, void* stream)
{
    if (int rc = check_index(ix)) return rc;
    if (nprobe < 1 || nprobe > HR_NPROBE_MAX) return fail(HR_ERR_ARG, "nprobe=%d must be in 1..%d", nprobe, HR_NPROBE_MAX);
    int np_plan = nprobe > ix->nlist ? (int)ix->nlist : nprobe;
    if (int rc = check_batch(ix, nq, np_plan, k, metric, true)) return rc;
    if (nq == 0) return HR_OK;
    if (!queries || !probe_ids || !io_ids || !io_scores) return fail(HR_ERR_ARG, "queries / probe_ids / state null");
    const Plan p = make_plan(ix, nq, nprobe, k, both_parts(ix, metric));
    if (int rc = check_ws(p, workspace, workspace_bytes)) return rc;
    char* ws = (char*)workspace;
    hipStream_t s = (hipStream_t)stream;
    HR_HIP(launch_prep_queries(prep_args(ix, p, ws, queries, nq, false, true), s));
    return enqueue_scan(ix, p, ws, queries, nq, probe_ids, nprobe, k, metric, io_ids, io_scores, s, true, io_rows);
}

int hr_ivf_scan_step(const hr_ivf_index* ix, const float* queries, int64_t nq, const int32_t* probe_ids,
                     int32_t nprobe, int32_t k, int32_t metric, int64_t* io_ids, float* io_scores,
                     void* workspace, size_t workspace_bytes, void* stream)
{
    return scan_step(ix, queries, nq, probe_ids, nprobe, k, metric, io_ids, io_scores, nullptr, workspace, workspace_bytes, stream);
}

int hr_ivf_scan_step_rows(const hr_ivf_index* ix, const float* queries, int64_t nq, const int32_t* probe_ids,
                          int32_t nprobe, int32_t k, int32_t metric, int64_t* io_ids, float* io_scores,
                          int32_t* io_rows, void* workspace, size_t workspace_bytes, void* stream)
{
    if (int rc = check_index(ix)) return rc;
    if (nq > 0 && !io_rows) return fail(HR_ERR_ARG, "io_rows is null");
    return scan_step(ix, queries, nq, probe_ids, nprobe, k, metric, io_ids, io_scores, io_rows, workspace, workspace_bytes, stream);
}

int hr_ivf_rescore(const hr_ivf_index* ix, const float* queries, int64_t nq, const int32_t* rows, int32_t m,
                   int32_t k, int32_t metric, int64_t* out_ids, float* out_scores, int32_t* out_rows, void* stream)
{
    if (int rc = check_index(ix)) return rc;
    if (nq < 0 || nq > (1 << 24)) return fail(HR_ERR_ARG, "nq=%lld out of range", (long long)nq);
    if (m < 1 || m > HR_K_MAX) return fail(HR_ERR_ARG, "m=%d must be in 1..%d", m, HR_K_MAX);
    if (k < 1 || k > HR_K_MAX) return fail(HR_ERR_ARG, "k=%d must be in 1..%d", k, HR_K_MAX);
    if (metric != HR_METRIC_IP && metric != HR_METRIC_L2) return fail(HR_ERR_ARG, "unknown metric %d", metric);
    if (nq == 0) return HR_OK;
    if (!queries || !rows || !out_ids || !out_scores || !out_rows) return fail(HR_ERR_ARG, "queries / rows / outputs null");
    HR_HIP(launch_rescore(queries, nq, ix->d, row_dtype(ix), row_table(ix), ix->d_row_norm, ix->ids, ix->N, rows, m, k,
                          metric == HR_METRIC_L2, out_ids, out_scores, out_rows, (hipStream_t)stream));
    return HR_OK;
}

int hr_ivf_lists_of_rows(const hr_ivf_index* ix, const int32_t* rows, int64_t n, int32_t* out_lists, void* stream)
{
    if (int rc = check_index(ix)) return rc;
    if (n < 0) return fail(HR_ERR_ARG, "n=%lld is negative", (long long)n);
    if (n == 0) return HR_OK;
    if (!rows || !out_lists) return fail(HR_ERR_ARG, "rows / out_lists null");
    HR_HIP(launch_lists_of_rows(rows, n, ix->d_list_off, (int)ix->nlist, out_lists, (hipStream_t)stream));
    return HR_OK;
}

int hr_ivf_reorder_probes(const int32_t* probe, int64_t nq, int32_t nprobe, const int32_t* prev, int32_t nprev,
                          const int32_t* hot, int32_t nhot, int32_t* out_probe, void* stream)
{
    if (nq < 0 || nq > (1 << 24)) return fail(HR_ERR_ARG, "nq=%lld out of range", (long long)nq);
    if (nprobe < 1 || nprobe > HR_NPROBE_MAX) return fail(HR_ERR_ARG, "nprobe=%d must be in 1..%d", nprobe, HR_NPROBE_MAX);
    if (nprev < 0 || nprev > HR_NPROBE_MAX) return fail(HR_ERR_ARG, "nprev=%d must be in 0..%d", nprev, HR_NPROBE_MAX);
    if (nhot < 0 || nhot > HR_K_MAX) return fail(HR_ERR_ARG, "nhot=%d must be in 0..%d", nhot, HR_K_MAX);
    if (nq == 0) return HR_OK;
    if (!probe || !out_probe) return fail(HR_ERR_ARG, "probe / out_probe null");
    if (probe == out_probe) return fail(HR_ERR_ARG, "out_probe must not be probe");
    HR_HIP(launch_reorder_probes(probe, nprobe, nprev > 0 ? prev : nullptr, nprev, nhot > 0 ? hot : nullptr, nhot, nq,
                                 out_probe, (hipStream_t)stream));
    return HR_OK;
}

int hr_ivf_list_hits(const hr_ivf_index* ix, int64_t* out_hits, int32_t reset, void* stream)
{
    if (int rc = check_index(ix)) return rc;
    if (!out_hits) return fail(HR_ERR_ARG, "out_hits is null");
    HR_HIP(launch_read_hits(ix->d_hits, ix->nlist, out_hits, reset != 0, (hipStream_t)stream));
    return HR_OK;
}

int hr_ivf_hot_lists(const hr_ivf_index* ix, int32_t gc, int32_t* out_lists, void* stream)
{
    if (int rc = check_index(ix)) return rc;
    if (gc < 1 || gc > ix->nlist) return fail(HR_ERR_ARG, "gc=%d must be in 1..nlist=%lld", gc, (long long)ix->nlist);
    if (ix->nlist > 65536) return fail(HR_ERR_UNSUPPORTED, "hr_ivf_hot_lists ranks by counting: nlist=%lld > 65536", (long long)ix->nlist);
    if (!out_lists) return fail(HR_ERR_ARG, "out_lists is null");
    HR_HIP(launch_hot_lists(ix->d_hits, (int)ix->nlist, gc, out_lists, (hipStream_t)stream));
    return HR_OK;
}

int hr_ivf_set_resident(hr_ivf_index* ix, const int32_t* lists, int64_t n, int32_t resident, void* stream)
{
    if (int rc = check_index(ix)) return rc;
    if (n < 0) return fail(HR_ERR_ARG, "n=%lld is negative", (long long)n);
    if (lists == nullptr) n = ix->nlist;                     // all lists
    HR_HIP(launch_set_resident(ix->d_resident, (int)ix->nlist, lists, n, resident != 0 ? 1 : 0, (hipStream_t)stream));
    return HR_OK;
}

int hr_ivf_split_probes(const hr_ivf_index* ix, const int32_t* probe_ids, int64_t nq, int32_t nprobe,
                        int32_t* out_resident, int32_t* out_missing, void* stream)
{
    if (int rc = check_index(ix)) return rc;
    if (nq < 0 || nq > (1 << 24)) return fail(HR_ERR_ARG, "nq=%lld out of range", (long long)nq);
    if (nprobe < 1 || nprobe > HR_NPROBE_MAX) return fail(HR_ERR_ARG, "nprobe=%d must be in 1..%d", nprobe, HR_NPROBE_MAX);
    if (nq == 0) return HR_OK;
    if (!probe_ids || !out_resident || !out_missing) return fail(HR_ERR_ARG, "probe_ids / outputs null");
    if (probe_ids == out_resident || probe_ids == out_missing || out_resident == out_missing)
        return fail(HR_ERR_ARG, "the three arrays must be distinct");
    HR_HIP(launch_split_probes(probe_ids, nq, nprobe, ix->d_resident, (int)ix->nlist, ix->d_hits, out_resident, out_missing,
                               (hipStream_t)stream));
    return HR_OK;
}

}  // extern "C"

// The report word of one refresh, cleared, its own until the call returns: calls on other threads and streams report in other
// words.  (With one word per index the call that reads it first takes another's report and clears it, and that other call
// finds none.)  A sixty-fifth call waits for one of the others.
class OverflowWord {
public:
    explicit OverflowWord(hr_ivf_index* ix) : ix_(ix)
    {
        uint64_t used = ix->over_used.load();
        for (;;) {
            if (used == ~0ull) { std::this_thread::yield(); used = ix->over_used.load(); continue; }
            at_ = __builtin_ctzll(~used);
            if (ix->over_used.compare_exchange_weak(used, used | 1ull << at_)) break;
        }
        ((volatile int*)ix->h_over)[at_] = 0;
    }
    ~OverflowWord() { ix_->over_used.fetch_and(~(1ull << at_)); }
    OverflowWord(const OverflowWord&) = delete;
    int* on_device() const { return ix_->d_over + at_; }
    int value() const { return ((volatile int*)ix_->h_over)[at_]; }
private:
    hr_ivf_index* ix_;
    int at_;
};

extern "C" {

int hr_ivf_refresh_rows(hr_ivf_index* ix, int64_t row_begin, int64_t row_end, void* stream)
{
    if (int rc = check_index(ix)) return rc;
    if (row_begin < 0 || row_end < row_begin || row_end > ix->N)
        return fail(HR_ERR_ARG, "rows %lld..%lld outside 0..N=%lld", (long long)row_begin, (long long)row_end, (long long)ix->N);
    const int64_t n = row_end - row_begin;
    if (n == 0) return HR_OK;
    hipStream_t s = (hipStream_t)stream;
    const size_t esize = ix->dtype == HR_F32 ? 4 : 2;
    const char* rows = (const char*)ix->vectors + (size_t)row_begin * ix->d * esize;
    if (ix->d_vec16) {
        // (the only case in which this call waits for the stream: a new value beyond binary16 cannot go into the
        // table, and a later search must not read an infinity there.  The kernel reports it in host memory, so the wait is all
        // there is: with two launches and a copy of the flag as well, a batch that swaps eight ranges in took 753 us, now 643)
        const OverflowWord word(ix);
        HR_HIP(launch_refresh_bf16(rows, n, ix->d, ix->d_row_norm + row_begin, (char*)ix->d_vec16 + (size_t)row_begin * ix->d * 2,
                                   word.on_device(), s));
        HR_HIP(hipStreamSynchronize(s));
        if (word.value())
            return fail(HR_ERR_UNSUPPORTED, "a refreshed bfloat16 value exceeds 65504 and does not fit the binary16 row table: "
                                            "replace the rows again, or load the index without HR_LOAD_ROW_TABLES");
        return HR_OK;
    }
    if (ix->d_list_bound) {
        // the lists that have some of the rows, and those of which all rows are new
        const int *off = ix->h_list_off, *end = off + ix->nlist + 1;
        const int l0 = (int)(std::upper_bound(off, end, (int)row_begin) - off) - 1, l1 = (int)(std::lower_bound(off, end, (int)row_end) - off);
        const int whole0 = (int)(std::lower_bound(off, end, (int)row_begin) - off), whole1 = (int)(std::upper_bound(off, end, (int)row_end) - off) - 1;
        const ListArgs a{(const float*)ix->vectors, row_begin, n, ix->d_list_off, (int)ix->nlist, ix->d, l0, l1 - l0, ix->d_row_norm, ix->d_list_bound,
                         ix->d_vec_hi, ix->d_spread, ix->d_tight, ix->d_flag + 2, whole0, whole1};
        HR_HIP(launch_list_bounds(a, s));
        // (looked over when a 64th of the rows are new, or more: 16 us for 1024 lists)
        if (whole1 > whole0 && (both_parts(ix, HR_METRIC_IP) || both_parts(ix, HR_METRIC_L2)) &&
            (ix->replaced += off[whole1] - off[whole0]) * kWindowShare >= ix->N) {
            ix->replaced = 0;
            HR_HIP(launch_wide_windows(a, s));
        }
    } else
        HR_HIP(launch_row_norms(rows, ix->dtype, n, ix->d, ix->d_row_norm + row_begin, s));
    return HR_OK;
}

int hr_ivf_workspace_layout(const hr_ivf_index* ix, int64_t nq, int32_t nprobe, int32_t k, int64_t* out, int32_t cap,
                            int32_t* n)
{
    if (int rc = check_index(ix)) return rc;
    if (!out || !n || cap < 0) return fail(HR_ERR_ARG, "out / n is null");
    if (nprobe < 1 || nprobe > HR_NPROBE_MAX) return fail(HR_ERR_ARG, "nprobe=%d must be in 1..%d", nprobe, HR_NPROBE_MAX);
    if (int rc = check_batch(ix, nq, nprobe > ix->nlist ? (int)ix->nlist : nprobe, k, HR_METRIC_IP, true)) return rc;
    const Plan p = make_plan(ix, nq, nprobe, k, false);
    *n = p.nreg;
    for (int i = 0; i < p.nreg && i < cap; i++) { out[2 * i] = (int64_t)p.reg_off[i]; out[2 * i + 1] = (int64_t)p.reg_len[i]; }
    return HR_OK;
}

int hr_ivf_stats(const hr_ivf_index* ix, const void* workspace, size_t workspace_bytes, int64_t nq,
                 int32_t nprobe, int32_t k, int64_t out[4])
{
    if (int rc = check_index(ix)) return rc;
    if (!out) return fail(HR_ERR_ARG, "out is null");
    if (int rc = check_batch(ix, nq, nprobe > ix->nlist ? (int)ix->nlist : nprobe, k, HR_METRIC_IP, true)) return rc;
    const Plan p = make_plan(ix, nq, nprobe, k, false);
    if (int rc = check_ws(p, workspace, workspace_bytes)) return rc;
    int dyn[DYN_COUNT];
    HR_HIP(hipMemcpy(dyn, (const char*)workspace + p.o_zero + (size_t)ix->nlist * 4, sizeof dyn, hipMemcpyDeviceToHost));
    out[0] = dyn[DYN_ITEMS];
    out[1] = dyn[DYN_SEG_ROWS];
    out[2] = ((int64_t)(uint32_t)dyn[DYN_ROWS_HI] << 32) | (uint32_t)dyn[DYN_ROWS_LO];
    out[3] = dyn[DYN_PAIRS];
    return HR_OK;
}

}  // extern "C"
