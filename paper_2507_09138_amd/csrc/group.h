// Grouping of a batch's (query, list) pairs by list: what the kernels that do it have in common, and the whole of it for a batch
// that one workgroup can group.
#pragma once
#include "wave.h"

namespace hr {

// Exclusive prefix sums of N values over the T threads of a workgroup (16 waves at most); totals returned to all.  One
// barrier: every wave adds up the waves' sums for itself; s_wave is written by this call alone.
template <int T, int N>
__device__ __forceinline__ void block_scan(const int (&v)[N], int (&before)[N], int (&total)[N], int (*s_wave)[16])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int incl[N];
#pragma unroll
    for (int n = 0; n < N; n++) {
        incl[n] = wave_prefix_sum(v[n]);
        if (lane == 63) s_wave[n][wave] = incl[n];
    }
    __syncthreads();
#pragma unroll
    for (int n = 0; n < N; n++) {
        const int x = lane < T / 64 ? s_wave[n][lane] : 0, upto = wave_prefix_sum(x);
        total[n] = __shfl(upto, T / 64 - 1);
        before[n] = __shfl(upto - x, wave) + incl[n] - v[n];
    }
}

__device__ __forceinline__ long long wave_sum_ll(long long v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Work items and their order of execution.  Items are numbered list-major (segment-major,
// query tile minor inside a list).  The order of execution is given by eight queues, one per
// XCD: all query tiles of one (list, segment) go to the same queue, next to each other, so the
// workgroups that re-read that segment run on one XCD at about the same time and share it
// through that XCD's L2.  Inside a queue the segments are ordered in rounds.  The longest list
// has eight segments per round, in order: its segments are spread over the whole run, and the
// later ones start from the lower bounds that the earlier ones have published.  The segments
// of a shorter list are spread evenly over the same rounds from a start that depends on the
// list (a list of one segment lands in a round of its own choosing).  So every stretch of a
// queue holds the same mix of items that many queries share (long lists of popular clusters:
// bound by the matrix pipes) and items of a few queries (bound by the row stream from HBM), and
// the two kinds run side by side on the compute units of an XCD for the whole run; with all
// short lists in the first round the device streams rows with idle matrix pipes first and
// multiplies with an idle HBM afterwards.  (Within a round the order is that of arrival;
// results do not depend on the order.)
// (kRounds, the most rounds a queue has, is declared with the device scalars in common.h)

// segment s of the nseg segments of list l: queue and round (R rounds in use)
__device__ __forceinline__ int queue_of(int l, int s) { return (l + s) & 7; }
__device__ __forceinline__ int round_of(int l, int s, int nseg, int R)
{
    const unsigned u = ((unsigned)l * 2654435761u) >> 16;            // start of the list inside its first stretch, in 65536ths
    return (int)((((long long)s << 16) + u) * R / ((long long)nseg << 16));
}

// Records of the query tiles of segment s of list l (w queries, len rows from row_first on) from place pos of queue x on.
__device__ __forceinline__ void write_items(const BucketArgs& a, int x, int pos, int l, int s, int nqt, int w, int row_first, int len,
                                            int seg, int boff, long long sbase)
{
    const int row0 = row_first + s * seg, nrows = min(len - s * seg, seg);
    for (int t = 0; t < nqt; t++) {
        // first result slot of the item: entries t*cw .. of segment s (the last tile of a bucket has fewer
        // than cw entries; what lies behind them belongs to the next segment and is never touched)
        const long long first = sbase + (long long)s * w + (long long)t * a.cw;
        // (the guards cannot fail: the host sizes the tables from the same bounds)
        if (pos + t < a.item_cap && first + min(a.cw, w - t * a.cw) <= a.slot_cap) {
            int4* rec = a.xq_rec + ((size_t)x * a.item_cap + pos + t) * 2;
            rec[0] = make_int4(row0, nrows, boff, w);
            rec[1] = make_int4(t, (int)first, l, s);
        }
    }
}

// One workgroup of T threads: bucket offsets, rows per segment for this batch, first result slot of every list, rounds in use.
// (PER > 0: every thread owns at most PER lists and reads their widths and lengths once, all loads in flight
// together, into registers; the passes below then run without touching memory again.  PER == 0: any number of
// lists per thread, read from memory in every pass.)
// WHOLE: the whole grouping in this one workgroup (launch_bucketing says when): the pairs are counted in LDS before the
// passes and put in place after them, and the work items are written with the (list, segment) units spread flat over the
// threads.  Bound: latency; the four other kernels of the chain are each a launch, a drain and a few dependent loads.
// With one barrier per group of sums (was three per sum): one request over 16 of 256 lists 118.6 -> 110.7 us a call, 64
// requests 210.6 -> 201.5; 544 requests in four sub-stages of two lists 1381 -> 1346.
template <int T, int PER, bool WHOLE>
__device__ __forceinline__ void group_pairs(const BucketArgs& a)
{
    static_assert(!WHOLE || PER == kWholeLists / T, "the lists of a thread sit in registers");
    constexpr int NL = WHOLE ? kWholeLists : 1, NP = WHOLE ? kWholePairs / T : 1;
    __shared__ int s_w[NL], s_boff[NL], s_slot[NL], s_unit[NL + 1];      // width, bucket, first slot, first unit of every list
    __shared__ int s_round[WHOLE ? 8 * kRounds : 1], s_cur[WHOLE ? 8 * kRounds : 1];
    int pl[NP], pe[NP];                                // list (-1: none) of this thread's pairs, place inside its bucket
    __shared__ int s_sums1[1][16], s_sums2[3][16];
    __shared__ long long s_cost[16], s_fine[16], s_rows[16];
    __shared__ int s_maxseg;
    const int t = threadIdx.x;
    if (t == 0) s_maxseg = 0;
    const int per = (a.nlist + T - 1) / T;
    const int l0 = min(a.nlist, t * per), l1 = min(a.nlist, l0 + per);
    constexpr int NR = PER > 0 ? PER : 1;
    constexpr int UN = NR;                              // loops over a thread's lists: unrolled when they sit in registers
    int wv[NR], lv[NR];
    if constexpr (WHOLE) {
        const int pairs = a.nq * a.nprobe;
        for (int l = t; l < a.nlist; l += T) s_w[l] = 0;
        for (int i = t; i < 8 * kRounds; i += T) { s_round[i] = 0; s_cur[i] = 0; }
#pragma unroll
        for (int j = 0; j < NP; j++) pl[j] = j * T + t < pairs ? a.probe[j * T + t] : -1;
        int res[NP];
#pragma unroll
        for (int j = 0; j < NP; j++) {
            if (pl[j] >= a.nlist) pl[j] = -1;
            res[j] = pl[j] >= 0 ? a.resident[pl[j]] : 0;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < NP; j++) {
            pe[j] = -1;
            if (pl[j] >= 0) {
                if (res[j] != 0) pe[j] = atomicAdd(&s_w[pl[j]], 1);
                else if (a.hits != nullptr) atomicAdd(&a.hits[pl[j]], 1ull);       // (as in k_bucket_count)
            }
            if (j * T + t < pairs) a.pair_entry[j * T + t] = pe[j];
        }
        __syncthreads();
    }
    if constexpr (PER > 0) {
#pragma unroll
        for (int i = 0; i < PER; i++) {
            const int l = min(l0 + i, a.nlist - 1);
            wv[i] = WHOLE ? s_w[l] : a.list_w[l];
            lv[i] = a.list_off[l + 1] - a.list_off[l];
        }
    }
    auto width = [&](int l) __attribute__((always_inline)) -> int {
        if constexpr (PER > 0) {
            int r = 0;
#pragma unroll
            for (int i = 0; i < PER; i++) r = (l - l0 == i) ? wv[i] : r;
            return r;
        } else {
            return a.list_w[l];
        }
    };
    auto length = [&](int l) __attribute__((always_inline)) -> int {
        if constexpr (PER > 0) {
            int r = 0;
#pragma unroll
            for (int i = 0; i < PER; i++) r = (l - l0 == i) ? lv[i] : r;
            return r;
        } else {
            return a.list_off[l + 1] - a.list_off[l];
        }
    };

    // pass 1: bucket offsets, cost = sum rows * query tiles (fine: half as wide tiles, where those are counted), rows streamed, pairs
    int w_sum = 0;
    const bool finer = a.half_tiles != 0;
    long long cost = 0, fine = 0, rows = 0;
#pragma unroll UN
    for (int i = 0; i < (PER > 0 ? PER : per); i++) {
        const int l = l0 + i;
        if (l >= l1) break;
        int w = width(l);
        long long len = length(l);
        if (a.hits != nullptr && w > 0) atomicAdd(&a.hits[l], (unsigned long long)w);     // access frequency of the list
        w_sum += w;
        cost += len * ((w + a.cw - 1) >> a.cw_log2);
        if (finer) fine += len * ((w + (a.cw >> 1) - 1) >> (a.cw_log2 - 1));
        if (w > 0) rows += len;
        if (w > 0 && len > 0) rows += (long long)((w + a.cw - 1) >> a.cw_log2) << 32;      // (fewer than 2^31 rows: the tiles above them)
    }
    cost = wave_sum_ll(cost);
    fine = finer ? wave_sum_ll(fine) : cost;
    rows = wave_sum_ll(rows);
    if ((t & 63) == 0) { s_cost[t >> 6] = cost; s_fine[t >> 6] = fine; s_rows[t >> 6] = rows; }
    {
        int v[1] = {w_sum}, before[1], total[1];
        block_scan<T>(v, before, total, s_sums1);
        int run = before[0];
#pragma unroll UN
        for (int i = 0; i < (PER > 0 ? PER : per); i++) {
            const int l = l0 + i;
            if (l >= l1) break;
            a.bucket_off[l] = run;
            if constexpr (WHOLE) s_boff[l] = run;
            run += width(l);
        }
        if (t == 0) { a.bucket_off[a.nlist] = total[0]; a.dyn[DYN_PAIRS] = total[0]; }
    }
    long long c = 0, cf = 0, r = 0;
#pragma unroll
    for (int i = 0; i < T / 64; i++) { c += s_cost[i]; cf += s_fine[i]; r += s_rows[i]; }
    // rows per segment: about item_target items at most; and, since every item costs some ten
    // microseconds whatever its size, segments of up to 1024 rows as long as that leaves 1024 items
    // (one million rows in 1024 lists: 1024 items of 1024 rows, 0.60 ms; 4096 items of 256 rows, 0.65 ms).  Counted in tiles
    // of 64 queries where a tile holds two operands per query: its items take twice as long, and the merge walks every
    // segment of every query (128 queries over all of 512 lists of 1024 bfloat16 rows, d = 768: with segments of 512 rows
    // 513 us, of 1024 rows 478; 1500 queries over 32 of them 426 and 400)
    long long segll = (c + a.item_target - 1) / a.item_target;
    const long long fewer = cf / 1024 < 1024 ? cf / 1024 : 1024;
    if (segll < fewer) segll = fewer;
    segll = (segll + 15) & ~15LL;
    // small batches of long vectors: shorter segments, as long as every workgroup still has one item at most (min_rows says
    // for which, and with which figures)
    const int tiles = (int)(r >> 32), room = a.few_items - tiles;
    r &= 0xffffffffLL;
    int least = a.base_rows;
    if (room > 0 && c < (long long)room * a.base_rows) least = max(a.min_rows, (int)(((unsigned)c + room - 1) / (unsigned)room + 15) & ~15);
    if (segll < least) segll = least;
    if (segll > 0x7ffffff0LL) segll = 0x7ffffff0LL;          // (a list has fewer than 2^31 rows: one segment then)
    const int seg = (int)segll;
    if (t == 0) {
        a.dyn[DYN_SEG_ROWS] = seg;
        a.dyn[DYN_ROWS_LO] = (int)(r & 0xffffffffLL);
        a.dyn[DYN_ROWS_HI] = (int)(r >> 32);
    }

    // pass 2: work items of a list = segments * query tiles; result slots per list = segments * bucket width
    // (one slot per (segment, query of the bucket): slot of entry e of segment s = slot_base[l] + s * w + e)
    auto list_items = [&](int l, int& nseg, int& nqt) __attribute__((always_inline)) {
        const int w = width(l);
        const int len = length(l);
        nseg = (w > 0 && len > 0) ? (len + seg - 1) / seg : 0;
        nqt = (w + a.cw - 1) >> a.cw_log2;
    };
    int items = 0, slots = 0, maxseg = 0, units = 0;
#pragma unroll UN
    for (int i = 0; i < (PER > 0 ? PER : per); i++) {
        const int l = l0 + i;
        if (l >= l1) break;
        int nseg, nqt; list_items(l, nseg, nqt);
        items += nseg * nqt; slots += nseg * width(l); maxseg = max(maxseg, nseg); units += nseg;
    }
    if (maxseg > 0) atomicMax(&s_maxseg, maxseg);
    int v2[3] = {items, slots, units}, before[3], total[3];
    block_scan<T>(v2, before, total, s_sums2);
    {
        int run = before[1];
#pragma unroll UN
        for (int i = 0; i < (PER > 0 ? PER : per); i++) {
            const int l = l0 + i;
            if (l >= l1) break;
            a.slot_base[l] = run;
            if constexpr (WHOLE) s_slot[l] = run;
            int nseg, nqt; list_items(l, nseg, nqt);
            run += nseg * width(l);
        }
        if (t == 0) {
            a.slot_base[a.nlist] = total[1];
            a.dyn[DYN_SLOTS] = total[1];
            // never more than the table holds (cannot happen: the host sizes it from the same bound)
            a.dyn[DYN_ITEMS] = min(total[0], a.item_cap);
        }
    }
    // rounds of the queues: the longest list has eight segments per round
    const int R = max(1, min(kRounds, (s_maxseg + 7) / 8));
    if (t == 0) a.dyn[DYN_ROUNDS] = R;
    if constexpr (WHOLE) {
        int run = before[2];
#pragma unroll
        for (int i = 0; i < PER; i++) {
            const int l = l0 + i;
            if (i >= per || l >= l1) break;
            s_unit[l] = run;
            int nseg, nqt; list_items(l, nseg, nqt);
            run += nseg;
        }
        if (t == 0) s_unit[a.nlist] = total[2];
        __syncthreads();
        // pairs to their places
#pragma unroll
        for (int j = 0; j < NP; j++)
            if (pe[j] >= 0) a.bucket_q[s_boff[pl[j]] + pe[j]] = (j * T + t) / a.nprobe;
        // list and segment of a unit: the last list whose first unit is not behind it (lists without units share theirs
        // with the next one, so that one is never theirs)
        auto unit = [&](int u, int& l, int& s, int& slot, int& nqt) __attribute__((always_inline)) {
            int lo = 0, hi = a.nlist;                    // s_unit[lo] <= u < s_unit[hi]
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (s_unit[mid] <= u) lo = mid; else hi = mid;
            }
            l = lo; s = u - s_unit[lo];
            slot = queue_of(l, s) * kRounds + round_of(l, s, s_unit[lo + 1] - s_unit[lo], R);
            nqt = (s_w[l] + a.cw - 1) >> a.cw_log2;
        };
        for (int u = t; u < total[2]; u += T) {
            int l, s, slot, nqt; unit(u, l, s, slot, nqt);
            atomicAdd(&s_round[slot], nqt);
        }
        __syncthreads();
        // one wave per queue: where every round starts in it
        static_assert(kRounds == 64, "a lane per round");
        if (t < 8 * kRounds) {
            const int c = s_round[t], incl = wave_prefix_sum(c);
            s_round[t] = incl - c;
            if ((t & 63) == 63) a.xq_count[t >> 6] = min(incl, a.item_cap);
        }
        __syncthreads();
        for (int u = t; u < total[2]; u += T) {
            int l, s, slot, nqt; unit(u, l, s, slot, nqt);
            const int w = s_w[l], row_first = a.list_off[l], len = a.list_off[l + 1] - row_first;
            const int pos = s_round[slot] + atomicAdd(&s_cur[slot], nqt);
            write_items(a, slot / kRounds, pos, l, s, nqt, w, row_first, len, seg, s_boff[l], s_slot[l]);
        }
    }
}

}  // namespace hr
