// Cluster-major list scan with in-kernel top-k selection (gfx950, wave64, MFMA 16x16x32).
//
// One work item = (a segment of consecutive rows of one inverted list) x (a tile of the
// queries bucketed to that list).  The rows are streamed once through LDS in blocks of 16 (short vectors: up to 64)
// and every wave multiplies each block with the query operand it keeps in registers, so a
// staged block is reused by all queries of the tile (the cross-request sharing of one pass
// over a probed cluster: Sections 4.4 and 5 of the paper; the per-pair similarity is the
// one of Section 2.2).  Each wave owns a fixed set of query columns and keeps, per column,
// a small candidate buffer in LDS that is pruned to the k best whenever it fills up; what
// is left at the end of the item goes to the item's slots for the per-query merge.
//
// Storage types:
//   HR_F16   rows are binary16; the query is rounded to binary16; one MFMA per k-step.
//   HR_BF16  rows are bfloat16; the query is split into bfloat16 hi + lo parts, each an operand in registers of its
//            own (d <= 768), or the two in two MFMA columns (lanes j and j+8 of each 16-lane row); the same products
//            in the same order either way, summed after the MFMA.
//   HR_F32   rows are float32 and rounded to binary16 as they are read from LDS, the query likewise; the key is that product
//            plus what the roundings can have taken from it (an upper bound, see scan_slack), and the merge computes the
//            exact float32 scores of the rows that may be among the k best.  All four products of (hi + lo) parts, which this
//            replaces, multiplied for every row what decides for a few: 1024 queries, 32 of 1024 lists of 1024 rows,
//            d = 768, scan 601 -> 498 us (6.4 TB/s of rows), 3000 queries over 16 of 256 lists, d = 64, k 100, 1020 -> 803 a call.
//   HR_F16HI (internal) the same with rows that were rounded beforehand: half the bytes (600 -> 290 us of the first).
//   HR_F32X2 (internal) float32 rows of which every block is split into binary16 hi and 2^11-scaled lo parts where it lies in LDS, by the
//            waves that requested it, the query likewise; the four partial products as in HR_F16X2, and a bound of what those leave
//            over, a hundredth of what HR_F32 leaves out.  For rows that are so close to each other, or so long against the distances
//            between them, that the bounds of HR_F32 leave too many of them (see score_window): the first of the above 698 us a call
//            instead of 613; rows within 2 % of each other, 1024 queries over 16 of 256 lists of 1024, d = 768, 803 -> 334.
//   HR_F16X2 (internal) rows that were split into binary16 hi and 2^11-scaled lo tables beforehand, the query likewise; the
//            four partial products are recombined with their scales, which keeps about 22 bits of each factor with
//            float32 accumulation (the centroid table: the coarse step of Section 2.2 runs this kernel
//            in "dense" mode, all queries against all rows, and writes every key out).
#pragma once
#include "group.h"
#include "wave.h"

namespace hr {

// Lower edge of histogram bin b of a query whose bin 0 starts at base and whose bins are w
// wide; one expression, used wherever a key is binned or a bound is derived, so that a key
// counted in bin b is never below the edge that later readers compute for b.
__device__ __forceinline__ float hist_edge(float base, float w, int b) { return __builtin_fmaf((float)b, w, base); }

// Keep the k best of the n (> k) candidates in buf[0..n): afterwards buf[0..k) holds them, in
// no particular order.  Order: key descending, then label ascending (label = row number when
// ids == nullptr; labels are only fetched when equal keys straddle the k-th place).
// Binary radix select on the key bits.  What bounds it is a serial chain, one ballot and count per entry slot and bit,
// so it walks as few bits as decide: from the highest bit in which two of the keys differ (keys of one query share
// sign, exponent and more) down to where as many entries are left as are wanted, about log2 n + 2 bits instead of 32.
// Called by a whole converged wave with wave-uniform arguments.  Returns the k-th best key.
// Label of a candidate for tie-breaking and output: rows with the top bit set are entries of
// a carried result (index into ext), the others stored rows.
constexpr uint32_t kCarried = 0x80000000u;
__device__ __forceinline__ int64_t label_of(uint32_t row, const int64_t* ids, const int64_t* ext)
{
    if (row & kCarried) return ext[row & ~kCarried];
    return ids ? ids[row] : (int64_t)row;
}

template <int CAPE>   // entries held per lane: CAPE * 64 >= n
__device__ __forceinline__ uint32_t wave_select(Cand* buf, int n, int k, const int64_t* ids, const int64_t* ext, const int lane)
{
    Cand e[CAPE];
    unsigned long long alive[CAPE], kept[CAPE];
#pragma unroll
    for (int m = 0; m < CAPE; m++) {
        const int idx = lane + 64 * m;
        const bool valid = idx < n;
        e[m] = valid ? buf[idx] : Cand{0u, 0u};
        alive[m] = __builtin_amdgcn_ballot_w64(valid);
        kept[m] = 0;
    }
    // the bits above the highest one in which two keys differ decide nothing: start below them
    uint32_t has1 = 0, has0 = 0;
#pragma unroll
    for (int m = 0; m < CAPE; m++)
        if ((alive[m] >> lane) & 1) { has1 |= e[m].key; has0 |= ~e[m].key; }
    has1 = wave_or(has1);
    const uint32_t differ = has1 & wave_or(has0);
    int need = k;              // how many of the entries still alive belong to the k best
    int left = n;              // entries still alive
    int b = differ ? 31 - __builtin_clz(differ) : -1;
    uint32_t T = has1 & ~(uint32_t)((2ull << (b < 0 ? 0 : b)) - 1);     // k-th best key, built from bit b down
    if (b < 0) T = has1;
    for (; b >= 0 && left != need; b--) {
        const uint32_t bit = 1u << b;
        unsigned long long ones[CAPE];
        int c1 = 0;
#pragma unroll
        for (int m = 0; m < CAPE; m++) {
            ones[m] = alive[m] & __builtin_amdgcn_ballot_w64((e[m].key & bit) != 0);
            c1 += __builtin_popcountll(ones[m]);
        }
        if (c1 >= need) {
            T |= bit;
            left = c1;
#pragma unroll
            for (int m = 0; m < CAPE; m++) alive[m] = ones[m];
        } else {
            need -= c1;
            left -= c1;
#pragma unroll
            for (int m = 0; m < CAPE; m++) { kept[m] |= ones[m]; alive[m] &= ~ones[m]; }
        }
    }
    if (b >= 0) {
        // everything still alive belongs to the k best: the k-th is the smallest of it
        uint32_t low = ~0u;
#pragma unroll
        for (int m = 0; m < CAPE; m++)
            if ((alive[m] >> lane) & 1) low = min(low, e[m].key);
        T = wave_min(low);
    }
    // `need` of the entries still alive complete the k best (more alive than that: their keys all equal T)
    if (left > need) {
        // equal keys on both sides of the k-th place: take the lowest labels
        int64_t label[CAPE];
        int rank[CAPE];
#pragma unroll
        for (int m = 0; m < CAPE; m++) {
            const bool mine = (alive[m] >> lane) & 1;
            label[m] = mine ? label_of(e[m].row, ids, ext) : INT64_MAX;
            rank[m] = 0;
        }
#pragma unroll
        for (int m2 = 0; m2 < CAPE; m2++) {
            unsigned long long mask = alive[m2];
            while (mask) {
                const int L = __builtin_ctzll(mask);
                mask &= mask - 1;
                const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)label[m2], L);
                const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)((uint64_t)label[m2] >> 32), L);
                const int64_t other = (int64_t)(((uint64_t)hi << 32) | lo);
#pragma unroll
                for (int m = 0; m < CAPE; m++) rank[m] += (other < label[m]) ? 1 : 0;
            }
        }
#pragma unroll
        for (int m = 0; m < CAPE; m++)
            alive[m] &= __builtin_amdgcn_ballot_w64(rank[m] < need);
    }
    wave_sync();
    int base = 0;
#pragma unroll
    for (int m = 0; m < CAPE; m++) {
        const unsigned long long both = kept[m] | alive[m];
        if ((both >> lane) & 1) buf[base + lanes_below(both)] = e[m];
        base += __builtin_popcountll(both);
    }
    wave_sync();
    return T;
}

template <int CAPE>
__device__ __forceinline__ uint32_t wave_select(Cand* buf, int n, int k, const int64_t* ids, const int64_t* ext = nullptr)
{
    return wave_select<CAPE>(buf, n, k, ids, ext, lane_id());
}

template <int DT> struct StoreTraits;
template <> struct StoreTraits<HR_F32>  { static constexpr int esize = 4, planes = 1; };
template <> struct StoreTraits<HR_F16>  { static constexpr int esize = 2, planes = 1; };
template <> struct StoreTraits<HR_BF16> { static constexpr int esize = 2, planes = 1; };
template <> struct StoreTraits<HR_F16HI> { static constexpr int esize = 2, planes = 1; };
template <> struct StoreTraits<HR_F16X2> { static constexpr int esize = 2, planes = 2; };
template <> struct StoreTraits<HR_F32X2> { static constexpr int esize = 4, planes = 1; };

// Eight waves per workgroup: two per SIMD with 256 registers each, so that one wave's MFMAs run while the other selects or
// waits, or, two workgroups on a unit, four with 128 (see groups_per_cu).  Every wave owns nc query columns, so a work item
// covers 8 * nc queries of a bucket; all waves share the staged rows.
//
// A block of rows (16, or up to 64 short ones: see block_groups) is staged by global_load_lds, which moves 16-byte
// chunks from HBM straight into LDS, no registers and no LDS store instructions in between.  Such a load writes the 64 chunks
// of a wave next to each other, so rows cannot be padded; instead chunk c of row r sits at position c ^ (r & 15) of its
// row (rows of 8 chunks: r & 7), which spreads the 16 rows of an MFMA fragment read over all banks.  Up to four blocks
// are in flight or waiting in LDS ahead of the one in use.

template <int DT, int KSTEPS>
struct ScanShape {
    static constexpr int nw = kScanWaves;
    static constexpr int d = KSTEPS * 32;
    static constexpr bool dense = DT == HR_F16X2;                  // the coarse step: every key written out, nothing selected
    static constexpr bool bounded = scan_bounded(DT);              // keys are upper bounds: see k_scan
    static constexpr int nc = cols_per_set(DT, d);                 // query columns per wave
    static constexpr int qp = operand_parts(DT, d);                // parts of the query operand in registers of their own
    static constexpr int na = 2 * qp;                              // accumulators per group of rows (independent MFMA chains)
    static constexpr int planes = StoreTraits<DT>::planes;
    static constexpr int raw = stored_f32(DT) ? 2 : planes;         // 16-byte reads from LDS per row fragment of a k-step
    static constexpr int rb = block_groups(DT, d);                 // groups of 16 rows per block
    static constexpr int br = kMfmaRows * rb;                      // rows per block
    static constexpr int rowb = d * StoreTraits<DT>::esize;        // bytes of one stored row
    static constexpr int cpr = rowb / 16;                          // 16-byte chunks per stored row
    static constexpr int swz = (cpr < 16 ? cpr : 16) - 1;          // row bits xor-ed into the chunk position
    static constexpr int chunks = br * cpr;                        // 16-byte chunks per block
    static constexpr int nld = (chunks + nw * 64 - 1) / (nw * 64); // chunks per thread per block
    // (every wave always issues nld loads, so a buffer is a whole number of them)
    static constexpr int plane_bytes = nld * nw * 1024;
    static constexpr int buf_bytes = plane_bytes * planes;
    static constexpr int nnl = (br + 63) / 64;                     // loads of the norms of a block's rows
    static constexpr int lpf = planes * nld + nnl;                 // loads per wave per block (chunks + norms)
    // k-steps whose row fragments are fetched from LDS together, ahead of their MFMAs
    static constexpr int grp = scan_group(DT, KSTEPS);
    // a wave whose operand fills the register file: what the rare paths need is computed there (see lane_now), and
    // the fragment addresses come from one register.  The others have registers to spare and lose by it: binary16,
    // 4096 queries x 4096 lists, d = 768, 2.46 -> 2.74 ms; 1024 queries, 524288 rows of d = 1024: binary16 1.45 -> 1.46.
    static constexpr bool lean = qp == 2 && KSTEPS >= 16;
    // two blocks of a pair as one MFMA chain (see mfma_pair): twice the accumulators, which a wave that holds both
    // parts of 24 k-steps has no registers for.
    static constexpr bool chain = !dense && rb == 1 && (KSTEPS / grp) % 2 == 0 && grp * 2 <= KSTEPS && qp * KSTEPS < 48;
    static constexpr int cw = nc * nw;                             // query columns per item
};

// s_waitcnt immediate that waits for all but n vector-memory operations (n <= 63) and for
// nothing else
__host__ __device__ constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0F70; }

// eight float32 values as binary16
__device__ __forceinline__ half8 round8(const u32x4 (&raw)[2])
{
    typedef float floatx8 __attribute__((ext_vector_type(8)));
    const floatx4 x0 = __builtin_bit_cast(floatx4, raw[0]), x1 = __builtin_bit_cast(floatx4, raw[1]);
    const floatx8 x = __builtin_shufflevector(x0, x1, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_convertvector(x, half8);
}

// eight float32 values as binary16, and what that rounding left over, times 2^11
__device__ __forceinline__ void split8(const u32x4 (&raw)[2], half8& hi, half8& lo)
{
    const floatx4 x0 = __builtin_bit_cast(floatx4, raw[0]), x1 = __builtin_bit_cast(floatx4, raw[1]);
#pragma unroll
    for (int i = 0; i < 8; i++) {
        const float x = i < 4 ? x0[i & 3] : x1[i & 3];
        hi[i] = (_Float16)x;
        lo[i] = (_Float16)((x - (float)hi[i]) * 2048.0f);
    }
}

// The products of one row fragment with the query operand of a wave (fragments of k-step t).
template <int DT, typename S>
__device__ __forceinline__ void mfma_step(const u32x4 (&row)[S::raw], const u32x4 q_hi, const u32x4 q_lo, const int t, floatx4 (&acc)[S::na])
{
    auto f16 = [](half8 x, u32x4 q, floatx4& c) __attribute__((always_inline)) { c = __builtin_amdgcn_mfma_f32_16x16x32_f16(x, __builtin_bit_cast(half8, q), c, 0, 0, 0); };
    if constexpr (DT == HR_F16 || DT == HR_F16HI) {
        f16(__builtin_bit_cast(half8, row[0]), q_hi, acc[t & 1]);
    } else if constexpr (DT == HR_F32) {
        f16(round8(row), q_hi, acc[t & 1]);
    } else if constexpr (DT == HR_BF16) {
        auto bf16 = [&](u32x4 q, floatx4& c) __attribute__((always_inline)) {
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, row[0]), __builtin_bit_cast(bf16x8, q), c, 0, 0, 0);
        };
        bf16(q_hi, acc[t & 1]);
        if constexpr (S::qp == 2) bf16(q_lo, acc[2 + (t & 1)]);
    } else {
        // (in one column: hi q x hi and lo rows, lo q x hi and lo rows; in two columns each lane has its part of the query)
        f16(__builtin_bit_cast(half8, row[0]), q_hi, acc[0]);
        f16(__builtin_bit_cast(half8, row[1]), q_hi, acc[1]);
        if constexpr (S::qp == 2) {
            f16(__builtin_bit_cast(half8, row[0]), q_lo, acc[2]);
            f16(__builtin_bit_cast(half8, row[1]), q_lo, acc[3]);
        }
    }
}

// The staged rows x the wave's query columns x d: the MFMA chains of one block.  acc[j][*] are the partial
// accumulators of the j-th 16 rows.  The row fragments are fetched from LDS a group of k-steps ahead of the MFMAs that
// use them (the scheduling barriers keep the compiler from sinking each read next to its use, which would expose the
// LDS latency 24 times per block).  The fragment of k-step t of the first 16 rows is at ap[t & 3] + (t >> 2) * 256
// (float32: its halves at ap[2 (t & 1)] and ap[2 (t & 1) + 1], + (t >> 1) * 256); the four bases are permuted per lane
// by the xor-ed chunk positions of the staging.
template <int DT, int KSTEPS, typename S>
__device__ __forceinline__ void mfma_block(const char* const (&ap)[4], const u32x4 (&bfrag)[S::qp][KSTEPS], floatx4 (&acc)[S::rb][S::na])
{
    constexpr int G = S::grp;                        // k-steps per group
    constexpr int NT = S::rb * KSTEPS;               // k-steps of the groups of 16 rows, one after the other
    constexpr int NG = NT / G;
    static_assert(NT % G == 0, "k-steps must split into whole groups");
    static_assert(KSTEPS % G == 0 || S::rb > 1, "k-steps must split into whole groups");
#pragma unroll
    for (int j = 0; j < S::rb; j++)
#pragma unroll
        for (int i = 0; i < S::na; i++) acc[j][i] = floatx4{0.f, 0.f, 0.f, 0.f};
    u32x4 af[2][G][S::raw];
    auto fetch = [&](int gi, int i) __attribute__((always_inline)) {
        const int u = gi * G + i, t = u % KSTEPS, j = u / KSTEPS;
#pragma unroll
        for (int r = 0; r < S::raw; r++) {
            if constexpr (stored_f32(DT)) af[gi & 1][i][r] = *(const u32x4*)(ap[(t & 1) * 2 + r] + (t >> 1) * 256 + j * kMfmaRows * S::rowb);
            else                          af[gi & 1][i][r] = *(const u32x4*)(ap[t & 3] + r * S::plane_bytes + (t >> 2) * 256 + j * kMfmaRows * S::rowb);
        }
    };
#pragma unroll
    for (int i = 0; i < G; i++) fetch(0, i);
#pragma unroll
    for (int gi = 0; gi < NG; gi++) {
        if (gi + 1 < NG) {
#pragma unroll
            for (int i = 0; i < G; i++) fetch(gi + 1, i);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < G; i++) {
            const int t = (gi * G + i) % KSTEPS, j = (gi * G + i) / KSTEPS;
            mfma_step<DT, S>(af[gi & 1][i], bfrag[0][t], bfrag[S::qp - 1][t], t, acc[j]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Two blocks that lie ready in LDS, multiplied back to back as one chain of 2 * KSTEPS k-steps: the first
// fragments of the second block are fetched while the last MFMAs of the first are issued (a block started on
// its own begins with a round trip to LDS during which the wave has nothing to issue), and `between` (the
// filter of the first block) runs after the first MFMAs of the second block have been handed to the matrix pipe.
template <int DT, int KSTEPS, typename S, typename F>
__device__ __forceinline__ void mfma_pair(const char* const (&ap0)[4], const char* const (&ap1)[4], const u32x4 (&bfrag)[S::qp][KSTEPS],
                                          floatx4 (&acc0)[S::rb][S::na], floatx4 (&acc1)[S::rb][S::na], F&& between)
{
    constexpr int G = S::grp;
    constexpr int NG = KSTEPS / G;
    static_assert(KSTEPS % G == 0, "k-steps must split into whole groups");
    static_assert(NG % 2 == 0, "the fragment buffers alternate: an even number of groups per block");
#pragma unroll
    for (int i = 0; i < S::na; i++) { acc0[0][i] = floatx4{0.f, 0.f, 0.f, 0.f}; acc1[0][i] = floatx4{0.f, 0.f, 0.f, 0.f}; }
    u32x4 af[2][G][S::raw];
    // (every index below is a compile-time constant: the loop over the groups is unrolled by the type system,
    // so that the operand and accumulator arrays stay in registers)
    auto fetch = [&](auto gc) __attribute__((always_inline)) {       // group gg of the 2 * NG groups of the pair
        constexpr int gg = decltype(gc)::value;
        constexpr int g0 = (gg < NG ? gg : gg - NG) * G;
#pragma unroll
        for (int i = 0; i < G; i++)
#pragma unroll
            for (int r = 0; r < S::raw; r++) {
                const int t = g0 + i;
                const char* b = stored_f32(DT) ? (gg < NG ? ap0[(t & 1) * 2 + r] : ap1[(t & 1) * 2 + r]) + (t >> 1) * 256
                                             : (gg < NG ? ap0[t & 3] : ap1[t & 3]) + r * S::plane_bytes + (t >> 2) * 256;
                af[gg & 1][i][r] = *(const u32x4*)b;
            }
    };
    auto group = [&](auto gc, floatx4 (&acc)[S::rb][S::na]) __attribute__((always_inline)) {
        constexpr int gg = decltype(gc)::value;
#pragma unroll
        for (int i = 0; i < G; i++) {
            const int t = (gg < NG ? gg : gg - NG) * G + i;
            mfma_step<DT, S>(af[gg & 1][i], bfrag[0][t], bfrag[S::qp - 1][t], t, acc[0]);
        }
    };
    fetch(std::integral_constant<int, 0>{});
    static_for<2 * NG>([&](auto gc) __attribute__((always_inline)) {
        constexpr int gg = decltype(gc)::value;
        if constexpr (gg + 1 < 2 * NG) fetch(std::integral_constant<int, gg + 1>{});
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (gg < NG) group(gc, acc0); else group(gc, acc1);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (gg == NG) between();
    });
}

// items at the head of queue x that the workgroups of its XCD start with, without asking
__device__ __forceinline__ int given_items(int x) { return ((int)gridDim.x + 7 - x) >> 3; }

// prune with as few register slots per lane as the buffer capacity needs
__device__ __forceinline__ uint32_t select_k(Cand* buf, int n, int k, int cap, const int64_t* ids, int lane)
{
    if (cap <= 64) return wave_select<1>(buf, n, k, ids, nullptr, lane);
    if (cap <= 128) return wave_select<2>(buf, n, k, ids, nullptr, lane);
    if (cap <= 192) return wave_select<3>(buf, n, k, ids, nullptr, lane);
    return wave_select<4>(buf, n, k, ids, nullptr, lane);
}

// what is xor-ed into the address of a lane's row fragment of k-step 0 for base j of mfma_block
template <int DT>
__device__ __forceinline__ constexpr int frag_step(int j) { return stored_f32(DT) ? 128 * (j >> 1) + 16 * (j & 1) : 64 * j; }

// Bounded types: the scan leaves parts of rows and query out, and the key of a row is that product's plus what they can
// add at most, |x.y| <= |x| |y|: an upper bound of its exact key, and less two slacks a lower one.
// bound: of the list's rows (ListBound).  q, q_lo: norms of the query and of its low part (infinite: no bound).  Two hundredths more for the
// roundings of the norms and for the product of the low parts, 2^-19 |q| |x| for the float32 sums of key and exact
// key; with squared L2 a key is twice the product less the squared norm, both rounded.
// split: both parts are multiplied (HR_F32X2).  What they leave over of an element is at most 2^-22 of it, or 2^-36 of one that is
// small itself.
__device__ __forceinline__ float scan_slack(float q, float q_lo, const ListBound bound, int l2, bool split, int d)
{
    const float n2 = fmaxf(bound_value(bound.norm2), 1e-18f), norm = sqrtf(n2);   // (squares of smaller numbers may have vanished)
    float s = split ? 4.9e-07f * q * norm + 1.5e-11f * sqrtf((float)d) * (q + norm) : 1.02f * (q_lo * norm + q * sqrtf(bound_value(bound.left2)));
    if (!(q_lo < __builtin_inff())) s = __builtin_inff();
    s += 1.9073486328125e-06f * q * norm;
    if (l2) s = 2.0f * s + n2 * 9.5367431640625e-07f;
    return s < __builtin_inff() ? s : __builtin_inff();          // (also for NaN)
}

// Order-preserving image of the key that lies w below the one with image u.
__device__ __forceinline__ uint32_t key_below(uint32_t u, float w)
{
    const float f = dec_key(u) - w;
    return f == f ? enc_key(f) : kKeyNegInf;                     // (an infinite key less an infinite slack)
}

// Of the n candidates in buf those that may be among the k best, given that a key is at most w above the exact one: all within w
// of the k-th largest key.  bound: set to a key that the k-th best exact one reaches; best: how many keys at the head of buf are the
// k largest (and those equal to the k-th).  Returns how many are left in buf.
template <int CAPE>   // entries held per lane: CAPE * 64 >= n
__device__ __forceinline__ int wave_window(Cand* buf, int n, int k, float w, uint32_t& bound, int& best, const int lane)
{
    Cand e[CAPE];
    unsigned long long alive[CAPE];
    uint32_t has1 = 0, has0 = 0;
#pragma unroll
    for (int m = 0; m < CAPE; m++) {
        const bool valid = lane + 64 * m < n;
        e[m] = valid ? buf[lane + 64 * m] : Cand{0u, 0u};
        alive[m] = __builtin_amdgcn_ballot_w64(valid);
        if (valid) { has1 |= e[m].key; has0 |= ~e[m].key; }
    }
    // the k-th largest key (or, once as many keys are left as are wanted, what is below all of them and above the others)
    has1 = wave_or(has1);
    const uint32_t differ = has1 & wave_or(has0);
    int b = differ ? 31 - __builtin_clz(differ) : -1;
    uint32_t T = b < 0 ? has1 : has1 & ~(uint32_t)((2ull << b) - 1);
    for (int need = k, left = n; b >= 0 && left != need; b--) {
        unsigned long long ones[CAPE];
        int c1 = 0;
#pragma unroll
        for (int m = 0; m < CAPE; m++) {
            ones[m] = alive[m] & __builtin_amdgcn_ballot_w64((e[m].key >> b) & 1u);
            c1 += __builtin_popcountll(ones[m]);
        }
        const bool up = c1 >= need;
        if (up) { T |= 1u << b; left = c1; } else { need -= c1; left -= c1; }
#pragma unroll
        for (int m = 0; m < CAPE; m++) alive[m] = up ? ones[m] : alive[m] & ~ones[m];
    }
    bound = key_below(T, w);
    wave_sync();
    int left = 0;
#pragma unroll
    for (int part = 0; part < 2; part++) {
#pragma unroll
        for (int m = 0; m < CAPE; m++) {
            const bool keep = lane + 64 * m < n && (part == 0 ? e[m].key >= T : e[m].key < T && e[m].key >= bound);
            const unsigned long long mask = __builtin_amdgcn_ballot_w64(keep);
            if (keep) buf[left + lanes_below(mask)] = e[m];
            left += __builtin_popcountll(mask);
        }
        if (part == 0) best = left;
    }
    wave_sync();
    return left;
}

// The exact keys of the entries first, first + step, .. of the n in buf, in place of their bounds: rows and query in float32, one
// wave, CH chunks of 256 elements of AT rows on their way together (past the end of a row its first elements again, times zero:
// a load under a condition would wait for the one before).  Every lane adds up its elements of the whole row in order, then the
// lanes are added up: the same sum whatever CH and AT, so a key is the same bits wherever it is computed, and a row that is left out for
// its exact key is behind k others in the final order too.  Entries of a carried result stay as they are.
template <int AT, int CH>
__device__ __forceinline__ void exact_keys(Cand* buf, int n, int first, int step, const float* rows, const float* row_norm, const float* query, int d, int l2)
{
    constexpr bool whole = CH * 256 >= 1024;                    // (the longest supported row)
    const int lane = lane_now();
    if (first >= n) return;
    floatx4 y[CH];
    int at[CH];
    auto part = [&](int c0) __attribute__((always_inline)) {    // the query's elements from c0 on
#pragma unroll
        for (int c = 0; c < CH; c++) {
            const int i = c0 + c * 256 + lane * 4;
            at[c] = i < d ? i : 0;
            y[c] = floatx4{0.f, 0.f, 0.f, 0.f};
            if (i < d) y[c] = floatx4{query[i], query[i + 1], query[i + 2], query[i + 3]};       // (the caller's: any alignment)
        }
    };
    if (whole) part(0);
#pragma unroll 1
    for (int e0 = first; e0 < n; e0 += AT * step) {
        uint32_t r[AT];
        float norm[AT], dot[AT];
#pragma unroll
        for (int j = 0; j < AT; j++) {
            r[j] = __builtin_amdgcn_readfirstlane(buf[min(e0 + j * step, n - 1)].row);
            dot[j] = 0.f;
        }
#pragma unroll 1
        for (int c0 = 0; c0 < (whole ? 1 : d); c0 += CH * 256) {
            floatx4 x[AT][CH];
            if (!whole) part(c0);
#pragma unroll
            for (int j = 0; j < AT; j++) {
                const float* p = rows + (size_t)(r[j] & kCarried ? 0u : r[j]) * d;
#pragma unroll
                for (int c = 0; c < CH; c++) x[j][c] = *(const floatx4*)(p + at[c]);
                if (c0 == 0) norm[j] = l2 ? row_norm[r[j] & kCarried ? 0u : r[j]] : 0.f;
            }
#pragma unroll
            for (int j = 0; j < AT; j++)
#pragma unroll
                for (int c = 0; c < CH; c++)
#pragma unroll
                    for (int m = 0; m < 4; m++) dot[j] = __builtin_fmaf(x[j][c][m], y[c][m], dot[j]);
        }
#pragma unroll
        for (int j = 0; j < AT; j++) dot[j] = wave_add(dot[j]);
#pragma unroll
        for (int j = 0; j < AT; j++) {
            const int e = e0 + j * step;
            if (lane == 63 && e < n && !(r[j] & kCarried)) buf[e].key = enc_key(l2 ? 2.0f * dot[j] - norm[j] : dot[j]);
        }
    }
    wave_sync();
}

__device__ __forceinline__ int window_k(Cand* buf, int n, int k, int cap, float w, uint32_t& bound, int lane)
{
    int best;
    if (cap <= 64) return wave_window<1>(buf, n, k, w, bound, best, lane);
    if (cap <= 128) return wave_window<2>(buf, n, k, w, bound, best, lane);
    if (cap <= 192) return wave_window<3>(buf, n, k, w, bound, best, lane);
    return wave_window<4>(buf, n, k, w, bound, best, lane);
}

// GROUPS = a.dense_groups > 0 (an instance of its own: both orders in one made the shortest coarse calls up to 0.5 us
// longer, 200 queries, 1024 centroids, d = 64, 15.6 and 16.1)
template <int DT, int KSTEPS, bool GROUPS = false>
__global__ __launch_bounds__(kScanWaves * 64, groups_per_cu(DT, KSTEPS * 32) == 2 ? 4 : 1) void k_scan(ScanArgs a)
{
    using S = ScanShape<DT, KSTEPS>;
    constexpr int NW = S::nw;
    constexpr int NC = S::nc;
    constexpr int QP = S::qp;
    constexpr bool DENSE = S::dense;
    constexpr int NLD = S::nld;
    constexpr int RB = S::rb, BR = S::br;
    extern __shared__ __align__(16) char smem[];
    // staging buffers in LDS: a.nbuf of them; block blk of an item uses buffer blk % NB, and the blocks up to blk + NB - 1 are
    // on their way meanwhile.
    // With 4 or 6 buffers the blocks go in pairs: one barrier per two blocks, the next pair
    // on its way meanwhile.  A barrier per block keeps the two waves of a SIMD in step (both
    // want the matrix pipeline, then both the vector ALU); between the barriers of a pair they
    // drift apart and overlap.
    const int NB = a.nbuf;
    const bool pairs = NB == 4 || NB == 6;
    const int D = pairs ? NB - 2 : NB - 1;         // blocks requested ahead of the one in use
    // LDS: [NB staging buffers][row norms NB x BR][item].  The selection buffers are the item's result slots in global
    // memory: a wave alone writes and reads the buffers of its columns, candidates are few, and LDS is left to the rows.
    char* stage = smem;
    float* nstage = (float*)(smem + NB * S::buf_bytes);
    int* s_item = (int*)(nstage + NB * BR);

    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4;                       // k-group / output row group
    const int jcol = lane & (NC - 1);              // column inside a set
    const int part = (NC == 8) ? ((lane >> 3) & 1) : 0;   // 0 = hi, 1 = lo operand column
    const bool owner = (NC == 16) || part == 0;    // lane whose accumulator holds the full dot
    const int seg_rows = a.dense_seg_rows;                   // (dense mode only: the items of the lists carry their rows)
    const int myx = blockIdx.x & 7;                // workgroups are dealt round-robin to the 8 XCDs
    bool started = false, own = true;              // first item taken; own queue not seen empty yet
    // Bounds are passed on from item to item through the histograms; where every workgroup has its only item from the
    // start there is nobody to pass them to.
    const bool keep_hist = !DENSE && a.hist != nullptr && a.dyn[DYN_ITEMS] > (int)gridDim.x;

    auto lane_here = [&]() __attribute__((always_inline)) { return S::lean ? lane_now() : lane; };

    // ---- per-lane constants of the staging layout
    // row fragment of k-step t of this lane: abase[t & 3] + (t >> 2) * 256 inside a buffer
    int abase[4];
    // byte offset inside a stored block of the chunk that load m of this lane moves
    uint32_t goff[NLD];
    {
        const int i = lane & 15;
        static_assert(!S::lean || S::rowb % 256 == 0, "the xor below stays inside a row");
        if constexpr (S::lean) {
            // (a row is a multiple of 256 bytes: the address of step j is that of step 0 with frag_step(j) xor-ed in)
            abase[0] = i * S::rowb + 16 * ((stored_f32(DT) ? 2 * g : g) ^ (i & S::swz));
            abase[1] = abase[2] = abase[3] = 0;
        } else {
#pragma unroll
            for (int j = 0; j < 4; j++) abase[j] = i * S::rowb + ((16 * ((stored_f32(DT) ? 2 * g : g) ^ (i & S::swz))) ^ frag_step<DT>(j));
        }
#pragma unroll
        for (int m = 0; m < NLD; m++) {
            const int L = (m * S::nw + wave) * 64 + lane;  // chunk position inside the buffer
            const int r = L / S::cpr, pos = L % S::cpr;
            goff[m] = (uint32_t)(min(r, BR - 1) * S::cpr + (pos ^ (r & S::swz))) * 16u;
        }
    }

    // ---- the next item.  The first one is the workgroup's place in the order: 256 workgroups asking eight counters
    // at once are served one after the other, 25 ns each and eight counters per workgroup that finds none.  Later ones
    // are asked for: in the own XCD's queue first (its items share list segments through this XCD's L2), then, once
    // that is empty, wherever a look at all eight heads together finds some left (heads only grow, so an empty queue
    // stays empty).  A queue entry is the whole record of the item.  (Every workgroup asking every counter, one after the
    // other: one request over 16 of 256 lists 111.3 us, now 70.3; 64 requests 200.5, 140.8; 512 requests, 32 of 4096
    // lists, 1162, 1091; the end of the largest batches is no shorter.)
    // The last wave asks, as soon as the blocks are done: its columns are the first to be empty, so that the two round
    // trips run while other waves hand over their results (the first wave after the barrier, waiting for its own stores
    // as well: searches of 55 .. 230 us 1 .. 2 % longer).  With many neighbours the handing over takes so long that an item
    // taken before it is missed elsewhere at the end (k 100, 500 queries, 200 lists, 308 -> 328 us): there after the barrier.
    auto next_item = [&]() __attribute__((always_inline)) {
        const int lane = lane_now();
        int item = -1;
        if (DENSE) {
            // (in groups: the workgroups of an XCD start with items that lie one behind the other)
            const int each = (int)gridDim.x >> 3, odd = (int)gridDim.x & 7;
            if (!started) item = !GROUPS ? (int)blockIdx.x : myx * each + min(myx, odd) + ((int)blockIdx.x >> 3);
            else if (lane == 0 && (int)gridDim.x < a.dense_items) item = gridDim.x + atomicAdd(a.work_counter, 1);
            if (item >= a.dense_items) item = -1;
        } else {
            const int lx = lane & 7;
            int x = myx, pos = started ? 0x7fffffff : (int)(blockIdx.x >> 3), count = 0;
            if (!started || own) {
                if (started) {
                    if (lane == 0) pos = given_items(x) + atomicAdd(&a.xq_head[x], 1);
                    pos = __builtin_amdgcn_readfirstlane(pos);
                }
                count = a.xq_count[x];
            }
            while (pos >= count) {
                own = false;
                const int head = __hip_atomic_load(&a.xq_head[lx], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const int all = a.xq_count[lx];
                const uint32_t left = (uint32_t)__builtin_amdgcn_ballot_w64(given_items(lx) + head < all) & 255u;
                if (left == 0) { x = -1; break; }
                x = (myx + __builtin_ctz(left >> myx | left << (8 - myx))) & 7;
                if (lane == 0) pos = given_items(x) + atomicAdd(&a.xq_head[x], 1);
                pos = __builtin_amdgcn_readfirstlane(pos);
                count = __builtin_amdgcn_readlane(all, x);
            }
            if (x >= 0) {
                const int* rec = (const int*)(a.xq_rec + ((size_t)x * a.xq_stride + pos) * 2);
                if (lane < 7) s_item[1 + lane] = rec[lane];
                item = 0;
            }
        }
        if (lane == 0) s_item[0] = item;
        started = true;
    };
    if (wave == NW - 1) next_item();
    __syncthreads();
    for (;;) {
        const int item = __builtin_amdgcn_readfirstlane(s_item[0]);
        if (item < 0) break;

        // ---- decode the work item
        int qt, row0, row_end, w, boff, slot0 = 0, list = 0;
        if (DENSE) {
            // plain order: all tiles of a segment, then those of the next.  In groups: tiles g, g + groups, g + 2 groups, .. of all
            // segments, then those of the next group; the first `more` groups have one tile more than the others.
            int seg;
            if (!GROUPS) {
                seg = item / a.dense_nqt;
                qt = item - seg * a.dense_nqt;
            } else {
                const int nseg = a.dense_items / a.dense_nqt;
                const int fewer = a.dense_nqt / a.dense_groups, more = a.dense_nqt - fewer * a.dense_groups;
                const int wide = more * (fewer + 1) * nseg;             // items of those groups
                const int tiles = item < wide ? fewer + 1 : fewer, at = item < wide ? item : item - wide;
                const int grp = at / (tiles * nseg), rest = at - grp * tiles * nseg;
                seg = rest / tiles;
                qt = (item < wide ? grp : more + grp) + (rest - seg * tiles) * a.dense_groups;
            }
            row0 = seg * seg_rows;
            row_end = min(a.dense_nrows, row0 + seg_rows);
            w = a.nq;
            boff = 0;
        } else {
            row0 = __builtin_amdgcn_readfirstlane(s_item[1]);
            row_end = row0 + __builtin_amdgcn_readfirstlane(s_item[2]);
            boff = __builtin_amdgcn_readfirstlane(s_item[3]);
            w = __builtin_amdgcn_readfirstlane(s_item[4]);
            qt = __builtin_amdgcn_readfirstlane(s_item[5]);
            slot0 = __builtin_amdgcn_readfirstlane(s_item[6]);
            list = __builtin_amdgcn_readfirstlane(s_item[7]);
        }
        const int nrows = row_end - row0;
        const int nblk = (nrows + BR - 1) / BR;
        // queries per wave (dense: see make_plan).  Bounded types with more than a few neighbours: a tile that is at most half full goes
        // on twice the waves, which share its selections: 250 queries over 16 of 512 lists, k 128, float32 rows of d = 768 266 -> 221
        // us, with row tables 255 -> 209, d = 64 419 -> 365, 128 queries over 32, k 24, d = 1024 183 -> 170 (k 10, 1024 queries over 32
        // of 1024 lists of 1024 rows 620 -> 626: there more waves read the same rows from LDS).
        constexpr bool SOME = (DENSE && QP == 2 && KSTEPS >= 16) || S::bounded;
        const int tile = S::bounded ? a.tile : S::cw;
        const int cpw = DENSE ? (SOME ? a.dense_cols : NC) : (S::bounded && (tile < S::cw || (a.k > 12 && w - qt * tile <= S::cw / 2)) ? NC / 2 : NC);
        Cand* const sel = a.slot_ent + ((size_t)slot0 + wave * cpw) * (size_t)a.cap;    // selection buffers of this wave's columns
        const char* src = (const char*)a.rows + (size_t)row0 * S::rowb;
        const char* src_lo = S::planes == 2 ? (const char*)a.rows_lo + (size_t)row0 * S::rowb : src;

        // ---- staging.  Requests for a block past the end of the segment fetch its last block again, or, where
        // blocks have several groups of rows, one chunk for all lanes, as a short list is past its end from the
        // start (nobody reads the copy): every wave then has the same, fixed number of loads in flight at every
        // point of the loop, which is what the wait counts below rely on.
        //
        // Block blk -> buffer buf, straight from HBM, and the squared norms of its rows (64 .. 256 bytes) beside it
        const bool stream_once = !DENSE && w <= (S::bounded ? a.tile : S::cw);   // the only work item that reads these rows
        auto fill = [&](int blk, int buf) __attribute__((always_inline)) {
            if (RB > 1 && blk >= nblk) {
#pragma unroll
                for (int m = 0; m < NLD * S::planes; m++)
                    lds_dma16(src, 0u, lds_addr(stage) + buf * S::buf_bytes + (m / NLD) * S::plane_bytes + wave * 1024 + (m % NLD) * S::nw * 1024);
                if (a.l2) {
#pragma unroll
                    for (int j = 0; j < S::nnl; j++)
                        if (lane_here() + 64 * j < BR) lds_dma4(a.row_norm + row0, 0u, lds_addr(nstage) + buf * (BR * 4) + 256 * j);
                }
                return;
            }
            const int bl = min(blk, nblk - 1);
            const int valid = min(nrows - bl * BR, BR);
#pragma unroll
            for (int pl = 0; pl < S::planes; pl++) {
                const char* bsrc = (pl == 0 ? src : src_lo) + (size_t)bl * BR * S::rowb;
                const uint32_t dst = lds_addr(stage) + buf * S::buf_bytes + pl * S::plane_bytes + wave * 1024;
                if (valid == BR) {
                    if (stream_once) {
#pragma unroll
                        for (int m = 0; m < NLD; m++) lds_dma16_nt(bsrc, goff[m], dst + m * S::nw * 1024);
                    } else {
#pragma unroll
                        for (int m = 0; m < NLD; m++) lds_dma16(bsrc, goff[m], dst + m * S::nw * 1024);
                    }
                } else {
                    // ragged last block: rows past the end repeat the last valid one (their scores
                    // are masked out of the selection)
#pragma unroll
                    for (int m = 0; m < NLD; m++) {
                        const int L = (m * S::nw + wave) * 64 + lane_here();
                        const int r = L / S::cpr, pos = L % S::cpr;
                        const uint32_t o = (uint32_t)(min(r, valid - 1) * S::cpr + (pos ^ (r & S::swz))) * 16u;
                        lds_dma16(bsrc, o, dst + m * S::nw * 1024);
                    }
                }
            }
            // (every wave writes the same norms: the same number of loads per wave; the inner
            // product needs none)
            if (a.l2) {
#pragma unroll
                for (int j = 0; j < S::nnl; j++) {
                    const int ln = lane_here() + 64 * j;
                    if (ln < BR) lds_dma4(a.row_norm + row0 + bl * BR, (uint32_t)min(ln, valid - 1) * 4u, lds_addr(nstage) + buf * (BR * 4) + 256 * j);
                }
            }
        };
        // HR_F32X2: what this wave has requested of block blk lies in buffer buf: eight elements, 32 bytes, become their hi and
        // their scaled lo parts in the same place, before the barrier that hands the block to all waves.  (Every wave splits an
        // eighth; split while the fragments are read, all of them would split all of it.)
        auto split_block = [&](int buf) __attribute__((always_inline)) {
            if constexpr (DT == HR_F32X2) {
                static_assert(NLD % 2 == 0, "half of the lanes for each of two requests");
                const int ln = lane_here();
#pragma unroll 1
                for (int m0 = 0; m0 < NLD; m0 += 2) {
                    const int m = m0 + (ln >> 5);
                    const int odd = ((m * NW + wave) * 64 + (ln & 31) * 2) / S::cpr & 1;      // (odd rows: the two chunks are swapped)
                    char* const at = stage + buf * S::buf_bytes + (m * NW + wave) * 1024 + (ln & 31) * 32;
                    u32x4* const first = (u32x4*)(at + odd * 16);
                    u32x4* const second = (u32x4*)(at + 16 - odd * 16);
                    const u32x4 x[2] = {*first, *second};
                    half8 hi, lo;
                    split8(x, hi, lo);
                    *first = __builtin_bit_cast(u32x4, hi);
                    *second = __builtin_bit_cast(u32x4, lo);
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
        };
        // ---- first row blocks on their way before anything else
        for (int i = 0; i < D; i++) fill(i, i);

        // ---- query operands of this lane's columns into registers (B fragments)
        const int ecol = (DENSE ? qt * NW * cpw : qt * tile) + wave * cpw + jcol;      // entry inside the bucket
        u32x4 bfrag[QP][KSTEPS];
        const bool col_ok = ecol < w && (!SOME || jcol < cpw);
        int q = 0;
        if (col_ok) q = DENSE ? ecol : a.bucket_q[boff + ecol];
        // operand rows of a query: both parts where they are in registers or in two columns, and of bounded types
        constexpr int QROWS = DT == HR_F16 ? 1 : 2;
        const char* const qrow = (const char*)a.qop + ((size_t)q * QROWS + (NC == 8 ? part : 0)) * (size_t)(S::d * 2) + g * 16;
        if (DENSE && a.queries != nullptr) {
            // (the same split as k_prep_queries makes; DENSE is HR_F16X2: hi and lo, in two operands or two columns)
            const float* qp = a.queries + (size_t)q * S::d + g * 8;
#pragma unroll
            for (int t = 0; t < KSTEPS; t++) {
                const u32x4 x[2] = {*(const u32x4*)(qp + t * 32), *(const u32x4*)(qp + t * 32 + 4)};
                half8 hi, lo;
                split8(x, hi, lo);
                const u32x4 none = {0, 0, 0, 0};
                if constexpr (QP == 2) {
                    bfrag[0][t] = col_ok ? __builtin_bit_cast(u32x4, hi) : none;
                    bfrag[QP - 1][t] = col_ok ? __builtin_bit_cast(u32x4, lo) : none;
                } else {
                    bfrag[0][t] = col_ok ? (part == 0 ? __builtin_bit_cast(u32x4, hi) : __builtin_bit_cast(u32x4, lo)) : none;
                }
            }
        } else {
#pragma unroll
            for (int h = 0; h < QP; h++) {
#pragma unroll
                for (int t = 0; t < KSTEPS; t++)
                    bfrag[h][t] = col_ok ? *(const u32x4*)(qrow + (size_t)h * (S::d * 2) + t * 64) : u32x4{0, 0, 0, 0};
            }
        }
        float thr = (!DENSE && owner && col_ok) ? dec_key(a.thr[q]) : __builtin_inff();
        // how far the key of a row of this list can lie above its exact key, halved (see scan_slack; infinite: every row is kept)
        float slack = 0.f;
        if constexpr (S::bounded) {
            if (col_ok) {
                const float lo = a.qlo[q];
                slack = scan_slack(sqrtf(a.qnorm[q]), lo, a.list_bound[list], a.l2, scan_split(DT), S::d);
                if (lo != lo) thr = __builtin_inff();            // (a query beyond binary16)
            }
        }
        // candidates buffered per column: kept in a register by every lane of the column (the
        // lanes of a column see the same ballots, so they stay in step without LDS traffic)
        int ccnt = 0;
        // (a wave without columns only helps to stage rows)
        const bool active = __builtin_amdgcn_ballot_w64(col_ok) != 0;
        // The query operands and thresholds are waited for here, once (the first blocks
        // with them): if the compiler still counted them as in flight inside the loop it
        // would wait for "everything" at their first use in every iteration, and that
        // includes the blocks on their way to LDS.
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));

        // ---- the blocks of the segment.  Per block (direct staging): (1) this wave's part of
        // the block has landed, (2) barrier: so has everybody's, and nobody reads the previous
        // block any more, (3) request block blk + D into the buffer the previous block leaves,
        // (4) multiply, (5) select.
        //
        // ---- dense scoring: the keys of a block are written out at the start of the next
        // step, right after the barrier.  Stores count in vmcnt like the requests for blocks,
        // and may complete in any order relative to them, so the wait at the top of a step has
        // to assume they are still outstanding; issued here they have a whole step to complete.
        floatx4 held[RB];
        int held_rbase = -1;
        auto flush_keys = [&]() __attribute__((always_inline)) {
            if (held_rbase < 0) return;
            if (active && owner && col_ok) {
#pragma unroll
                for (int j = 0; j < RB; j++) {
                    const int first = held_rbase + j * kMfmaRows;
                    float* out = a.key_out + (size_t)q * a.dense_nrows + first;
                    if (first + 3 < row_end && (a.dense_nrows & 3) == 0) {
                        *(floatx4*)out = held[j];
                    } else {
#pragma unroll
                        for (int r = 0; r < 4; r++)
                            if (first + r < row_end) out[r] = held[j][r];
                    }
                }
            }
            held_rbase = -1;
        };

        // where the row fragments of this lane start in a staged block (mfma_block's ap)
        auto frag_bases = [&](const char* (&ap)[4], const char* cur) __attribute__((always_inline)) {
            if constexpr (S::lean) {
                int a0 = abase[0];
                asm volatile("" : "+v"(a0));                     // (one register across the loop instead of four)
#pragma unroll
                for (int j = 0; j < 4; j++) ap[j] = cur + (a0 ^ frag_step<DT>(j));
            } else {
#pragma unroll
                for (int j = 0; j < 4; j++) ap[j] = cur + abase[j];
            }
        };

        // ---- selection over the scores of block blk in buffer buf: acc = accumulators of the block, nrm =
        // squared norms of this lane's 4 rows of every group
        auto select_block = [&](floatx4 (&acc)[RB][S::na], const floatx4 (&nrm)[RB], const int blk, const int buf) __attribute__((always_inline)) {
            const int brow = row0 + blk * BR;
            float keys[RB][4];
            auto make_keys = [&](auto dot) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < RB; j++) {
#pragma unroll
                    for (int r = 0; r < 4; r++) keys[j][r] = dot(acc[j], r);
                    if (a.l2) {
#pragma unroll
                        for (int r = 0; r < 4; r++) keys[j][r] = 2.0f * keys[j][r] - nrm[j][r];
                    }
                }
            };
            auto largest = [&]() __attribute__((always_inline)) {
                float best = fmaxf(fmaxf(keys[0][0], keys[0][1]), fmaxf(keys[0][2], keys[0][3]));
#pragma unroll
                for (int j = 1; j < RB; j++) best = fmaxf(best, fmaxf(fmaxf(keys[j][0], keys[j][1]), fmaxf(keys[j][2], keys[j][3])));
                return best;
            };
            make_keys([](const floatx4 (&c)[S::na], int r) __attribute__((always_inline)) {
                if constexpr (!scan_split(DT) && QP == 1) {
                    const float v = c[0][r] + c[1][r];
                    return NC == 8 ? v + lane_xor8(v) : v;
                } else if constexpr (!scan_split(DT)) {
                    return (c[0][r] + c[1][r]) + (c[2][r] + c[3][r]);
                } else if constexpr (QP == 2) {
                    return c[0][r] + (c[2][r] + c[1][r]) * (1.0f / 2048.0f) + c[3][r] * (1.0f / 4194304.0f);
                } else {
                    const float t0 = lane_xor8(c[0][r]);      // hi rows x lo query
                    const float t1 = lane_xor8(c[1][r]);      // lo rows x lo query
                    return c[0][r] + (t0 + c[1][r]) * (1.0f / 2048.0f) + t1 * (1.0f / 4194304.0f);
                }
            });
            if (DENSE) {
                // dense scoring only: every key goes to its place in the [query, row] table,
                // one block late (see flush_keys)
#pragma unroll
                for (int j = 0; j < RB; j++) held[j] = floatx4{keys[j][0], keys[j][1], keys[j][2], keys[j][3]};
                held_rbase = brow + g * 4;
                return;
            }
            // ---- keys of this lane's 4 (row, column) pairs in every group.  The common case is
            // that none reaches the column's threshold: that is decided with one compare
            // of the largest of them (thr is +inf in lanes that own no query column).
            if (__builtin_amdgcn_ballot_w64(largest() >= (S::bounded ? thr - slack : thr)) == 0) return;
            // ---- append what reaches the column's threshold, one group of 16 rows after the other
#pragma unroll 1
            for (int j = 0; j < RB; j++) {
                float key[4];
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    key[r] = keys[0][r];
#pragma unroll
                    for (int i = 1; i < RB; i++) key[r] = j == i ? keys[i][r] : key[r];
                }
                if (RB > 1 && __builtin_amdgcn_ballot_w64(fmaxf(fmaxf(key[0], key[1]), fmaxf(key[2], key[3])) >= (S::bounded ? thr - slack : thr)) == 0) continue;
                const int lane = lane_here();
                const int jcol = lane & (NC - 1);
                const int rbase = brow + j * kMfmaRows + (lane >> 4) * 4;           // first of this lane's rows
                const unsigned long long colmask = 0x0001000100010001ULL << jcol;   // lanes of my column
                bool pass[4];
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    // (a row beyond binary16, whose product is infinite, has no key)
                    pass[r] = (S::bounded ? key[r] >= thr - slack && key[r] < __builtin_inff() : key[r] >= thr) && (rbase + r < row_end);
                    if (S::bounded) key[r] += slack;
                }
                // slot of each new candidate = column count + candidates of the same
                // column in earlier row slots and in lower lanes of this row slot
                int add = 0;
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const unsigned long long mine = __builtin_amdgcn_ballot_w64(pass[r]) & colmask;
                    if (pass[r]) sel[jcol * a.cap + ccnt + add + lanes_below(mine)] = Cand{enc_key(key[r]), (uint32_t)(rbase + r)};
                    add += __builtin_popcountll(mine);
                }
                static_assert(kAppendMax >= kMfmaRows, "a column has room for what one group of rows appends");
                ccnt += add;
                unsigned long long full = __builtin_amdgcn_ballot_w64(lane < NC && ccnt > a.cap - kAppendMax);
                if (full) wave_sync();
                while (full) {
                    int col = __builtin_ctzll(full);
                    full &= full - 1;
                    int n = __builtin_amdgcn_readlane(ccnt, col);
                    uint32_t kth;
                    int left = a.k;
                    if constexpr (S::bounded) {
                        const float w = 2.0f * __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, slack), col));
                        left = window_k(sel + col * a.cap, n, a.k, a.cap, w, kth, lane);
                        if (left > a.cap - kAppendMax - kRoomAfterCut) {
                            // more rows than that are within the slack of the k-th best: the best by their exact keys
                            const int qc = __builtin_amdgcn_readlane(q, col);
                            exact_keys<scan_split(DT) ? 2 : 4, 1>(sel + col * a.cap, left, 0, 1, a.rows_f32, a.row_norm, a.queries + (size_t)qc * S::d, S::d, a.l2);
                            kth = select_k(sel + col * a.cap, left, a.k, a.cap, a.row_ids, lane);
                            left = a.k;
                        }
                    } else {
                        kth = select_k(sel + col * a.cap, n, a.k, a.cap, a.row_ids, lane);
                    }
                    float nt = 0.f;
                    if (lane == col) {
                        uint32_t old = atomicMax(&a.thr[q], kth);
                        nt = dec_key(kth > old ? kth : old);
                    }
                    nt = __shfl(nt, col);
                    if (jcol == col) { thr = fmaxf(thr, nt); ccnt = left; }
                }
            }
        };

        int bi = 0;                                              // blk % NB
        floatx4 accs[2][RB][S::na];
        floatx4 nrms[2][RB] = {};
        auto get_norms = [&](floatx4 (&nrm)[RB], int buf) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < RB; j++) nrm[j] = *(const floatx4*)(nstage + buf * BR + j * kMfmaRows + (lane_here() >> 4) * 4);
        };
        auto multiply = [&](int blk, int buf) __attribute__((always_inline)) {
            const char* ap[4];
            frag_bases(ap, stage + buf * S::buf_bytes);
            if (a.l2) get_norms(nrms[0], buf);
            mfma_block<DT, KSTEPS, S>(ap, bfrag, accs[0]);
            select_block(accs[0], nrms[0], blk, buf);
        };
        // (1) this wave's part of block blk has landed, (2) barrier: so has
        // everybody's, and nobody reads block blk-1 any more, (3) request block blk+D into the
        // buffer that one leaves, (4) multiply, (5) select
        auto step_one = [&](int blk) __attribute__((always_inline)) {
            // all but the D-1 youngest requests of this wave (S::lpf loads each) are done
            if (a.l2) {
                switch (D) {
                case 1: wait_vmcnt<0>(); break;
                case 2: wait_vmcnt<S::lpf>(); break;
                case 3: wait_vmcnt<2 * S::lpf>(); break;
                default: wait_vmcnt<3 * S::lpf>(); break;
                }
            } else {
                switch (D) {
                case 1: wait_vmcnt<0>(); break;
                case 2: wait_vmcnt<S::lpf - S::nnl>(); break;
                case 3: wait_vmcnt<2 * (S::lpf - S::nnl)>(); break;
                default: wait_vmcnt<3 * (S::lpf - S::nnl)>(); break;
                }
            }
            split_block(bi);
            __builtin_amdgcn_s_barrier();
            if (DENSE) flush_keys();
            fill(blk + D, bi == 0 ? NB - 1 : bi - 1);
            if (active) multiply(blk, bi);
            bi = bi + 1 == NB ? 0 : bi + 1;
        };
        // 4 or 6 buffers: blocks blk and blk+1 between two barriers, blocks blk+2 and
        // blk+3 requested into the two buffers the previous pair leaves
        auto step_pair = [&](int blk) __attribute__((always_inline)) {
            // (6 buffers: the requests of the pair after the next one may still be on their way)
            if (NB != 6) wait_vmcnt<0>();
            else if (a.l2) wait_vmcnt<2 * S::lpf>();
            else wait_vmcnt<2 * (S::lpf - S::nnl)>();
            split_block(bi);
            split_block(bi + 1);
            __builtin_amdgcn_s_barrier();
            // (the requests of all waves at once keep the address unit busy for a while, and a
            // wave cannot go on before its own are accepted: half of the waves send theirs
            // now, the other half after their first block, when the first half multiplies)
            const bool early = wave < NW / 2 || !active;
            auto requests = [&]() __attribute__((always_inline)) {
                const int fb = bi + D >= NB ? bi + D - NB : bi + D;     // the buffers the pair before this one used
                fill(blk + D, fb);
                fill(blk + D + 1, fb + 1);
            };
            if (early) requests();
            if (S::chain && active && blk + 1 < nblk) {
                // both blocks of the pair as one chain (see mfma_pair); the late requests go out with the
                // filter of the first block
                const char* c0 = stage + bi * S::buf_bytes;
                const char* c1 = c0 + S::buf_bytes;
                if (a.l2) {
                    get_norms(nrms[0], bi);
                    get_norms(nrms[1], bi + 1);
                }
                const char* ap0[4];
                frag_bases(ap0, c0);
                const char* ap1[4];
                frag_bases(ap1, c1);
                if constexpr (S::chain) {
                    mfma_pair<DT, KSTEPS, S>(ap0, ap1, bfrag, accs[0], accs[1], [&]() __attribute__((always_inline)) {
                        if (!early) requests();
                        select_block(accs[0], nrms[0], blk, bi);
                    });
                }
                select_block(accs[1], nrms[1], blk + 1, bi + 1);
            } else {
#pragma unroll
                for (int h = 0; h < 2; h++) {
                    if (active && blk + h < nblk) multiply(blk + h, bi + h);
                    if (h == 0 && !early) requests();
                }
            }
            bi = bi + 2 == NB ? 0 : bi + 2;
        };
        if (pairs) {
            for (int blk = 0; blk < nblk; blk += 2) step_pair(blk);
        } else {
            for (int blk = 0; blk < nblk; blk++) step_one(blk);
        }

        // (everybody has read this item's record: that was before the barrier of the first block)
        const bool early_next = DENSE || a.k <= 24;
        if (early_next && wave == NW - 1) next_item();
        if (DENSE) flush_keys();
        // ---- what is left in the selection buffers is in the item's slots already: every column's count
        wave_sync();
        if (!DENSE) {
            const int lane = lane_here();
            const int n = ccnt;                                  // (lanes below NC: of column `lane` of this wave)
            const bool ok = col_ok && lane < NC;
            if (ok) a.slot_cnt[(size_t)slot0 + wave * cpw + lane] = n;
            // ---- what this item found tightens the lower bounds of its queries for the items
            // still to come.  Every query has a histogram of the keys reported so far over
            // fixed key ranges above its seed; each reported key is a distinct row (an item
            // owns its rows), so "k keys in the bins from b up" proves that the k-th best of
            // the query is at least the lower edge of bin b.  Counts only grow, so a reader
            // that misses concurrent additions merely gets a weaker bound.
            if (keep_hist) {
                const int qcol = q;
                const bool have = ok && n > 0;
                float base = 0.f, wd = 0.f;
                uint32_t now = 0;
                if (have) {
                    base = a.hpar[2 * (size_t)qcol];
                    wd = a.hpar[2 * (size_t)qcol + 1];
                    // keys under the bound other items have reached meanwhile cannot raise it
                    now = __hip_atomic_load(&a.thr[qcol], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                int added = 0;
                {
                    // the entries of all columns of this wave side by side over the lanes (entry e of the
                    // wave = entry e - start[c] of column c): one load and one addition per entry, all
                    // of a pass in flight together
                    const int cnt = (have && wd > 0.f) ? n : 0;
                    const int incl = wave_prefix_sum(cnt);
                    const int total = __builtin_amdgcn_readlane(incl, 63);
                    unsigned long long gained = 0;                   // columns whose histogram got an addition
                    for (int e0 = 0; e0 < total; e0 += 64) {
                        const int e = e0 + lane;
                        const bool live = e < total;
                        int c = 0;                                   // column of entry e: columns that end at or before e
#pragma unroll
                        for (int cl = 0; cl < NC; cl++) c += (__builtin_amdgcn_readlane(incl, cl) <= e) ? 1 : 0;
                        c = live ? c : 0;
                        const int start = __shfl(incl - cnt, c);
                        const float cbase = __shfl(base, c), cwd = __shfl(wd, c);
                        const uint32_t cnow = (uint32_t)__shfl((int)now, c);
                        const float cslack = S::bounded ? __shfl(slack, c) : 0.f;
                        const int qc = __shfl(qcol, c);
                        bool did = false;
                        if (live) {
                            uint32_t ek = sel[c * a.cap + (e - start)].key;
                            if constexpr (S::bounded) ek = key_below(ek, 2.0f * cslack);          // (what the exact key reaches)
                            if (ek >= cnow) {
                                const float key = dec_key(ek);
                                int b = (int)fminf(fmaxf((key - cbase) * (1.0f / cwd), 0.f), (float)(kHistBins - 1));
                                if (hist_edge(cbase, cwd, b) > key) b--;
                                else if (b < kHistBins - 1 && hist_edge(cbase, cwd, b + 1) <= key) b++;
                                // (the returned value is used so that the additions have been performed
                                // before the counts are read back below)
                                if (b >= 0) did = atomicAdd(&a.hist[(size_t)qc * kHistBins + b], 1) >= 0;
                            }
                        }
#pragma unroll
                        for (int cl = 0; cl < NC; cl++)
                            if (__builtin_amdgcn_ballot_w64(did && c == cl) != 0) gained |= 1ull << cl;
                    }
                    if (lane < NC && ((gained >> lane) & 1)) added = 1;
                }
                const unsigned long long todo = __builtin_amdgcn_ballot_w64(added > 0);
                // lane i looks at bin 63 - i: the prefix sum over lanes then counts the keys
                // from the top bin down (all columns' loads go out before the first is used)
                int h[NC];
#pragma unroll
                for (int cl = 0; cl < NC; cl++) {
                    const int qc = __builtin_amdgcn_readlane(qcol, cl);
                    h[cl] = 0;
                    if ((todo >> cl) & 1)
                        h[cl] = __hip_atomic_load(&a.hist[(size_t)qc * kHistBins + (kHistBins - 1 - lane)], __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT);
                }
#pragma unroll
                for (int cl = 0; cl < NC; cl++) {
                    if (!((todo >> cl) & 1)) continue;
                    const unsigned long long reach = __builtin_amdgcn_ballot_w64(wave_prefix_sum(h[cl]) >= a.k);
                    if (reach) {
                        const int b = kHistBins - 1 - __builtin_ctzll(reach);
                        const int qc = __builtin_amdgcn_readlane(qcol, cl);
                        const float cb0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, base), cl));
                        const float cw0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, wd), cl));
                        if (b > 0 && lane == 0) atomicMax(&a.thr[qc], enc_key(hist_edge(cb0, cw0, b)));
                    }
                }
            }
        }
        __syncthreads();
        if (!early_next) {
            if (wave == NW - 1) next_item();
            __syncthreads();
        }
    }
}

template <int DT, bool GROUPS = false>
inline hipError_t launch_scan_shape(int d, const ScanArgs& a, int grid, size_t lds, hipStream_t s)
{
#define HR_SCAN_CASE(KS)                                                                           \
    case KS * 32: {                                                                                \
        auto kern = k_scan<DT, KS, GROUPS>;                                           \
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); \
        if (e != hipSuccess) return e;                                                             \
        hipLaunchKernelGGL(kern, dim3(grid), dim3(kScanWaves * 64), lds, s, a);                            \
        return hipGetLastError();                                                                  \
    }
    switch (d) {
        HR_SCAN_CASE(2)
        HR_SCAN_CASE(4)
        HR_SCAN_CASE(8)
        HR_SCAN_CASE(16)
        HR_SCAN_CASE(24)
        HR_SCAN_CASE(32)
    default: return hipErrorInvalidValue;
    }
#undef HR_SCAN_CASE
}

template <int DT>
inline hipError_t launch_scan_dtype(int d, const ScanArgs& a, int grid, size_t lds, hipStream_t s)
{
    // (HR_F16X2 is the centroid table in the coarse step, every key written out)
    if ((a.key_out != nullptr) != (DT == HR_F16X2)) return hipErrorInvalidValue;
    if constexpr (DT == HR_F16X2) {
        if (a.dense_groups > 0) return launch_scan_shape<DT, true>(d, a, grid, lds, s);
    }
    return launch_scan_shape<DT>(d, a, grid, lds, s);
}

// Key (larger is better) of an entry of a carried result, from its reported score: the score
// itself for the inner product; |q|^2 - distance for squared L2 (the inverse of what the merge
// reports, up to rounding).
__device__ __forceinline__ float key_of_score(float score, float qn, int l2) { return l2 ? qn - score : score; }

// ------------------------------------------------------------------------------------------
// Threshold seeding.  One workgroup per query scores the first rows of the query's best-ranked
// list (with the very MFMA sequence of k_scan, so the keys are the ones the scan will compute
// for these rows) and publishes the k-th best of them as the query's starting lower bound.
// On clustered data that bound already excludes nearly every row of the other probed lists,
// which then cost the scan one compare per score instead of a candidate insertion.  Any k
// real candidates give a valid bound, so the result of the search does not depend on this.
// The kernel is a chain of round trips to memory (probe row, list offsets, rows), so what
// matters is how few there are one after the other: each wave takes every fourth 16-row
// block and asks for the whole block at once (the query operand waits in LDS meanwhile,
// not in registers), wave 0 then picks the k-th key.
constexpr int kSeedRowsMax = 192;

template <int DT, int KSTEPS, int NW>      // NW waves
__device__ __forceinline__ void seed_query(const SeedArgs& a, const int64_t q)
{
    using T = StoreTraits<DT>;
    constexpr int NC = DT == HR_F16 ? 16 : 8;           // (hi and lo rows of an operand in two columns)
    constexpr int d = KSTEPS * 32;
    constexpr int rowb = d * T::esize;
    constexpr int QP = (NC == 8) ? 2 : 1;               // operand rows per query (bfloat16: hi and lo)
    __shared__ uint32_t s_keys[kSeedRowsMax];
    __shared__ u32x4 s_q[QP * KSTEPS * 4];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    // Carried results as starting lower bounds: a query whose carried result is full starts the scan at the key of its
    // worst entry (minus a margin for the rounding of key_of_score).  (A launch of its own before: 4.6 us of every sub-stage.)
    if (a.state_ids != nullptr && threadIdx.x == 0 && a.state_ids[q * a.k + a.k - 1] >= 0) {       // (best first, empty places last)
        const float sc = a.state_scores[q * a.k + a.k - 1];
        const float qn = a.l2 ? a.qnorm[q] : 0.f;
        const float margin = a.l2 ? 4.0e-7f * fmaxf(fabsf(qn), fabsf(sc)) : 0.f;
        atomicMax(&a.thr[q], enc_key(key_of_score(sc, qn, a.l2) - margin));
    }
    // the best-ranked list of the query whose vectors are in place (among the first 64 places of its row);
    // every wave finds it for itself (same loads, same answer: what follows is uniform over the workgroup)
    int l = -1;
    {
        const int c = lane < a.nprobe ? a.probe[q * a.nprobe + lane] : -1;
        const unsigned long long ok = __builtin_amdgcn_ballot_w64(c >= 0 && c < a.nlist && a.resident[c] != 0);
        if (ok == 0) return;
        l = __builtin_amdgcn_readlane(c, __builtin_ctzll(ok));
    }
    const int row0 = a.list_off[l];
    const int nrows = min(a.list_off[l + 1] - row0, a.seed_rows);
    if (nrows < a.k) return;
    for (int i = threadIdx.x; i < QP * KSTEPS * 4; i += NW * 64)
        s_q[i] = ((const u32x4*)((const char*)a.qop + (size_t)q * QP * (size_t)(d * 2)))[i];
    const int g = lane >> 4;
    const int part = (NC == 8) ? ((lane >> 3) & 1) : 0;
    const bool bcol = (lane & (NC - 1)) == 0;          // MFMA column 0 (and its lo twin)
    const u32x4* qfrag = s_q + part * (KSTEPS * 4) + g;
    __syncthreads();
    const int nblk = (nrows + 15) / 16;
    for (int blk = wave; blk < nblk; blk += NW) {
        const int r = row0 + blk * 16 + (lane & 15);
        const bool rv = r < row0 + nrows;
        const char* rp = (const char*)a.rows + (size_t)(rv ? r : row0) * rowb;
        floatx4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
        if constexpr (DT == HR_F32) {
            constexpr int H = KSTEPS / 2;               // half a row at a time: 8 registers per k-step
#pragma unroll
            for (int h = 0; h < 2; h++) {
                u32x4 v0[H], v1[H];
#pragma unroll
                for (int t = 0; t < H; t++) {
                    v0[t] = *(const u32x4*)(rp + (h * H + t) * 128 + g * 32);
                    v1[t] = *(const u32x4*)(rp + (h * H + t) * 128 + g * 32 + 16);
                }
#pragma unroll
                for (int t = 0; t < H; t++) {
                    const floatx4 f0 = __builtin_bit_cast(floatx4, v0[t]), f1 = __builtin_bit_cast(floatx4, v1[t]);
                    float x[8];
#pragma unroll
                    for (int i = 0; i < 4; i++) { x[i] = rv ? f0[i] : 0.f; x[4 + i] = rv ? f1[i] : 0.f; }
                    half8 hi, lo;
#pragma unroll
                    for (int i = 0; i < 8; i++) {
                        _Float16 hh = (_Float16)x[i];
                        hi[i] = hh;
                        lo[i] = (_Float16)((x[i] - (float)hh) * 2048.0f);
                    }
                    const half8 b = __builtin_bit_cast(half8, bcol ? qfrag[(h * H + t) * 4] : u32x4{0, 0, 0, 0});
                    acc0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(hi, b, acc0, 0, 0, 0);
                    acc1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(lo, b, acc1, 0, 0, 0);
                }
            }
        } else {
            u32x4 v[KSTEPS];
#pragma unroll
            for (int t = 0; t < KSTEPS; t++) v[t] = *(const u32x4*)(rp + t * 64 + g * 16);
#pragma unroll
            for (int t = 0; t < KSTEPS; t++) {
                const u32x4 x = rv ? v[t] : u32x4{0, 0, 0, 0};
                const u32x4 bq = bcol ? qfrag[t * 4] : u32x4{0, 0, 0, 0};
                if constexpr (DT == HR_F16) {
                    const half8 b = __builtin_bit_cast(half8, bq);
                    if (t & 1) acc1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, x), b, acc1, 0, 0, 0);
                    else       acc0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, x), b, acc0, 0, 0, 0);
                } else {
                    const bf16x8 b = __builtin_bit_cast(bf16x8, bq);
                    if (t & 1) acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x), b, acc1, 0, 0, 0);
                    else       acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x), b, acc0, 0, 0, 0);
                }
            }
        }
#pragma unroll
        for (int r4 = 0; r4 < 4; r4++) {
            float dot;
            if constexpr (DT == HR_F32) {
                float t0 = lane_xor8(acc0[r4]);
                float t1 = lane_xor8(acc1[r4]);
                dot = acc0[r4] + (t0 + acc1[r4]) * (1.0f / 2048.0f) + t1 * (1.0f / 4194304.0f);
            } else if constexpr (DT == HR_BF16) {
                float v2 = acc0[r4] + acc1[r4];
                dot = v2 + lane_xor8(v2);
            } else {
                dot = acc0[r4] + acc1[r4];
            }
            const int row = row0 + blk * 16 + g * 4 + r4;
            if ((lane & 15) == 0 && row < row0 + nrows) {
                float key = a.l2 ? (2.0f * dot - a.row_norm[row]) : dot;
                s_keys[blk * 16 + g * 4 + r4] = enc_key(key);
            }
        }
    }
    __syncthreads();
    if (wave != 0) return;
    const uint32_t* keys = s_keys;
    // k-th largest of the nrows keys (binary radix select, as in wave_select)
    uint32_t e[3];
    unsigned long long alive[3];
#pragma unroll
    for (int m = 0; m < 3; m++) {
        const int idx = lane + 64 * m;
        e[m] = idx < nrows ? keys[idx] : 0u;
        alive[m] = __builtin_amdgcn_ballot_w64(idx < nrows);
    }
    int need = a.k;
    uint32_t kth = 0;
    for (int b = 31; b >= 0; b--) {
        const uint32_t bit = 1u << b;
        unsigned long long ones[3];
        int c1 = 0;
#pragma unroll
        for (int m = 0; m < 3; m++) {
            ones[m] = alive[m] & __builtin_amdgcn_ballot_w64((e[m] & bit) != 0);
            c1 += __builtin_popcountll(ones[m]);
        }
        if (c1 >= need) {
            kth |= bit;
#pragma unroll
            for (int m = 0; m < 3; m++) alive[m] = ones[m];
        } else {
            need -= c1;
#pragma unroll
            for (int m = 0; m < 3; m++) alive[m] &= ~ones[m];
        }
    }
    // a few units in the last place lower, in case a later pass rounds a sum differently
    uint32_t pub = kth > 8u ? kth - 8u : 0u;
    if constexpr (DT == HR_F32) {
        // (the scores that count are exact ones: other sums of products of about 22 bits per factor, half of the 2^-19 |q| |x| that
        // scan_slack counts for both; and elements below 2^-36 or so vanish in the low parts.  A bound too high by that would keep
        // rows of lists with shorter rows out)
        const float qn = a.qnorm[q], xn = bound_value(a.list_bound[l].norm2);
        float lost = 2.9103830456733704e-11f * sqrtf((float)d) * (sqrtf(qn) + sqrtf(xn)) + 9.5367431640625e-07f * sqrtf(qn) * sqrtf(xn);
        if (a.l2) lost = 2.0f * lost + xn * 4.76837158203125e-07f;
        pub = qn > 1e-30f && xn > 1e-30f ? key_below(pub, lost) : 0u;
    }
    if (lane == 0) atomicMax(&a.thr[q], pub);
    // key ranges of the query's histogram in the scan: from the seed upwards, an eighth of
    // the distance between the seed and the best key of the sample per bin
    if (a.hpar != nullptr) {
        uint32_t mx = 0;
#pragma unroll
        for (int m = 0; m < 3; m++) mx = max(mx, e[m]);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mx = max(mx, (uint32_t)__shfl_xor((int)mx, o));
        if (lane == 0) {
            const float base = dec_key(pub);
            const float wd = (dec_key(mx) - base) * 0.125f;
            const bool fine = wd > 0.f && wd < 3.0e38f && base > -3.0e38f;
            a.hpar[2 * q] = fine ? base : 0.f;
            a.hpar[2 * q + 1] = fine ? wd : 0.f;
        }
    }
}

template <int DT, int KSTEPS>
__global__ __launch_bounds__(256) void k_seed(SeedArgs a) { seed_query<DT, KSTEPS, 4>(a, blockIdx.x); }

// A small batch: the first workgroup groups the probes by list, the others seed a query each.  Neither needs the other and both
// are chains of round trips, 9 and 11 us of the 52 that one request takes.  Two launches and this one, us a call: one request over 16
// of 512 lists, float32 of d = 768 57.4 and 48.5, binary16 of d = 128 45.7 and 39.0, bfloat16 of d = 1024 61.1 and 52.3; 250 over 16
// 155 and 144, 155 and 150, 141 and 130.  512 threads: with 1024 a wave has 128 registers, too few for the rows that the seeding
// asks for at once.
//
// A larger batch: the one workgroup between the counting of the probes and the work items goes beside the seeding of 256 threads a
// query (PER: lists of its threads, whose widths sit in registers).  777 queries over 33 of 1000 lists 192 -> 181 us a call (with
// k_scatter_count, a launch less), 214 over 23 of 199 112 -> 102, 1024 over 32 of 1024 629 -> 614.  Up to 4096 lists: 64 lists a thread
// take 256 registers, which the seeding misses (466 over 15 of 12754 lists 468 -> 485, 8192 over 128 of 16384 15.6 -> 15.8 ms).
template <int DT, int KSTEPS, int T, int PER>
__global__ __launch_bounds__(T) void k_group_seed(BucketArgs b, SeedArgs a)
{
    if (blockIdx.x == 0) group_pairs<T, PER, T == 512>(b);
    else seed_query<DT, KSTEPS, T / 64>(a, blockIdx.x - 1);
}

// group: the grouping of the batch rides along, or nullptr
template <int DT>
inline hipError_t launch_seed_dtype(int d, const SeedArgs& a, const BucketArgs* group, hipStream_t s)
{
    if (a.nq <= 0) return hipSuccess;
    const dim3 grid((unsigned)a.nq + (group ? 1 : 0));
    auto launch = [&](auto ks) {
        constexpr int KS = decltype(ks)::value;
        if (!group) hipLaunchKernelGGL((k_seed<DT, KS>), grid, dim3(256), 0, s, a);
        else if (grouped_whole(*group)) hipLaunchKernelGGL((k_group_seed<DT, KS, 512, kWholeLists / 512>), grid, dim3(512), 0, s, *group, a);
        else hipLaunchKernelGGL((k_group_seed<DT, KS, 256, kWholeLists / 256>), grid, dim3(256), 0, s, *group, a);
        return hipGetLastError();
    };
#define HR_SEED_CASE(KS) case KS * 32: return launch(std::integral_constant<int, KS>{});
    switch (d) {
        HR_SEED_CASE(2)
        HR_SEED_CASE(4)
        HR_SEED_CASE(8)
        HR_SEED_CASE(16)
        HR_SEED_CASE(24)
        HR_SEED_CASE(32)
    default: return hipErrorInvalidValue;
    }
#undef HR_SEED_CASE
}

}  // namespace hr
