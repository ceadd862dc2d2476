// Small kernels around the list scan: query operand preparation, row norms, grouping of
// (query, list) probes by list, and the per-query merge of the scan's partial results.
#include <algorithm>
#include <type_traits>

#include "group.h"
#include "scan_kernel.h"

namespace hr {

// ------------------------------------------------------------------------------------------
__global__ void k_fill_i32(int* p, int64_t n, int v)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

hipError_t launch_fill_i32(int* p, int64_t n, int v, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

// float32 -> binary16 hi + 2^11-scaled binary16 lo (the split the scan applies to float32 rows)
__global__ void k_split_f32(const float* x, int64_t n, _Float16* hi, _Float16* lo)
{
    // (grid-stride: a launch may not have 2^32 threads or more)
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float v = x[i];
        const _Float16 h = (_Float16)v;
        hi[i] = h;
        lo[i] = (_Float16)((v - (float)h) * 2048.0f);
    }
}

// bfloat16 -> binary16 (exact for magnitudes from 2^-14 to 65504: 8 significant bits fit in 11;
// below that the result is rounded to a multiple of 2^-24; above, the flag is raised)
__global__ void k_bf16_to_f16(const uint16_t* x, int64_t n, _Float16* out, int* overflow)
{
    bool over = false;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float v = __builtin_bit_cast(float, ((uint32_t)x[i]) << 16);
        over |= !(fabsf(v) <= 65504.0f);                       // (also for NaN)
        out[i] = (_Float16)v;
    }
    if (over) atomicOr(overflow, 1);
}

hipError_t launch_bf16_to_f16(const void* x, int64_t n, void* out, int* overflow, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_bf16_to_f16, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 1 << 20)), dim3(256), 0, s, (const uint16_t*)x, n, (_Float16*)out, overflow);
    return hipGetLastError();
}

// Labels must be non-negative: a negative id marks an empty place in results and carried results.
__global__ void k_check_labels(const int64_t* ids, int64_t n, int* negative)
{
    bool neg = false;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) neg |= ids[i] < 0;
    if (neg) atomicOr(negative, 1);
}

hipError_t launch_check_labels(const int64_t* ids, int64_t n, int* negative, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_check_labels, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 1 << 16)), dim3(256), 0, s, ids, n, negative);
    return hipGetLastError();
}

hipError_t launch_split_f32(const float* x, int64_t n, void* hi, void* lo, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_split_f32, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 1 << 20)), dim3(256), 0, s, x, n, (_Float16*)hi, (_Float16*)lo);
    return hipGetLastError();
}

// Per-list access counters (how often each list was probed: the frequency a cache of hot
// clusters is driven by, Section 4.4 of the paper): copy out, optionally start again from zero.
__global__ void k_read_hits(unsigned long long* hits, int64_t n, int64_t* out, int reset)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    out[i] = (int64_t)(reset ? atomicExch(&hits[i], 0ull) : hits[i]);
}

hipError_t launch_read_hits(unsigned long long* hits, int64_t n, int64_t* out, int reset, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_read_hits, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, hits, n, out, reset);
    return hipGetLastError();
}

// Partial residency (Section 4.4 of the paper: only the most frequently accessed clusters are kept in GPU memory, the
// searches of the others are served elsewhere and the partial results merged).  A flag per list says whether its
// vectors are in place; the grouping of probes drops the probes of the other lists.
__global__ void k_set_resident(int* resident, int nlist, const int32_t* lists, int64_t n, int value)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    if (lists == nullptr) { resident[i] = value; return; }
    const int l = lists[i];
    if (l >= 0 && l < nlist) resident[l] = value;
}

hipError_t launch_set_resident(int* resident, int nlist, const int32_t* lists, int64_t n, int value, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_set_resident, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, resident, nlist, lists, n, value);
    return hipGetLastError();
}

// Every query's probe list split into the lists whose vectors are in place and the others, each part in the given
// order, the rest of both rows filled with -1 (entries outside 0..nlist-1 go to neither).  The lists of the second
// part are counted as accessed here: no scan will see them.  One wave per query.
__global__ __launch_bounds__(256) void k_split_probes(const int32_t* probe, int64_t nq, int np, const int* resident, int nlist,
                                                      unsigned long long* hits, int32_t* out_res, int32_t* out_mis)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t q = (int64_t)blockIdx.x * 4 + wave;
    if (q >= nq) return;
    int nres = 0, nmis = 0;
    for (int i0 = 0; i0 < np; i0 += 64) {
        const int i = i0 + lane;
        const int l = i < np ? probe[q * np + i] : -1;
        const bool valid = l >= 0 && l < nlist;
        const bool here = valid && resident[l] != 0;
        const unsigned long long mr = __builtin_amdgcn_ballot_w64(here), mm = __builtin_amdgcn_ballot_w64(valid && !here);
        if (here) out_res[q * np + nres + lanes_below(mr)] = l;
        if (valid && !here) {
            out_mis[q * np + nmis + lanes_below(mm)] = l;
            if (hits != nullptr) atomicAdd(&hits[l], 1ull);
        }
        nres += __builtin_popcountll(mr);
        nmis += __builtin_popcountll(mm);
    }
    for (int i = nres + lane; i < np; i += 64) out_res[q * np + i] = -1;
    for (int i = nmis + lane; i < np; i += 64) out_mis[q * np + i] = -1;
}

hipError_t launch_split_probes(const int32_t* probe, int64_t nq, int np, const int* resident, int nlist, unsigned long long* hits,
                               int32_t* out_resident, int32_t* out_missing, hipStream_t s)
{
    if (nq <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_split_probes, dim3((unsigned)((nq + 3) / 4)), dim3(256), 0, s, probe, nq, np, resident, nlist, hits,
                       out_resident, out_missing);
    return hipGetLastError();
}

// The gc most frequently probed lists, most frequent first, equal counts by list number: the
// lists a cache of hot clusters would keep (Section 4.4).  Every list counts the lists that
// come before it; its rank is its place in the output.  Bound by the nlist^2 comparisons: 16 threads share the counting of
// a list, and in tiles of counters that lie wholly before or behind it one comparison does (a thread for each list and
// the list number compared every time: 2048 lists 125 us a call, 9903 lists 603, 65536 lists 3986; now 9.8, 27 and 555).
__global__ __launch_bounds__(256) void k_hot_lists(const unsigned long long* hits, int nlist, int gc, int32_t* out)
{
    constexpr int kTile = 1024, kLists = 16, kShare = 16;
    static_assert(kTile % kLists == 0, "the lists of a workgroup lie in one tile");
    __shared__ unsigned long long s_h[kTile];
    const int part = threadIdx.x & (kShare - 1), l = blockIdx.x * kLists + (threadIdx.x / kShare);
    const unsigned long long mine = l < nlist ? hits[l] : 0ull;
    const int own = l / kTile * kTile;
    int rank = 0;
    for (int j0 = 0; j0 < nlist; j0 += kTile) {
        const int n = min(kTile, nlist - j0);
        __syncthreads();
        for (int t = threadIdx.x; t < n; t += 256) s_h[t] = hits[j0 + t];
        __syncthreads();
        if (j0 < own) {
#pragma unroll 8
            for (int t = part; t < kTile; t += kShare) rank += s_h[t] >= mine ? 1 : 0;
        } else if (j0 > own) {
#pragma unroll 4
            for (int t = part; t < n; t += kShare) rank += s_h[t] > mine ? 1 : 0;
        } else {
            for (int t = part; t < n; t += kShare) {
                const unsigned long long h = s_h[t];
                rank += (h > mine || (h == mine && j0 + t < l)) ? 1 : 0;
            }
        }
    }
#pragma unroll
    for (int o = kShare / 2; o > 0; o >>= 1) rank += __shfl_xor(rank, o);
    if (part == 0 && l < nlist && rank < gc) out[rank] = l;
}

hipError_t launch_hot_lists(const unsigned long long* hits, int nlist, int gc, int32_t* out, hipStream_t s)
{
    hipLaunchKernelGGL(k_hot_lists, dim3((unsigned)((nlist + 15) / 16)), dim3(256), 0, s, hits, nlist, gc, out);
    return hipGetLastError();
}

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

__device__ __forceinline__ uint16_t bf16_rne(float f)
{
    uint32_t u = __builtin_bit_cast(uint32_t, f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf16_to_f32(uint16_t b)
{
    return __builtin_bit_cast(float, ((uint32_t)b) << 16);
}

// Squared norm of every stored row, float32 accumulation of the exact stored values; used by
// the squared-L2 metric in its expanded form |q|^2 + |x|^2 - 2 q.x.  One wave per row.
__global__ __launch_bounds__(256) void k_row_norms(const void* rows, int dtype, int64_t nrows, int d, float* out)
{
    int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= nrows) return;
    int lane = threadIdx.x & 63;
    float acc = 0.f;
    if (dtype == HR_F32) {
        const float* p = (const float*)rows + row * d;
        for (int i = lane; i < d; i += 64) acc += p[i] * p[i];
    } else if (dtype == HR_F16) {
        const _Float16* p = (const _Float16*)rows + row * d;
        for (int i = lane; i < d; i += 64) { float x = (float)p[i]; acc += x * x; }
    } else {
        const uint16_t* p = (const uint16_t*)rows + row * d;
        for (int i = lane; i < d; i += 64) { float x = bf16_to_f32(p[i]); acc += x * x; }
    }
    acc = wave_sum(acc);
    if (lane == 0) out[row] = acc;
}

// What the bounds of a list's scores tell: the window (two slacks) that the high parts alone leave to a score, in deviations of the scores
// of the list's rows, whose tail the best ones are (dev: see list_spread; norm2, left2: of the longest row and of the largest rounding
// residue; what rounding leaves over of a query is about 1.4e-4 of it).  1024 queries over 16 lists, high parts and both parts (HR_F32X2), us
// a call, by the window of all lists: d = 768, 256 lists of 1024 rows of norm 1, inner product, k 10, 0.37 269 and 340, 0.71 297 and 339,
// 1.4 736 and 340, 8 2130 and 342; k 50, 0.71 422 and 415, 1.4 1463 and 415; squared distance, 0.63 293 and 352, 0.97 457 and 351; d = 1024,
// 0.82 219 and 230, 1.6 496 and 229; d = 128, 512 lists, 0.31 197 and 209, 0.58 213 and 208, 0.90 295 and 209; d = 64, 2000 queries, k 20,
// 0.31 229 and 226, 0.52 261 and 226.  A few lists are as slow as all, their queries hold up the batch: one in twenty, d = 768, 0.71 271 and
// 342, 1.4 414 and 340, d = 128, 0.58 199 and 209, 0.90 241 and 208; one list, d = 768, 1.4 285 and 341, 2.2 306 and 340, 3.8 390 and 341, k
// 50, 1.4 531 and 416; d = 128, 1.6 211 and 209.  So both parts are multiplied where a 64th of the rows (kWindowShare) is in lists whose
// window is wider than the line, 0.7 for long rows and 0.4 for short ones, which both parts take little longer for, and where one list
// is kWindowAny times as wide.
constexpr float kWindowAny = 2.2f;
__device__ __forceinline__ float score_window(float norm2, float left2, float dev, int d)      // (in units of the line)
{
    const float over = 4.1f * (sqrtf(left2) + 1.4e-4f * sqrtf(norm2)) / (d >= 512 ? 0.7f : 0.4f);
    return dev > 0.f ? over / dev : 0.f;                          // (rows that are all the same: both parts tell no more)
}

// Some list's window is too wide for the high parts alone.  (Said to the host once: a store into its memory takes 0.3 us, and one from every
// wave that finds it made k_list_bounds take 11.9 ms for 1048576 close rows of d = 768, now 1.0.)
__device__ __forceinline__ void tell_wide(const ListArgs& a, int m)
{
    if (__hip_atomic_load(&a.told[m], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0 && atomicExch(&a.told[m], 1) == 0) ((volatile int*)a.tight)[m] = 1;
}

// Whether both parts are multiplied, from the windows of all lists as they are now: at load, and where whole lists have been replaced since
// (see hr_ivf_refresh_rows): one cluster of close rows that has come and gone would leave an index with row tables at half its speed for
// good.  One workgroup: what has been said so far is taken back before it looks, and said again if a refresh on another stream has said
// so meanwhile.
__global__ __launch_bounds__(1024) void k_wide_windows(ListArgs a)
{
    __shared__ unsigned long long s_rows[2];
    __shared__ int s_any[2];
    if (threadIdx.x < 2) {
        s_rows[threadIdx.x] = 0;
        s_any[threadIdx.x] = 0;
        atomicExch(&a.told[threadIdx.x], 0);
    }
    __threadfence();
    __syncthreads();
    unsigned long long rows[2] = {0, 0};
    bool any[2] = {false, false};
    for (int64_t l = threadIdx.x; l < a.nlist; l += 1024) {
        const float norm2 = bound_value(__hip_atomic_load(&a.bound[l].norm2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        const float left2 = bound_value(__hip_atomic_load(&a.bound[l].left2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        for (int m = 0; m < 2; m++) {
            const float w = score_window(norm2, left2, m == HR_METRIC_L2 ? a.spread[l].y : a.spread[l].x, a.d);
            if (w > 1.0f) rows[m] += a.list_off[l + 1] - a.list_off[l];
            any[m] |= w > kWindowAny;
        }
    }
    for (int m = 0; m < 2; m++) {
        if (rows[m]) atomicAdd(&s_rows[m], rows[m]);
        if (any[m]) s_any[m] = 1;
    }
    __syncthreads();
    if (threadIdx.x >= 2) return;
    const int m = threadIdx.x;
    if (s_any[m] || s_rows[m] * kWindowShare > (unsigned long long)a.list_off[a.nlist]) tell_wide(a, m);
    else {
        ((volatile int*)a.tight)[m] = 0;
        __threadfence_system();
        if (__hip_atomic_load(&a.told[m], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) ((volatile int*)a.tight)[m] = 1;
    }
}

hipError_t launch_wide_windows(const ListArgs& a, hipStream_t s)
{
    hipLaunchKernelGGL(k_wide_windows, dim3(1), dim3(1024), 0, s, a);
    return hipGetLastError();
}

constexpr int kBoundWaves = 8, kPairs = 16;
// squared norms of row p and of what rounding it to binary16 leaves over (hi: its place in the table, or nullptr), four loads on their
// way together
__device__ __forceinline__ float2 row_squares(const float* p, _Float16* hi, int d, int lane)
{
    float sum = 0.f, left = 0.f;
    for (int j0 = lane; j0 < d; j0 += 256) {
        float x[4];
#pragma unroll
        for (int t = 0; t < 4; t++) x[t] = j0 + t * 64 < d ? p[j0 + t * 64] : 0.f;
#pragma unroll
        for (int t = 0; t < 4; t++) {
            const _Float16 h = (_Float16)x[t];
            const float r = x[t] - (float)h;
            if (hi && j0 + t * 64 < d) hi[j0 + t * 64] = h;
            sum += x[t] * x[t];
            left += r * r;
        }
    }
    return float2{wave_sum(sum), wave_sum(left)};
}
// their bits (NaN counts as infinite)
__device__ __forceinline__ uint32_t square_bits(float v) { return __builtin_bit_cast(uint32_t, v < __builtin_inff() ? v : __builtin_inff()); }

// How far apart the scores of the rows of list l are, in deviations for a query of norm 1, from 16 pairs of rows that are half a list from
// each other (infinite for a list of fewer than 16 rows), two for each wave.  With squared distances, of a query that is as far
// from the rows as these are from each other: sqrt(2 / d) times half the median squared distance of a pair over the norm, whatever the
// rows have in common; with the inner product, which is half of what the two norms leave of that distance, as far as the norms are as well (1.05: the
// deviation of one from the median difference of two).
__device__ __forceinline__ void list_spread(const ListArgs& a, int l)
{
    __shared__ float s_dist[kPairs], s_apart[kPairs], s_norm[kPairs];
    __shared__ float s_longest;
    __shared__ uint32_t s_most[2];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int first = a.list_off[l], half = (a.list_off[l + 1] - first) / 2, pairs = min(half, kPairs);
    if (half < kPairs / 2) {
        if (threadIdx.x == 0) a.spread[l] = float2{__builtin_inff(), __builtin_inff()};
        return;
    }
    const bool whole = l >= a.whole0 && l < a.whole1;
    // (one thread asks: other workgroups may raise it meanwhile, and the branch on it has barriers)
    if (threadIdx.x == 0) s_longest = whole ? bound_value(__hip_atomic_load(&a.bound[l].norm2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) : 0.f;
    constexpr int P = kPairs / kBoundWaves;
    const float* p[P];
    float dist[P], norm[P], other[P];
#pragma unroll
    for (int j = 0; j < P; j++) {
        p[j] = a.rows + (first + (int64_t)min(wave * P + j, pairs - 1) * half / pairs) * a.d;
        dist[j] = norm[j] = other[j] = 0.f;
    }
#pragma unroll 4
    for (int i = lane; i < a.d; i += 64)
#pragma unroll
        for (int j = 0; j < P; j++) {
            const float x = p[j][i], y = p[j][i + (size_t)half * a.d];
            dist[j] += (x - y) * (x - y);
            norm[j] += x * x;
            other[j] += y * y;
        }
#pragma unroll
    for (int j = 0; j < P; j++) {
        dist[j] = wave_add(dist[j]);
        norm[j] = sqrtf(wave_add(norm[j]));
        other[j] = sqrtf(wave_add(other[j]));
        if (lane == 63) { s_dist[wave * P + j] = dist[j]; s_apart[wave * P + j] = fabsf(norm[j] - other[j]); s_norm[wave * P + j] = norm[j]; }
    }
    __syncthreads();
    // Bounds only grow, row by row.  Where all rows of a list are new and its bound is that of rows twice as long as those met here, it
    // starts anew, from all of them.  (In whichever order the waves that see the rows one by one raise it: none is above this one.)
    if (whole) {
        float met = 0.f;
        for (int t = 0; t < kPairs; t++) met = fmaxf(met, s_norm[t]);
        if (s_longest > 4.0f * met * met) {
            if (threadIdx.x == 0) s_most[0] = s_most[1] = 0;
            __syncthreads();
            uint32_t most = 0, most_left = 0;
            for (int64_t row = first + wave; row < a.list_off[l + 1]; row += kBoundWaves) {
                const float2 v = row_squares(a.rows + row * a.d, nullptr, a.d, lane);
                most = max(most, square_bits(v.x));
                most_left = max(most_left, square_bits(v.y));
            }
            if (lane == 0) { atomicMax(&s_most[0], most); atomicMax(&s_most[1], most_left); }
            __syncthreads();
            if (threadIdx.x == 0) { atomicExch(&a.bound[l].norm2, s_most[0]); atomicExch(&a.bound[l].left2, s_most[1]); }
        }
    }
    if (threadIdx.x >= 64) return;
    // (the median ones, to all lanes; none is negative, so their bits are in order)
    auto median = [&](const float* v) __attribute__((always_inline)) {
        const uint32_t mine = lane < pairs ? __builtin_bit_cast(uint32_t, v[lane]) : ~0u;
        int rank = 0;
#pragma unroll
        for (int t = 0; t < kPairs; t++) {
            const uint32_t other = __builtin_amdgcn_readlane(mine, t);
            rank += other < mine || (other == mine && t < lane) ? 1 : 0;
        }
        const unsigned long long at = __builtin_amdgcn_ballot_w64(lane < pairs && rank == pairs / 2);     // (one lane)
        return __builtin_bit_cast(float, __builtin_amdgcn_readlane(mine, __builtin_ctzll(at)));
    };
    const float spread2 = 0.5f * median(s_dist), apart = 1.05f * median(s_apart), typical = median(s_norm);
    const float l2 = typical > 0.f ? 1.4f * spread2 / (sqrtf((float)a.d) * typical) : 0.f, ip = sqrtf(l2 * l2 + apart * apart);
    if (lane == 0) {
        a.spread[l] = float2{ip, l2};
        // (the window that these rows alone make)
        for (int m = 0; m < 2; m++)
            if (score_window(typical * typical, typical * typical * 2e-8f, m == HR_METRIC_L2 ? l2 : ip, a.d) > kWindowAny) tell_wide(a, m);
    }
}

// float32 rows: how far the scores of every list are apart (the first `blocks` workgroups, whose chain is the longest), and the squared norm of
// every row, its image in the table and the bounds of its list (the others, `each` rows a wave, one after the other, asking once per
// list for all of them).  A refresh of some 400 rows of d = 256 takes 5.8 us (6.0 without the spread, one load of a row after the other).
__global__ __launch_bounds__(kBoundWaves * 64) void k_list_bounds(ListArgs a, int each, unsigned blocks)
{
    if (blockIdx.x < blocks) {
        for (unsigned l = blockIdx.x; l < (unsigned)a.lists; l += blocks) {
            list_spread(a, a.l0 + (int)l);
            __syncthreads();
        }
        return;
    }
    const int lane = threadIdx.x & 63;
    const int64_t first = ((int64_t)(blockIdx.x - blocks) * kBoundWaves + (threadIdx.x >> 6)) * each;
    if (first >= a.nrows) return;
    _Float16* const hi = (_Float16*)a.hi;
    const int n = (int)min((int64_t)each, a.nrows - first);
    int lo = 0;                                                 // list of the row: the last one that starts at it or before
    for (int end = a.nlist; end - lo > 1;) {
        const int step = (end - lo + 63) >> 6, at = lo + lane * step;
        const int less = __builtin_popcountll(__builtin_amdgcn_ballot_w64(at < end && a.list_off[at] <= a.row0 + first));     // (at least 1)
        lo += (less - 1) * step;
        end = min(end, lo + step);
    }
    uint32_t most = 0, most_left = 0;
    // (additions to one address go one after the other: most rows are below what is known already)
    auto raise = [](uint32_t* at, uint32_t v) __attribute__((always_inline)) {
        if (v > __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(at, v);
    };
    auto report = [&]() __attribute__((always_inline)) {
        if (lane == 0) {
            raise(&a.bound[lo].norm2, most);
            raise(&a.bound[lo].left2, most_left);
            // (a list of which all rows are new: its spread may be that of the rows before)
            for (int m = 0; m < 2 && !(lo >= a.whole0 && lo < a.whole1); m++)
                if (score_window(bound_value(most), bound_value(most_left), m == HR_METRIC_L2 ? a.spread[lo].y : a.spread[lo].x, a.d) > kWindowAny) tell_wide(a, m);
        }
        most = most_left = 0;
    };
    for (int i = 0; i < n; i++) {
        const int64_t row = a.row0 + first + i;
        while (row >= a.list_off[lo + 1]) { if (most) report(); lo++; }
        const float2 v = row_squares(a.rows + row * a.d, hi ? hi + row * a.d : nullptr, a.d, lane);
        if (lane == 0) a.row_norm[row] = v.x;
        most = max(most, square_bits(v.x));
        most_left = max(most_left, square_bits(v.y));
    }
    report();
}

hipError_t launch_list_bounds(const ListArgs& a, hipStream_t s)
{
    if (a.nrows <= 0) return hipSuccess;
    // (rows of a wave: as many as the device has no waves for; 84 queries with eight lists of some 70 rows of d = 256 swapped in, 16 rows
    // a wave 335 us a batch, one 181)
    const int each = a.nrows <= 16384 ? 1 : (a.nrows <= 262144 ? 4 : 16);
    // (a launch may not have 2^32 threads or more)
    const unsigned blocks = (unsigned)std::min(a.lists, 1 << 20), rows = (unsigned)((a.nrows + (int64_t)each * kBoundWaves - 1) / (each * kBoundWaves));
    hipLaunchKernelGGL(k_list_bounds, dim3(blocks + rows), dim3(kBoundWaves * 64), 0, s, a, each, blocks);
    return hipGetLastError();
}

// Replaced bfloat16 rows: their norms and their copy in the binary16 table in one pass (k_row_norms and k_bf16_to_f16 on the
// same rows).  A value that does not fit is reported in host memory, which the caller reads once the stream is empty.
__global__ __launch_bounds__(256) void k_refresh_bf16(const uint16_t* rows, int64_t nrows, int d, float* norm, _Float16* table, volatile int* overflow)
{
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= nrows) return;
    const int lane = threadIdx.x & 63;
    const uint16_t* p = rows + row * d;
    float acc = 0.f;
    bool over = false;
    for (int i0 = lane; i0 < d; i0 += 256) {
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; j++) v[j] = i0 + j * 64 < d ? bf16_to_f32(p[i0 + j * 64]) : 0.f;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            if (i0 + j * 64 >= d) break;
            acc += v[j] * v[j];
            over |= !(fabsf(v[j]) <= 65504.0f);                       // (also for NaN)
            table[row * d + i0 + j * 64] = (_Float16)v[j];
        }
    }
    acc = wave_sum(acc);
    if (lane == 0) norm[row] = acc;
    if (over) *overflow = 1;
}

hipError_t launch_refresh_bf16(const void* rows, int64_t nrows, int d, float* norm, void* table, int* overflow, hipStream_t s)
{
    if (nrows <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_refresh_bf16, dim3((unsigned)((nrows + 3) / 4)), dim3(256), 0, s, (const uint16_t*)rows, nrows, d, norm, (_Float16*)table, overflow);
    return hipGetLastError();
}

hipError_t launch_row_norms(const void* rows, int dtype, int64_t nrows, int d, float* out, hipStream_t s)
{
    if (nrows <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_row_norms, dim3((unsigned)((nrows + 3) / 4)), dim3(256), 0, s, rows, dtype, nrows, d, out);
    return hipGetLastError();
}

// Query operands.  Coarse step and float32 storage: binary16 hi row and 2^11-scaled binary16
// lo row per query.  binary16 storage: the query rounded to binary16.  bfloat16 storage:
// bfloat16 hi and lo rows.  The squared norms are those of the operand actually multiplied,
// so that the expanded L2 form cancels consistently.  One wave per query.
// The same launch clears what a call needs cleared in its workspace (counters, histograms: zero; the per-query
// lower bounds: the key of -inf): one small launch less in front of every search.
__device__ __forceinline__ float prep_query(const PrepArgs& a, int64_t row, int lane)
{
    const int d = a.d;
    const float* p = a.q + row * d;
    float n32 = 0.f, ns = 0.f, nl = 0.f;
    // (four loads in flight: waiting for each would be twelve round trips at d = 768)
    for (int i0 = lane; i0 < d; i0 += 256) {
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; j++) v[j] = i0 + j * 64 < d ? p[i0 + j * 64] : 0.f;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int i = i0 + j * 64;
            if (i >= d) break;
            const float x = v[j];
            n32 += x * x;
            if (a.qop_coarse) {
                _Float16 h = (_Float16)x;
                const _Float16 l = (_Float16)((x - (float)h) * 2048.0f);
                a.qop_coarse[(row * 2) * d + i] = h;
                a.qop_coarse[(row * 2 + 1) * d + i] = l;
                nl += ((float)l * (1.0f / 2048.0f)) * ((float)l * (1.0f / 2048.0f));
            }
            if (a.qop_scan) {
                if (a.dtype == HR_F16) {
                    _Float16 h = (_Float16)x;
                    ((_Float16*)a.qop_scan)[row * d + i] = h;
                    ns += (float)h * (float)h;
                } else if (a.dtype == HR_BF16) {
                    uint16_t hi = bf16_rne(x);
                    uint16_t lo = bf16_rne(x - bf16_to_f32(hi));
                    ((uint16_t*)a.qop_scan)[(row * 2) * d + i] = hi;
                    ((uint16_t*)a.qop_scan)[(row * 2 + 1) * d + i] = lo;
                    float e = bf16_to_f32(hi) + bf16_to_f32(lo);
                    ns += e * e;
                }
            }
        }
    }
    n32 = wave_sum(n32);
    ns = wave_sum(ns);
    if (a.qlo) nl = wave_sum(nl);
    if (lane == 0) {
        // (a query so small that squares of parts that matter vanish has no bound; one that is beyond binary16 has no keys)
        if (a.qlo) a.qlo[row] = !(nl < __builtin_inff()) ? __builtin_nanf("") : (n32 >= 1e-18f ? sqrtf(nl) : __builtin_inff());
        if (a.qnorm_coarse) a.qnorm_coarse[row] = n32;
        if (a.qnorm_scan) a.qnorm_scan[row] = (a.dtype == HR_F32) ? n32 : ns;
    }
    return n32;
}

// what a call needs cleared, shared out over the threads of a launch
__device__ __forceinline__ void prep_clear(const PrepArgs& a)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n_zero; i += (int64_t)gridDim.x * blockDim.x) a.zero[i] = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n_neg; i += (int64_t)gridDim.x * blockDim.x) a.neg[i] = a.neg_value;
}

__global__ __launch_bounds__(256) void k_prep_queries(PrepArgs a)
{
    prep_clear(a);
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row < a.nq) prep_query(a, row, threadIdx.x & 63);
}

hipError_t launch_prep_queries(const PrepArgs& a, hipStream_t s)
{
    if (a.nq <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_prep_queries, dim3((unsigned)((a.nq + 3) / 4)), dim3(256), 0, s, a);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Grouping of the nq*nprobe (query, list) pairs by list (the cross-request grouping behind
// the variable-length cluster search interface, Section 5 of the paper).

// pair -> its position inside the list's bucket (order of arrival; results do not depend on it)
__global__ void k_bucket_count(BucketArgs a)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)a.nq * a.nprobe) return;
    int l = a.probe[i];
    const bool valid = l >= 0 && l < a.nlist;
    const bool here = valid && a.resident[l] != 0;
    // (a list whose vectors are not in place is not scanned; the probe still counts as an access)
    if (valid && !here && a.hits != nullptr) atomicAdd(&a.hits[l], 1ull);
    a.pair_entry[i] = here ? atomicAdd(&a.list_w[l], 1) : -1;
}

// The same where a list is probed by many: a workgroup counts its pairs (2048, of large batches 8192) per list in LDS
// first and asks for the places of all of a list's pairs at once.  Additions to one address go one after the other, 25 ns
// each, so the most popular list decides how long the plain kernel takes.  Searches of given lists (lists of 16 rows, k 1), plain
// and shared: 10^6 pairs of 64 lists 1820 and 682 us, of 4097 lists 792 and 737, probed as 1 / rank 1472 and 797.  The line, 16
// pairs per list, is where evenly spread probes begin to gain: 16384 pairs of 1000 lists 95 and 97, 40000 103 and 97; 40000 of
// 4097 251 and 254, 131072 298 and 293 (1 / rank: 249 and 224, 380 and 293).  kCountLists: the counters fit 64 KB of LDS.
constexpr int kCountShare = 16, kCountLists = 16384;
template <int PER>                                      // pairs per thread
__global__ __launch_bounds__(1024) void k_bucket_count_shared(BucketArgs a)
{
    extern __shared__ int s_count[];                    // [nlist] pairs of the list, then the first of their places
    const int64_t pairs = (int64_t)a.nq * a.nprobe, first = (int64_t)blockIdx.x * (PER * 1024) + threadIdx.x;
    for (int l = threadIdx.x; l < a.nlist; l += 1024) s_count[l] = 0;
    int pl[PER], pe[PER];                               // list of the pair (-1: none), place among the workgroup's pairs of it
#pragma unroll
    for (int j = 0; j < PER; j++) pl[j] = first + j * 1024 < pairs ? a.probe[first + j * 1024] : -1;
#pragma unroll
    for (int j = 0; j < PER; j++) {
        const bool valid = pl[j] >= 0 && pl[j] < a.nlist;
        const bool here = valid && a.resident[pl[j]] != 0;
        if (valid && !here && a.hits != nullptr) atomicAdd(&a.hits[pl[j]], 1ull);       // (as in k_bucket_count)
        if (!here) pl[j] = -1;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; j++) pe[j] = pl[j] >= 0 ? atomicAdd(&s_count[pl[j]], 1) : -1;
    __syncthreads();
    for (int l0 = threadIdx.x; l0 < a.nlist; l0 += 4096) {
        int c[4];
#pragma unroll
        for (int j = 0; j < 4; j++) c[j] = l0 + j * 1024 < a.nlist ? s_count[l0 + j * 1024] : 0;
#pragma unroll
        for (int j = 0; j < 4; j++)
            if (c[j] > 0) c[j] = atomicAdd(&a.list_w[l0 + j * 1024], c[j]);
#pragma unroll
        for (int j = 0; j < 4; j++)
            if (l0 + j * 1024 < a.nlist) s_count[l0 + j * 1024] = c[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; j++)
        if (first + j * 1024 < pairs) a.pair_entry[first + j * 1024] = pl[j] >= 0 ? s_count[pl[j]] + pe[j] : -1;
}

template <int PER, bool WHOLE>
__global__ __launch_bounds__(1024) void k_bucket_scan(BucketArgs a) { group_pairs<1024, PER, WHOLE>(a); }

// Pairs to their places in the buckets (the first `scatter` workgroups), and items per queue and round (one wave per list, its
// segments over the lanes): neither needs the other.
__global__ __launch_bounds__(256) void k_scatter_count(BucketArgs a, unsigned scatter)
{
    if (blockIdx.x < scatter) {
        const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
        if (i >= (int64_t)a.nq * a.nprobe) return;
        const int e = a.pair_entry[i];
        if (e < 0) return;
        a.bucket_q[a.bucket_off[a.probe[i]] + e] = (int)(i / a.nprobe);
        return;
    }
    const int l = (blockIdx.x - scatter) * 4 + (threadIdx.x >> 6);
    if (l >= a.nlist) return;
    int lane = threadIdx.x & 63;
    int w = a.list_w[l];
    int len = a.list_off[l + 1] - a.list_off[l];
    if (w <= 0 || len <= 0) return;
    int seg = a.dyn[DYN_SEG_ROWS];
    int nqt = (w + a.cw - 1) >> a.cw_log2;
    int nseg = (len + seg - 1) / seg;
    const int R = a.dyn[DYN_ROUNDS];
    for (int s = lane; s < nseg; s += 64) atomicAdd(&a.round_cnt[queue_of(l, s) * kRounds + round_of(l, s, nseg, R)], nqt);
}

// (every workgroup turns the 8 x kRounds counts into where every round starts in its queue, for itself; the
// first one also writes the queue lengths)
__global__ __launch_bounds__(256) void k_item_expand(BucketArgs a)
{
    __shared__ int s_start[8 * kRounds];
    for (int i = threadIdx.x; i < 8 * kRounds; i += 256) s_start[i] = a.round_cnt[i];
    __syncthreads();
    if (threadIdx.x < 8) {
        int run = 0;
        for (int r = 0; r < kRounds; r++) { const int c = s_start[threadIdx.x * kRounds + r]; s_start[threadIdx.x * kRounds + r] = run; run += c; }
        if (blockIdx.x == 0) a.xq_count[threadIdx.x] = min(run, a.item_cap);
    }
    __syncthreads();
    int l = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (l >= a.nlist) return;
    int lane = threadIdx.x & 63;
    int w = a.list_w[l];
    int len = a.list_off[l + 1] - a.list_off[l];
    if (w <= 0 || len <= 0) return;
    int seg = a.dyn[DYN_SEG_ROWS];
    int nqt = (w + a.cw - 1) >> a.cw_log2;
    int nseg = (len + seg - 1) / seg;
    const long long sbase = a.slot_base[l];
    const int R = a.dyn[DYN_ROUNDS];
    const int row_first = a.list_off[l], boff = a.bucket_off[l];
    for (int s = lane; s < nseg; s += 64) {
        const int x = queue_of(l, s), slot = x * kRounds + round_of(l, s, nseg, R);
        const int pos = s_start[slot] + atomicAdd(&a.round_cur[slot], nqt);
        write_items(a, x, pos, l, s, nqt, w, row_first, len, seg, boff, sbase);
    }
}

hipError_t launch_bucketing_before(const BucketArgs& a, hipStream_t s)
{
    const int64_t pairs = (int64_t)a.nq * a.nprobe;
    if (pairs >= (int64_t)kCountShare * a.nlist && a.nlist <= kCountLists) {
        if (pairs <= 131072) hipLaunchKernelGGL(k_bucket_count_shared<2>, dim3((unsigned)((pairs + 2047) / 2048)), dim3(1024), (size_t)a.nlist * 4, s, a);
        else hipLaunchKernelGGL(k_bucket_count_shared<8>, dim3((unsigned)((pairs + 8191) / 8192)), dim3(1024), (size_t)a.nlist * 4, s, a);
    } else
        hipLaunchKernelGGL(k_bucket_count, dim3((unsigned)((pairs + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_bucketing_behind(const BucketArgs& a, hipStream_t s)
{
    const unsigned gp = (unsigned)(((int64_t)a.nq * a.nprobe + 255) / 256), gl = (unsigned)((a.nlist + 3) / 4);
    hipLaunchKernelGGL(k_scatter_count, dim3(gp + gl), dim3(256), 0, s, a, gp);
    hipLaunchKernelGGL(k_item_expand, dim3(gl), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_bucketing(const BucketArgs& a, hipStream_t s)
{
    if (grouped_whole(a)) {
        hipLaunchKernelGGL((k_bucket_scan<kWholeLists / 1024, true>), dim3(1), dim3(1024), 0, s, a);
        return hipGetLastError();
    }
    hipError_t e = launch_bucketing_before(a, s);
    if (e != hipSuccess) return e;
    // (up to kWholeLists lists this rides on the seeding)
    const int per = (a.nlist + 1023) / 1024;
    if (per <= 16) hipLaunchKernelGGL((k_bucket_scan<16, false>), dim3(1), dim3(1024), 0, s, a);
    else hipLaunchKernelGGL((k_bucket_scan<0, false>), dim3(1), dim3(1024), 0, s, a);
    e = hipGetLastError();
    return e != hipSuccess ? e : launch_bucketing_behind(a, s);
}

// ------------------------------------------------------------------------------------------
// Per-query merge of the scan's partial results (the reduction step of the cluster search of
// Section 5 and the per-request merge of Section 4.4): a wave, or four, walk the slots that hold a query's
// candidates, keep the k best in LDS buffers pruned as in the scan; the first then orders the
// survivors by (key, label) and writes the output row.
// candidates buffered per wave: k <= 128 and up to 64 appended per step, with upper bounds also what is within their slack of the k-th
__host__ __device__ constexpr int merge_cap(bool bounded) { return bounded ? 384 : 256; }

// W waves share the slots of a query, 64 slots at a time in turn, each with a buffer of its own; the first takes in what
// the others kept.  Bound by a wave's chain of loads and cuts, so one wave per query is enough only where the queries
// fill the device.  Searches with one and with four (d = 64): 40 queries over 6 of 208 lists, 624000 rows, k 83, 418 and 345 us;
// 256 over 30 of 60 lists, 2 M rows, k 100, 782 and 674; 512 over 32 of 1024, k 10, 239 and 239.  The line: 1024 queries 705 and
// 584, 126 and 126, 2048 999 and 886, 142 and 150, 8192 256 and 272 (sixteen waves are slower than four).
constexpr int kMergeShare = 1024;  // most queries that get four waves each
// BOUNDED: the slots hold upper bounds; a cut keeps what is within twice the slack of the k-th, and the exact keys of what is left in
// the end, k rows and a few more, are computed by all W waves.
template <int W, bool BOUNDED>
__global__ __launch_bounds__(256) void k_merge(MergeArgs a)
{
    constexpr int NW = 4, Q = NW / W;                  // waves and queries of a workgroup
    constexpr int AT = W > 1 ? 8 : 4;                  // rows on their way together while exact keys are computed
    constexpr int CAP = merge_cap(BOUNDED), CE = CAP / 64;
    const int cap = BOUNDED && a.k <= 64 ? 256 : CAP;  // (a cut takes longer the more it looks at)
    __shared__ Cand s_buf[NW][CAP];
    __shared__ int64_t s_tie[Q][HR_K_MAX];         // labels of the last entries
    __shared__ int s_pref[Q][HR_NPROBE_MAX + 1];
    __shared__ int s_cnt[NW];
    __shared__ uint32_t s_thr[Q];
    __shared__ int s_total[Q];
    __shared__ float s_slack[Q];                    // largest slack of the probed lists
    __shared__ int s_first[NW][64];
    __shared__ size_t s_slot[NW][64];
    __shared__ int64_t s_ext_id[Q][HR_K_MAX];
    __shared__ float s_ext_score[Q][HR_K_MAX];
    __shared__ int s_ext_row[Q][HR_K_MAX];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int own = wave / W, part = wave % W;         // query of the workgroup, place among its waves
    const int64_t q = (int64_t)blockIdx.x * Q + own;
    const bool live = q < a.nq;
    if (W == 1 && !live) return;                       // (no barrier below)
    auto together = [&]() __attribute__((always_inline)) { if (W == 1) wave_sync(); else __syncthreads(); };
    int64_t* ext_id = s_ext_id[own];
    int* ext_row = s_ext_row[own];               // rows of the carried entries (-1: empty place or rows not carried)
    float* ext_score = s_ext_score[own];
    Cand* buf = s_buf[wave];
    int64_t* tie = s_tie[own];
    int* pref = s_pref[own];
    int* first = s_first[wave];
    size_t* slot_of = s_slot[wave];
    const int k = a.k;
    const int seg_rows = a.dyn[DYN_SEG_ROWS];

    // ---- how many segments (= slots) does each probed list contribute
    if (lane == 0) s_cnt[wave] = 0;
    if (part == 0 && live) {
        int run = 0;
        float slack = 0.f;
        const float qn = BOUNDED ? sqrtf(a.qnorm[q]) : 0.f, ql = BOUNDED ? a.qlo[q] : 0.f;
        for (int p0 = 0; p0 < a.nprobe; p0 += 64) {
            int p = p0 + lane;
            int ns = 0;
            if (p < a.nprobe) {
                int l = a.probe[q * a.nprobe + p];
                if (l >= 0 && l < a.nlist && a.pair_entry[q * a.nprobe + p] >= 0) {
                    int len = a.list_off[l + 1] - a.list_off[l];
                    ns = (len + seg_rows - 1) / seg_rows;
                    if (BOUNDED) slack = fmaxf(slack, scan_slack(qn, ql, a.list_bound[l], a.l2, a.split != 0, a.d));
                }
            }
            const int inc = wave_prefix_sum(ns);
            if (p < a.nprobe) pref[p + 1] = run + inc;
            run += __builtin_amdgcn_readlane(inc, 63);
        }
        if (BOUNDED) slack = wave_max(slack);
        if (lane == 0) { pref[0] = 0; s_thr[own] = 0; s_total[own] = run; s_slack[own] = slack; }
    }
    wave_sync();
    // ---- a carried result joins as one more partial result (read whole before anything of
    // this query is written: the same arrays take the merged result)
    const float qn0 = (live && a.l2 && a.qnorm) ? a.qnorm[q] : 0.f;
    if (a.carried && part == 0 && live) {
        for (int j0 = 0; j0 < k; j0 += 64) {
            const int j = j0 + lane;
            const int64_t id = j < k ? a.out_ids[(size_t)q * k + j] : -1;
            const bool have = id >= 0;
            const unsigned long long m = __builtin_amdgcn_ballot_w64(have);
            if (j < k) ext_row[j] = (have && a.io_rows) ? a.io_rows[(size_t)q * k + j] : -1;
            if (have) {
                const float sc = a.out_scores[(size_t)q * k + j];
                ext_id[j] = id;
                ext_score[j] = sc;
                buf[s_cnt[wave] + lanes_below(m)] = Cand{enc_key(key_of_score(sc, qn0, a.l2)), kCarried | (uint32_t)j};
            }
            wave_sync();
            if (lane == 0) s_cnt[wave] += __builtin_popcountll(m);
            wave_sync();
        }
    }
    together();

    // (what the scan knew in the end: k rows of the query, or its whole carried result, reach this key, so nothing below it counts;
    // from zero on, with 64 entries asked for at a time, 40 queries over 6 of 208 lists, k 83, took 343 us, now 305)
    uint32_t thr = live ? a.thr[q] : 0;
    int n = __builtin_amdgcn_readfirstlane(s_cnt[wave]);
    const int total = live ? s_total[own] : 0;
    const float slack2 = BOUNDED && live ? 2.0f * s_slack[own] : 0.f;
    auto window = [&](Cand* b, int n, uint32_t& bound, int& best) __attribute__((always_inline)) {
        if (n <= 64) return wave_window<1>(b, n, k, slack2, bound, best, lane);
        if (n <= 256) return wave_window<4>(b, n, k, slack2, bound, best, lane);
        return wave_window<CE>(b, n, k, slack2, bound, best, lane);
    };
    // a full buffer is cut to the k best (BOUNDED: and what is too close to them to tell, unless that is too much); the k-th of
    // any k candidates is a bound for all waves of the query
    auto cut = [&](Cand* b, int n) __attribute__((always_inline)) {
        uint32_t kth;
        int left = k;
        if constexpr (BOUNDED) {
            int best;
            left = window(b, n, kth, best);
            if (left > cap - 64) {
                exact_keys<8, 1>(b, left, 0, 1, a.rows_f32, a.row_norm, a.queries + (size_t)q * a.d, a.d, a.l2);
                kth = wave_select<CE>(b, left, k, a.row_ids, ext_id);
                left = k;
            }
        } else {
            kth = wave_select<4>(b, n, k, a.row_ids, ext_id);
        }
        thr = kth > thr ? kth : thr;
        if (W > 1 && lane == 0) atomicMax(&s_thr[own], kth);
        return left;
    };
    // (every W-th slot: the segments of a list lie side by side, and most of a query's entries are in those of one list)
    for (int f0 = 0; f0 < total; f0 += W * 64) {
        const int f = f0 + lane * W + part;
        int c = 0;
        size_t slot = 0;
        if (f < total) {
            {
                int lo = 0, hi = a.nprobe;        // largest p with pref[p] <= f
                while (hi - lo > 1) {
                    int mid = (lo + hi) >> 1;
                    if (pref[mid] <= f) lo = mid; else hi = mid;
                }
                int p = lo;
                int s = f - pref[p];
                int l = a.probe[q * a.nprobe + p];
                int e = a.pair_entry[q * a.nprobe + p];
                int w = a.bucket_off[l + 1] - a.bucket_off[l];
                slot = (size_t)a.slot_base[l] + (size_t)s * w + (size_t)e;
            }
            c = a.slot_cnt[slot];
        }
        // the entries of these 64 slots, 64 at a time whichever slot they sit in (a loop over the fullest slot's
        // entries would be one round trip to memory per entry: the slot of a query's own cluster holds up to k)
        const int inc = wave_prefix_sum(c);
        const int tot = __builtin_amdgcn_readlane(inc, 63);
        first[lane] = inc - c;
        slot_of[lane] = slot;
        wave_sync();
        // (256 entries are asked for together: a round trip to memory for every 64 was most of the time of a query with many)
        for (int e0 = 0; e0 < tot; e0 += 256) {
            Cand got[4];
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const int e = e0 + j * 64 + lane;
                int lo = 0, hi = 64;                  // largest lane o with first[o] <= e: the slot that holds entry e
                while (hi - lo > 1) {
                    int mid = (lo + hi) >> 1;
                    if (first[mid] <= e) lo = mid; else hi = mid;
                }
                got[j] = e < tot ? a.slot_ent[slot_of[lo] * a.slot_stride + (e - first[lo])] : Cand{0u, 0u};
            }
#pragma unroll
            for (int j = 0; j < 4; j++) {
                if (e0 + j * 64 >= tot) break;
                if (W > 1) thr = max(thr, __hip_atomic_load(&s_thr[own], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
                const Cand cd = got[j];
                bool take = e0 + j * 64 + lane < tot && cd.key >= thr;
                // a row the carried result already holds (it came from a cache of earlier results
                // and its list is scanned now) is not taken a second time
                if (take && a.io_rows && a.carried)
                    for (int t = 0; t < k; t++) take = take && ext_row[t] != (int)cd.row;
                const unsigned long long mask = __builtin_amdgcn_ballot_w64(take);
                if (mask == 0) continue;
                if (take) buf[n + lanes_below(mask)] = cd;
                n += __builtin_popcountll(mask);
                wave_sync();
                if (n > cap - 64) n = cut(buf, n);
            }
        }
        wave_sync();
    }
    wave_sync();
    if (W > 1 && n > max(k, 64)) n = cut(buf, n);      // (few are handed over as they are: a cut takes 0.5 .. 2 us)
    if (W > 1) {
        if (lane == 0) s_cnt[wave] = n;
        __syncthreads();
        if (!BOUNDED && (part != 0 || !live)) return;  // (no barrier of the workgroup below)
        thr = max(thr, s_thr[own]);
        for (int o = 1; o < W && part == 0; o++) {
            const int m = s_cnt[wave + o];
            for (int e0 = 0; e0 < m; e0 += 64) {
                const Cand cd = e0 + lane < m ? s_buf[wave + o][e0 + lane] : Cand{0u, 0u};
                const bool take = e0 + lane < m && cd.key >= thr;
                const unsigned long long mask = __builtin_amdgcn_ballot_w64(take);
                if (take) buf[n + lanes_below(mask)] = cd;
                n += __builtin_popcountll(mask);
                wave_sync();
                if (n > cap - 64) n = cut(buf, n);
            }
        }
    }
    wave_sync();
    if constexpr (BOUNDED) {
        // the k largest bounds are made exact first; of the others, only those that reach the least of these keys can matter
        int best = n;
        if (part == 0 && n > k && n > W * AT) {        // (else all in one go)
            uint32_t bound;
            n = window(buf, n, bound, best);
            if (n <= W * AT) best = n;
        }
        if (W > 1) {
            if (part == 0 && lane == 0) { s_cnt[0] = best; s_cnt[1] = n; }
            __syncthreads();
            best = s_cnt[0];
            n = s_cnt[1];
        }
        for (int from = 0;;) {
            exact_keys<AT, 4>(s_buf[wave - part] + from, best - from, part, W, a.rows_f32, a.row_norm, a.queries + (size_t)q * a.d, a.d, a.l2);
            together();
            if (best == n) break;
            if (part == 0) {
                uint32_t least = ~0u;
                for (int e0 = 0; e0 < best; e0 += 64) least = min(least, wave_min(e0 + lane < best ? buf[e0 + lane].key : ~0u));
                int m = best;
                for (int e0 = best; e0 < n; e0 += 64) {
                    const Cand cd = e0 + lane < n ? buf[e0 + lane] : Cand{0u, 0u};
                    const bool keep = e0 + lane < n && cd.key >= least;
                    const unsigned long long mask = __builtin_amdgcn_ballot_w64(keep);
                    if (keep) buf[m + lanes_below(mask)] = cd;
                    m += __builtin_popcountll(mask);
                    wave_sync();
                }
                n = m;
            }
            if (W > 1) {
                if (part == 0 && lane == 0) s_cnt[1] = n;
                __syncthreads();
                n = s_cnt[1];
            }
            from = best;
            best = n;
        }
        if (W > 1 && part != 0) return;
    }
    if (n > HR_K_MAX) { wave_select<CE>(buf, n, k, a.row_ids, ext_id); n = k; }
    wave_sync();

    // ---- final order by (key descending, label ascending), the first k of it: two entries per lane
    Cand e[2];
    int64_t id[2];
#pragma unroll
    for (int m = 0; m < 2; m++) {
        int idx = lane + 64 * m;
        e[m] = (idx < n) ? buf[idx] : Cand{0u, 0u};
        id[m] = (idx < n) ? label_of(e[m].row, a.row_ids, ext_id) : INT64_MAX;
        if (idx < n) tie[idx] = id[m];
    }
    wave_sync();
    int pos[2] = {0, 0};
#pragma unroll 8
    for (int i = 0; i < n; i++) {
        uint32_t so = buf[i].key;
        int64_t oid = tie[i];
#pragma unroll
        for (int m = 0; m < 2; m++)
            pos[m] += (so > e[m].key || (so == e[m].key && oid < id[m])) ? 1 : 0;
    }
    const float qn = (a.l2 && a.qnorm) ? a.qnorm[q] : 0.f;
#pragma unroll
    for (int m = 0; m < 2; m++) {
        int idx = lane + 64 * m;
        if (idx < n && pos[m] < k) {
            float key = dec_key(e[m].key);
            float score = a.l2 ? fmaxf(qn - key, 0.f) : key;
            if (e[m].row & kCarried) score = ext_score[e[m].row & ~kCarried];     // (as it was reported)
            size_t o = (size_t)q * k + pos[m];
            if (a.out_ids) a.out_ids[o] = id[m];
            if (a.out_scores) a.out_scores[o] = score;
            if (a.io_rows) a.io_rows[o] = (e[m].row & kCarried) ? ext_row[e[m].row & ~kCarried] : (int)e[m].row;
        }
    }
    for (int idx = n + lane; idx < k; idx += 64) {     // fewer than k candidates: pad
        size_t o = (size_t)q * k + idx;
        if (a.out_ids) a.out_ids[o] = -1;
        if (a.out_scores) a.out_scores[o] = a.l2 ? __builtin_inff() : -__builtin_inff();
        if (a.io_rows) a.io_rows[o] = -1;
    }
}

// ------------------------------------------------------------------------------------------
// Top-k of one row of keys per wave (coarse step: the nprobe best centroids of a query out of
// the nlist keys the dense scan wrote; Section 2.2: the closest clusters are the ones probed).
// Exact: radix select on the order-preserving 32-bit image of the key, one 8-bit digit per pass
// with a 256-bin histogram in LDS, then the entries above the k-th key and, of those equal to
// it, the ones with the lowest index, ordered best first (equal keys: lower index first).
struct TopkArgs {
    const float* keys;          // [nq, n] larger is better
    const float* qnorm;         // [nq] squared query norms (L2 only)
    int32_t* out_ids;           // [nq, k]
    float* out_scores;          // [nq, k] or nullptr
    int nq, n, k, l2;
    TopkSample sample;          // (computed on the host: its square root and divisions cost each wave a microsecond)
    PrepArgs prep;              // PREP: what k_prep_queries would have done
};

// PREP: the preparation of the queries rides on this launch (the dense scoring before it took the queries as they are)
template <bool PREP>
__global__ __launch_bounds__(256, 4) void k_topk_rows(TopkArgs a)
{
    constexpr int kCollect = kTopkCollect;          // entries one wave can collect in LDS
    static_assert(kCollect >= HR_NPROBE_MAX, "the best of a row must fit");
    __shared__ int s_hist[4][256];
    __shared__ Cand s_ent[4][kCollect];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int64_t q = (int64_t)blockIdx.x * 4 + wave;
    if (PREP) prep_clear(a.prep);
    if (q >= a.nq) return;
    float norm = 0.f;
    if (PREP) norm = prep_query(a.prep, q, lane);
    const float* row = a.keys + (size_t)q * a.n;
    int* hist = s_hist[wave];
    Cand* ent = s_ent[wave];
    const int k = min(a.k, a.n);

    // ---- the quick way, one pass over the row: a lower bound t0 from keys spread over the row (topk_sample says how
    // many and which of them), every key >= t0 collected in LDS, the k best of those selected there.  It is exact
    // whenever at least k and at most kCollect keys were collected (all keys >= the k-th best are then among them).
    // Too few: a lower one of the sampled keys and another pass.  Too many: the k-th best of those that did fit is a
    // bound that at least k keys reach and few others do, and another pass.  Only rows of many equal keys, or keys in
    // an order that misleads the sample twice, are left to the radix passes below, some eight times slower, and one such
    // row is what the whole launch waits for (65536 keys, k 16, 100 rows of which one collected too many: 567 us a call
    // when that row took the radix passes, 160 with another pass over it).
    bool done = false;
    {
        uint32_t t0 = 0;                            // (below every encoded key: short rows are collected whole)
        const TopkSample sm = a.sample;
        auto sample = [&](auto per, int want, const int lane) __attribute__((always_inline)) {
            constexpr int C = decltype(per)::value, S = C * 64;
            uint32_t sv[C];
#pragma unroll
            for (int j = 0; j < C; j++) sv[j] = enc_key(row[(int)(((long long)(j * 64 + lane) * a.n) / S)]);
            unsigned long long alive[C];
#pragma unroll
            for (int j = 0; j < C; j++) alive[j] = ~0ull;
            uint32_t t = 0;
            for (int b = 31, left = S; b >= 0 && left != want; b--) {
                unsigned long long ones[C];
                int c1 = 0;
#pragma unroll
                for (int j = 0; j < C; j++) {
                    ones[j] = alive[j] & __builtin_amdgcn_ballot_w64((sv[j] >> b) & 1u);
                    c1 += __builtin_popcountll(ones[j]);
                }
                if (c1 >= want) {
                    t |= 1u << b;
                    left = c1;
#pragma unroll
                    for (int j = 0; j < C; j++) alive[j] = ones[j];
                } else {
                    want -= c1;
                    left -= c1;
#pragma unroll
                    for (int j = 0; j < C; j++) alive[j] &= ~ones[j];
                }
            }
            return t;
        };
        int want = sm.want;
        bool look = sm.size > 0;                    // t0 comes from the sample (else: as it is)
        for (int tries = 0; tries < 3 && !done; tries++) {
            const int lane = lane_now();                // (what follows from it is not kept in registers from one pass to the next)
            if (look) {
                if (sm.size == 1024) t0 = sample(std::integral_constant<int, 16>{}, want, lane);
                else if (sm.size == 512) t0 = sample(std::integral_constant<int, 8>{}, want, lane);
                else t0 = sample(std::integral_constant<int, 4>{}, want, lane);
            }
            int cnt = 0;
            auto collect = [&](float key, int i, bool valid) __attribute__((always_inline)) {
                const uint32_t u = enc_key(key);
                const bool take = valid && u >= t0;
                const unsigned long long m = __builtin_amdgcn_ballot_w64(take);
                if (m == 0) return;
                const int pos = cnt + lanes_below(m);
                if (take && pos < kCollect) ent[pos] = Cand{u, (uint32_t)i};
                cnt += __builtin_popcountll(m);
            };
            // (what hides the latency of the loads is how many are in flight: 8 of 16 bytes per
            // lane when the rows allow it; the order of collection does not matter)
            if ((a.n & 3) == 0) {
                const float4* row4 = (const float4*)row;
                const int n4 = a.n >> 2;
                for (int i0 = 0; i0 < n4; i0 += 64 * 8) {
                    float4 v[8];
#pragma unroll
                    for (int j = 0; j < 8; j++) v[j] = row4[min(i0 + j * 64 + lane, n4 - 1)];
#pragma unroll
                    for (int j = 0; j < 8; j++) {
                        const int i4 = i0 + j * 64 + lane;
                        collect(v[j].x, i4 * 4, i4 < n4);
                        collect(v[j].y, i4 * 4 + 1, i4 < n4);
                        collect(v[j].z, i4 * 4 + 2, i4 < n4);
                        collect(v[j].w, i4 * 4 + 3, i4 < n4);
                    }
                }
            } else {
                for (int i0 = 0; i0 < a.n; i0 += 64 * 8) {
                    float v[8];
#pragma unroll
                    for (int j = 0; j < 8; j++) { const int i = i0 + j * 64 + lane; v[j] = row[min(i, a.n - 1)]; }
#pragma unroll
                    for (int j = 0; j < 8; j++) collect(v[j], i0 + j * 64 + lane, i0 + j * 64 + lane < a.n);
                }
            }
            wave_sync();
            if (cnt < k) {                              // (of the sampled keys as well: nothing lower to try)
                if (!look || want == sm.size) break;
                want = min(sm.size, want + want / 2 + 4);
                continue;
            }
            // (equal keys: lower index first; the select walks as many 64-entry chunks as were collected, not
            // as many as the buffer holds)
            const int held = min(cnt, kCollect);
            uint32_t kth = t0;                      // (asked for where the buffer is full alone)
            if (held > k) {
                if (held <= 256) wave_select<4>(ent, held, k, nullptr);
                else if (held <= 512) wave_select<8>(ent, held, k, nullptr);
                else kth = wave_select<kCollect / 64>(ent, held, k, nullptr);
            }
            done = cnt <= kCollect;
            if (!done && kth == t0) break;              // (too many equal keys)
            t0 = kth;
            look = false;
        }
    }

    uint32_t prefix = 0, mask = 0;
    int need = k;                                   // entries still to take among those matching the prefix
    for (int shift = 24; shift >= 0 && !done; shift -= 8) {
#pragma unroll
        for (int j = 0; j < 4; j++) hist[lane * 4 + j] = 0;
        wave_sync();
        // (8 loads in flight per lane: the row is read once per pass and nothing else hides
        // the latency of a load)
        for (int i0 = 0; i0 < a.n; i0 += 64 * 8) {
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; j++) { const int i = i0 + j * 64 + lane; v[j] = row[min(i, a.n - 1)]; }
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const uint32_t u = enc_key(v[j]);
                const bool in = i0 + j * 64 + lane < a.n && (u & mask) == prefix;
                const int dg = (u >> shift) & 255;
                // keys of one row mostly share their leading digits: the lanes whose digit is
                // that of the first counted lane are added in one go, only the others one by
                // one (64 atomic additions to one LDS word would go one after the other)
                const unsigned long long min_ = __builtin_amdgcn_ballot_w64(in);
                if (min_ == 0) continue;
                const int d0 = __builtin_amdgcn_readlane(dg, __builtin_ctzll(min_));
                const unsigned long long same = __builtin_amdgcn_ballot_w64(in && dg == d0);
                if (lane == 0) atomicAdd(&hist[d0], (int)__builtin_popcountll(same));
                if (in && dg != d0) atomicAdd(&hist[dg], 1);
            }
        }
        wave_sync();
        // lane L holds digits 255-4L .. 252-4L: the prefix sum over lanes counts from the top digit down
        int c[4], tot = 0;
#pragma unroll
        for (int j = 0; j < 4; j++) { c[j] = hist[255 - (lane * 4 + j)]; tot += c[j]; }
        const int incl = wave_prefix_sum(tot);
        const unsigned long long reach = __builtin_amdgcn_ballot_w64(incl >= need);
        const int L = __builtin_ctzll(reach);       // (need <= number of matching entries, so some lane reaches it)
        int digit = 0, above = 0;
        if (lane == L) {
            int run = incl - tot;
#pragma unroll
            for (int j = 0; j < 4; j++) {
                if (run < need && run + c[j] >= need) { digit = 255 - (lane * 4 + j); above = run; }
                run += c[j];
            }
        }
        digit = __builtin_amdgcn_readlane(digit, L);
        above = __builtin_amdgcn_readlane(above, L);
        need -= above;
        prefix |= (uint32_t)digit << shift;
        mask |= 255u << shift;
        wave_sync();
    }
    // prefix = k-th best key; `need` of the entries equal to it are taken, lowest index first
    int n_gt = 0, n_eq = 0;
    for (int i0 = 0; i0 < a.n && !done; i0 += 64 * 8) {
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; j++) { const int i = i0 + j * 64 + lane; v[j] = row[min(i, a.n - 1)]; }
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const int i = i0 + j * 64 + lane;
            const uint32_t u = enc_key(v[j]);
            const bool gt = i < a.n && u > prefix;
            const bool eq = i < a.n && u == prefix;
            const unsigned long long mg = __builtin_amdgcn_ballot_w64(gt), me = __builtin_amdgcn_ballot_w64(eq);
            if (gt) ent[n_gt + lanes_below(mg)] = Cand{u, (uint32_t)i};
            n_gt += __builtin_popcountll(mg);
            // the equal ones go to the far end, in index order, until enough are taken
            const int r = n_eq + lanes_below(me);
            if (eq && r < need) ent[k - 1 - r] = Cand{u, (uint32_t)i};
            n_eq += __builtin_popcountll(me);
        }
    }
    wave_sync();
    // order: key descending, index ascending (rank of every entry = entries ahead of it)
    const float qn = !a.l2 ? 0.f : (PREP ? norm : a.qnorm ? a.qnorm[q] : 0.f);
    auto emit = [&](auto per) __attribute__((always_inline)) {
        constexpr int PER = decltype(per)::value;       // entries per lane
        uint64_t e[PER];                                // key, then the complement of the row: the larger is ahead
        int pos[PER];
#pragma unroll
        for (int m = 0; m < PER; m++) {
            const Cand c = lane + 64 * m < k ? ent[lane + 64 * m] : Cand{0u, 0u};
            e[m] = (uint64_t)c.key << 32 | (uint32_t)~c.row;
            pos[m] = 0;
        }
        // (bound by the comparisons: one of 64 bits and one addition per pair.  Comparing key and row by themselves, three
        // comparisons and the logic between them, the 512 best of 512 keys took 91 us a call, now 32)
#pragma unroll 8
        for (int i = 0; i < k; i++) {
            const Cand c = ent[i];
            const uint64_t o = (uint64_t)c.key << 32 | (uint32_t)~c.row;
#pragma unroll
            for (int m = 0; m < PER; m++) pos[m] += o > e[m] ? 1 : 0;
        }
#pragma unroll
        for (int m = 0; m < PER; m++) {
            if (lane + 64 * m < k) {
                const float key = dec_key((uint32_t)(e[m] >> 32));
                const size_t o = (size_t)q * a.k + pos[m];
                a.out_ids[o] = (int32_t)~(uint32_t)e[m];
                if (a.out_scores) a.out_scores[o] = a.l2 ? fmaxf(qn - key, 0.f) : key;
            }
        }
    };
    if (k <= 64) emit(std::integral_constant<int, 1>{});
    else if (k <= 128) emit(std::integral_constant<int, 2>{});
    else if (k <= 256) emit(std::integral_constant<int, 4>{});
    else emit(std::integral_constant<int, HR_NPROBE_MAX / 64>{});
    for (int idx = k + lane; idx < a.k; idx += 64) {       // fewer than k rows: pad
        const size_t o = (size_t)q * a.k + idx;
        a.out_ids[o] = -1;
        if (a.out_scores) a.out_scores[o] = a.l2 ? __builtin_inff() : -__builtin_inff();
    }
}

hipError_t launch_topk_rows(const float* keys, const float* qnorm, int32_t* out_ids, float* out_scores,
                            int64_t nq, int n, int k, int l2, const PrepArgs* prep, hipStream_t s)
{
    if (nq <= 0) return hipSuccess;
    TopkArgs a{keys, qnorm, out_ids, out_scores, (int)nq, n, k, l2, topk_sample(n, k < n ? k : n), prep ? *prep : PrepArgs{}};
    if (prep) hipLaunchKernelGGL(k_topk_rows<true>, dim3((unsigned)((nq + 3) / 4)), dim3(256), 0, s, a);
    else hipLaunchKernelGGL(k_topk_rows<false>, dim3((unsigned)((nq + 3) / 4)), dim3(256), 0, s, a);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Reuse of the previous retrieval of a request (Section 4.3 of the paper: consecutive queries
// v, v' of a request are close, so the results of v' tend to lie among a larger top-k of v, in
// the clusters H_v that held v's results, and in clusters probed both times).

// List of every given row (binary search in the row offsets); -1 for rows outside the index.
__global__ void k_lists_of_rows(const int32_t* rows, int64_t n, const int* list_off, int nlist, int32_t* out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int r = rows[i];
    int res = -1;
    if (r >= 0 && r < list_off[nlist]) {
        int lo = 0, hi = nlist;                 // largest l with list_off[l] <= r (lists may be empty)
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (list_off[mid] <= r) lo = mid; else hi = mid;
        }
        res = lo;
    }
    out[i] = res;
}

hipError_t launch_lists_of_rows(const int32_t* rows, int64_t n, const int* list_off, int nlist, int32_t* out, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_lists_of_rows, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, rows, n, list_off, nlist, out);
    return hipGetLastError();
}

// Search order of the new probe lists C' of every query: first those in H_v, then those of
// the previous probe lists C that are not in H_v, then the rest, each group in its given
// (rank) order; absent entries (-1) last.  One wave per query.
struct ReorderArgs {
    const int32_t* probe;       // [nq, np]
    const int32_t* prev;        // [nq, pp] or nullptr
    const int32_t* hot;         // [nq, nh] or nullptr
    int32_t* out;               // [nq, np]
    int nq, np, pp, nh;
};

__global__ __launch_bounds__(256) void k_reorder_probes(ReorderArgs a)
{
    __shared__ int s_prev[4][HR_NPROBE_MAX];
    __shared__ int s_hot[4][HR_K_MAX];
    __shared__ unsigned char s_cls[4][HR_NPROBE_MAX];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t q = (int64_t)blockIdx.x * 4 + wave;
    if (q >= a.nq) return;
    int* prev = s_prev[wave];
    int* hot = s_hot[wave];
    unsigned char* cls = s_cls[wave];
    for (int i = lane; i < a.pp; i += 64) prev[i] = a.prev[q * a.pp + i];
    for (int i = lane; i < a.nh; i += 64) hot[i] = a.hot[q * a.nh + i];
    wave_sync();
    int count[4] = {0, 0, 0, 0};                // entries per group (whole wave holds the same values)
    for (int i0 = 0; i0 < a.np; i0 += 64) {
        const int i = i0 + lane;
        int c = 4;                              // (past the end)
        if (i < a.np) {
            const int l = a.probe[q * a.np + i];
            c = 3;
            if (l >= 0) {
                c = 2;
                for (int t = 0; t < a.pp; t++) if (prev[t] == l) { c = 1; break; }
                for (int t = 0; t < a.nh; t++) if (hot[t] == l) { c = 0; break; }
            }
            cls[i] = (unsigned char)c;
        }
#pragma unroll
        for (int g = 0; g < 4; g++) count[g] += __builtin_popcountll(__builtin_amdgcn_ballot_w64(c == g));
    }
    wave_sync();
    int base[4] = {0, count[0], count[0] + count[1], count[0] + count[1] + count[2]};
    for (int i0 = 0; i0 < a.np; i0 += 64) {
        const int i = i0 + lane;
        const int c = i < a.np ? cls[i] : 4;
#pragma unroll
        for (int g = 0; g < 4; g++) {
            const unsigned long long m = __builtin_amdgcn_ballot_w64(c == g);
            if (c == g) a.out[q * a.np + base[g] + lanes_below(m)] = a.probe[q * a.np + i];
            base[g] += __builtin_popcountll(m);
        }
    }
}

hipError_t launch_reorder_probes(const int32_t* probe, int np, const int32_t* prev, int pp, const int32_t* hot, int nh,
                                 int64_t nq, int32_t* out, hipStream_t s)
{
    if (nq <= 0) return hipSuccess;
    ReorderArgs a{probe, prev, hot, out, (int)nq, np, prev ? pp : 0, hot ? nh : 0};
    hipLaunchKernelGGL(k_reorder_probes, dim3((unsigned)((nq + 3) / 4)), dim3(256), 0, s, a);
    return hipGetLastError();
}

// The local cache of a request: the rows a previous retrieval returned (a larger top-k of v)
// are scored against the new query v' and the k best become the starting result of v's
// successor.  One workgroup of up to four waves per query, 16 lanes per row, four rows per wave at a time; bound by
// round trips to memory, so a lane asks for four steps of its row together and the waves share the rows (one wave per query, each
// step waited for, and serial comparisons at the end: 512 queries, d = 768, 20 rows each 47.9 us a call, now 14.5; 128 rows 338 and
// 56; 4000 queries, 20 rows, 129 and 35); the query is rounded
// as the scan's operand is (binary16 for binary16 lists, bfloat16 hi + lo for bfloat16 lists),
// products and sums in float32.  Rows listed twice count once; -1 = no row.
struct RescoreArgs {
    const float* q;             // [nq, d]
    const void* rows;           // stored rows
    const float* row_norm;      // [N]
    const int64_t* row_ids;     // labels or nullptr
    const int32_t* cand;        // [nq, m] row numbers
    int64_t* out_ids;           // [nq, k]
    float* out_scores;          // [nq, k]
    int32_t* out_rows;          // [nq, k]
    int64_t nrows;
    int nq, m, k, d, dtype, l2;
};

__device__ __forceinline__ float rounded_like_operand(float x, int dtype)
{
    if (dtype == HR_F16) return (float)(_Float16)x;
    if (dtype == HR_BF16) {
        const uint16_t hi = bf16_rne(x);
        return bf16_to_f32(hi) + bf16_to_f32(bf16_rne(x - bf16_to_f32(hi)));
    }
    return x;
}

__global__ __launch_bounds__(256) void k_rescore(RescoreArgs a)
{
    __shared__ __align__(16) float s_q[1024];            // the query, rounded (the longest supported)
    __shared__ float key[HR_K_MAX];
    __shared__ int row[HR_K_MAX];
    __shared__ int64_t lab[HR_K_MAX];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, threads = blockDim.x;
    const int64_t q = blockIdx.x;
    const float* qp = a.q + q * a.d;
    const int sub = lane & 15, grp = lane >> 4;
    for (int i = threadIdx.x; i < a.d; i += threads) s_q[i] = rounded_like_operand(qp[i], a.dtype);
    __syncthreads();
    for (int j0 = wave * 4; j0 < a.m; j0 += threads / 16) {
        const int j = j0 + grp;
        int r = j < a.m ? a.cand[q * a.m + j] : -1;
        if (r < 0 || r >= a.nrows) r = -1;
        float dot = 0.f;
        if (r >= 0) {
            // 8 elements per lane and step, the 16 lanes of a group side by side
#pragma unroll 4
            for (int e = sub * 8; e < a.d; e += 128) {
                float x[8];
                if (a.dtype == HR_F32) {
                    const float4* p = (const float4*)((const float*)a.rows + (size_t)r * a.d + e);
                    const float4 u = p[0], v = p[1];
                    x[0] = u.x; x[1] = u.y; x[2] = u.z; x[3] = u.w; x[4] = v.x; x[5] = v.y; x[6] = v.z; x[7] = v.w;
                } else {
                    const uint4 u = *(const uint4*)((const uint16_t*)a.rows + (size_t)r * a.d + e);
                    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
                    for (int t = 0; t < 4; t++) {
                        if (a.dtype == HR_F16) {
                            x[2 * t] = (float)__builtin_bit_cast(_Float16, (uint16_t)(w[t] & 0xffffu));
                            x[2 * t + 1] = (float)__builtin_bit_cast(_Float16, (uint16_t)(w[t] >> 16));
                        } else {
                            x[2 * t] = bf16_to_f32((uint16_t)(w[t] & 0xffffu));
                            x[2 * t + 1] = bf16_to_f32((uint16_t)(w[t] >> 16));
                        }
                    }
                }
#pragma unroll
                for (int t = 0; t < 8; t++) dot = __builtin_fmaf(x[t], s_q[e + t], dot);
            }
        }
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) dot += __shfl_xor(dot, o);
        if (sub == 0 && j < a.m) {
            row[j] = r;
            key[j] = r < 0 ? 0.f : (a.l2 ? 2.0f * dot - a.row_norm[r] : dot);
            lab[j] = r < 0 ? INT64_MAX : (a.row_ids ? a.row_ids[r] : (int64_t)r);
        }
    }
    __syncthreads();
    float qn = 0.f;
    for (int i = lane; i < a.d; i += 64) qn += s_q[i] * s_q[i];
    qn = wave_sum(qn);
    // rows listed twice: the first copy counts, the others become "no row"
    constexpr int PER = HR_K_MAX / 64;               // rows of a thread, where the workgroup is one wave
    bool dup[PER];
#pragma unroll
    for (int c = 0; c < PER; c++) {
        const int j = c * threads + threadIdx.x;
        dup[c] = false;
        if (j < a.m) {
            const int r = row[j];
#pragma unroll 8
            for (int u = 0; u < j; u++) dup[c] |= row[u] == r;
        }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < PER; c++)
        if (dup[c]) row[c * threads + threadIdx.x] = -1;
    __syncthreads();
    // rank among the valid rows: better key first, equal keys by label
    int nvalid = 0;
    for (int j0 = 0; j0 < a.m; j0 += 64) nvalid += __builtin_popcountll(__builtin_amdgcn_ballot_w64(j0 + lane < a.m && row[j0 + lane] >= 0));
    for (int j = threadIdx.x; j < a.m; j += threads) {
        const int r = row[j];
        if (r < 0) continue;
        const float kj = key[j];
        const int64_t lj = lab[j];
        int rank = 0;
#pragma unroll 8
        for (int t = 0; t < a.m; t++) rank += (row[t] >= 0 && (key[t] > kj || (key[t] == kj && lab[t] < lj))) ? 1 : 0;
        if (rank < a.k) {
            const size_t o = (size_t)q * a.k + rank;
            a.out_ids[o] = lj;
            a.out_scores[o] = a.l2 ? fmaxf(qn - kj, 0.f) : kj;
            a.out_rows[o] = r;
        }
    }
    for (int i = nvalid + threadIdx.x; i < a.k; i += threads) {      // fewer than k rows: the other places stay empty
        const size_t o = (size_t)q * a.k + i;
        a.out_ids[o] = -1;
        a.out_scores[o] = a.l2 ? __builtin_inff() : -__builtin_inff();
        a.out_rows[o] = -1;
    }
}

hipError_t launch_rescore(const float* q, int64_t nq, int d, int dtype, const void* rows, const float* row_norm,
                          const int64_t* row_ids, int64_t nrows, const int32_t* cand, int m, int k, int l2,
                          int64_t* out_ids, float* out_scores, int32_t* out_rows, hipStream_t s)
{
    if (nq <= 0) return hipSuccess;
    RescoreArgs a{q, rows, row_norm, row_ids, cand, out_ids, out_scores, out_rows, nrows, (int)nq, m, k, d, dtype, l2};
    // (a wave takes four rows at a time; where the queries alone fill the device, one wave each)
    const int waves = nq > 1024 ? 1 : std::min(4, (m + 3) / 4);
    hipLaunchKernelGGL(k_rescore, dim3((unsigned)nq), dim3(64 * waves), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_merge(const MergeArgs& a, hipStream_t s)
{
    if (a.nq <= 0) return hipSuccess;
    auto launch = [&](auto bounded) {
        constexpr bool B = decltype(bounded)::value;
        if (a.nq <= kMergeShare) hipLaunchKernelGGL((k_merge<4, B>), dim3((unsigned)a.nq), dim3(256), 0, s, a);
        else hipLaunchKernelGGL((k_merge<1, B>), dim3((unsigned)((a.nq + 3) / 4)), dim3(256), 0, s, a);
        return hipGetLastError();
    };
    return a.rows_f32 != nullptr ? launch(std::true_type{}) : launch(std::false_type{});
}

}  // namespace hr
