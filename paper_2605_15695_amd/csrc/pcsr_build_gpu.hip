// PCSR generation on the GPU (Section 4.2, "PCSR Generation"): the same two steps as the
// host builder - vectorised blocking into V x 1 nonzero vectors, then the optional
// workload split - but with the CSR arrays already in device memory, so nothing crosses
// PCIe except a handful of scalars.  The arrays it produces are bit-identical to the
// host builder's.
//
// What bounds it: the arrays are read and written a few times at memory speed (16 M nonzeros:
// 20-60 us a pass), so passes, launches (about 5 us each with the gaps) and waits of the host
// (12-15 us each) are what is counted here.  No pass gives one thread a whole row: rows of
// power-law graphs are up to a thousand times longer than the average, and the one thread
// that had the longest took 5.3 ms to validate a graph whose average row takes microseconds.
#include <hip/hip_runtime.h>
#include <hipcub/hipcub.hpp>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>

#include "../../include/pcsr.h"
#include "pcsr_build_gpu.h"
#include "pcsr_gpu_util.h"
#include "pcsr_sort_gpu.h"

namespace pcsr {
namespace {

// ---- validation and row statistics

// What the host learns from one pass over the row pointer and one over the columns.
struct Checked {
    int bad;         // a row pointer or column out of range, a column that does not ascend
    int first, last; // rowptr[0], rowptr[n_rows]
    int longest;     // longest row
    int nonempty;
    unsigned long long common[2]; // cluster_probe's sums
};

// Monotone row pointer inside [0, nnz], row statistics, the row at the start of each slice.  Few, large
// workgroups: each ends in atomics to one line of memory (1,048,576 rows: 9 us, 27 with 1024 workgroups of 256).
constexpr int kRowThreads = 1024, kRowBlocks = 128;
__global__ void __launch_bounds__(kRowThreads) check_rows_kernel(int64_t n_rows, int64_t nnz, const int32_t *rowptr,
                                                                 int32_t *slices, Checked *out)
{
    int bad = 0, longest = 0, nonempty = 0;
    constexpr int N = 4; // rows in flight
    const int64_t stride = (int64_t)gridDim.x * kRowThreads;
    for (int64_t i0 = (int64_t)blockIdx.x * kRowThreads + threadIdx.x; i0 < n_rows; i0 += N * stride) {
        int32_t s[N], e[N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const int64_t i = i0 + k * stride;
            s[k] = i < n_rows ? rowptr[i] : 0;
            e[k] = i < n_rows ? rowptr[i + 1] : 0;
        }
#pragma unroll
        for (int k = 0; k < N; ++k) {
            if (s[k] < 0 || s[k] > e[k] || e[k] > nnz) {
                bad = 1;
            } else if (e[k] > s[k]) {
                ++nonempty;
                longest = e[k] - s[k] > longest ? e[k] - s[k] : longest;
                note_slices(slices, i0 + k * stride, s[k], e[k]);
            }
        }
    }
    typedef hipcub::BlockReduce<int, kRowThreads> Reduce;
    __shared__ typename Reduce::TempStorage t2, t3, t4;
    const int b = Reduce(t2).Sum(bad);
    const int n = Reduce(t3).Sum(nonempty);
    const int l = Reduce(t4).Reduce(longest, hipcub::Max());
    if (threadIdx.x == 0) {
        if (b) out->bad = 1;
        if (n) atomicAdd(&out->nonempty, n);
        if (l) atomicMax(&out->longest, l);
        if (blockIdx.x == 0) {
            out->first = rowptr[0];
            out->last = rowptr[n_rows];
        }
    }
}

// Columns in range and ascending inside every row (check); the arrays copied (pcol, with V = 1; vals null: the columns alone).  One pass
// for both: 16 M nonzeros 49 us (5.2 TB/s), where a check that met every row start on its own took 77 and the copies 45.
__global__ void __launch_bounds__(kThreads) check_copy_kernel(int64_t n_rows, int64_t n_cols, int64_t nnz,
                                                              const int32_t *rowptr, const int32_t *colidx,
                                                              const float *vals, const int32_t *slices, int check,
                                                              int32_t *pcol, float *pval, Checked *out)
{
    __shared__ int32_t starts_lds[kSlice];
    __shared__ int32_t last_col[kThreads + 1];
    const int tid = threadIdx.x;
    const int64_t t0 = (int64_t)blockIdx.x * kSlice, t1 = t0 + kSlice < nnz ? t0 + kSlice : nnz;
    const int64_t t = t0 + tid * kPerThread;
    int4u c = {0, 0, 0, 0};
    if (t + kPerThread <= t1) {
        c = *reinterpret_cast<const int4u *>(colidx + t);
        if (pcol) *reinterpret_cast<int4u *>(pcol + t) = c;
        if (pcol && vals) *reinterpret_cast<float4u *>(pval + t) = *reinterpret_cast<const float4u *>(vals + t);
    } else {
        for (int k = 0; k < kPerThread && t + k < t1; ++k) {
            c[k] = colidx[t + k];
            if (pcol) pcol[t + k] = c[k];
            if (pcol && vals) pval[t + k] = vals[t + k];
        }
    }
    if (!check) return; // the whole grid
    last_col[tid + 1] = c[kPerThread - 1];
    if (tid == 0) last_col[0] = t0 > 0 ? colidx[t0 - 1] : -1;
    RowStarts rows{starts_lds};
    rows.find(rowptr, n_rows, slices[blockIdx.x], t0, t1);
    bool bad = false;
    int32_t before = last_col[tid];
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
        if (t + k < t1) {
            bad |= c[k] < 0 || c[k] >= n_cols;
            if (c[k] <= before && t + k > 0) { // fine where a row starts
                bad |= !rows.starts_row(rowptr, n_rows, t0, t + k);
            }
        }
        before = c[k];
    }
    if (__syncthreads_or(bad) && tid == 0) out->bad = 1;
}

// number of entries of colidx[b, e) smaller than c
__device__ __forceinline__ int64_t count_below(const int32_t *colidx, int64_t b, int64_t e, int32_t c)
{
    int64_t lo = b, hi = e;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (colidx[mid] < c)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo - b;
}

// ---- V = 2.  The vectors of panel p are the sorted union of the columns of rows 2p ("even")
// and 2p+1 ("odd"); an element's place in the union follows from two counts: the elements of
// its own row before it, and those of the other row that are smaller and not already counted
// (columns present in both rows are counted with the even row).

// whether nonzero t of row r is an odd row's column that the even row of its panel has too
__device__ __forceinline__ bool shared_column(const int32_t *rowptr, const int32_t *colidx, int64_t r, int64_t t)
{
    if (!(r & 1)) return false;
    const int64_t a0 = rowptr[r - 1], a1 = rowptr[r];
    const int32_t c = colidx[t];
    const int64_t k = count_below(colidx, a0, a1, c);
    return a0 + k < a1 && colidx[a0 + k] == c;
}

// shared[t] = 1 for such a nonzero, else 0; shared[nnz] = 0 (scanned together with the rest)
__global__ void __launch_bounds__(kThreads) union_shared_kernel(int64_t n_rows, int64_t nnz, const int32_t *rowptr,
                                                                const int32_t *colidx, int32_t *shared)
{
    __shared__ RowSlice slice;
    const int64_t t0 = (int64_t)blockIdx.x * kSlice, t1 = t0 + kSlice < nnz ? t0 + kSlice : nnz;
    if (t0 < nnz) slice.find(rowptr, n_rows, t0, t1);
    for (int64_t t = t0 + threadIdx.x; t < t1; t += kThreads)
        shared[t] = shared_column(rowptr, colidx, slice.row(rowptr, n_rows, t), t) ? 1 : 0;
    if (nnz >= t0 && nnz < t0 + kSlice && threadIdx.x == 0) shared[nnz] = 0;
}

// vectors per panel: both rows' nonzeros minus the columns they share; cnt[P] = 0
__global__ void union_count_kernel(int64_t P, int64_t n_rows, const int32_t *rowptr, const int32_t *shared_scan,
                                   int32_t *cnt)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p > P) return;
    if (p == P) {
        cnt[P] = 0; // scanned together with the panels: prow[P] becomes the total
        return;
    }
    const int64_t r0 = 2 * p;
    const int64_t a0 = rowptr[r0], a1 = rowptr[r0 + 1];
    const int64_t b1 = (r0 + 1 < n_rows) ? rowptr[r0 + 2] : a1;
    cnt[p] = (int32_t)((b1 - a0) - (shared_scan[b1] - shared_scan[a1]));
}

// every nonzero writes its vector (ascending column, +0.0f padding); a column that both
// rows hold is written by the even row's nonzero
__global__ void __launch_bounds__(kThreads) union_fill_kernel(int64_t n_rows, int64_t nnz, const int32_t *rowptr,
                                                              const int32_t *colidx, const float *vals,
                                                              const int32_t *shared_scan, const int32_t *prow,
                                                              int32_t *out_col, float *out_val)
{
    __shared__ RowSlice slice;
    const int64_t t0 = (int64_t)blockIdx.x * kSlice, t1 = t0 + kSlice < nnz ? t0 + kSlice : nnz;
    slice.find(rowptr, n_rows, t0, t1);
    for (int64_t t = t0 + threadIdx.x; t < t1; t += kThreads) {
        const int64_t r = slice.row(rowptr, n_rows, t);
        const int64_t p = r >> 1;
        const int32_t c = colidx[t];
        const int64_t a0 = rowptr[2 * p], a1 = rowptr[2 * p + 1];
        const int64_t b1 = (2 * p + 1 < n_rows) ? rowptr[2 * p + 2] : a1;
        if (!(r & 1)) {
            const int64_t k = count_below(colidx, a1, b1, c);           // odd-row columns below c
            const int64_t both = shared_scan[a1 + k] - shared_scan[a1]; // of which also in this row
            const int64_t o = prow[p] + (t - a0) + (k - both);
            const bool twin = a1 + k < b1 && colidx[a1 + k] == c;
            if (o >= prow[p + 1]) continue; // only with rows that are not sorted (validation skipped)
            out_col[o] = c;
            out_val[2 * o] = vals[t];
            out_val[2 * o + 1] = twin ? vals[a1 + k] : 0.0f;
        } else if (shared_scan[t + 1] == shared_scan[t]) { // not shared
            const int64_t k = count_below(colidx, a0, a1, c); // even-row columns below c
            const int64_t o = prow[p] + k + ((t - a1) - (shared_scan[t] - shared_scan[a1]));
            if (o >= prow[p + 1]) continue;
            out_col[o] = c;
            out_val[2 * o] = 0.0f;
            out_val[2 * o + 1] = vals[t];
        }
    }
}

// non-empty panels and longest panel (V = 2; check_rows_kernel has them for V = 1)
__global__ void __launch_bounds__(kThreads) panel_stats_kernel(int64_t P, const int32_t *prow, Checked *out)
{
    int n = 0, l = 0;
    for (int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x; p < P; p += (int64_t)gridDim.x * kThreads) {
        const int len = prow[p + 1] - prow[p];
        n += len > 0;
        l = len > l ? len : l;
    }
    typedef hipcub::BlockReduce<int, kThreads> Reduce;
    __shared__ typename Reduce::TempStorage t1, t2;
    const int ne = Reduce(t1).Sum(n);
    const int mx = Reduce(t2).Reduce(l, hipcub::Max());
    if (threadIdx.x == 0) {
        if (ne) atomicAdd(&out->nonempty, ne);
        if (mx) atomicMax(&out->longest, mx);
    }
}

// ---- workload split

// What a panel adds to the four running counts of the split; one scan does for all of them.
struct SplitCount {
    int items;  // max(1, ceil(len / SG))
    int split;  // 1 if that is more than one
    int slots;  // its items then
    int longp;  // 1 if it has more than kLongPanelSlots items
};
struct SplitSum {
    __device__ SplitCount operator()(const SplitCount &a, const SplitCount &b) const
    {
        return {a.items + b.items, a.split + b.split, a.slots + b.slots, a.longp + b.longp};
    }
};
__device__ __forceinline__ SplitCount split_count(const int32_t *prow, int64_t p, int64_t P, int32_t sg)
{
    if (p >= P) return {0, 0, 0, 0};
    const int len = prow[p + 1] - prow[p];
    int it = (int)(((long)len + sg - 1) / sg);
    it = it > 1 ? it : 1;
    return {it, it > 1, it > 1 ? it : 0, it > kLongPanelSlots};
}
constexpr int kSplitPanels = 1024; // panels per workgroup

__global__ void __launch_bounds__(kThreads) split_sums_kernel(int64_t P, const int32_t *prow, int32_t sg,
                                                              SplitCount *sums)
{
    typedef hipcub::BlockReduce<SplitCount, kThreads> Reduce;
    __shared__ typename Reduce::TempStorage tmp;
    SplitCount c = {0, 0, 0, 0};
    for (int i = 0; i < kSplitPanels / kThreads; ++i)
        c = SplitSum()(c, split_count(prow, (int64_t)blockIdx.x * kSplitPanels + i * kThreads + threadIdx.x, P, sg));
    c = Reduce(tmp).Reduce(c, SplitSum());
    if (threadIdx.x == 0) sums[blockIdx.x] = c;
}

// exclusive scan in place by one workgroup; the total goes to sums[n]
__global__ void __launch_bounds__(1024) split_scan_kernel(int n, SplitCount *sums)
{
    typedef hipcub::BlockScan<SplitCount, 1024> Scan;
    __shared__ typename Scan::TempStorage tmp;
    SplitCount before = {0, 0, 0, 0};
    for (int base = 0; base < n; base += 1024) {
        const int i = base + threadIdx.x;
        SplitCount c = {0, 0, 0, 0}, ex, total;
        if (i < n) c = sums[i];
        Scan(tmp).ExclusiveScan(c, ex, SplitCount{0, 0, 0, 0}, SplitSum(), total);
        if (i < n) sums[i] = SplitSum()(before, ex);
        before = SplitSum()(before, total);
        __syncthreads();
    }
    if (threadIdx.x == 0) sums[n] = before;
}

struct SplitOut {
    int32_t *rowptr, *trow, *item_slot;        // per item (rowptr one more)
    int32_t *split_panels, *split_slot, *long_list;
    int32_t *long_key, *long_item, *short_item; // column-ordered schedule (may be null)
};

// Rewritten rowPtr, TRow, workspace slots, the tables of split panels and, for the schedule, the
// lists of items of split panels (with their first column) and of the others.  A workgroup
// numbers its 1024 panels, then its threads take the items one by one: a panel of a
// thousand items is no longer one thread's.
__global__ void __launch_bounds__(kThreads) split_fill_kernel(int64_t P, const int32_t *prow, const int32_t *colidx,
                                                              int32_t sg, const SplitCount *sums, SplitOut o)
{
    constexpr int N = kSplitPanels / kThreads;
    typedef hipcub::BlockScan<SplitCount, kThreads> Scan;
    __shared__ typename Scan::TempStorage tmp;
    __shared__ int32_t first[kSplitPanels + 1]; // first item of each panel
    __shared__ int32_t slot[kSplitPanels];      // slots handed out before it
    const int64_t p0 = (int64_t)blockIdx.x * kSplitPanels;
    const SplitCount base = sums[blockIdx.x];
    SplitCount mine[N], ex, own = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < N; ++i) {
        mine[i] = split_count(prow, p0 + threadIdx.x * N + i, P, sg);
        own = SplitSum()(own, mine[i]);
    }
    Scan(tmp).ExclusiveScan(own, ex, SplitCount{0, 0, 0, 0}, SplitSum());
    ex = SplitSum()(base, ex);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int k = threadIdx.x * N + i;
        const int64_t p = p0 + k;
        first[k] = ex.items;
        slot[k] = ex.slots;
        if (mine[i].split) {
            o.split_panels[ex.split] = (int32_t)p;
            o.split_slot[ex.split] = ex.slots;
            if (mine[i].longp) o.long_list[ex.longp] = ex.split;
        }
        ex = SplitSum()(ex, mine[i]);
        if (p == P - 1) {
            o.rowptr[ex.items] = prow[P];
            o.split_slot[ex.split] = ex.slots;
        }
    }
    if (threadIdx.x == kThreads - 1) first[kSplitPanels] = ex.items;
    __syncthreads();
    const int panels = (int)(P - p0 < kSplitPanels ? P - p0 : kSplitPanels);
    for (int it = first[0] + threadIdx.x; it < first[panels]; it += kThreads) {
        int lo = 0, hi = panels; // first[lo] <= it
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (first[mid] <= it)
                lo = mid;
            else
                hi = mid;
        }
        const int k = it - first[lo];
        const bool split = first[lo + 1] - first[lo] > 1;
        const int32_t s = prow[p0 + lo] + k * sg;
        const int sl = split ? slot[lo] + k : -1;
        o.rowptr[it] = s;
        o.trow[it] = (int32_t)(p0 + lo);
        o.item_slot[it] = sl;
        if (o.long_key) {
            if (split) {
                o.long_key[sl] = colidx[s]; // items of split panels are never empty
                o.long_item[sl] = it;
            } else {
                o.short_item[it - slot[lo]] = it;
            }
        }
    }
}

// ---- column-ordered schedule (same result as the host builder's schedule_by_column)

// work of an item in a list: its vectors + 8
__device__ __forceinline__ int sched_weight(const int32_t *list, const int32_t *rowptr, int64_t i, int64_t n)
{
    return i < n ? rowptr[list[i] + 1] - rowptr[list[i]] + 8 : 0;
}
constexpr int kSchedChunk = 1024;

// work of each chunk of 1024 entries: chunks of the long list first, then of the short one
__global__ void __launch_bounds__(kThreads) sched_sums_kernel(int64_t nl, const int32_t *longs, int64_t ns,
                                                              const int32_t *shorts, const int32_t *rowptr,
                                                              long long *sums)
{
    const int64_t cl = (nl + kSchedChunk - 1) / kSchedChunk;
    const bool is_long = blockIdx.x < cl;
    const int32_t *list = is_long ? longs : shorts;
    const int64_t n = is_long ? nl : ns, c = is_long ? blockIdx.x : blockIdx.x - cl;
    long long w = 0;
    for (int i = threadIdx.x; i < kSchedChunk; i += kThreads) w += sched_weight(list, rowptr, c * kSchedChunk + i, n);
    typedef hipcub::BlockReduce<long long, kThreads> Reduce;
    __shared__ typename Reduce::TempStorage tmp;
    const long long t = Reduce(tmp).Sum(w);
    if (threadIdx.x == 0) sums[blockIdx.x] = t;
}

// exclusive scan in place of one list's chunk sums, total behind them; workgroup 0 the long
// list's (n0 sums at sums[0]), workgroup 1 the short one's (n1 at sums[n0], written from
// scan[n0 + 1])
__global__ void __launch_bounds__(1024) sched_scan_kernel(int n0, int n1, const long long *sums, long long *scan)
{
    typedef hipcub::BlockScan<long long, 1024> Scan;
    __shared__ typename Scan::TempStorage tmp;
    const int n = blockIdx.x ? n1 : n0;
    const long long *in = blockIdx.x ? sums + n0 : sums;
    long long *out = blockIdx.x ? scan + n0 + 1 : scan;
    long long before = 0;
    for (int base = 0; base < n; base += 1024) {
        const int i = base + threadIdx.x;
        long long c = i < n ? in[i] : 0, ex, total;
        Scan(tmp).ExclusiveSum(c, ex, total);
        if (i < n) out[i] = before + ex;
        before += total;
        __syncthreads();
    }
    if (threadIdx.x == 0) out[n] = before;
}

// 8 contiguous equal-work slices of both lists: workgroup x < 9 finds boundary x of the long
// list, 9 + x that of the short one: the first index whose work before it reaches x eighths.
__global__ void __launch_bounds__(kThreads) sched_bounds_kernel(int64_t nl, const int32_t *longs, int64_t ns,
                                                                const int32_t *shorts, const int32_t *rowptr,
                                                                const long long *scan, int32_t *bounds)
{
    const bool is_long = blockIdx.x < 9;
    const int x = is_long ? blockIdx.x : blockIdx.x - 9;
    const int64_t n = is_long ? nl : ns, cl = (nl + kSchedChunk - 1) / kSchedChunk;
    const int64_t chunks = (n + kSchedChunk - 1) / kSchedChunk;
    const int32_t *list = is_long ? longs : shorts;
    const long long *cum = is_long ? scan : scan + cl + 1;
    const long long target = cum[chunks] * x / 8;
    if (x == 0 || x == 8 || target <= 0) {
        if (threadIdx.x == 0) bounds[blockIdx.x] = (int32_t)(x == 8 ? n : 0);
        return;
    }
    int64_t lo = 0, hi = chunks; // the last chunk with less work before it than the target
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (cum[mid] < target)
            lo = mid;
        else
            hi = mid;
    }
    constexpr int N = kSchedChunk / kThreads;
    typedef hipcub::BlockScan<long long, kThreads> Scan;
    __shared__ typename Scan::TempStorage tmp;
    __shared__ int found;
    if (threadIdx.x == 0) found = kSchedChunk;
    long long w[N], own = 0, ex;
#pragma unroll
    for (int i = 0; i < N; ++i) own += w[i] = sched_weight(list, rowptr, lo * kSchedChunk + threadIdx.x * N + i, n);
    Scan(tmp).ExclusiveSum(own, ex);
    __syncthreads();
    long long at = cum[lo] + ex;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        at += w[i]; // work before entry threadIdx.x*N + i + 1
        if (at >= target) {
            atomicMin(&found, threadIdx.x * N + i + 1);
            break;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int64_t i = lo * kSchedChunk + found;
        bounds[blockIdx.x] = (int32_t)(i < n ? i : n);
    }
}

// one record per launch position: XCD x runs its slice of the column-ordered list, then
// its slice of the others.  bounds: lb[9], sb[9].
__global__ void __launch_bounds__(kThreads) sched_emit_kernel(int64_t nl, const int32_t *longs, int64_t ns,
                                                              const int32_t *shorts, const int32_t *bounds,
                                                              const int32_t *rowptr, const int32_t *trow,
                                                              const int32_t *item_slot, int4 *sched)
{
    const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (t >= nl + ns) return;
    const bool is_short = t >= nl;
    const int64_t i = is_short ? t - nl : t;
    const int32_t *lb = bounds, *sb = bounds + 9;
    const int32_t *mine = is_short ? sb : lb;
    int x = 0;
    while (x < 7 && i >= mine[x + 1]) ++x;
    const int64_t pos = is_short ? (int64_t)lb[x + 1] + i : (int64_t)sb[x] + i;
    const int it = is_short ? shorts[i] : longs[i];
    const int start = rowptr[it];
    sched[pos] = make_int4(start, rowptr[it + 1] - start, trow[it], item_slot[it]);
}

// 8 contiguous item ranges of equal work (vectors + 8 per item); same rule as the host builder
__global__ void xcd_bounds_kernel(int32_t M, const int32_t *rowptr, int32_t *xb)
{
    const int x = threadIdx.x;
    if (x > 8) return;
    if (x == 0) {
        xb[0] = 0;
        return;
    }
    if (x == 8) {
        xb[8] = M;
        return;
    }
    const long total = (long)rowptr[M] + 8L * M;
    const long target = total * x / 8;
    long lo = 0, hi = M;
    while (lo < hi) {
        const long mid = (lo + hi) / 2;
        if ((long)rowptr[mid] + 8L * mid >= target)
            hi = mid;
        else
            lo = mid + 1;
    }
    xb[x] = (int32_t)lo;
}

// ---- Table 3 features on the GPU: one pass over the panels of two rows, one over the rows
constexpr unsigned kPanelBlocks = 512, kDevBlocks = 512;
constexpr int kPanelThreads = 1024;

struct RowPart { // per workgroup of the pass over the panels
    long long n_hat, nonempty2, shared, near;
    double bw_sum, bw_max;
    int d_max, pad;
};
struct DevPart { // per workgroup of the second
    double ss, ss_hat;
    long long M1, M2;
};
struct FeatAcc {
    long long n_hat, nnz2, nonempty2, M1, M2, near;
    double bw_sum, bw_max, ss, ss_hat;
    int d_max, pad;
};
struct RowPartSum {
    __device__ RowPart operator()(const RowPart &a, const RowPart &b) const
    {
        return {a.n_hat + b.n_hat, a.nonempty2 + b.nonempty2, a.shared + b.shared, a.near + b.near, a.bw_sum + b.bw_sum,
                a.bw_max > b.bw_max ? a.bw_max : b.bw_max, a.d_max > b.d_max ? a.d_max : b.d_max, 0};
    }
};
struct DevPartSum {
    __device__ DevPart operator()(const DevPart &a, const DevPart &b) const
    {
        return {a.ss + b.ss, a.ss_hat + b.ss_hat, a.M1 + b.M1, a.M2 + b.M2};
    }
};

// Panels that eight lanes would take too long for, in units of 64 nonzeros of the shorter row, and the columns found in
// both rows of them.
constexpr int kFarBlocks = 1024;
constexpr int kMostPanels = 1024; // of a workgroup
__device__ __forceinline__ bool far_panel(int32_t shorter, int32_t longer) { return shorter > 64 || (shorter > 8 && longer > 256); }
struct FarList {
    int32_t n, pad;
    unsigned long long shared;
};

// Statistics of the rows and, per panel, how many columns both of its rows have (shared).  Eight lanes take a panel:
// the nonzeros of its shorter row are looked up in the longer one (whose few lines of memory are in the vector cache
// by the second step), and four of the lanes find the ends of the two rows' stretches within 512 columns of the
// diagonal.  What bounds it is the chain of loads per panel, so as many panels as fit are in flight.  With
// features_far_kernel 56 us for 250,000 rows of 48 and 105 for R-MAT scale 20 (16 M nonzeros), where passes over
// the nonzeros and over the rows took 100 and 125.
__global__ void __launch_bounds__(kPanelThreads) features_panels_kernel(int64_t n_rows, int64_t nnz, const int32_t *rowptr,
                                                                        const int32_t *colidx, int32_t *shared, int64_t room,
                                                                        int2 *units, FarList *far, RowPart *parts)
{
    constexpr int G = 8;
    __shared__ int32_t held[kMostPanels];
    __shared__ int n_held;
    if (threadIdx.x == 0) n_held = 0;
    __syncthreads();
    const int l = threadIdx.x % G;
    const int64_t P = (n_rows + 1) / 2, step = (int64_t)gridDim.x * (kPanelThreads / G);
    RowPart a = {0, 0, 0, 0, 0.0, 0.0, 0, 0};
    for (int64_t p = (int64_t)blockIdx.x * (kPanelThreads / G) + threadIdx.x / G; p < P; p += step) {
        const int64_t r = 2 * p;
        const int32_t s = rowptr[r], m = rowptr[r + 1], e = r + 1 < n_rows ? rowptr[r + 2] : m;
        if (s < 0 || s > m || m > e || e > nnz) continue; // (no CSR)
        // lanes 0 and 1: first and last column of the even row, 2 and 3: of the odd one
        const int32_t row0 = l & 2 ? m : s, row1 = l & 2 ? e : m;
        const int32_t own_col = l < 4 && row1 > row0 ? colidx[l & 1 ? row1 - 1 : row0] : 0;
        // the shorter row
        const bool odd = e - m <= m - s;
        const int32_t own0 = odd ? m : s, own1 = odd ? e : m, in0 = odd ? s : m, in1 = odd ? m : e;
        const bool near_by = !far_panel(own1 - own0, in1 - in0);
        int both = 0;
        int32_t near_lo = row0, near_hi = l < 4 ? row1 : row0; // (lanes 0 to 3, beside the first of the look-ups)
        const int64_t bound = r + (l >> 1) + (l & 1 ? 512 : -511);
        for (int32_t t = own0 + l;; t += G) {
            const bool more = near_by && t < own1;
            const int32_t c = more ? colidx[t] : 0;
            int32_t lo = in0, hi = more ? in1 : in0;
            while (lo < hi || near_lo < near_hi) {
                narrow(colidx, c, lo, hi);
                narrow(colidx, bound, near_lo, near_hi);
            }
            if (!more) break;
            both += lo < in1 && colidx[lo] == c;
        }
        if (!near_by && l == 0) held[atomicAdd(&n_held, 1)] = (int32_t)p; // (the grid leaves it kMostPanels at most)
#pragma unroll
        for (int k = 1; k < G; k <<= 1) both += __shfl_xor(both, k);
        const int32_t other_col = __shfl_xor(own_col, 1), other_lo = __shfl_xor(near_lo, 1);
        if (l == 0) {
            shared[p] = both;
            a.shared += both;
            a.nonempty2 += e > s;
        }
        if ((l == 0 || l == 2) && row1 > row0) {
            ++a.n_hat;
            a.d_max = row1 - row0 > a.d_max ? row1 - row0 : a.d_max;
            const double bw = (double)other_col - (double)own_col;
            a.bw_sum += bw;
            a.bw_max = bw > a.bw_max ? bw : a.bw_max;
            a.near += other_lo - near_lo;
        }
    }
    typedef hipcub::BlockReduce<RowPart, kPanelThreads> Reduce;
    __shared__ typename Reduce::TempStorage tmp;
    a = Reduce(tmp).Reduce(a, RowPartSum());
    if (threadIdx.x == 0) parts[blockIdx.x] = a;
    __syncthreads();
    // the panels set aside: one atomic for all of them
    const int n_mine = n_held;
    if (n_mine == 0) return; // uniform
    typedef hipcub::BlockScan<int, kPanelThreads> Scan;
    __shared__ typename Scan::TempStorage scan;
    __shared__ int base;
    int n = 0, at, total;
    if ((int)threadIdx.x < n_mine) {
        const int64_t r = 2 * (int64_t)held[threadIdx.x];
        const int32_t s = rowptr[r], m = rowptr[r + 1], e = rowptr[r + 2];
        n = ((e - m <= m - s ? e - m : m - s) + 63) / 64;
    }
    Scan(scan).ExclusiveSum(n, at, total);
    if (threadIdx.x == 0) base = atomicAdd(&far->n, total);
    __syncthreads();
    for (int k = 0; k < n; ++k)
        if (base + at + k < room) units[base + at + k] = make_int2(held[threadIdx.x], k);
}

// The listed units, a wavefront each.
__global__ void __launch_bounds__(kThreads) features_far_kernel(int64_t n_rows, const int32_t *rowptr, const int32_t *colidx,
                                                                int64_t room, const int2 *units, FarList *far,
                                                                int32_t *shared)
{
    const int64_t n = far->n < room ? far->n : room;
    const int lane = threadIdx.x & 63;
    int found = 0;
    for (int64_t u = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6); u < n; u += kFarBlocks * (kThreads / 64)) {
        const int2 unit = units[u];
        const int64_t r = 2 * (int64_t)unit.x;
        const int32_t s = rowptr[r], m = rowptr[r + 1], e = rowptr[r + 2]; // both rows have nonzeros
        const bool odd = e - m <= m - s;
        const int32_t own0 = odd ? m : s, own1 = odd ? e : m, in0 = odd ? s : m, in1 = odd ? m : e;
        const int64_t t = own0 + 64 * (int64_t)unit.y + lane;
        bool both = false;
        if (t < own1) {
            const int32_t c = colidx[t];
            int32_t lo = in0, hi = in1;
            while (lo < hi) narrow(colidx, c, lo, hi);
            both = lo < in1 && colidx[lo] == c;
        }
        const int c = __popcll(__ballot(both));
        if (lane == 0 && c) atomicAdd(&shared[unit.x], c);
        found += c;
    }
    if (lane == 0 && found) atomicAdd(&far->shared, (unsigned long long)found);
}

__device__ __forceinline__ long panel_len(const int32_t *rowptr, const int32_t *shared, int64_t p, int64_t n_rows)
{
    const int64_t end = 2 * p + 2 < n_rows ? 2 * p + 2 : n_rows;
    return (long)rowptr[end] - rowptr[2 * p] - shared[p];
}

// sums over the panels, the same in every workgroup that asks (result in thread 0)
__device__ RowPart sum_row_parts(const RowPart *parts, int n, const FarList *far)
{
    typedef hipcub::BlockReduce<RowPart, kThreads> Reduce;
    __shared__ typename Reduce::TempStorage tmp;
    RowPart a = {0, 0, 0, 0, 0.0, 0.0, 0, 0};
    for (int i = threadIdx.x; i < n; i += kThreads) a = RowPartSum()(a, parts[i]);
    a = Reduce(tmp).Reduce(a, RowPartSum());
    a.shared += (long long)far->shared;
    return a;
}

// Eq. (3)
__device__ __forceinline__ long eq3_sg(long v, long nonempty, long omega)
{
    return (v == 0 || nonempty == 0) ? omega : ((v + nonempty * omega - 1) / (nonempty * omega)) * omega;
}

// squared deviations of the degrees and the item counts under Eq. (3)'s SG
__global__ void __launch_bounds__(kThreads) features_deviation_kernel(int64_t n_rows, int64_t nnz, const int32_t *rowptr,
                                                                      const int32_t *shared, const RowPart *parts,
                                                                      int n_parts, const FarList *far, int32_t omega,
                                                                      DevPart *out)
{
    __shared__ double s_d, s_d_hat;
    __shared__ long s_sg1, s_sg2;
    const RowPart r = sum_row_parts(parts, n_parts, far);
    if (threadIdx.x == 0) {
        s_d = (double)nnz / (double)n_rows;
        s_d_hat = r.n_hat ? (double)nnz / (double)r.n_hat : 0.0;
        s_sg1 = eq3_sg(nnz, r.n_hat, omega);
        s_sg2 = eq3_sg(nnz - r.shared, r.nonempty2, omega);
    }
    __syncthreads();
    const double d = s_d, d_hat = s_d_hat;
    const long sg1 = s_sg1, sg2 = s_sg2;
    DevPart a = {0.0, 0.0, 0, 0};
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n_rows; i += (int64_t)gridDim.x * kThreads) {
        const int l = rowptr[i + 1] - rowptr[i];
        a.ss += ((double)l - d) * ((double)l - d);
        if (l > 0) a.ss_hat += ((double)l - d_hat) * ((double)l - d_hat);
        const long m1 = (l + sg1 - 1) / sg1;
        a.M1 += m1 < 1 ? 1 : m1;
        if ((i & 1) == 0) {
            const long m2 = (panel_len(rowptr, shared, i >> 1, n_rows) + sg2 - 1) / sg2;
            a.M2 += m2 < 1 ? 1 : m2;
        }
    }
    typedef hipcub::BlockReduce<DevPart, kThreads> Reduce;
    __shared__ typename Reduce::TempStorage tmp;
    a = Reduce(tmp).Reduce(a, DevPartSum());
    if (threadIdx.x == 0) out[blockIdx.x] = a;
}

__global__ void __launch_bounds__(kThreads) features_final_kernel(int64_t nnz, const RowPart *parts, int n_parts,
                                                                  const FarList *far, const DevPart *devs, int n_devs,
                                                                  FeatAcc *out)
{
    const RowPart r = sum_row_parts(parts, n_parts, far);
    typedef hipcub::BlockReduce<DevPart, kThreads> ReduceD;
    __shared__ typename ReduceD::TempStorage t1;
    DevPart d = {0.0, 0.0, 0, 0};
    for (int i = threadIdx.x; i < n_devs; i += kThreads) d = DevPartSum()(d, devs[i]);
    d = ReduceD(t1).Reduce(d, DevPartSum());
    if (threadIdx.x == 0)
        *out = {r.n_hat, nnz - r.shared, r.nonempty2, d.M1, d.M2, r.near, r.bw_sum, r.bw_max, d.ss, d.ss_hat, r.d_max, 0};
}

// Where the rows' columns pass into each band but the first: how many lie below the start of each of kColumnBands equal parts of
// the columns.  Counted, 16 lanes a row, as that reads the columns once and in order (300,000 rows of 134: 80 us, most of it the
// table; a search for each start takes 290); and the ends ascend and cover the row whatever order its columns have.
__global__ void __launch_bounds__(kThreads) bands_kernel(int64_t n_rows, int64_t n_cols, const int32_t *rowptr, const int32_t *colidx,
                                                         int32_t *bands)
{
    constexpr int kLanes = 16, kEnds = kColumnBands - 1;
    static_assert(kEnds <= kLanes);
    const int lane = threadIdx.x % kLanes;
    int32_t start[kEnds];
#pragma unroll
    for (int b = 0; b < kEnds; ++b) start[b] = (int32_t)((n_cols * (b + 1) + kColumnBands - 1) / kColumnBands);
    for (int64_t row = ((int64_t)blockIdx.x * kThreads + threadIdx.x) / kLanes; row < n_rows;
         row += (int64_t)gridDim.x * (kThreads / kLanes)) {
        const int32_t head = rowptr[row], tail = rowptr[row + 1];
        int32_t below[kEnds] = {};
        for (int64_t t = (int64_t)head + lane; t < tail; t += kLanes) {
            const int32_t c = colidx[t];
#pragma unroll
            for (int b = 0; b < kEnds; ++b) below[b] += c < start[b];
        }
        int32_t mine = 0;
#pragma unroll
        for (int b = 0; b < kEnds; ++b) {
#pragma unroll
            for (int step = 1; step < kLanes; step *= 2) below[b] += __shfl_xor(below[b], step);
            if (lane == b) mine = below[b];
        }
        if (lane < kEnds) bands[lane * n_rows + row] = head + mine;
    }
}

__global__ void __launch_bounds__(64) deliver_kernel(unsigned *to, const unsigned *from, int words, unsigned *flag, unsigned seq)
{
    for (int i = threadIdx.x; i < words; i += 64) to[i] = from[i];
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(flag, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

hipError_t exclusive_scan(const int32_t *in, int32_t *out, int64_t n, Scratch &sc)
{
    size_t bytes = 0;
    hipError_t e = hipcub::DeviceScan::ExclusiveSum(nullptr, bytes, in, out, (int)n, setup_stream());
    if (e != hipSuccess) return e;
    void *tmp = nullptr;
    e = sc.alloc(&tmp, bytes);
    if (e != hipSuccess) return e;
    return hipcub::DeviceScan::ExclusiveSum(tmp, bytes, in, out, (int)n, setup_stream());
}

// The check of the CSR, and its columns and values copied to pcol / pval where these are given.
int check_device(int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t *d_rowptr, const int32_t *d_colidx,
                 const float *d_vals, bool validate, bool probe, int32_t *pcol, float *pval, Scratch &sc, Checked **d_out,
                 Checked *h, int *hip_err)
{
    Checked *d = nullptr;
    int32_t *slices = nullptr;
    const int64_t n_slices = (nnz + kSlice - 1) / kSlice;
    HIP_TRY(sc.alloc((void **)&d, sizeof(Checked)));
    HIP_TRY(sc.alloc((void **)&slices, sizeof(int32_t) * (n_slices + 1)));
    HIP_TRY(hipMemsetAsync(d, 0, sizeof(Checked), setup_stream()));
    const int64_t row_blocks = (n_rows + kRowThreads - 1) / kRowThreads;
    hipLaunchKernelGGL(check_rows_kernel, dim3((unsigned)(row_blocks < 1 ? 1 : (row_blocks > kRowBlocks ? kRowBlocks : row_blocks))),
                       dim3(kRowThreads), 0, setup_stream(), n_rows, nnz, d_rowptr, slices, d);
    HIP_TRY(hipGetLastError());
    if (nnz > 0 && n_rows > 0 && (validate || pcol)) {
        hipLaunchKernelGGL(check_copy_kernel, dim3((unsigned)n_slices), dim3(kThreads), 0, setup_stream(), n_rows, n_cols, nnz, d_rowptr,
                           d_colidx, d_vals, slices, validate ? 1 : 0, pcol, pval, d);
        HIP_TRY(hipGetLastError());
    }
    if (probe) HIP_TRY(cluster_probe(n_rows, nnz, d_rowptr, d_colidx, d->common));
    HIP_TRY(setup_copy(h, d, sizeof(Checked), hipMemcpyDeviceToHost));
    *d_out = d;
    if (h->first != 0 || h->last != nnz) return PCSR_E_BAD_CSR;
    if (validate && h->bad) return PCSR_E_BAD_CSR;
    return PCSR_OK;
}

} // namespace

hipError_t deliver(void *to, const void *from, int words, unsigned *flag, unsigned seq, hipStream_t stream)
{
    hipLaunchKernelGGL(deliver_kernel, dim3(1), dim3(64), 0, stream, static_cast<unsigned *>(to),
                       static_cast<const unsigned *>(from), words, flag, seq);
    return hipGetLastError();
}

int validate_device(int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t *d_rowptr, const int32_t *d_colidx,
                    int *hip_err)
{
    Scratch sc;
    Checked *d = nullptr, h;
    return check_device(n_rows, n_cols, nnz, d_rowptr, d_colidx, nullptr, true, false, nullptr, nullptr, sc, &d, &h,
                        hip_err);
}

namespace {
struct LabelsGuard { // what cluster_rows made, given back on scope exit
    int32_t *p = nullptr;
    ~LabelsGuard()
    {
        if (!p) return;
        (void)setup_wait();
        pool_free(p);
    }
};
} // namespace

int build_device(int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t *d_rowptr,
                 const int32_t *d_colidx, const float *d_vals, int32_t V, int32_t S, int32_t SG,
                 int32_t omega, bool validate, bool column_order, bool clusters, bool windows, bool bands, const RowStats *known, Late *late,
                 DeviceBuild *out, int *hip_err)
{
    if (V != 1 && V != 2) return PCSR_E_UNSUPPORTED;
    if (omega == 0) omega = 64;
    Scratch sc;
    const int64_t P = (n_rows + V - 1) / V;

    // ---- vectorised blocking
    int32_t *prow = nullptr, *pcol = nullptr;
    const int32_t *panels = d_rowptr; // row pointer of the panels
    float *pval = nullptr;
    int64_t nnz_v = nnz;
    if (V == 1) { // the arrays as they are
        HIP_TRY(sc.alloc((void **)&pcol, sizeof(int32_t) * (nnz + 1)));
        HIP_TRY(sc.alloc((void **)&pval, sizeof(float) * (nnz + 1)));
    }
    Checked *d_check = nullptr, check = {};
    clusters = clusters && V == 1 && n_rows == n_cols && nnz > 0;
    int rc = PCSR_OK;
    if (known && !clusters) {
        check.longest = (int)known->longest;
        check.nonempty = (int)known->nonempty;
        HIP_TRY(sc.alloc((void **)&d_check, sizeof(Checked)));
        if (pcol && nnz > 0)
            HIP_TRY(hipMemcpyAsync(pcol, d_colidx, sizeof(int32_t) * nnz, hipMemcpyDeviceToDevice, setup_stream()));
        if (pval && !late && nnz > 0)
            HIP_TRY(hipMemcpyAsync(pval, d_vals, sizeof(float) * nnz, hipMemcpyDeviceToDevice, setup_stream()));
    } else {
        rc = check_device(n_rows, n_cols, nnz, d_rowptr, d_colidx, late ? nullptr : d_vals, validate, clusters, pcol, pval, sc,
                          &d_check, &check, hip_err);
        if (rc != PCSR_OK) return rc;
    }
    LabelsGuard labels;
    double label_size = 0.0;
    if (clusters && cluster_probe_says(check.common, n_rows)) {
        rc = cluster_rows(n_rows, d_rowptr, d_colidx, &labels.p, &label_size, hip_err);
        if (rc != PCSR_OK && rc != PCSR_E_OOM) return rc; // without the memory for it: the order asked for otherwise
        out->dropped |= rc == PCSR_E_OOM;
        if (labels.p) {
            S = 1;
            SG = kClusterItem;
            column_order = true;
            out->clustered = true;
        }
    }
    // Communities of over kRowsMost rows lie in several blocks, and from twice that on fewer than half of the vectors are
    // inside theirs: then not even tried (250,000 rows in communities of 1000: 0.2 ms for nothing).
    if (windows && labels.p && check.longest <= kClusterItem && label_size <= 1.5 * kRowsMost) {
        if (late) HIP_TRY(late->wait());
        rc = cluster_windows(n_rows, nnz, d_rowptr, d_colidx, d_vals, labels.p, out, hip_err);
        if (rc != PCSR_OK && rc != PCSR_E_OOM) return rc; // without the memory for them: the order alone
        out->dropped |= rc == PCSR_E_OOM;
    }
    if (V == 1) {
        if (!S) {
            HIP_TRY(sc.alloc((void **)&prow, sizeof(int32_t) * (P + 1)));
            HIP_TRY(hipMemcpyAsync(prow, d_rowptr, sizeof(int32_t) * (n_rows + 1), hipMemcpyDeviceToDevice, setup_stream()));
            panels = prow;
        }
    } else {
        if (nnz + 1 > 0x7fffffffLL) return PCSR_E_TOO_LARGE; // the scan below counts in int32
        int32_t *cnt = nullptr, *shared = nullptr, *shared_scan = nullptr;
        HIP_TRY(sc.alloc((void **)&prow, sizeof(int32_t) * (P + 1)));
        panels = prow;
        HIP_TRY(sc.alloc((void **)&cnt, sizeof(int32_t) * (P + 1)));
        HIP_TRY(sc.alloc((void **)&shared, sizeof(int32_t) * (nnz + 1)));
        HIP_TRY(sc.alloc((void **)&shared_scan, sizeof(int32_t) * (nnz + 1)));
        const unsigned slices = (unsigned)((nnz + 1 + kSlice - 1) / kSlice);
        hipLaunchKernelGGL(union_shared_kernel, dim3(slices), dim3(kThreads), 0, setup_stream(), n_rows, nnz, d_rowptr, d_colidx,
                           shared);
        HIP_TRY(hipGetLastError());
        HIP_TRY(exclusive_scan(shared, shared_scan, nnz + 1, sc));
        hipLaunchKernelGGL(union_count_kernel, dim3(blocks_for(P + 1)), dim3(kThreads), 0, setup_stream(), P, n_rows,
                           d_rowptr, shared_scan, cnt);
        HIP_TRY(hipGetLastError());
        HIP_TRY(exclusive_scan(cnt, prow, P + 1, sc));
        HIP_TRY(hipMemsetAsync(d_check, 0, sizeof(Checked), setup_stream()));
        hipLaunchKernelGGL(panel_stats_kernel, dim3(strided_blocks(P, 1024)), dim3(kThreads), 0, setup_stream(), P, prow, d_check);
        HIP_TRY(hipGetLastError());
        int32_t total = 0;
        HIP_TRY(setup_copy(&total, prow + P, sizeof(int32_t), hipMemcpyDeviceToHost));
        HIP_TRY(setup_copy(&check, d_check, sizeof(Checked), hipMemcpyDeviceToHost));
        nnz_v = total;
        HIP_TRY(sc.alloc((void **)&pcol, sizeof(int32_t) * (nnz_v + 1)));
        HIP_TRY(sc.alloc((void **)&pval, sizeof(float) * (2 * nnz_v + 1)));
        if (late) HIP_TRY(late->wait());
        if (nnz > 0) {
            hipLaunchKernelGGL(union_fill_kernel, dim3((unsigned)((nnz + kSlice - 1) / kSlice)), dim3(kThreads), 0, setup_stream(),
                               n_rows, nnz, d_rowptr, d_colidx, d_vals, shared_scan, prow, pcol, pval);
            HIP_TRY(hipGetLastError());
        }
    }

    // ---- Eq. (3) from the panel lengths
    int64_t sg = SG;
    if (sg <= 0) {
        const int64_t nonempty = check.nonempty;
        sg = (nnz_v == 0 || nonempty == 0) ? omega : ((nnz_v + nonempty * omega - 1) / (nonempty * omega)) * omega;
    }
    if (sg >= (int64_t(1) << 31)) return PCSR_E_TOO_LARGE;

    out->P = P;
    out->nnz_v = nnz_v;
    out->S = S;
    out->SG = (int32_t)sg;
    int32_t *d_bounds = nullptr;
    HIP_TRY(sc.alloc((void **)&d_bounds, 27 * sizeof(int32_t)));

    if (!S) {
        out->M = P;
        out->max_item_len = check.longest;
        hipLaunchKernelGGL(xcd_bounds_kernel, dim3(1), dim3(64), 0, setup_stream(), (int32_t)P, prow, d_bounds);
        HIP_TRY(hipGetLastError());
        HIP_TRY(setup_copy(out->xcd_bounds, d_bounds, 9 * sizeof(int32_t), hipMemcpyDeviceToHost));
    } else {
        if (P + nnz_v / sg >= (int64_t(1) << 31) - 2) return PCSR_E_TOO_LARGE;
        const int64_t chunks = (P + kSplitPanels - 1) / kSplitPanels;
        SplitCount *sums = nullptr, total = {0, 0, 0, 0};
        HIP_TRY(sc.alloc((void **)&sums, sizeof(SplitCount) * (chunks + 1)));
        if (P > 0) {
            hipLaunchKernelGGL(split_sums_kernel, dim3((unsigned)chunks), dim3(kThreads), 0, setup_stream(), P, panels, (int32_t)sg,
                               sums);
            HIP_TRY(hipGetLastError());
            hipLaunchKernelGGL(split_scan_kernel, dim3(1), dim3(1024), 0, setup_stream(), (int)chunks, sums);
            HIP_TRY(hipGetLastError());
            HIP_TRY(setup_copy(&total, sums + chunks, sizeof(total), hipMemcpyDeviceToHost));
        }
        const int64_t M = total.items, n_long = total.slots, n_short = M - n_long;
        SplitOut o = {};
        HIP_TRY(sc.alloc((void **)&o.rowptr, sizeof(int32_t) * (M + 1)));
        HIP_TRY(sc.alloc((void **)&o.trow, sizeof(int32_t) * (M + 1)));
        HIP_TRY(sc.alloc((void **)&o.item_slot, sizeof(int32_t) * (M + 1)));
        HIP_TRY(sc.alloc((void **)&o.split_panels, sizeof(int32_t) * (total.split + 1)));
        HIP_TRY(sc.alloc((void **)&o.split_slot, sizeof(int32_t) * (total.split + 1)));
        if (total.longp) HIP_TRY(sc.alloc((void **)&o.long_list, sizeof(int32_t) * total.longp));
        if (column_order) {
            HIP_TRY(sc.alloc((void **)&o.long_key, sizeof(int32_t) * (n_long + 1)));
            HIP_TRY(sc.alloc((void **)&o.long_item, sizeof(int32_t) * (n_long + 1)));
            HIP_TRY(sc.alloc((void **)&o.short_item, sizeof(int32_t) * (n_short + 1)));
        }
        if (P > 0) {
            hipLaunchKernelGGL(split_fill_kernel, dim3((unsigned)chunks), dim3(kThreads), 0, setup_stream(), P, panels, pcol,
                               (int32_t)sg, sums, o);
            HIP_TRY(hipGetLastError());
        } else {
            HIP_TRY(hipMemsetAsync(o.rowptr, 0, sizeof(int32_t), setup_stream()));
            HIP_TRY(hipMemsetAsync(o.split_slot, 0, sizeof(int32_t), setup_stream()));
        }
        int32_t *sched = nullptr;
        if (column_order) {
            HIP_TRY(sc.alloc((void **)&sched, sizeof(int32_t) * 4 * (M + 1)));
            int32_t *sorted = nullptr;
            if (n_long > 0) {
                // stable: equal first columns stay in item order, as on the host
                int32_t *key_sorted = nullptr;
                HIP_TRY(sc.alloc((void **)&key_sorted, sizeof(int32_t) * n_long));
                HIP_TRY(sc.alloc((void **)&sorted, sizeof(int32_t) * n_long));
                HIP_TRY(sort_pairs_u32(reinterpret_cast<const uint32_t *>(o.long_key),
                                       reinterpret_cast<uint32_t *>(key_sorted),
                                       reinterpret_cast<const uint32_t *>(o.long_item),
                                       reinterpret_cast<uint32_t *>(sorted), n_long, key_bits(n_cols), sc));
            }
            const int32_t *shorts = o.short_item;
            if (out->win.blocks && n_short == n_rows && M == n_rows) {
                shorts = out->win.rows; // an item is a row, and these are sorted already
            } else if (labels.p && n_short > 0) { // the rows of a community side by side
                uint32_t *key = nullptr, *key_sorted = nullptr, *ordered = nullptr;
                HIP_TRY(sc.alloc((void **)&key, sizeof(uint32_t) * n_short));
                HIP_TRY(sc.alloc((void **)&key_sorted, sizeof(uint32_t) * n_short));
                HIP_TRY(sc.alloc((void **)&ordered, sizeof(uint32_t) * n_short));
                HIP_TRY(cluster_keys(n_rows, labels.p, n_short, o.short_item, o.trow, key));
                HIP_TRY(sort_pairs_u32(key, key_sorted, reinterpret_cast<const uint32_t *>(o.short_item), ordered, n_short,
                                       cluster_key_bits(n_rows), sc));
                shorts = reinterpret_cast<const int32_t *>(ordered);
            }
            const int64_t cl = (n_long + kSchedChunk - 1) / kSchedChunk, cs = (n_short + kSchedChunk - 1) / kSchedChunk;
            long long *wsum = nullptr, *wscan = nullptr;
            HIP_TRY(sc.alloc((void **)&wsum, sizeof(long long) * (cl + cs + 1)));
            HIP_TRY(sc.alloc((void **)&wscan, sizeof(long long) * (cl + cs + 2)));
            if (cl + cs > 0) {
                hipLaunchKernelGGL(sched_sums_kernel, dim3((unsigned)(cl + cs)), dim3(kThreads), 0, setup_stream(), n_long, sorted,
                                   n_short, shorts, o.rowptr, wsum);
                HIP_TRY(hipGetLastError());
            }
            hipLaunchKernelGGL(sched_scan_kernel, dim3(2), dim3(1024), 0, setup_stream(), (int)cl, (int)cs, wsum, wscan);
            HIP_TRY(hipGetLastError());
            hipLaunchKernelGGL(sched_bounds_kernel, dim3(18), dim3(kThreads), 0, setup_stream(), n_long, sorted, n_short,
                               shorts, o.rowptr, wscan, d_bounds);
            HIP_TRY(hipGetLastError());
            if (M > 0) {
                hipLaunchKernelGGL(sched_emit_kernel, dim3(blocks_for(M)), dim3(kThreads), 0, setup_stream(), n_long, sorted, n_short,
                                   shorts, d_bounds, o.rowptr, o.trow, o.item_slot,
                                   reinterpret_cast<int4 *>(sched));
                HIP_TRY(hipGetLastError());
            }
            int32_t b[18];
            HIP_TRY(setup_copy(b, d_bounds, sizeof(b), hipMemcpyDeviceToHost));
            for (int x = 0; x < 9; ++x) out->xcd_bounds[x] = b[x] + b[9 + x];
        } else {
            hipLaunchKernelGGL(xcd_bounds_kernel, dim3(1), dim3(64), 0, setup_stream(), (int32_t)M, o.rowptr, d_bounds);
            HIP_TRY(hipGetLastError());
            HIP_TRY(setup_copy(out->xcd_bounds, d_bounds, 9 * sizeof(int32_t), hipMemcpyDeviceToHost));
        }
        out->M = M;
        out->n_split = total.split;
        out->n_split_items = total.slots;
        out->n_long = total.longp;
        out->max_item_len = std::min<int64_t>(sg, check.longest);
        out->trow = o.trow;
        out->split = o.split_panels;
        out->item_slot = o.item_slot;
        out->split_slot = o.split_slot;
        out->long_list = o.long_list;
        out->sched = sched;
        for (void *q : {(void *)o.trow, (void *)o.split_panels, (void *)o.item_slot, (void *)o.split_slot,
                        (void *)o.long_list, (void *)sched})
            sc.release(q);
        prow = o.rowptr;
    }
    if (bands && V == 1 && !S && n_rows > 0 && nnz > 0) {
        int32_t *b = nullptr;
        if (sc.alloc((void **)&b, sizeof(int32_t) * (kColumnBands - 1) * n_rows) == hipSuccess) {
            hipLaunchKernelGGL(bands_kernel, dim3(strided_blocks(16 * n_rows, 4096)), dim3(kThreads), 0, setup_stream(), n_rows, n_cols,
                               prow, pcol, b);
            HIP_TRY(hipGetLastError());
            out->bands = b;
            sc.release(b);
        } else {
            (void)hipGetLastError(); // products without them
            out->dropped = true;
        }
    }
    out->vals_due = late && V == 1;
    out->rowptr = prow;
    out->colidx = pcol;
    out->val = pval;
    sc.release(prow);
    sc.release(pcol);
    sc.release(pval);
    return PCSR_OK;
}

int features_device(int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t *d_rowptr,
                    const int32_t *d_colidx, int32_t omega, double *out, int *hip_err)
{
    if (omega == 0) omega = 64;
    FeatAcc h;
    memset(&h, 0, sizeof(h));
    const int64_t P2 = (n_rows + 1) / 2;
    if (n_rows > 0) {
        Scratch sc;
        const int64_t room = nnz / 9 + 64; // units there can be at most: of 9 nonzeros or more
        const int64_t groups = kPanelThreads / 8;
        const unsigned pb = (unsigned)std::max(std::min<int64_t>((P2 + groups - 1) / groups, kPanelBlocks),
                                               (P2 + kMostPanels - 1) / kMostPanels);
        const unsigned db = strided_blocks(n_rows, kDevBlocks);
        int32_t *shared = nullptr;
        int2 *units = nullptr;
        FarList *far = nullptr;
        RowPart *rows = nullptr;
        DevPart *devs = nullptr;
        FeatAcc *acc = nullptr;
        HIP_TRY(sc.alloc((void **)&shared, sizeof(int32_t) * P2));
        HIP_TRY(sc.alloc((void **)&units, sizeof(int2) * room));
        HIP_TRY(sc.alloc((void **)&far, sizeof(FarList)));
        HIP_TRY(sc.alloc((void **)&rows, sizeof(RowPart) * pb));
        HIP_TRY(sc.alloc((void **)&devs, sizeof(DevPart) * db));
        HIP_TRY(sc.alloc((void **)&acc, sizeof(FeatAcc)));
        HIP_TRY(hipMemsetAsync(far, 0, sizeof(FarList), setup_stream()));
        hipLaunchKernelGGL(features_panels_kernel, dim3(pb), dim3(kPanelThreads), 0, setup_stream(), n_rows, nnz, d_rowptr, d_colidx, shared,
                           room, units, far, rows);
        HIP_TRY(hipGetLastError());
        hipLaunchKernelGGL(features_far_kernel, dim3(kFarBlocks), dim3(kThreads), 0, setup_stream(), n_rows, d_rowptr, d_colidx, room,
                           units, far, shared);
        HIP_TRY(hipGetLastError());
        hipLaunchKernelGGL(features_deviation_kernel, dim3(db), dim3(kThreads), 0, setup_stream(), n_rows, nnz, d_rowptr, shared, rows,
                           (int)pb, far, omega, devs);
        HIP_TRY(hipGetLastError());
        hipLaunchKernelGGL(features_final_kernel, dim3(1), dim3(kThreads), 0, setup_stream(), nnz, rows, (int)pb, far, devs, (int)db, acc);
        HIP_TRY(hipGetLastError());
        HIP_TRY(setup_copy(&h, acc, sizeof(h), hipMemcpyDeviceToHost));
    }
    const double d = n_rows ? double(nnz) / double(n_rows) : 0.0;
    const double d_hat = h.n_hat ? double(nnz) / double(h.n_hat) : 0.0;
    out[0] = double(n_rows);
    out[1] = double(h.n_hat);
    out[2] = double(nnz);
    out[3] = n_rows ? double(h.n_hat) / double(n_rows) : 0.0;
    out[4] = d;
    out[5] = d_hat;
    out[6] = double(h.d_max);
    out[7] = d > 0 ? sqrt(h.ss / double(n_rows)) / d : 0.0;
    out[8] = h.n_hat ? sqrt(h.ss_hat / double(h.n_hat)) / d_hat : 0.0;
    out[9] = n_rows ? double(h.M1) / double(n_rows) : 1.0;
    out[10] = P2 ? double(h.M2) / double(P2) : 1.0;
    out[11] = (n_rows && n_cols) ? double(nnz) / (double(n_rows) * double(n_cols)) : 0.0;
    out[12] = n_rows ? h.bw_sum / double(n_rows) : 0.0;
    out[13] = h.bw_max;
    out[14] = 0.0;
    out[15] = h.nnz2 ? 1.0 - double(nnz) / (double(h.nnz2) * 2.0) : 0.0;
    out[16] = nnz ? double(h.near) / double(nnz) : 0.0;
    return PCSR_OK;
}

} // namespace pcsr
