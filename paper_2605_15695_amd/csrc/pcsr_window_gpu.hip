// Column-window blocking on the GPU: the blocks and windows choose_windows picks on the host, from
// PCSR arrays in device memory.
#include <hipcub/hipcub.hpp>

#include "pcsr_build_gpu.h"
#include "pcsr_gpu_util.h"

namespace pcsr {
namespace {

constexpr int kCutThreads = 1024;
constexpr int kProbe = 32;        // as in choose_windows
constexpr int kSegment = 8192;    // as in choose_windows
constexpr int kSortMax = 8192;    // columns a workgroup sorts in LDS
constexpr int kMaxWindow = 2048;
constexpr int kBins = 3 * kMaxWindow;
constexpr int kOwnGroups = 16;
constexpr int kMaxPasses = 8;     // of densest_binned before it sorts
constexpr int kSegBlocks = kSegment / kProbe + 1; // every block but a segment's last has kProbe items or more

struct CutArgs {
    int64_t M, n_cols;
    int32_t win;
    const int32_t *rowptr, *colidx;
    int32_t *ptr_end, *start; // kSegBlocks per segment; start: the probe window until window_own_kernel
    int32_t *count;           // blocks per segment
    unsigned long long *hits; // over all of them
    int *gave_up;             // a stretch too large to sort in LDS: the host builder takes over
};

struct CutShared {
    union {
        int32_t sorted[kSortMax];
        int32_t bins[kBins];
    };
    int32_t coarse[kBins]; // entries per `win` columns
    int red[kCutThreads / 64];
    typename hipcub::BlockScan<int, kCutThreads>::TempStorage scan;
};

// the largest v of the workgroup (v >= 0), in every thread
__device__ __forceinline__ int cut_max(CutShared &sh, int v)
{
    // inside a row of 16 lanes on the vector ALU (row_ror), then across the four rows
    v = max(v, __builtin_amdgcn_mov_dpp(v, 0x121, 0xf, 0xf, true));
    v = max(v, __builtin_amdgcn_mov_dpp(v, 0x122, 0xf, 0xf, true));
    v = max(v, __builtin_amdgcn_mov_dpp(v, 0x124, 0xf, 0xf, true));
    v = max(v, __builtin_amdgcn_mov_dpp(v, 0x128, 0xf, 0xf, true));
    v = max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
            max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
    __syncthreads(); // red is free
    if ((threadIdx.x & 63) == 0) sh.red[threadIdx.x >> 6] = v;
    __syncthreads();
    v = sh.red[0];
#pragma unroll
    for (int i = 1; i < kCutThreads / 64; ++i) v = max(v, sh.red[i]);
    return v;
}
__device__ __forceinline__ int cut_sum(CutShared &sh, int v)
{
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) v += __shfl_xor(v, m);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh.red[threadIdx.x >> 6] = v;
    __syncthreads();
    v = 0;
#pragma unroll
    for (int i = 0; i < kCutThreads / 64; ++i) v += sh.red[i];
    return v;
}

// A window, by how many entries it holds and where it ends.  Of two the one with more is better,
// then the one that ends first.
struct Window {
    int count, end;
};
__device__ __forceinline__ bool better(Window a, Window b) { return a.count > b.count || (a.count == b.count && a.end < b.end); }
__device__ __forceinline__ Window cut_best(CutShared &sh, Window w)
{
    const int count = cut_max(sh, w.count);
    return {count, INT32_MAX - cut_max(sh, w.count == count ? INT32_MAX - w.end : 0)};
}

// entries of colidx[s, e) per column of [base, base + bins), as inclusive sums: bins[b] = entries in
// columns base .. base + b
__device__ __forceinline__ void binned_sums(CutShared &sh, const int32_t *colidx, int64_t s, int64_t e, int64_t base, int bins)
{
    const int tid = threadIdx.x;
    for (int b = tid; b < bins; b += kCutThreads) sh.bins[b] = 0;
    __syncthreads();
    constexpr int N4 = 8; // loads in flight
    for (int64_t t = s + tid; t < e; t += N4 * kCutThreads) {
        int64_t at[N4];
#pragma unroll
        for (int k = 0; k < N4; ++k) at[k] = t + k * kCutThreads < e ? (int64_t)colidx[t + k * kCutThreads] - base : -1;
#pragma unroll
        for (int k = 0; k < N4; ++k)
            if (at[k] >= 0 && at[k] < bins) atomicAdd(&sh.bins[at[k]], 1);
    }
    __syncthreads();
    constexpr int N = kBins / kCutThreads;
    const int per = (bins + kCutThreads - 1) / kCutThreads;
    int v[N], own = 0, ex;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const int b = tid * per + k;
        v[k] = k < per && b < bins ? sh.bins[b] : 0;
        own += v[k];
    }
    hipcub::BlockScan<int, kCutThreads>(sh.scan).ExclusiveSum(own, ex);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const int b = tid * per + k;
        ex += v[k];
        if (k < per && b < bins) sh.bins[b] = ex;
    }
    __syncthreads();
}
__device__ __forceinline__ int upto(const CutShared &sh, int bins, int b) { return b < 0 ? 0 : sh.bins[b < bins ? b : bins - 1]; }

// best window of w columns that ends at an occupied column of bin `first` or later; end: its bin
__device__ __forceinline__ Window best_end(CutShared &sh, int first, int bins, int32_t w)
{
    Window mine = {0, INT32_MAX};
    for (int b = first + threadIdx.x; b < bins; b += kCutThreads) {
        const int at = upto(sh, bins, b);
        const Window here = {at - upto(sh, bins, b - w), b};
        if (at != upto(sh, bins, b - 1) && better(here, mine)) mine = here;
    }
    return cut_best(sh, mine);
}
// first occupied column of the window that ends in bin `end`: the first bin after end - w whose sum exceeds
// the one there
__device__ __forceinline__ int64_t first_occupied(const CutShared &sh, int end, int bins, int32_t w, int64_t base)
{
    int lo = end - w + 1, hi = end;
    const int before = upto(sh, bins, end - w);
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (upto(sh, bins, mid) > before)
            hi = mid;
        else
            lo = mid + 1;
    }
    return base + lo;
}
// Column c0 of the densest window of `win` columns over the vectors [s, e), as the host builder
// defines it: the window that ends at the smallest column where the count is largest, and
// starts at its first occupied column.  By sorting in LDS; n = e - s <= kSortMax.
__device__ int32_t densest_sorted(CutShared &sh, const int32_t *colidx, int64_t s, int n, int32_t win)
{
    const int tid = threadIdx.x;
    int m = 64;
    while (m < n) m <<= 1;
    for (int i = tid; i < m; i += kCutThreads) sh.sorted[i] = i < n ? colidx[s + i] : INT32_MAX;
    __syncthreads();
    for (int k = 2; k <= m; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = tid; i < m; i += kCutThreads) {
                const int o = i ^ j;
                if (o > i) {
                    const int32_t a = sh.sorted[i], b = sh.sorted[o];
                    if ((a > b) == ((i & k) == 0)) {
                        sh.sorted[i] = b;
                        sh.sorted[o] = a;
                    }
                }
            }
            __syncthreads();
        }
    Window mine = {0, INT32_MAX}; // ends by position: ascending as the columns
    for (int r = tid; r < n; r += kCutThreads) {
        const int64_t low = (int64_t)sh.sorted[r] - win; // columns above it are in the window
        int lo = 0, hi = r;                              // first of them
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (sh.sorted[mid] > low)
                hi = mid;
            else
                lo = mid + 1;
        }
        const Window here = {r - lo + 1, r};
        if (better(here, mine)) mine = here;
    }
    const Window best = cut_best(sh, mine);
    const int32_t c0 = sh.sorted[best.end - best.count + 1];
    __syncthreads(); // sorted may be overwritten
    return c0;
}

// The same without a sort.  A first histogram counts `win` columns to a bin.  A window that ends in bin k
// holds at most what bins k - 1 and k hold together, and the best one at least what the fullest
// bin holds, so only ends in bins with enough around them are looked at, column by column, two bins at a
// time.  Where many bins qualify (scattered columns) it is sorted after all.
__device__ int32_t densest_binned(CutShared &sh, const int32_t *colidx, int64_t s, int n, int32_t win, int n_coarse)
{
    const int tid = threadIdx.x;
    const int shift = 31 - __builtin_clz((unsigned)win);
    for (int k = tid; k < n_coarse; k += kCutThreads) sh.coarse[k] = 0;
    __syncthreads();
    for (int t = tid; t < n; t += kCutThreads) {
        const unsigned k = (unsigned)colidx[s + t] >> shift;
        if (k < (unsigned)n_coarse) atomicAdd(&sh.coarse[k], 1); // (it is, short of unchecked arrays)
    }
    __syncthreads();
    int most = 0;
    for (int k = tid; k < n_coarse; k += kCutThreads) most = max(most, sh.coarse[k]);
    const int fullest = cut_max(sh, most);
    int best = 0;
    int64_t c0 = 0;
    int from = 0; // bins below are done
    for (int pass = 0;; ++pass) {
        int next = 0; // first bin that qualifies, by its distance from the end
        for (int k = tid; k < n_coarse; k += kCutThreads)
            if (k >= from && sh.coarse[k] > 0 && sh.coarse[k] + (k ? sh.coarse[k - 1] : 0) >= max(fullest, best + 1)) {
                next = n_coarse - k;
                break;
            }
        next = cut_max(sh, next);
        if (next == 0) break;
        if (pass == kMaxPasses) return densest_sorted(sh, colidx, s, n, win);
        const int k = n_coarse - next;
        const int64_t base = (int64_t)(k - 1) * win;
        const int bins = 3 * win;
        binned_sums(sh, colidx, s, s + n, base, bins);
        const Window w = best_end(sh, win, bins, win);
        if (w.count > best) { // uniform; earlier passes end earlier
            best = w.count;
            c0 = first_occupied(sh, w.end, bins, win, base);
        }
        __syncthreads(); // bins are read
        from = k + 2;
    }
    return (int32_t)c0;
}

// A workgroup cuts one segment of items into blocks, one after the other (where a block ends
// decides where the next begins), so the chain of a segment's 17 or so steps is what the kernel takes: only what the
// chain needs is done here, and a step is a few round trips to memory and barriers, everything in it spread over the
// threads.  250,000 rows of 48 (31 segments): 198 us, and 30 for the blocks' own windows below, where 860 were spent
// with both in the chain, the probe's columns sorted in LDS (66 barriers a step) and one contended counter.
__global__ void __launch_bounds__(kCutThreads) window_cut_kernel(CutArgs a)
{
    __shared__ CutShared sh;
    __shared__ int s_at;
    const int tid = threadIdx.x;
    const int64_t seg0 = (int64_t)blockIdx.x * kSegment;
    const int64_t seg_end = seg0 + kSegment < a.M ? seg0 + kSegment : a.M;
    const int32_t w = a.win;
    const int64_t last_start = a.n_cols > w ? a.n_cols - w : 0;
    const int64_t coarse = (a.n_cols + w - 1) / w; // too many for LDS: the probe's columns are sorted
    int blocks = 0;

    for (int64_t i = seg0; i < seg_end;) { // all of this is uniform over the workgroup
        const int64_t probe_end = i + kProbe < seg_end ? i + kProbe : seg_end;
        const int64_t limit = i + w < seg_end ? i + w : seg_end;
        // this thread's item of those the block may grow by, and the column in its middle, requested before the
        // window is known
        const int64_t own = probe_end + tid;
        int32_t own_b = 0, own_e = 0, own_mid = 0;
        if (own < limit) {
            own_b = a.rowptr[own];
            own_e = a.rowptr[own + 1];
        }
        const int64_t s = a.rowptr[i], pe = a.rowptr[probe_end];
        if (own_e > own_b) own_mid = a.colidx[own_b + ((own_e - own_b) >> 1)];
        if (pe - s > kSortMax) {
            if (tid == 0) *a.gave_up = 1;
            return;
        }
        int64_t j = probe_end, c_probe = -1;
        if (pe > s) {
            c_probe = coarse <= kBins ? densest_binned(sh, a.colidx, s, (int)(pe - s), w, (int)coarse)
                                      : densest_sorted(sh, a.colidx, s, (int)(pe - s), w);
            c_probe = c_probe < last_start ? c_probe : last_start;
            // the block grows while at least half of an item's vectors lie in that window
            if (tid == 0) s_at = (int)(limit - i);
            __syncthreads();
            for (int64_t k = own; k < limit; k += kCutThreads) {
                const bool first = k == own;
                const int32_t b = first ? own_b : a.rowptr[k], e = first ? own_e : a.rowptr[k + 1];
                if (e <= b) continue;
                // first positions of columns >= c_probe and >= c_probe + w, searched side by side
                const int32_t mid = b + ((e - b) >> 1);
                const int32_t c = first ? own_mid : a.colidx[mid];
                int32_t lo0 = b, hi0 = e, lo1 = b, hi1 = e;
                c < c_probe ? lo0 = mid + 1 : hi0 = mid;
                c < c_probe + w ? lo1 = mid + 1 : hi1 = mid;
                while (lo0 < hi0 || lo1 < hi1) {
                    const int32_t m0 = lo0 + ((hi0 - lo0) >> 1), m1 = lo1 + ((hi1 - lo1) >> 1);
                    const int32_t c0 = a.colidx[lo0 < hi0 ? m0 : b], c1 = a.colidx[lo1 < hi1 ? m1 : b];
                    if (lo0 < hi0) c0 < c_probe ? lo0 = m0 + 1 : hi0 = m0;
                    if (lo1 < hi1) c1 < c_probe + w ? lo1 = m1 + 1 : hi1 = m1;
                }
                if (2 * (int64_t)(lo1 - lo0) < e - b) atomicMin(&s_at, (int)(k - i));
            }
            __syncthreads();
            const int64_t stop = i + s_at;
            j = stop > probe_end ? stop : probe_end;
        }
        if (tid == 0) {
            a.start[blockIdx.x * kSegBlocks + blocks] = (int32_t)c_probe;
            a.ptr_end[blockIdx.x * kSegBlocks + blocks] = (int32_t)j;
        }
        ++blocks;
        i = j;
        __syncthreads(); // s_at is read
    }
    if (tid == 0) a.count[blockIdx.x] = blocks;
}

// The window of a whole block, kOwnGroups workgroups to a segment's blocks: from a histogram of the 3 * win
// columns around the probe window where that one already holds more than half of the block's
// vectors (a better window then has to overlap it), else sorted.
__global__ void __launch_bounds__(kCutThreads) window_own_kernel(CutArgs a)
{
    __shared__ CutShared sh;
    const int tid = threadIdx.x;
    const int32_t w = a.win;
    const int64_t last_start = a.n_cols > w ? a.n_cols - w : 0;
    const int64_t seg0 = (int64_t)blockIdx.x * kSegment;
    const int blocks = a.count[blockIdx.x];
    unsigned long long hits_total = 0;
    for (int q = blockIdx.y; q < blocks; q += kOwnGroups) { // uniform over the workgroup
        const int64_t at = blockIdx.x * kSegBlocks + q;
        const int64_t i = q ? a.ptr_end[at - 1] : seg0, j = a.ptr_end[at], c_probe = a.start[at];
        const int64_t s = a.rowptr[i], e = a.rowptr[j], n = e - s;
        int64_t c0 = -1;
        int hits = 0;
        if (n > 0) {
            // (c_probe < 0 means that the first kProbe items are empty, and then they are the block)
            const int64_t base = c_probe - w + 1; // column of bin 0
            const int bins = 3 * w - 2;
            binned_sums(sh, a.colidx, s, e, base, bins);
            // entries in the probe window, whose first column is that of bin w - 1
            if (2 * (int64_t)(upto(sh, bins, 2 * w - 2) - upto(sh, bins, w - 2)) > n) {
                const Window best = best_end(sh, w - 1, bins, w);
                c0 = first_occupied(sh, best.end, bins, w, base);
                c0 = c0 < last_start ? c0 : last_start;
                const int b0 = (int)(c0 - base);
                hits = upto(sh, bins, b0 + w - 1) - upto(sh, bins, b0 - 1);
                __syncthreads();
            } else {
                __syncthreads(); // the bins are read
                if (n > kSortMax) {
                    if (tid == 0) *a.gave_up = 1;
                    return;
                }
                c0 = densest_sorted(sh, a.colidx, s, (int)n, w);
                c0 = c0 < last_start ? c0 : last_start;
                int in = 0;
                for (int64_t t = s + tid; t < e; t += kCutThreads) {
                    const int64_t c = a.colidx[t];
                    in += c >= c0 && c < c0 + w;
                }
                hits = cut_sum(sh, in);
            }
        }
        if (tid == 0) {
            // staging costs `win` row reads: worth it from two uses per staged row
            const bool use = c0 >= 0 && hits >= 2 * w;
            a.start[at] = use ? (int32_t)c0 : -1;
            if (use) hits_total += hits;
        }
    }
    if (tid == 0 && hits_total) atomicAdd(a.hits, hits_total);
}

// blocks before each segment (in place), total behind them
__global__ void __launch_bounds__(1024) window_scan_kernel(int n, int32_t *count)
{
    typedef hipcub::BlockScan<int, 1024> Scan;
    __shared__ typename Scan::TempStorage tmp;
    int before = 0;
    for (int base = 0; base < n; base += 1024) {
        const int i = base + threadIdx.x;
        int c = i < n ? count[i] : 0, ex, total;
        Scan(tmp).ExclusiveSum(c, ex, total);
        if (i < n) count[i] = before + ex;
        before += total;
        __syncthreads();
    }
    if (threadIdx.x == 0) count[n] = before;
}

__global__ void __launch_bounds__(kThreads) window_compact_kernel(const int32_t *ptr_end, const int32_t *start,
                                                                  const int32_t *offset, int32_t *win_ptr,
                                                                  int32_t *win_start)
{
    const int o = offset[blockIdx.x], n = offset[blockIdx.x + 1] - o;
    for (int k = threadIdx.x; k < n; k += kThreads) {
        win_ptr[o + k + 1] = ptr_end[blockIdx.x * kSegBlocks + k];
        win_start[o + k] = start[blockIdx.x * kSegBlocks + k];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) win_ptr[0] = 0;
}

// the run of every item that lies inside its block's window
__global__ void __launch_bounds__(kThreads) window_runs_kernel(const int32_t *win_ptr, const int32_t *win_start,
                                                               int32_t win, const int32_t *rowptr,
                                                               const int32_t *colidx, int32_t *lo_out, int32_t *hi_out)
{
    const int64_t c0 = win_start[blockIdx.x];
    for (int it = win_ptr[blockIdx.x] + threadIdx.x; it < win_ptr[blockIdx.x + 1]; it += kThreads) {
        const int64_t s = rowptr[it], e = rowptr[it + 1];
        auto lower = [&](int64_t key) {
            int64_t lo = s, hi = e;
            while (lo < hi) {
                const int64_t mid = (lo + hi) >> 1;
                if (colidx[mid] < key)
                    lo = mid + 1;
                else
                    hi = mid;
            }
            return (int32_t)lo;
        };
        lo_out[it] = c0 < 0 ? (int32_t)s : lower(c0);
        hi_out[it] = c0 < 0 ? (int32_t)s : lower(c0 + win);
    }
}

} // namespace

int windows_device(int64_t M, int64_t n_cols, int32_t win, const int32_t *d_rowptr, const int32_t *d_colidx,
                   DeviceWindows *out, int *hip_err)
{
    if (win > kMaxWindow || M <= 0) return PCSR_E_UNSUPPORTED;
    Scratch sc;
    const int64_t n_seg = (M + kSegment - 1) / kSegment;
    CutArgs a;
    a.M = M;
    a.n_cols = n_cols;
    a.win = win;
    a.rowptr = d_rowptr;
    a.colidx = d_colidx;
    struct Totals {
        unsigned long long hits;
        int gave_up, pad;
    } *d_tot = nullptr, tot;
    HIP_TRY(sc.alloc((void **)&a.ptr_end, sizeof(int32_t) * n_seg * kSegBlocks));
    HIP_TRY(sc.alloc((void **)&a.start, sizeof(int32_t) * n_seg * kSegBlocks));
    HIP_TRY(sc.alloc((void **)&a.count, sizeof(int32_t) * (n_seg + 1)));
    HIP_TRY(sc.alloc((void **)&d_tot, sizeof(Totals)));
    HIP_TRY(hipMemsetAsync(d_tot, 0, sizeof(Totals), setup_stream()));
    HIP_TRY(hipMemsetAsync(a.count, 0, sizeof(int32_t) * (n_seg + 1), setup_stream()));
    a.hits = &d_tot->hits;
    a.gave_up = &d_tot->gave_up;
    hipLaunchKernelGGL(window_cut_kernel, dim3((unsigned)n_seg), dim3(kCutThreads), 0, setup_stream(), a);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(window_own_kernel, dim3((unsigned)n_seg, kOwnGroups), dim3(kCutThreads), 0, setup_stream(), a);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(window_scan_kernel, dim3(1), dim3(1024), 0, setup_stream(), (int)n_seg, a.count);
    HIP_TRY(hipGetLastError());
    int32_t nb = 0;
    HIP_TRY(setup_copy(&nb, a.count + n_seg, sizeof(nb), hipMemcpyDeviceToHost));
    HIP_TRY(setup_copy(&tot, d_tot, sizeof(tot), hipMemcpyDeviceToHost));
    if (tot.gave_up) return PCSR_E_UNSUPPORTED;
    int32_t *win_ptr = nullptr, *win_start = nullptr, *lo = nullptr, *hi = nullptr;
    HIP_TRY(sc.alloc((void **)&win_ptr, sizeof(int32_t) * (nb + 1)));
    HIP_TRY(sc.alloc((void **)&win_start, sizeof(int32_t) * (nb + 1)));
    HIP_TRY(sc.alloc((void **)&lo, sizeof(int32_t) * (M + 1)));
    HIP_TRY(sc.alloc((void **)&hi, sizeof(int32_t) * (M + 1)));
    hipLaunchKernelGGL(window_compact_kernel, dim3((unsigned)n_seg), dim3(kThreads), 0, setup_stream(), a.ptr_end, a.start, a.count,
                       win_ptr, win_start);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(window_runs_kernel, dim3((unsigned)nb), dim3(kThreads), 0, setup_stream(), win_ptr, win_start, win, d_rowptr,
                       d_colidx, lo, hi);
    HIP_TRY(hipGetLastError());
    HIP_TRY(setup_wait());
    out->ptr = win_ptr;
    out->start = win_start;
    out->lo = lo;
    out->hi = hi;
    out->blocks = nb;
    out->hits = (int64_t)tot.hits;
    for (int32_t *p : {win_ptr, win_start, lo, hi}) sc.release(p);
    return PCSR_OK;
}

} // namespace pcsr
