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
constexpr int kSegBlocks = kSegment / kProbe + 1; // every block but a segment's last has kProbe items or more

struct CutArgs {
    int64_t M, n_cols;
    int32_t win;
    const int32_t *rowptr, *colidx;
    int32_t *ptr_end, *start; // kSegBlocks per segment
    int32_t *count;           // blocks per segment
    unsigned long long *hits; // over all of them
    int *gave_up;             // a stretch too large to sort in LDS: the host builder takes over
};

union CutShared {
    int32_t sorted[kSortMax];
    int32_t bins[kBins];
};

// Column c0 of the densest window of `win` columns over the vectors [s, e), as the host builder
// defines it: the window that ends at the smallest column where the count is largest, and
// starts at its first occupied column.  Sorts in LDS; n = e - s <= kSortMax.
__device__ int32_t densest_sorted(CutShared &sh, unsigned long long &best, const int32_t *colidx, int64_t s, int n,
                                  int32_t win)
{
    const int tid = threadIdx.x;
    int m = 64;
    while (m < n) m <<= 1;
    for (int i = tid; i < m; i += kCutThreads) sh.sorted[i] = i < n ? colidx[s + i] : INT32_MAX;
    if (tid == 0) best = 0;
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
    unsigned long long mine = 0;
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
        // larger count first, then smaller r
        const unsigned long long key = ((unsigned long long)(r - lo + 1) << 32) | (0xffffffffu - (unsigned)r);
        mine = key > mine ? key : mine;
    }
    atomicMax(&best, mine);
    __syncthreads();
    const int r = (int)(0xffffffffu - (unsigned)(best & 0xffffffffu));
    const int l = r - (int)(best >> 32) + 1;
    const int32_t c0 = sh.sorted[l];
    __syncthreads(); // sorted and best may be overwritten
    return c0;
}

// A workgroup cuts one segment of items into blocks, one after the other (where a block ends
// decides where the next begins); everything inside a step is spread over its threads.  The
// window of a whole block comes from a histogram of the 3 * win columns around the probe
// window where that one already holds more than half of the block's vectors: a better window
// then has to overlap it.  250,000 rows of 48: 0.86 ms, where the host builder sorted every
// block's columns, 50 ms on 16 threads.
__global__ void __launch_bounds__(kCutThreads) window_cut_kernel(CutArgs a)
{
    __shared__ CutShared sh;
    __shared__ unsigned long long best;
    __shared__ int s_cnt, s_at;
    typedef hipcub::BlockScan<int, kCutThreads> Scan;
    __shared__ typename Scan::TempStorage tmp;
    const int tid = threadIdx.x;
    const int64_t seg0 = (int64_t)blockIdx.x * kSegment;
    const int64_t seg_end = seg0 + kSegment < a.M ? seg0 + kSegment : a.M;
    const int32_t w = a.win;
    const int64_t last_start = a.n_cols > w ? a.n_cols - w : 0;
    unsigned long long hits_total = 0;
    int blocks = 0;

    for (int64_t i = seg0; i < seg_end;) { // all of this is uniform over the workgroup
        const int64_t probe_end = i + kProbe < seg_end ? i + kProbe : seg_end;
        const int64_t s = a.rowptr[i], pe = a.rowptr[probe_end];
        if (pe - s > kSortMax) {
            if (tid == 0) *a.gave_up = 1;
            return;
        }
        int64_t j = probe_end, c_probe = -1;
        if (pe > s) {
            c_probe = densest_sorted(sh, best, a.colidx, s, (int)(pe - s), w);
            c_probe = c_probe < last_start ? c_probe : last_start;
            // the block grows while at least half of an item's vectors lie in that window
            const int64_t limit = i + w < seg_end ? i + w : seg_end;
            if (tid == 0) s_at = (int)(limit - i);
            __syncthreads();
            for (int64_t k = probe_end + tid; k < limit; k += kCutThreads) {
                const int64_t b = a.rowptr[k], e = a.rowptr[k + 1];
                auto lower = [&](int64_t key) {
                    int64_t lo = b, hi = e;
                    while (lo < hi) {
                        const int64_t mid = (lo + hi) >> 1;
                        if (a.colidx[mid] < key)
                            lo = mid + 1;
                        else
                            hi = mid;
                    }
                    return lo;
                };
                if (e > b && 2 * (lower(c_probe + w) - lower(c_probe)) < e - b) atomicMin(&s_at, (int)(k - i));
            }
            __syncthreads();
            const int64_t stop = i + s_at;
            j = stop > probe_end ? stop : probe_end;
            __syncthreads();
        }
        const int64_t e = a.rowptr[j], n = e - s;
        int64_t c0 = -1;
        int hits = 0;
        if (n > 0) {
            // (c_probe < 0 means that the first kProbe items are empty, and then they are the block)
            const int64_t base = c_probe - w + 1; // column of bin 0
            const int bins = 3 * w - 2;
            for (int b = tid; b < bins; b += kCutThreads) sh.bins[b] = 0;
            if (tid == 0) {
                s_cnt = 0;
                best = 0;
            }
            __syncthreads();
            int in_probe = 0;
            for (int64_t t = s + tid; t < e; t += kCutThreads) {
                const int64_t c = a.colidx[t];
                in_probe += c >= c_probe && c < c_probe + w;
                if (c >= base && c < base + bins) atomicAdd(&sh.bins[c - base], 1);
            }
            if (in_probe) atomicAdd(&s_cnt, in_probe);
            __syncthreads();
            if (2 * (int64_t)s_cnt > n) {
                // inclusive sums in place: bins[b] = vectors in columns up to that of bin b
                constexpr int N = kBins / kCutThreads;
                const int per = (bins + kCutThreads - 1) / kCutThreads;
                int v[N], own = 0, ex;
#pragma unroll
                for (int k = 0; k < N; ++k) {
                    const int b = tid * per + k;
                    v[k] = k < per && b < bins ? sh.bins[b] : 0;
                    own += v[k];
                }
                Scan(tmp).ExclusiveSum(own, ex);
                __syncthreads();
#pragma unroll
                for (int k = 0; k < N; ++k) {
                    const int b = tid * per + k;
                    ex += v[k];
                    if (k < per && b < bins) sh.bins[b] = ex;
                }
                __syncthreads();
                auto upto = [&](int b) { return b < 0 ? 0 : sh.bins[b < bins ? b : bins - 1]; };
                // windows that end at an occupied column c_probe or later
                for (int b = w - 1 + tid; b < bins; b += kCutThreads) {
                    if (upto(b) == upto(b - 1)) continue;
                    const unsigned long long key = ((unsigned long long)(upto(b) - upto(b - w)) << 32) |
                                                   (0xffffffffu - (unsigned)b);
                    atomicMax(&best, key);
                }
                __syncthreads();
                const int end = (int)(0xffffffffu - (unsigned)(best & 0xffffffffu));
                // its first occupied column: the first bin after end - w whose sum exceeds the one there
                int lo = end - w + 1, hi = end;
                const int before = upto(end - w);
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (upto(mid) > before)
                        hi = mid;
                    else
                        lo = mid + 1;
                }
                c0 = base + lo;
                c0 = c0 < last_start ? c0 : last_start;
                const int b0 = (int)(c0 - base);
                hits = upto(b0 + w - 1) - upto(b0 - 1);
                __syncthreads();
            } else {
                __syncthreads(); // s_cnt is read
                if (n > kSortMax) {
                    if (tid == 0) *a.gave_up = 1;
                    return;
                }
                c0 = densest_sorted(sh, best, a.colidx, s, (int)n, w);
                c0 = c0 < last_start ? c0 : last_start;
                if (tid == 0) s_cnt = 0;
                __syncthreads();
                int in = 0;
                for (int64_t t = s + tid; t < e; t += kCutThreads) {
                    const int64_t c = a.colidx[t];
                    in += c >= c0 && c < c0 + w;
                }
                if (in) atomicAdd(&s_cnt, in);
                __syncthreads();
                hits = s_cnt;
                __syncthreads();
            }
        }
        if (tid == 0) {
            // staging costs `win` row reads: worth it from two uses per staged row
            const bool use = c0 >= 0 && hits >= 2 * w;
            a.start[blockIdx.x * kSegBlocks + blocks] = use ? (int32_t)c0 : -1;
            a.ptr_end[blockIdx.x * kSegBlocks + blocks] = (int32_t)j;
            if (use) hits_total += hits;
        }
        ++blocks;
        i = j;
    }
    if (tid == 0) {
        a.count[blockIdx.x] = blocks;
        if (hits_total) atomicAdd(a.hits, hits_total);
    }
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
    HIP_TRY(hipMemsetAsync(d_tot, 0, sizeof(Totals), nullptr));
    HIP_TRY(hipMemsetAsync(a.count, 0, sizeof(int32_t) * (n_seg + 1), nullptr));
    a.hits = &d_tot->hits;
    a.gave_up = &d_tot->gave_up;
    hipLaunchKernelGGL(window_cut_kernel, dim3((unsigned)n_seg), dim3(kCutThreads), 0, 0, a);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(window_scan_kernel, dim3(1), dim3(1024), 0, 0, (int)n_seg, a.count);
    HIP_TRY(hipGetLastError());
    int32_t nb = 0;
    HIP_TRY(hipMemcpyAsync(&nb, a.count + n_seg, sizeof(nb), hipMemcpyDeviceToHost, nullptr));
    HIP_TRY(hipMemcpy(&tot, d_tot, sizeof(tot), hipMemcpyDeviceToHost));
    if (tot.gave_up) return PCSR_E_UNSUPPORTED;
    int32_t *win_ptr = nullptr, *win_start = nullptr, *lo = nullptr, *hi = nullptr;
    HIP_TRY(sc.alloc((void **)&win_ptr, sizeof(int32_t) * (nb + 1)));
    HIP_TRY(sc.alloc((void **)&win_start, sizeof(int32_t) * (nb + 1)));
    HIP_TRY(sc.alloc((void **)&lo, sizeof(int32_t) * (M + 1)));
    HIP_TRY(sc.alloc((void **)&hi, sizeof(int32_t) * (M + 1)));
    hipLaunchKernelGGL(window_compact_kernel, dim3((unsigned)n_seg), dim3(kThreads), 0, 0, a.ptr_end, a.start, a.count,
                       win_ptr, win_start);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(window_runs_kernel, dim3((unsigned)nb), dim3(kThreads), 0, 0, win_ptr, win_start, win, d_rowptr,
                       d_colidx, lo, hi);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(nullptr));
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
