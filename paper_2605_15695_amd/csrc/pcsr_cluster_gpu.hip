// Communities of a square CSR whose ids carry no locality, found while its handle is built, so that the product can
// run the rows of a community side by side (pcsr_build_gpu.hip: the schedule of PCSR_FLAG_CLUSTER_IF_USEFUL).
//
// Label propagation as in pcsr_reorder, cut down to what an order of the rows needs: 16 neighbours a row and round
// instead of all, six rounds.  On planted communities of 60 to 2000 nodes with 10 to 30 % of the nonzeros outside, that
// leaves all but 5 % of the inner nonzeros with one label (pcsr_reorder's rounds: all but 1 %).
// What bounds it: latency and requests to the labels, 4 bytes each out of L2.
#include <hip/hip_runtime.h>
#include <hipcub/hipcub.hpp>

#include "pcsr_build_gpu.h"
#include "pcsr_gpu_util.h"
#include "pcsr_sort_gpu.h"

namespace pcsr {
namespace {

constexpr int kRoundThreads = 1024, kRoundBlocks = 512;
constexpr int kRounds = 6;
constexpr int kSamples = 4096; // rows the probe looks at

// the integer mixer of pcsr_reorder: lowbias32, a published 32-bit hash (found by C. Wellons' hash-prospector search)
__device__ __forceinline__ uint32_t mix(uint32_t x)
{
    x ^= x >> 16;
    x *= 0x7feb352du;
    x ^= x >> 15;
    x *= 0x846ca68bu;
    x ^= x >> 16;
    return x;
}

// out[0]: columns that sampled rows have in common with the row of one of their columns; out[1]: n times
// what rows of uniform random columns would.  A wavefront takes a row.  Every index is checked: this runs beside the check of
// the arrays, before its result is known.
__global__ void __launch_bounds__(kThreads) cluster_probe_kernel(int64_t n, int64_t nnz, const int32_t *rowptr,
                                                                 const int32_t *colidx, unsigned long long *out)
{
    const int lane = threadIdx.x & 63;
    const int64_t q = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    unsigned common = 0;
    unsigned long long expected = 0;
    const int64_t r = (int64_t)((double)q * (double)n / kSamples);
    if (q < kSamples && r < n) {
        const int64_t s = rowptr[r], e = rowptr[r + 1];
        if (s >= 0 && e <= nnz && e > s) {
            const int64_t c = colidx[s + (int64_t)(mix((uint32_t)r) % (uint32_t)(e - s))];
            if (c >= 0 && c < n && c != r) {
                const int64_t s2 = rowptr[c], e2 = rowptr[c + 1];
                if (s2 >= 0 && e2 <= nnz && e2 > s2) {
                    const int64_t mine = e - s < 64 ? e - s : 64; // of a longer row, 64 spread over it
                    bool both = false;
                    if (lane < mine) {
                        const int32_t x = colidx[s + (e - s) * lane / mine];
                        int32_t lo = (int32_t)s2, hi = (int32_t)e2;
                        while (lo < hi) narrow(colidx, x, lo, hi);
                        both = lo < e2 && colidx[lo] == x;
                    }
                    common = __popcll(__ballot(both));
                    expected = (unsigned long long)mine * (unsigned long long)(e2 - s2);
                }
            }
        }
    }
    __shared__ unsigned long long sum[2][kThreads / 64];
    if (lane == 0) {
        sum[0][threadIdx.x >> 6] = common;
        sum[1][threadIdx.x >> 6] = expected;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        unsigned long long t = 0;
        for (int w = 0; w < kThreads / 64; ++w) t += sum[threadIdx.x][w];
        if (t) atomicAdd(&out[threadIdx.x], t);
    }
}

template <int K> __device__ __forceinline__ int rotated(int x) // lane l of every 16 gets lane l - K
{
    return __builtin_amdgcn_mov_dpp(x, 0x120 + K, 0xf, 0xf, true);
}
template <int K = 1> __device__ __forceinline__ int equals(int x)
{
    if constexpr (K == 16)
        return 1;
    else
        return (rotated<K>(x) == x) + equals<K + 1>(x);
}

struct RoundPart {
    unsigned long long same, sampled; // sampled neighbours with the label that won, all of them
};

// One round: a row takes the label most of 16 of its neighbours have (of equals the one it has, then the one with the
// smallest hash).  16 lanes to a row, a neighbour each; labels are compared by rotating them past each other.  Which
// neighbours are taken changes with the round.  250,000 rows: 24 us, bound by L2's rate for single words (4 M labels, 165
// per ns; requesting the next row's column ahead changed nothing).  lab null: every row its own label.
__global__ void __launch_bounds__(kRoundThreads) cluster_round_kernel(int64_t n, const int32_t *rowptr, const int32_t *colidx,
                                                                      int round, const int32_t *lab, int32_t *nxt,
                                                                      RoundPart *parts)
{
    const int lane = threadIdx.x & 63, l = lane & 15, shift = lane & 48;
    unsigned same = 0, sampled = 0;
    const int64_t step = (int64_t)gridDim.x * (kRoundThreads / 16);
    for (int64_t r0 = (int64_t)blockIdx.x * (kRoundThreads / 16) + threadIdx.x / 64 * 4; r0 < n; r0 += step) {
        const int64_t r = r0 + (shift >> 4); // (r0 is uniform over the wavefront)
        int32_t x = -1, own = -1;            // no label
        int64_t len = 0;
        if (r < n) {
            const int64_t s = rowptr[r];
            len = rowptr[r + 1] - s;
            own = lab ? lab[r] : (int32_t)r;
            if (l < len) {
                const int32_t c = colidx[s + (len <= 16 ? l : ((l * 8 + round) * len) >> 7)];
                if ((uint32_t)c < (uint64_t)n) x = lab ? lab[c] : c; // (it is, short of unchecked arrays)
            }
        }
        const unsigned count = equals(x);
        const unsigned rank = x < 0 ? 0 : count << 27 | (unsigned)(x == own) << 26 | (0x3ffffffu - (mix((uint32_t)x) >> 6));
        unsigned top = rank;
        top = max(top, (unsigned)rotated<1>((int)top));
        top = max(top, (unsigned)rotated<2>((int)top));
        top = max(top, (unsigned)rotated<4>((int)top));
        top = max(top, (unsigned)rotated<8>((int)top));
        const unsigned winners = (unsigned)(__ballot(rank == top && x >= 0) >> shift) & 0xffffu;
        const int first = winners ? __ffs(winners) - 1 : 0;
        if (r < n && l == first) {
            nxt[r] = winners ? x : own;
            same += winners ? count : 0;
            sampled += (unsigned)(len < 16 ? len : 16);
        }
    }
    if (parts) {
        typedef hipcub::BlockReduce<unsigned, kRoundThreads> Reduce;
        __shared__ typename Reduce::TempStorage t1, t2;
        const unsigned a = Reduce(t1).Sum(same), b = Reduce(t2).Sum(sampled);
        if (threadIdx.x == 0) parts[blockIdx.x] = {a, b};
    }
}

// What the rounds came to: the sums of the last one, and of kPairs pairs of rows how many have one label (n times
// their share is the size of the label a row has, to within what a decision needs).
struct Stats {
    unsigned long long same, sampled, pairs;
};
constexpr unsigned kPairs = 1u << 17;
__global__ void __launch_bounds__(kRoundThreads) cluster_stats_kernel(int64_t n, const int32_t *lab, int n_parts,
                                                                      const RoundPart *parts, Stats *out)
{
    const unsigned i = blockIdx.x * kRoundThreads + threadIdx.x;
    const int64_t a = (int64_t)((unsigned long long)mix(2 * i + 1) * (unsigned long long)n >> 32);
    const int64_t b = (int64_t)((unsigned long long)mix(~(2 * i)) * (unsigned long long)n >> 32);
    const int equal = i < kPairs && a != b && lab[a] == lab[b];
    typedef hipcub::BlockReduce<unsigned long long, kRoundThreads> Reduce;
    __shared__ typename Reduce::TempStorage t1, t2;
    const int found = __syncthreads_count(equal);
    if (threadIdx.x == 0 && found) atomicAdd(&out->pairs, (unsigned long long)found);
    if (blockIdx.x == 0) {
        const bool in = (int)threadIdx.x < n_parts;
        const unsigned long long x = Reduce(t1).Sum(in ? parts[threadIdx.x].same : 0);
        const unsigned long long y = Reduce(t2).Sum(in ? parts[threadIdx.x].sampled : 0);
        if (threadIdx.x == 0) {
            out->same = x;
            out->sampled = y;
        }
    }
}
static_assert(kRoundBlocks <= kRoundThreads, "a thread per part");

// sort key of every listed item: a hash of its row's label
__global__ void __launch_bounds__(kThreads) cluster_keys_kernel(int64_t n, const int32_t *items, const int32_t *rows,
                                                                const int32_t *lab, uint32_t mask, uint32_t *key)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n) key[i] = mix((uint32_t)lab[rows[items[i]]]) & mask;
}

// ---- windows of communities: the column-window kernel over rows sorted by label, which stages a block's own rows of B.
// From memory then come only the vectors that leave the block (250,000 rows of 48 in communities of 500, K = 256: 577 us
// in the order by community, bound by what L2 delivers, 378 so).  Set up in 0.11 ms of kernels.
constexpr int kSmall = kRowsMost / 2; // communities of at most this many rows share a block

// Rows of every label, as kSizeParts sums of n each: atomics on one line take turns, and communities have hundreds of
// rows (250,000 rows: 26 us with one sum, 15 so).
constexpr int kSizeParts = 8;
__global__ void __launch_bounds__(kThreads) cluster_sizes_kernel(int64_t n, const int32_t *lab, int32_t *sizes)
{
    const int64_t r = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (r < n) atomicAdd(&sizes[(blockIdx.x & (kSizeParts - 1)) * n + lab[r]], 1);
}
__device__ __forceinline__ int32_t size_of(const int32_t *sizes, int64_t n, uint32_t label)
{
    int32_t s = 0;
#pragma unroll
    for (int k = 0; k < kSizeParts; ++k) s += sizes[k * n + label];
    return s;
}

// small communities first, each side by label
__global__ void __launch_bounds__(kThreads) cluster_order_kernel(int64_t n, const int32_t *lab, const int32_t *sizes,
                                                                 uint32_t large, uint32_t *key, uint32_t *row)
{
    const int64_t r = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (r < n) {
        key[r] = (uint32_t)lab[r] | (size_of(sizes, n, (uint32_t)lab[r]) > kSmall ? large : 0u);
        row[r] = (uint32_t)r;
    }
}

// Where the blocks begin, in the sorted order: at a community of more than kSmall rows and, if it has more than kRowsMost, at
// every even piece of it; of the others, at the first one that begins in each kSmall places (the last of a block then
// ends fewer than kRowsMost places on).  Also the lengths of the rows in that order.
__global__ void __launch_bounds__(kThreads) cluster_cut_kernel(int64_t n, const uint32_t *key, const int32_t *rows,
                                                               const int32_t *sizes, uint32_t large, const int32_t *rowptr,
                                                               int32_t *len, uint8_t *cut)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i > n) return;
    if (i == n) {
        len[i] = 0;
        return;
    }
    const int32_t r = rows[i];
    len[i] = rowptr[r + 1] - rowptr[r];
    const uint32_t k = key[i], before = i ? key[i - 1] : ~k;
    const int32_t s = size_of(sizes, n, k & (large - 1));
    bool c = k != before;
    if (s > kRowsMost) {
        int64_t lo = 0, hi = i; // the first place of this community
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (key[mid] < k)
                lo = mid + 1;
            else
                hi = mid;
        }
        const int32_t pieces = (s + kRowsMost - 1) / kRowsMost;
        c = (i - lo) % ((s + pieces - 1) / pieces) == 0;
    } else if (c && i && !(k & large)) {
        c = i / kSmall != (i - size_of(sizes, n, before & (large - 1))) / kSmall;
    }
    cut[i] = c;
}

struct WindowCount {
    unsigned long long hits;
    int32_t blocks;
};

// A workgroup per block, 16 lanes per row: a row's vectors inside the block go to its front as places, the others to its end
// from the back.  Whether a column is a row of the block is looked up in LDS: 250,000 rows of 48 105 us with an array of
// places in memory (12 M single words, L2's rate for those), 58 so, bound by the round trips of a row's chunks.
constexpr int kTable = 4 * kRowsMost;
constexpr int kAhead = 4; // chunks of 16 vectors of a row requested at a time
__global__ void __launch_bounds__(kRoundThreads) cluster_fill_kernel(int64_t n, const int32_t *ptr_in, WindowCount *count,
                                                                     const int32_t *rows, const int32_t *rowptr,
                                                                     const int32_t *colidx, const float *vals,
                                                                     const int32_t *new_rowptr,
                                                                     int32_t *ptr, int32_t *new_colidx, float *new_vals,
                                                                     int32_t *inner_end)
{
    const int blocks = count->blocks, b = blockIdx.x;
    if (b >= blocks) return;
    const int32_t b0 = ptr_in[b], b1 = b + 1 < blocks ? ptr_in[b + 1] : (int32_t)n;
    if (threadIdx.x == 0) {
        ptr[b] = b0;
        if (b + 1 == blocks) ptr[blocks] = (int32_t)n;
    }
    const int lane = threadIdx.x & 63, l = lane & 15, shift = lane & 48;
    const unsigned below = (1u << l) - 1;
    // the block's rows by their number: open addressing, at most a quarter full
    __shared__ int32_t held[kTable], at[kTable];
    for (int k = threadIdx.x; k < kTable; k += kRoundThreads) held[k] = -1;
    __syncthreads();
    for (int32_t i = b0 + threadIdx.x; i < b1; i += kRoundThreads) {
        const int32_t r = rows[i];
        unsigned k = mix((uint32_t)r) & (kTable - 1);
        while (atomicCAS(&held[k], -1, r) != -1) k = (k + 1) & (kTable - 1);
        at[k] = i;
    }
    __syncthreads();
    auto place_of = [&](int32_t c) {
        unsigned k = mix((uint32_t)c) & (kTable - 1);
        int32_t x = held[k];
        while (x != c && x != -1) {
            k = (k + 1) & (kTable - 1);
            x = held[k];
        }
        return x == c ? at[k] : -1;
    };
    constexpr int step = kRoundThreads / 16;
    unsigned hits = 0;
    int32_t i = b0 + threadIdx.x / 16, s = 0, e = 0, front = 0, back = 0;
    auto fetch = [&](int32_t j, int32_t &js, int32_t &je, int32_t &jf, int32_t &jb) {
        if (j >= b1) return;
        const int32_t r = rows[j];
        jf = new_rowptr[j];
        jb = new_rowptr[j + 1];
        js = rowptr[r];
        je = rowptr[r + 1];
    };
    fetch(i, s, e, front, back);
    while (i < b1) {
        int32_t s_next = 0, e_next = 0, front_next = 0, back_next = 0;
        fetch(i + step, s_next, e_next, front_next, back_next);
        const int32_t first = front;
        for (int32_t t = s; t < e; t += 16 * kAhead) {
            int32_t c[kAhead], p[kAhead];
            float v[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int32_t q = t + u * 16 + l;
                c[u] = q < e ? colidx[q] : -1;
                v[u] = q < e ? vals[q] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u) p[u] = c[u] >= 0 ? place_of(c[u]) : -1;
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const bool have = t + u * 16 + l < e, in = p[u] >= 0;
                const unsigned ins = (unsigned)(__ballot(in) >> shift) & 0xffffu;
                const unsigned outs = (unsigned)(__ballot(have && !in) >> shift) & 0xffffu;
                if (have) {
                    const int32_t to = in ? front + __popc(ins & below) : back - 1 - __popc(outs & below);
                    new_colidx[to] = in ? p[u] : c[u];
                    new_vals[to] = v[u];
                }
                front += __popc(ins);
                back -= __popc(outs);
            }
        }
        if (l == 0) {
            inner_end[i] = front;
            hits += (unsigned)(front - first);
        }
        i += step;
        s = s_next;
        e = e_next;
        front = front_next;
        back = back_next;
    }
    typedef hipcub::BlockReduce<unsigned, kRoundThreads> Reduce;
    __shared__ typename Reduce::TempStorage tmp;
    const unsigned all = Reduce(tmp).Sum(hits);
    if (threadIdx.x == 0 && all) atomicAdd(&count->hits, (unsigned long long)all);
}

} // namespace

hipError_t cluster_probe(int64_t n, int64_t nnz, const int32_t *d_rowptr, const int32_t *d_colidx, unsigned long long *d_out)
{
    hipLaunchKernelGGL(cluster_probe_kernel, dim3(kSamples / (kThreads / 64)), dim3(kThreads), 0, setup_stream(), n, nnz, d_rowptr,
                       d_colidx, d_out);
    return hipGetLastError();
}

bool cluster_probe_says(const unsigned long long found[2], int64_t n)
{
    // 64: a few times what chance leaves on small counts
    return (double)found[0] > 4.0 * (double)found[1] / (double)n + 64.0;
}

int cluster_rows(int64_t n, const int32_t *d_rowptr, const int32_t *d_colidx, int32_t **labels, double *mean_size, int *hip_err)
{
    *labels = nullptr;
    Scratch sc;
    int32_t *lab[2] = {nullptr, nullptr};
    RoundPart *parts = nullptr;
    Stats *d_stats = nullptr, h;
    for (int b = 0; b < 2; ++b) HIP_TRY(sc.alloc((void **)&lab[b], sizeof(int32_t) * n));
    HIP_TRY(sc.alloc((void **)&parts, sizeof(RoundPart) * kRoundBlocks));
    HIP_TRY(sc.alloc((void **)&d_stats, sizeof(Stats)));
    HIP_TRY(hipMemsetAsync(d_stats, 0, sizeof(Stats), setup_stream()));
    const int64_t need = (n + kRoundThreads / 16 - 1) / (kRoundThreads / 16);
    const int blocks = (int)(need < kRoundBlocks ? need : kRoundBlocks);
    for (int k = 0; k < kRounds; ++k) {
        hipLaunchKernelGGL(cluster_round_kernel, dim3(blocks), dim3(kRoundThreads), 0, setup_stream(), n, d_rowptr, d_colidx, k,
                           k ? lab[(k - 1) & 1] : (const int32_t *)nullptr, lab[k & 1],
                           k == kRounds - 1 ? parts : (RoundPart *)nullptr);
        HIP_TRY(hipGetLastError());
    }
    int32_t *const made = lab[(kRounds - 1) & 1];
    hipLaunchKernelGGL(cluster_stats_kernel, dim3(kPairs / kRoundThreads), dim3(kRoundThreads), 0, setup_stream(), n, made, blocks, parts,
                       d_stats);
    HIP_TRY(hipGetLastError());
    HIP_TRY(setup_copy(&h, d_stats, sizeof(h), hipMemcpyDeviceToHost));
    // Worth it where most neighbours share the row's label and the label's rows of B (64 columns of them at a time)
    // take up no more than half of an XCD's L2.
    const double mean = (double)h.pairs / kPairs * (double)n; // size of the label a row has
    if (2 * h.same >= h.sampled && h.sampled > 0 && mean <= 8192.0 && mean * 8 <= (double)n) {
        *labels = made;
        *mean_size = mean;
        sc.release(made);
    }
    return PCSR_OK;
}

int cluster_windows(int64_t n, int64_t nnz, const int32_t *d_rowptr, const int32_t *d_colidx, const float *d_vals,
                    const int32_t *d_labels, DeviceBuild *out, int *hip_err)
{
    Scratch sc;
    int32_t *sizes, *len, *ptr_in, *ptr, *new_rowptr, *new_colidx, *inner_end;
    uint32_t *key, *key_sorted, *row, *rows;
    float *new_vals;
    uint8_t *cut;
    WindowCount *count, h;
    void *tmp;
    size_t select_bytes = 0, scan_bytes = 0;
    // a large community's blocks have more than kSmall rows, and there is at most one of small ones per kSmall places
    const int64_t most = n / kSmall + n / kSmall + 2;
    const int bits = key_bits(n);
    const uint32_t large = 1u << bits;
    hipcub::CountingInputIterator<int32_t> places(0);
    HIP_TRY(sc.alloc((void **)&sizes, sizeof(int32_t) * kSizeParts * n));
    HIP_TRY(sc.alloc((void **)&key, sizeof(uint32_t) * n));
    HIP_TRY(sc.alloc((void **)&key_sorted, sizeof(uint32_t) * n));
    HIP_TRY(sc.alloc((void **)&row, sizeof(uint32_t) * n));
    HIP_TRY(sc.alloc((void **)&rows, sizeof(uint32_t) * n));
    HIP_TRY(sc.alloc((void **)&len, sizeof(int32_t) * (n + 1)));
    HIP_TRY(sc.alloc((void **)&cut, n));
    HIP_TRY(sc.alloc((void **)&ptr_in, sizeof(int32_t) * n));
    HIP_TRY(sc.alloc((void **)&ptr, sizeof(int32_t) * (most + 1)));
    HIP_TRY(sc.alloc((void **)&count, sizeof(WindowCount)));
    HIP_TRY(sc.alloc((void **)&new_rowptr, sizeof(int32_t) * (n + 1)));
    HIP_TRY(sc.alloc((void **)&new_colidx, sizeof(int32_t) * (nnz + 1)));
    HIP_TRY(sc.alloc((void **)&new_vals, sizeof(float) * (nnz + 1)));
    HIP_TRY(sc.alloc((void **)&inner_end, sizeof(int32_t) * n));
    HIP_TRY(hipcub::DeviceSelect::Flagged(nullptr, select_bytes, places, cut, ptr_in, &count->blocks, (int)n, setup_stream()));
    HIP_TRY(hipcub::DeviceScan::ExclusiveSum(nullptr, scan_bytes, len, new_rowptr, (int)(n + 1), setup_stream()));
    HIP_TRY(sc.alloc(&tmp, select_bytes > scan_bytes ? select_bytes : scan_bytes));
    HIP_TRY(hipMemsetAsync(sizes, 0, sizeof(int32_t) * kSizeParts * n, setup_stream()));
    HIP_TRY(hipMemsetAsync(count, 0, sizeof(WindowCount), setup_stream()));
    hipLaunchKernelGGL(cluster_sizes_kernel, dim3(blocks_for(n)), dim3(kThreads), 0, setup_stream(), n, d_labels, sizes);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(cluster_order_kernel, dim3(blocks_for(n)), dim3(kThreads), 0, setup_stream(), n, d_labels, sizes, large, key,
                       row);
    HIP_TRY(hipGetLastError());
    HIP_TRY(sort_pairs_u32(key, key_sorted, row, rows, n, bits + 1, sc));
    hipLaunchKernelGGL(cluster_cut_kernel, dim3(blocks_for(n + 1)), dim3(kThreads), 0, setup_stream(), n, key_sorted,
                       reinterpret_cast<const int32_t *>(rows), sizes, large, d_rowptr, len, cut);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipcub::DeviceSelect::Flagged(tmp, select_bytes, places, cut, ptr_in, &count->blocks, (int)n, setup_stream()));
    HIP_TRY(hipcub::DeviceScan::ExclusiveSum(tmp, scan_bytes, len, new_rowptr, (int)(n + 1), setup_stream()));
    hipLaunchKernelGGL(cluster_fill_kernel, dim3((unsigned)most), dim3(kRoundThreads), 0, setup_stream(), n, ptr_in, count,
                       reinterpret_cast<const int32_t *>(rows), d_rowptr, d_colidx, d_vals, new_rowptr, ptr, new_colidx, new_vals,
                       inner_end);
    HIP_TRY(hipGetLastError());
    HIP_TRY(setup_copy(&h, count, sizeof(h), hipMemcpyDeviceToHost));
    // as the column windows: half of the vectors inside, and blocks that are worth a workgroup
    if (2 * h.hits < (unsigned long long)nnz || n < 128 * (int64_t)h.blocks || h.blocks > most) return PCSR_OK;
    HIP_TRY(prepare_row_windows());
    out->win.rowptr = new_rowptr;
    out->win.colidx = new_colidx;
    out->win.val = new_vals;
    out->win.rows = reinterpret_cast<int32_t *>(rows);
    out->win.ptr = ptr;
    out->win.hi = inner_end;
    out->win.blocks = h.blocks;
    for (void *q : {(void *)new_rowptr, (void *)new_colidx, (void *)new_vals, (void *)rows, (void *)ptr, (void *)inner_end})
        sc.release(q);
    return PCSR_OK;
}

int cluster_key_bits(int64_t n)
{
    // Ten bits of the label's hash, one pass of the sort: rows of a few communities then alternate, whose rows of B
    // still fit an XCD's L2 together (n / 1024 rows, 64 columns at a time); above 8 M rows, twenty.
    return n <= (int64_t(1) << 23) ? 10 : 20;
}

hipError_t cluster_keys(int64_t n, const int32_t *d_labels, int64_t n_items, const int32_t *d_items, const int32_t *d_rows,
                        uint32_t *d_key)
{
    hipLaunchKernelGGL(cluster_keys_kernel, dim3(blocks_for(n_items)), dim3(kThreads), 0, setup_stream(), n_items, d_items, d_rows, d_labels,
                       (1u << cluster_key_bits(n)) - 1, d_key);
    return hipGetLastError();
}

} // namespace pcsr
