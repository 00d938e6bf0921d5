// Relabelling pre-step and transpose on the GPU (see pcsr_relabel_gpu.h).
#include "pcsr_relabel_gpu.h"

#include <hipcub/hipcub.hpp>

#include "pcsr_build_gpu.h"
#include "pcsr_gpu_util.h"

namespace pcsr {
namespace {

// ---- transpose

// (row, value) of every nonzero, the payload of the sort by column
__global__ void __launch_bounds__(kThreads) row_value_kernel(int64_t n_rows, int64_t nnz, const int32_t *rowptr,
                                                             const float *vals, uint2 *out)
{
    __shared__ RowSlice slice;
    const int64_t t0 = (int64_t)blockIdx.x * kSlice, t1 = t0 + kSlice < nnz ? t0 + kSlice : nnz;
    slice.find(rowptr, n_rows, t0, t1);
    for (int64_t t = t0 + threadIdx.x; t < t1; t += kThreads)
        out[t] = make_uint2((unsigned)slice.row(rowptr, n_rows, t), __float_as_uint(vals[t]));
}

// rowptr of sorted keys: the first position of a key >= c, for every c <= n
__global__ void __launch_bounds__(kThreads) lower_bounds_kernel(int64_t n, int64_t nnz, const int32_t *keys,
                                                                int32_t *rowptr)
{
    const int64_t c = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (c > n) return;
    int64_t lo = 0, hi = nnz;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (keys[mid] < c)
            lo = mid + 1;
        else
            hi = mid;
    }
    rowptr[c] = (int32_t)lo;
}

__global__ void __launch_bounds__(kThreads) split_pairs_kernel(int64_t nnz, const uint2 *in, int32_t *colidx, float *vals)
{
    const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (t >= nnz) return;
    const uint2 p = in[t];
    colidx[t] = (int32_t)p.x;
    vals[t] = __uint_as_float(p.y);
}

// ---- label propagation

// deterministic tie-break priority of a label in a given round (as on the host: lowbias32)
__device__ __forceinline__ uint32_t mix(uint32_t x, uint32_t round)
{
    x ^= round * 0x9E3779B9u;
    x ^= x >> 16;
    x *= 0x7feb352du;
    x ^= x >> 15;
    x *= 0x846ca68bu;
    x ^= x >> 16;
    return x;
}

// Order of the candidates of a row: more neighbours with the label, then the label the node
// has, then the smaller hash.  mix is a bijection, so no two labels of a row are equal.
__device__ __forceinline__ unsigned long long label_rank(int count, uint32_t label, uint32_t own, uint32_t round)
{
    return ((unsigned long long)(unsigned)count << 33) | ((unsigned long long)(label == own) << 32) |
           (0xffffffffu - mix(label, round));
}

struct Rows {
    const int32_t *rowptr, *colidx;
    const int32_t *medium, *large; // rows of more than 64 / kMediumRow nonzeros
    int32_t *counts;               // how many of them: [0] medium, [1] large; [2] a bad array; [3] stuck
};
constexpr int kMediumRow = 1024;

// sound row pointer and columns; lists of the longer rows
__global__ void __launch_bounds__(kThreads) classify_kernel(int64_t n, int64_t n_cols, int64_t nnz, Rows r,
                                                            int32_t *medium, int32_t *large)
{
    const int64_t stride = (int64_t)gridDim.x * kThreads, i0 = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    bool bad = false;
    for (int64_t i = i0; i < n; i += stride) {
        const int64_t s = r.rowptr[i], e = r.rowptr[i + 1];
        if (s < 0 || s > e || e > nnz) {
            bad = true;
        } else if (medium) {
            if (e - s > kMediumRow)
                large[atomicAdd(&r.counts[1], 1)] = (int32_t)i;
            else if (e - s > 64)
                medium[atomicAdd(&r.counts[0], 1)] = (int32_t)i;
        }
    }
    for (int64_t t = medium ? nnz : i0; t < nnz; t += stride) { // columns: checked by the pass without lists
        const int32_t c = r.colidx[t];
        bad |= c < 0 || c >= n_cols;
    }
    if (bad) r.counts[2] = 1;
}

// whether the rounds before this one have converged (fewer than 0.5 % of the nodes moved)
__device__ __forceinline__ bool converged(const int32_t *changed, int round, int64_t n)
{
    return round > 0 && (int64_t)changed[round - 1] * 200 < n;
}

// One round for rows of up to 64 nonzeros, a wavefront per row: a lane holds one neighbour's
// label and counts its equals by having every lane's broadcast.  No sort, no LDS.
__global__ void __launch_bounds__(kThreads) propagate_short_kernel(int64_t n, Rows r, const int32_t *lab, int32_t *nxt,
                                                                   int slot, uint32_t round, int32_t *changed)
{
    if (converged(changed, slot, n)) return;
    const int lane = threadIdx.x & 63;
    int moved = 0;
    for (int64_t i = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6); i < n;
         i += (int64_t)gridDim.x * (kThreads / 64)) {
        const int s = __builtin_amdgcn_readfirstlane(r.rowptr[i]);
        const int len = __builtin_amdgcn_readfirstlane(r.rowptr[i + 1]) - s;
        if (len > 64) continue;
        const int32_t own = lab[i];
        int32_t best = own;
        if (len > 0) {
            const int32_t x = lane < len ? lab[r.colidx[s + lane]] : -1;
            int count = 0;
            for (int j = 0; j < len; ++j) count += __builtin_amdgcn_readlane(x, j) == x;
            const unsigned long long mine = lane < len ? label_rank(count, x, own, round) : 0;
            unsigned long long top = mine;
#pragma unroll
            for (int m = 1; m < 64; m <<= 1) {
                const unsigned long long o = __shfl_xor(top, m);
                top = o > top ? o : top;
            }
            best = __builtin_amdgcn_readlane(x, __builtin_ctzll(__ballot(mine == top)));
        }
        if (lane == 0) nxt[i] = best;
        moved += best != own;
    }
    __shared__ int sum[kThreads / 64];
    if (lane == 0) sum[threadIdx.x >> 6] = moved;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
        for (int w = 0; w < kThreads / 64; ++w) t += sum[w];
        if (t) atomicAdd(&changed[slot], t);
    }
}

// Longer rows, a workgroup per row: the labels are counted in an open-addressing table in LDS.
// A row with more labels than fit is taken in several passes, each over the labels whose
// hash falls into its share; the table is at most half full then.
template <int T, int TABLE>
__global__ void __launch_bounds__(T) propagate_long_kernel(int64_t n, Rows r, const int32_t *list, const int32_t *n_list,
                                                           const int32_t *lab, int32_t *nxt, int slot, uint32_t round,
                                                           int32_t *changed)
{
    if (converged(changed, slot, n)) return;
    __shared__ int32_t key[TABLE];
    __shared__ int32_t cnt[TABLE];
    __shared__ unsigned long long top;
    int moved = 0;
    for (int q = blockIdx.x; q < *n_list; q += gridDim.x) {
        const int64_t i = list[q];
        const int64_t s = r.rowptr[i], e = r.rowptr[i + 1];
        const int32_t own = lab[i];
        const unsigned passes = (unsigned)((e - s + TABLE / 2 - 1) / (TABLE / 2));
        if (threadIdx.x == 0) top = 0;
        for (unsigned pass = 0; pass < passes; ++pass) {
            for (int k = threadIdx.x; k < TABLE; k += T) {
                key[k] = -1;
                cnt[k] = 0;
            }
            __syncthreads();
            for (int64_t t = s + threadIdx.x; t < e; t += T) {
                const int32_t x = lab[r.colidx[t]];
                const uint32_t h = mix((uint32_t)x, 0x51ED27u);
                if (passes > 1 && (h >> 16) % passes != pass) continue;
                int k = h & (TABLE - 1), tries = 0;
                for (; tries < TABLE; ++tries, k = (k + 1) & (TABLE - 1)) {
                    const int32_t old = atomicCAS(&key[k], -1, x);
                    if (old == -1 || old == x) {
                        atomicAdd(&cnt[k], 1);
                        break;
                    }
                }
                if (tries == TABLE) r.counts[3] = 1; // does not happen short of a hash gone wrong: host
            }
            __syncthreads();
            for (int k = threadIdx.x; k < TABLE; k += T)
                if (key[k] >= 0) atomicMax(&top, label_rank(cnt[k], key[k], own, round));
            __syncthreads();
            // the label that leads so far; a later pass may overtake it
            for (int k = threadIdx.x; k < TABLE; k += T)
                if (key[k] >= 0 && label_rank(cnt[k], key[k], own, round) == top) nxt[i] = key[k];
            __syncthreads();
        }
        if (threadIdx.x == 0) moved += nxt[i] != own;
    }
    if (threadIdx.x == 0 && moved) atomicAdd(&changed[slot], moved);
}

__global__ void __launch_bounds__(kThreads) iota_kernel(int64_t n, int32_t *a, int32_t *b)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n) {
        a[i] = (int32_t)i;
        if (b) b[i] = (int32_t)i;
    }
}

// perm of a sorted order; number of distinct keys (may be null)
__global__ void __launch_bounds__(kThreads) number_kernel(int64_t n, const int32_t *order, const int32_t *key,
                                                          int32_t *perm, int32_t *distinct)
{
    const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    bool first = false;
    if (k < n) {
        perm[order[k]] = (int32_t)k;
        first = key && (k == 0 || key[k] != key[k - 1]);
    }
    if (key) {
        const int c = __popcll(__ballot(first));
        if ((threadIdx.x & 63) == 0 && c) atomicAdd(distinct, c);
    }
}

// ---- relabelled matrix

// inv of perm; flag[0] = 1 if perm is no permutation
__global__ void __launch_bounds__(kThreads) invert_kernel(int64_t n, const int32_t *perm, int32_t *inv, int32_t *flag)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    const int32_t p = perm[i];
    if (p < 0 || p >= n || atomicCAS(&inv[p], -1, (int32_t)i) != -1) *flag = 1;
}

__global__ void __launch_bounds__(kThreads) permuted_len_kernel(int64_t n, const int32_t *rowptr, const int32_t *inv,
                                                                int32_t *len)
{
    const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (k > n) return;
    len[k] = k < n ? rowptr[inv[k] + 1] - rowptr[inv[k]] : 0;
}

// sort key of every nonzero: new row, new column
__global__ void __launch_bounds__(kThreads) permuted_key_kernel(int64_t n, int64_t nnz, const int32_t *rowptr,
                                                                const int32_t *colidx, const int32_t *perm, int bits,
                                                                unsigned long long *key)
{
    __shared__ RowSlice slice;
    const int64_t t0 = (int64_t)blockIdx.x * kSlice, t1 = t0 + kSlice < nnz ? t0 + kSlice : nnz;
    slice.find(rowptr, n, t0, t1);
    for (int64_t t = t0 + threadIdx.x; t < t1; t += kThreads)
        key[t] = ((unsigned long long)(unsigned)perm[slice.row(rowptr, n, t)] << bits) | (unsigned)perm[colidx[t]];
}

// columns of the sorted keys; flag[0] = 1 if a row holds a column twice
__global__ void __launch_bounds__(kThreads) permuted_cols_kernel(int64_t nnz, const unsigned long long *key, int bits,
                                                                 int32_t *colidx, int32_t *flag)
{
    const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (t >= nnz) return;
    colidx[t] = (int32_t)(key[t] & ((1ull << bits) - 1));
    if (t > 0 && key[t] == key[t - 1]) *flag = 1;
}

__global__ void __launch_bounds__(kThreads) count_columns_kernel(int64_t nnz, const int32_t *colidx, uint32_t *refs)
{
    const int64_t stride = (int64_t)gridDim.x * kThreads;
    for (int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x; t < nnz; t += stride) atomicAdd(&refs[colidx[t]], 1u);
}

template <class K, class T>
hipError_t sort_pairs(const K *kin, K *kout, const T *vin, T *vout, int64_t n, int bits, bool descending, Scratch &sc)
{
    size_t bytes = 0;
    void *tmp = nullptr;
    auto go = [&]() {
        return descending ? hipcub::DeviceRadixSort::SortPairsDescending(tmp, bytes, kin, kout, vin, vout, (int)n, 0, bits)
                          : hipcub::DeviceRadixSort::SortPairs(tmp, bytes, kin, kout, vin, vout, (int)n, 0, bits);
    };
    hipError_t e = go();
    if (e != hipSuccess) return e;
    e = sc.alloc(&tmp, bytes);
    return e == hipSuccess ? go() : e;
}

// every failure of the GPU side leaves the work to the host
#define TRY_GPU(expr)                \
    do {                             \
        if ((expr) != hipSuccess) {  \
            (void)hipGetLastError(); \
            return kUseHost;         \
        }                            \
    } while (0)

// Host CSR pattern in device memory, with its rows classified.
struct DevicePattern {
    Rows r = {};
    int32_t *rowptr = nullptr, *colidx = nullptr, *medium = nullptr, *large = nullptr;
    int upload(int64_t n, int64_t n_cols, int64_t nnz, const int32_t *h_rowptr, const int32_t *h_colidx, bool lists,
               Scratch &sc)
    {
        int32_t *counts = nullptr;
        TRY_GPU(sc.alloc((void **)&rowptr, sizeof(int32_t) * (n + 1)));
        TRY_GPU(sc.alloc((void **)&colidx, sizeof(int32_t) * (nnz + 1)));
        TRY_GPU(sc.alloc((void **)&counts, sizeof(int32_t) * 4));
        if (lists) {
            // rows of more than 64 / kMediumRow nonzeros there can be at most
            TRY_GPU(sc.alloc((void **)&medium, sizeof(int32_t) * (nnz / 65 + 1)));
            TRY_GPU(sc.alloc((void **)&large, sizeof(int32_t) * (nnz / (kMediumRow + 1) + 1)));
        }
        TRY_GPU(copy_to_device(rowptr, h_rowptr, sizeof(int32_t) * (n + 1)));
        TRY_GPU(copy_to_device(colidx, h_colidx, sizeof(int32_t) * nnz));
        r.rowptr = rowptr;
        r.colidx = colidx;
        r.counts = counts;
        // rows first: with a broken row pointer the lists could overflow
        TRY_GPU(hipMemsetAsync(counts, 0, sizeof(int32_t) * 4, nullptr));
        hipLaunchKernelGGL(classify_kernel, dim3(strided_blocks(n > nnz ? n : nnz)), dim3(kThreads), 0, 0, n, n_cols,
                           nnz, r, (int32_t *)nullptr, (int32_t *)nullptr);
        TRY_GPU(hipGetLastError());
        int32_t h[4];
        TRY_GPU(hipMemcpy(h, counts, sizeof(h), hipMemcpyDeviceToHost));
        if (h[2]) return kUseHost;
        if (lists) {
            hipLaunchKernelGGL(classify_kernel, dim3(strided_blocks(n)), dim3(kThreads), 0, 0, n, n_cols, nnz, r, medium,
                               large);
            TRY_GPU(hipGetLastError());
            r.medium = medium;
            r.large = large;
        }
        return PCSR_OK;
    }
};

} // namespace

bool relabel_on_gpu(int64_t nnz)
{
    // below this the launches and waits cost more than the host threads take
    if (nnz < 200000) return false;
    static const bool there = [] {
        int count = 0;
        const bool ok = hipGetDeviceCount(&count) == hipSuccess && count > 0;
        if (!ok) (void)hipGetLastError();
        return ok;
    }();
    return there;
}

int transpose_device(int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t *d_rowptr, const int32_t *d_colidx,
                     const float *d_vals, int32_t **t_rowptr, int32_t **t_colidx, float **t_vals, int *hip_err)
{
    Scratch sc;
    int32_t *keys = nullptr, *rp = nullptr, *ci = nullptr;
    float *va = nullptr;
    uint2 *in = nullptr, *sorted = nullptr;
    HIP_TRY(sc.alloc((void **)&rp, sizeof(int32_t) * (n_cols + 1)));
    HIP_TRY(sc.alloc((void **)&ci, sizeof(int32_t) * (nnz + 1)));
    HIP_TRY(sc.alloc((void **)&va, sizeof(float) * (nnz + 1)));
    HIP_TRY(sc.alloc((void **)&keys, sizeof(int32_t) * (nnz + 1)));
    HIP_TRY(sc.alloc((void **)&in, sizeof(uint2) * (nnz + 1)));
    HIP_TRY(sc.alloc((void **)&sorted, sizeof(uint2) * (nnz + 1)));
    if (nnz > 0) {
        hipLaunchKernelGGL(row_value_kernel, dim3((unsigned)((nnz + kSlice - 1) / kSlice)), dim3(kThreads), 0, 0, n_rows,
                           nnz, d_rowptr, d_vals, in);
        HIP_TRY(hipGetLastError());
        // stable, and the nonzeros come in row order: every output row ends up ascending
        HIP_TRY(sort_pairs(d_colidx, keys, reinterpret_cast<const unsigned long long *>(in),
                           reinterpret_cast<unsigned long long *>(sorted), nnz, key_bits(n_cols), false, sc));
        hipLaunchKernelGGL(split_pairs_kernel, dim3(blocks_for(nnz)), dim3(kThreads), 0, 0, nnz, sorted, ci, va);
        HIP_TRY(hipGetLastError());
    }
    hipLaunchKernelGGL(lower_bounds_kernel, dim3(blocks_for(n_cols + 1)), dim3(kThreads), 0, 0, n_cols, nnz, keys, rp);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(nullptr));
    *t_rowptr = rp;
    *t_colidx = ci;
    *t_vals = va;
    sc.release(rp);
    sc.release(ci);
    sc.release(va);
    return PCSR_OK;
}

int transpose_gpu(int64_t n_rows, int64_t n_cols, const int32_t *rowptr, const int32_t *colidx, const float *vals,
                  int32_t *out_rowptr, int32_t *out_colidx, float *out_vals)
{
    const int64_t nnz = rowptr[n_rows];
    Scratch sc;
    DevicePattern m;
    int rc = m.upload(n_rows, n_cols, nnz, rowptr, colidx, false, sc), herr = 0;
    if (rc != PCSR_OK) return rc;
    int32_t *rp = nullptr, *ci = nullptr;
    float *d_vals = nullptr, *va = nullptr;
    TRY_GPU(sc.alloc((void **)&d_vals, sizeof(float) * nnz));
    TRY_GPU(copy_to_device(d_vals, vals, sizeof(float) * nnz));
    rc = transpose_device(n_rows, n_cols, nnz, m.rowptr, m.colidx, d_vals, &rp, &ci, &va, &herr);
    if (rc != PCSR_OK) return kUseHost;
    hipError_t e = copy_to_host(out_rowptr, rp, sizeof(int32_t) * (n_cols + 1));
    if (e == hipSuccess) e = copy_to_host(out_colidx, ci, sizeof(int32_t) * nnz);
    if (e == hipSuccess) e = copy_to_host(out_vals, va, sizeof(float) * nnz);
    (void)hipStreamSynchronize(nullptr);
    pool_free(rp);
    pool_free(ci);
    pool_free(va);
    TRY_GPU(e);
    return PCSR_OK;
}

int reorder_gpu(int64_t n, const int32_t *rowptr, const int32_t *colidx, int32_t max_rounds, int32_t *perm,
                int64_t *n_clusters)
{
    const int64_t nnz = rowptr[n];
    Scratch sc;
    DevicePattern m;
    const int rc = m.upload(n, n, nnz, rowptr, colidx, true, sc);
    if (rc != PCSR_OK) return rc;
    constexpr int kBatch = 8; // rounds enqueued before the host looks
    int32_t *lab[2] = {nullptr, nullptr}, *changed = nullptr, *ids = nullptr;
    for (int b = 0; b < 2; ++b) TRY_GPU(sc.alloc((void **)&lab[b], sizeof(int32_t) * n));
    TRY_GPU(sc.alloc((void **)&ids, sizeof(int32_t) * n));
    TRY_GPU(sc.alloc((void **)&changed, sizeof(int32_t) * (kBatch + 1)));
    hipLaunchKernelGGL(iota_kernel, dim3(blocks_for(n)), dim3(kThreads), 0, 0, n, lab[0], ids);
    TRY_GPU(hipGetLastError());
    int at = 0;
    const unsigned waves = (unsigned)((n + kThreads / 64 - 1) / (kThreads / 64));
    const unsigned blocks = waves < 2048 ? waves : 2048;
    for (int32_t done = 0; done < max_rounds;) {
        const int batch = max_rounds - done < kBatch ? max_rounds - done : kBatch;
        TRY_GPU(hipMemsetAsync(changed, 0, sizeof(int32_t) * (kBatch + 1), nullptr));
        for (int b = 0; b < batch; ++b) {
            const int32_t *from = lab[(at + b) & 1];
            int32_t *to = lab[(at + b + 1) & 1];
            const uint32_t round = (uint32_t)(done + b);
            hipLaunchKernelGGL(propagate_short_kernel, dim3(blocks), dim3(kThreads), 0, 0, n, m.r, from, to, b, round,
                               changed);
            TRY_GPU(hipGetLastError());
            hipLaunchKernelGGL((propagate_long_kernel<256, 2048>), dim3(2048), dim3(256), 0, 0, n, m.r, m.r.medium,
                               m.r.counts, from, to, b, round, changed);
            TRY_GPU(hipGetLastError());
            hipLaunchKernelGGL((propagate_long_kernel<1024, 8192>), dim3(512), dim3(1024), 0, 0, n, m.r, m.r.large,
                               m.r.counts + 1, from, to, b, round, changed);
            TRY_GPU(hipGetLastError());
        }
        int32_t h[kBatch], counts[4];
        TRY_GPU(hipMemcpyAsync(counts, m.r.counts, sizeof(counts), hipMemcpyDeviceToHost, nullptr));
        TRY_GPU(hipMemcpy(h, changed, sizeof(int32_t) * kBatch, hipMemcpyDeviceToHost));
        if (counts[3]) return kUseHost;
        int ran = batch;
        bool over = false;
        for (int b = 0; b < batch && !over; ++b)
            if ((int64_t)h[b] * 200 < n) {
                ran = b + 1;
                over = true;
            }
        at = (at + ran) & 1;
        done += ran;
        if (over) break;
    }
    // clusters in order of their label, members in original order
    int32_t *order = nullptr, *d_perm = nullptr, *distinct = nullptr, *sorted = lab[at ^ 1], clusters = 0;
    TRY_GPU(sc.alloc((void **)&order, sizeof(int32_t) * n));
    TRY_GPU(sc.alloc((void **)&d_perm, sizeof(int32_t) * n));
    TRY_GPU(sc.alloc((void **)&distinct, sizeof(int32_t)));
    TRY_GPU(hipMemsetAsync(distinct, 0, sizeof(int32_t), nullptr));
    TRY_GPU(sort_pairs(lab[at], sorted, ids, order, n, key_bits(n), false, sc));
    hipLaunchKernelGGL(number_kernel, dim3(blocks_for(n)), dim3(kThreads), 0, 0, n, order, sorted, d_perm, distinct);
    TRY_GPU(hipGetLastError());
    TRY_GPU(hipMemcpy(&clusters, distinct, sizeof(clusters), hipMemcpyDeviceToHost));
    TRY_GPU(copy_to_host(perm, d_perm, sizeof(int32_t) * n));
    if (n_clusters) *n_clusters = clusters;
    return PCSR_OK;
}

int degree_order_gpu(int64_t n, const int32_t *rowptr, const int32_t *colidx, int32_t *perm)
{
    const int64_t nnz = rowptr[n];
    Scratch sc;
    DevicePattern m;
    const int rc = m.upload(n, n, nnz, rowptr, colidx, false, sc);
    if (rc != PCSR_OK) return rc;
    uint32_t *refs = nullptr, *sorted = nullptr;
    int32_t *ids = nullptr, *order = nullptr, *d_perm = nullptr;
    TRY_GPU(sc.alloc((void **)&refs, sizeof(uint32_t) * n));
    TRY_GPU(sc.alloc((void **)&sorted, sizeof(uint32_t) * n));
    TRY_GPU(sc.alloc((void **)&ids, sizeof(int32_t) * n));
    TRY_GPU(sc.alloc((void **)&order, sizeof(int32_t) * n));
    TRY_GPU(sc.alloc((void **)&d_perm, sizeof(int32_t) * n));
    TRY_GPU(hipMemsetAsync(refs, 0, sizeof(uint32_t) * n, nullptr));
    hipLaunchKernelGGL(iota_kernel, dim3(blocks_for(n)), dim3(kThreads), 0, 0, n, ids, (int32_t *)nullptr);
    TRY_GPU(hipGetLastError());
    hipLaunchKernelGGL(count_columns_kernel, dim3(strided_blocks(nnz)), dim3(kThreads), 0, 0, nnz, m.colidx, refs);
    TRY_GPU(hipGetLastError());
    TRY_GPU(sort_pairs(refs, sorted, ids, order, n, key_bits(nnz + 1), true, sc)); // descending, stable
    hipLaunchKernelGGL(number_kernel, dim3(blocks_for(n)), dim3(kThreads), 0, 0, n, order, (const int32_t *)nullptr,
                       d_perm, (int32_t *)nullptr);
    TRY_GPU(hipGetLastError());
    TRY_GPU(copy_to_host(perm, d_perm, sizeof(int32_t) * n));
    return PCSR_OK;
}

int permute_gpu(int64_t n, const int32_t *rowptr, const int32_t *colidx, const float *vals, const int32_t *perm,
                int32_t *out_rowptr, int32_t *out_colidx, float *out_vals)
{
    const int64_t nnz = rowptr[n];
    Scratch sc;
    int32_t *d_perm = nullptr, *inv = nullptr, *flag = nullptr, *len = nullptr, *rp = nullptr, *ci = nullptr, bad = 0;
    float *va = nullptr, *va_out = nullptr;
    unsigned long long *key = nullptr, *sorted = nullptr;
    TRY_GPU(sc.alloc((void **)&d_perm, sizeof(int32_t) * n));
    TRY_GPU(sc.alloc((void **)&inv, sizeof(int32_t) * n));
    TRY_GPU(sc.alloc((void **)&flag, sizeof(int32_t)));
    TRY_GPU(sc.alloc((void **)&len, sizeof(int32_t) * (n + 1)));
    TRY_GPU(sc.alloc((void **)&rp, sizeof(int32_t) * (n + 1)));
    TRY_GPU(copy_to_device(d_perm, perm, sizeof(int32_t) * n));
    TRY_GPU(hipMemsetAsync(inv, 0xff, sizeof(int32_t) * n, nullptr));
    TRY_GPU(hipMemsetAsync(flag, 0, sizeof(int32_t), nullptr));
    hipLaunchKernelGGL(invert_kernel, dim3(blocks_for(n)), dim3(kThreads), 0, 0, n, d_perm, inv, flag);
    TRY_GPU(hipGetLastError());
    DevicePattern m;
    const int rc = m.upload(n, n, nnz, rowptr, colidx, false, sc);
    if (rc != PCSR_OK) return rc;
    TRY_GPU(hipMemcpy(&bad, flag, sizeof(bad), hipMemcpyDeviceToHost));
    if (bad) return kUseHost;
    hipLaunchKernelGGL(permuted_len_kernel, dim3(blocks_for(n + 1)), dim3(kThreads), 0, 0, n, m.rowptr, inv, len);
    TRY_GPU(hipGetLastError());
    size_t bytes = 0;
    void *tmp = nullptr;
    TRY_GPU(hipcub::DeviceScan::ExclusiveSum(nullptr, bytes, len, rp, (int)(n + 1)));
    TRY_GPU(sc.alloc(&tmp, bytes));
    TRY_GPU(hipcub::DeviceScan::ExclusiveSum(tmp, bytes, len, rp, (int)(n + 1)));
    TRY_GPU(sc.alloc((void **)&va, sizeof(float) * nnz));
    TRY_GPU(sc.alloc((void **)&va_out, sizeof(float) * nnz));
    TRY_GPU(sc.alloc((void **)&ci, sizeof(int32_t) * nnz));
    TRY_GPU(sc.alloc((void **)&key, sizeof(long long) * nnz));
    TRY_GPU(sc.alloc((void **)&sorted, sizeof(long long) * nnz));
    TRY_GPU(copy_to_device(va, vals, sizeof(float) * nnz));
    const int bits = key_bits(n);
    hipLaunchKernelGGL(permuted_key_kernel, dim3((unsigned)((nnz + kSlice - 1) / kSlice)), dim3(kThreads), 0, 0, n, nnz,
                       m.rowptr, m.colidx, d_perm, bits, key);
    TRY_GPU(hipGetLastError());
    TRY_GPU(sort_pairs(key, sorted, reinterpret_cast<const uint32_t *>(va), reinterpret_cast<uint32_t *>(va_out), nnz,
                       2 * bits, false, sc));
    hipLaunchKernelGGL(permuted_cols_kernel, dim3(blocks_for(nnz)), dim3(kThreads), 0, 0, nnz, sorted, bits, ci, flag);
    TRY_GPU(hipGetLastError());
    TRY_GPU(hipMemcpy(&bad, flag, sizeof(bad), hipMemcpyDeviceToHost));
    if (bad) return kUseHost; // a column twice in a row: their order is the host sort's business
    TRY_GPU(copy_to_host(out_rowptr, rp, sizeof(int32_t) * (n + 1)));
    TRY_GPU(copy_to_host(out_colidx, ci, sizeof(int32_t) * nnz));
    TRY_GPU(copy_to_host(out_vals, va_out, sizeof(float) * nnz));
    return PCSR_OK;
}

} // namespace pcsr
