// Relabelling pre-step and transpose on the GPU (see pcsr_relabel_gpu.h).
#include "pcsr_relabel_gpu.h"

#include <hipcub/hipcub.hpp>

#include "pcsr_build_gpu.h"
#include "pcsr_gpu_util.h"
#include "pcsr_sort_gpu.h"

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
    x ^= round * 0x9E3779B9u; // the rest: lowbias32, a published 32-bit hash (C. Wellons' hash-prospector)
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
    int32_t *counts;               // how many of them: [0] medium, [1] large; [2] a bad array; [3] stuck; [4] longest row
};
constexpr int kMediumRow = 1024;

// sound row pointer and columns; lists of the longer rows
__global__ void __launch_bounds__(kThreads) classify_kernel(int64_t n, int64_t n_cols, int64_t nnz, Rows r,
                                                            int32_t *medium, int32_t *large)
{
    const int64_t stride = (int64_t)gridDim.x * kThreads, i0 = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    bool bad = false;
    int longest = 0;
    for (int64_t i = i0; i < n; i += stride) {
        const int64_t s = r.rowptr[i], e = r.rowptr[i + 1];
        if (s < 0 || s > e || e > nnz) {
            bad = true;
        } else if (!medium) {
            longest = max(longest, (int)(e - s));
        } else {
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
    if (medium) return; // the whole grid
    typedef hipcub::BlockReduce<int, kThreads> Reduce;
    __shared__ typename Reduce::TempStorage tmp;
    longest = Reduce(tmp).Reduce(longest, hipcub::Max());
    // (most workgroups find the longest row so far there already)
    if (threadIdx.x == 0 && longest > *(volatile int32_t *)&r.counts[4]) atomicMax(&r.counts[4], longest);
}

// whether the rounds before this one have converged (fewer than 0.5 % of the nodes moved)
__device__ __forceinline__ bool converged(const int32_t *changed, int round, int64_t n)
{
    return round > 0 && (int64_t)changed[round - 1] * 200 < n;
}

template <int CTRL> __device__ __forceinline__ unsigned dpp(unsigned x)
{
    return (unsigned)__builtin_amdgcn_mov_dpp((int)x, CTRL, 0xf, 0xf, true);
}
__device__ __forceinline__ unsigned wave_max(unsigned x) // of all 64 lanes, uniform
{
    x = max(x, dpp<0x121>(x)); // row_ror 1, 2, 4, 8
    x = max(x, dpp<0x122>(x));
    x = max(x, dpp<0x124>(x));
    x = max(x, dpp<0x128>(x));
    return max(max((unsigned)__builtin_amdgcn_readlane((int)x, 0), (unsigned)__builtin_amdgcn_readlane((int)x, 16)),
               max((unsigned)__builtin_amdgcn_readlane((int)x, 32), (unsigned)__builtin_amdgcn_readlane((int)x, 48)));
}

// One round for rows of up to 64 nonzeros, a wavefront per row, a lane per neighbour.  Labels are taken one at a time and
// counted by a ballot until none that is left can lead: once communities have formed that is after a step or two.  Where
// kTries labels have not decided it, every lane's label is counted by having every lane's broadcast.  Bound by vector
// instructions: 10 M nonzeros 97 us a round on average over eight, 126 with all rows counted the second way.
constexpr int kTries = 6;
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
        const int32_t own = __builtin_amdgcn_readfirstlane(lab[i]);
        int32_t best = own;
        if (len > 0) {
            const int32_t x = lane < len ? lab[r.colidx[s + lane]] : -1;
            unsigned long long left = __ballot(lane < len);
            int most = 0;
            uint32_t best_hash = 0;
            int t = 0;
            for (; t < kTries && __popcll(left) >= max(most, 1); ++t) {
                const int32_t y = __builtin_amdgcn_readlane(x, __builtin_ctzll(left));
                const unsigned long long m = __ballot(x == y);
                const int count = __popcll(m);
                left &= ~m;
                if (count < most || (count == most && best == own)) continue;
                const uint32_t hash = mix((uint32_t)y, round);
                if (count > most || y == own || hash < best_hash) {
                    most = count;
                    best = y;
                    best_hash = hash;
                }
            }
            if (__popcll(left) >= max(most, 1)) {
                int count = 0;
                for (int j = 0; j < len; ++j) count += __builtin_amdgcn_readlane(x, j) == x;
                const unsigned mine = lane < len ? (unsigned)count : 0;
                const unsigned top = wave_max(mine);
                const bool leads = mine == top;
                if (__ballot(leads && x == own)) {
                    best = own;
                } else { // no two labels have one hash
                    const unsigned h = leads ? 0xffffffffu - mix((uint32_t)x, round) : 0;
                    const unsigned low = wave_max(h);
                    best = __builtin_amdgcn_readlane(x, __builtin_ctzll(__ballot(leads && h == low)));
                }
            }
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

// length and old first nonzero of every new row
__global__ void __launch_bounds__(kThreads) permuted_len_kernel(int64_t n, const int32_t *rowptr, const int32_t *inv,
                                                                int32_t *len, int32_t *from)
{
    const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (k > n) return;
    const int32_t s = k < n ? rowptr[inv[k]] : 0;
    len[k] = k < n ? rowptr[inv[k] + 1] - s : 0;
    from[k] = s;
}

struct PermutedRows {
    const int32_t *colidx, *perm, *from, *rowptr; // rowptr: of the new rows
    int32_t *out_col, *order; // order: the old nonzero of every new one
    int32_t *flag;            // 1 if a row holds a column twice
};

// New rows of up to 64 nonzeros, a wavefront each: a nonzero's place is how many of the row's new columns are smaller,
// counted against every lane's broadcast.  (All places are taken, and add up to that, unless a column comes twice.)  The next
// row's bounds are requested while this one is counted.  10 M nonzeros 125 us; a sort of all nonzeros by row and column took
// 590 with the passes around it.
__global__ void __launch_bounds__(kThreads) permute_short_kernel(int64_t n, PermutedRows a)
{
    const int lane = threadIdx.x & 63;
    const int64_t step = (int64_t)gridDim.x * (kThreads / 64);
    int64_t k = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    int from = 0, at = 0, end = 0;
    if (k < n) from = a.from[k], at = a.rowptr[k], end = a.rowptr[k + 1];
    bool twice = false;
    for (; k < n; k += step) {
        const int s = __builtin_amdgcn_readfirstlane(from), base = __builtin_amdgcn_readfirstlane(at);
        const int len = __builtin_amdgcn_readfirstlane(end) - base;
        if (k + step < n) from = a.from[k + step], at = a.rowptr[k + step], end = a.rowptr[k + step + 1];
        if (len > 64) continue;
        const bool in = lane < len;
        const int32_t c = in ? a.perm[a.colidx[s + lane]] : -1;
        int place = 0;
        for (int j = 0; j < len; ++j) place += __builtin_amdgcn_readlane(c, j) < c;
        if (in) {
            a.out_col[base + place] = c;
            a.order[base + place] = s + lane;
        }
        int sum = in ? place : 0;
        sum += (int)dpp<0x121>((unsigned)sum);
        sum += (int)dpp<0x122>((unsigned)sum);
        sum += (int)dpp<0x124>((unsigned)sum);
        sum += (int)dpp<0x128>((unsigned)sum);
        sum = __builtin_amdgcn_readlane(sum, 0) + __builtin_amdgcn_readlane(sum, 16) + __builtin_amdgcn_readlane(sum, 32) +
              __builtin_amdgcn_readlane(sum, 48);
        twice |= sum != len * (len - 1) / 2;
    }
    if (twice && lane == 0) *a.flag = 1;
}

// Longer rows, a workgroup each, sorted in LDS.  list: old rows of more than 64 nonzeros, at most MOST
template <int T, int MOST>
__global__ void __launch_bounds__(T) permute_long_kernel(const int32_t *list, const int32_t *n_list, PermutedRows a)
{
    __shared__ unsigned long long key[MOST]; // new column, place in the old row
    bool twice = false;
    for (int q = blockIdx.x; q < *n_list; q += gridDim.x) {
        const int k = a.perm[list[q]];
        const int s = a.from[k], base = a.rowptr[k], len = a.rowptr[k + 1] - base;
        int m = 64;
        while (m < len) m <<= 1;
        for (int i = threadIdx.x; i < m; i += T)
            key[i] = i < len ? (unsigned long long)(unsigned)a.perm[a.colidx[s + i]] << 32 | (unsigned)i : ~0ull;
        __syncthreads();
        for (int w = 2; w <= m; w <<= 1)
            for (int j = w >> 1; j > 0; j >>= 1) {
                for (int i = threadIdx.x; i < m; i += T) {
                    const int o = i ^ j;
                    if (o > i && (key[i] > key[o]) == ((i & w) == 0)) {
                        const unsigned long long t = key[i];
                        key[i] = key[o];
                        key[o] = t;
                    }
                }
                __syncthreads();
            }
        for (int i = threadIdx.x; i < len; i += T) {
            const int32_t c = (int32_t)(key[i] >> 32);
            a.out_col[base + i] = c;
            a.order[base + i] = s + (int)(unsigned)key[i];
            twice |= i > 0 && (int32_t)(key[i - 1] >> 32) == c;
        }
        __syncthreads();
    }
    if (twice) *a.flag = 1;
}
__global__ void __launch_bounds__(kThreads) permuted_vals_kernel(int64_t nnz, const int32_t *order, const float *vals,
                                                                 float *out)
{
    const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (t < nnz) out[t] = vals[order[t]];
}
constexpr int kLongestSorted = 8192; // in a row; where one is longer all nonzeros are sorted together

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
        return descending ? hipcub::DeviceRadixSort::SortPairsDescending(tmp, bytes, kin, kout, vin, vout, (int)n, 0, bits, setup_stream())
                          : hipcub::DeviceRadixSort::SortPairs(tmp, bytes, kin, kout, vin, vout, (int)n, 0, bits, setup_stream());
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
    int32_t longest = 0; // row
    int upload(int64_t n, int64_t n_cols, int64_t nnz, const int32_t *h_rowptr, const int32_t *h_colidx, bool lists,
               Scratch &sc)
    {
        int32_t *counts = nullptr;
        TRY_GPU(sc.alloc((void **)&rowptr, sizeof(int32_t) * (n + 1)));
        TRY_GPU(sc.alloc((void **)&colidx, sizeof(int32_t) * (nnz + 1)));
        TRY_GPU(sc.alloc((void **)&counts, sizeof(int32_t) * 5));
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
        TRY_GPU(hipMemsetAsync(counts, 0, sizeof(int32_t) * 5, setup_stream()));
        hipLaunchKernelGGL(classify_kernel, dim3(strided_blocks(n > nnz ? n : nnz)), dim3(kThreads), 0, setup_stream(), n, n_cols,
                           nnz, r, (int32_t *)nullptr, (int32_t *)nullptr);
        TRY_GPU(hipGetLastError());
        int32_t h[5];
        TRY_GPU(setup_copy(h, counts, sizeof(h), hipMemcpyDeviceToHost));
        if (h[2]) return kUseHost;
        longest = h[4];
        if (lists) {
            hipLaunchKernelGGL(classify_kernel, dim3(strided_blocks(n)), dim3(kThreads), 0, setup_stream(), n, n_cols, nnz, r, medium,
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
    if (transpose_in_two_passes(n_rows, n_cols, nnz)) {
        const int rc = transpose_two_passes(n_rows, n_cols, nnz, d_rowptr, d_colidx, d_vals, rp, ci, va, hip_err);
        if (rc != PCSR_OK) return rc;
        *t_rowptr = rp;
        *t_colidx = ci;
        *t_vals = va;
        for (void *q : {(void *)rp, (void *)ci, (void *)va}) sc.release(q);
        return PCSR_OK;
    }
    HIP_TRY(sc.alloc((void **)&keys, sizeof(int32_t) * (nnz + 1)));
    HIP_TRY(sc.alloc((void **)&in, sizeof(uint2) * (nnz + 1)));
    HIP_TRY(sc.alloc((void **)&sorted, sizeof(uint2) * (nnz + 1)));
    if (nnz > 0) {
        hipLaunchKernelGGL(row_value_kernel, dim3((unsigned)((nnz + kSlice - 1) / kSlice)), dim3(kThreads), 0, setup_stream(), n_rows,
                           nnz, d_rowptr, d_vals, in);
        HIP_TRY(hipGetLastError());
        // stable, and the nonzeros come in row order: every output row ends up ascending
        HIP_TRY(sort_pairs(d_colidx, keys, reinterpret_cast<const unsigned long long *>(in),
                           reinterpret_cast<unsigned long long *>(sorted), nnz, key_bits(n_cols), false, sc));
        hipLaunchKernelGGL(split_pairs_kernel, dim3(blocks_for(nnz)), dim3(kThreads), 0, setup_stream(), nnz, sorted, ci, va);
        HIP_TRY(hipGetLastError());
    }
    hipLaunchKernelGGL(lower_bounds_kernel, dim3(blocks_for(n_cols + 1)), dim3(kThreads), 0, setup_stream(), n_cols, nnz, keys, rp);
    HIP_TRY(hipGetLastError());
    HIP_TRY(setup_wait());
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
    (void)setup_wait();
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
    hipLaunchKernelGGL(iota_kernel, dim3(blocks_for(n)), dim3(kThreads), 0, setup_stream(), n, lab[0], ids);
    TRY_GPU(hipGetLastError());
    int at = 0;
    const unsigned waves = (unsigned)((n + kThreads / 64 - 1) / (kThreads / 64));
    const unsigned blocks = waves < 2048 ? waves : 2048;
    for (int32_t done = 0; done < max_rounds;) {
        const int batch = max_rounds - done < kBatch ? max_rounds - done : kBatch;
        TRY_GPU(hipMemsetAsync(changed, 0, sizeof(int32_t) * (kBatch + 1), setup_stream()));
        for (int b = 0; b < batch; ++b) {
            const int32_t *from = lab[(at + b) & 1];
            int32_t *to = lab[(at + b + 1) & 1];
            const uint32_t round = (uint32_t)(done + b);
            hipLaunchKernelGGL(propagate_short_kernel, dim3(blocks), dim3(kThreads), 0, setup_stream(), n, m.r, from, to, b, round,
                               changed);
            TRY_GPU(hipGetLastError());
            hipLaunchKernelGGL((propagate_long_kernel<256, 2048>), dim3(2048), dim3(256), 0, setup_stream(), n, m.r, m.r.medium,
                               m.r.counts, from, to, b, round, changed);
            TRY_GPU(hipGetLastError());
            hipLaunchKernelGGL((propagate_long_kernel<1024, 8192>), dim3(512), dim3(1024), 0, setup_stream(), n, m.r, m.r.large,
                               m.r.counts + 1, from, to, b, round, changed);
            TRY_GPU(hipGetLastError());
        }
        int32_t h[kBatch], counts[4];
        TRY_GPU(setup_copy(counts, m.r.counts, sizeof(counts), hipMemcpyDeviceToHost));
        TRY_GPU(setup_copy(h, changed, sizeof(int32_t) * kBatch, hipMemcpyDeviceToHost));
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
    TRY_GPU(hipMemsetAsync(distinct, 0, sizeof(int32_t), setup_stream()));
    TRY_GPU(sort_pairs_u32(reinterpret_cast<const uint32_t *>(lab[at]), reinterpret_cast<uint32_t *>(sorted),
                           reinterpret_cast<const uint32_t *>(ids), reinterpret_cast<uint32_t *>(order), n, key_bits(n), sc));
    hipLaunchKernelGGL(number_kernel, dim3(blocks_for(n)), dim3(kThreads), 0, setup_stream(), n, order, sorted, d_perm, distinct);
    TRY_GPU(hipGetLastError());
    TRY_GPU(setup_copy(&clusters, distinct, sizeof(clusters), hipMemcpyDeviceToHost));
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
    TRY_GPU(hipMemsetAsync(refs, 0, sizeof(uint32_t) * n, setup_stream()));
    hipLaunchKernelGGL(iota_kernel, dim3(blocks_for(n)), dim3(kThreads), 0, setup_stream(), n, ids, (int32_t *)nullptr);
    TRY_GPU(hipGetLastError());
    hipLaunchKernelGGL(count_columns_kernel, dim3(strided_blocks(nnz)), dim3(kThreads), 0, setup_stream(), nnz, m.colidx, refs);
    TRY_GPU(hipGetLastError());
    TRY_GPU(sort_pairs(refs, sorted, ids, order, n, key_bits(nnz + 1), true, sc)); // descending, stable
    hipLaunchKernelGGL(number_kernel, dim3(blocks_for(n)), dim3(kThreads), 0, setup_stream(), n, order, (const int32_t *)nullptr,
                       d_perm, (int32_t *)nullptr);
    TRY_GPU(hipGetLastError());
    TRY_GPU(copy_to_host(perm, d_perm, sizeof(int32_t) * n));
    return PCSR_OK;
}

int permute_gpu(int64_t n, const int32_t *rowptr, const int32_t *colidx, const float *vals, const int32_t *perm,
                int32_t *out_rowptr, int32_t *out_colidx, float *out_vals)
{
    const int64_t nnz = rowptr[n];
    // Beside the work: the values' upload during the columns' download (the link carries both ways at once).  10 M
    // nonzeros: 4.0 ms, 4.8 one after the other (the link takes 1.5 ms for 41 MB up and 41 MB down at once, 0.9 for
    // either).  Taking the faults of fresh output pages ahead, on threads of their own, costs more than it saves: 4.2 ms.
    Scratch sc;
    Upload values; // waits before the memory it writes is given back
    int32_t *d_perm = nullptr, *inv = nullptr, *flag = nullptr, *len = nullptr, *from = nullptr, *rp = nullptr, *ci = nullptr,
            *order = nullptr, bad = 0;
    float *va = nullptr, *va_out = nullptr;
    TRY_GPU(sc.alloc((void **)&d_perm, sizeof(int32_t) * n));
    TRY_GPU(sc.alloc((void **)&inv, sizeof(int32_t) * n));
    TRY_GPU(sc.alloc((void **)&flag, sizeof(int32_t)));
    TRY_GPU(sc.alloc((void **)&len, sizeof(int32_t) * (n + 1)));
    TRY_GPU(sc.alloc((void **)&from, sizeof(int32_t) * (n + 1)));
    TRY_GPU(sc.alloc((void **)&rp, sizeof(int32_t) * (n + 1)));
    TRY_GPU(copy_to_device(d_perm, perm, sizeof(int32_t) * n));
    TRY_GPU(hipMemsetAsync(inv, 0xff, sizeof(int32_t) * n, setup_stream()));
    TRY_GPU(hipMemsetAsync(flag, 0, sizeof(int32_t), setup_stream()));
    hipLaunchKernelGGL(invert_kernel, dim3(blocks_for(n)), dim3(kThreads), 0, setup_stream(), n, d_perm, inv, flag);
    TRY_GPU(hipGetLastError());
    DevicePattern m;
    const int rc = m.upload(n, n, nnz, rowptr, colidx, true, sc);
    if (rc != PCSR_OK) return rc;
    TRY_GPU(setup_copy(&bad, flag, sizeof(bad), hipMemcpyDeviceToHost));
    if (bad) return kUseHost;
    TRY_GPU(sc.alloc((void **)&va, sizeof(float) * nnz));
    values.start(va, vals, sizeof(float) * nnz);
    hipLaunchKernelGGL(permuted_len_kernel, dim3(blocks_for(n + 1)), dim3(kThreads), 0, setup_stream(), n, m.rowptr, inv, len, from);
    TRY_GPU(hipGetLastError());
    size_t bytes = 0;
    void *tmp = nullptr;
    TRY_GPU(hipcub::DeviceScan::ExclusiveSum(nullptr, bytes, len, rp, (int)(n + 1), setup_stream()));
    TRY_GPU(sc.alloc(&tmp, bytes));
    TRY_GPU(hipcub::DeviceScan::ExclusiveSum(tmp, bytes, len, rp, (int)(n + 1), setup_stream()));
    TRY_GPU(sc.alloc((void **)&va_out, sizeof(float) * nnz));
    TRY_GPU(sc.alloc((void **)&ci, sizeof(int32_t) * nnz));
    TRY_GPU(sc.alloc((void **)&order, sizeof(int32_t) * nnz));
    if (m.longest <= kLongestSorted) {
        const PermutedRows a = {m.colidx, d_perm, from, rp, ci, order, flag};
        const unsigned waves = (unsigned)((n + kThreads / 64 - 1) / (kThreads / 64));
        hipLaunchKernelGGL(permute_short_kernel, dim3(waves < 2048 ? waves : 2048), dim3(kThreads), 0, setup_stream(), n, a);
        TRY_GPU(hipGetLastError());
        if (m.longest > 64) {
            hipLaunchKernelGGL((permute_long_kernel<256, kMediumRow>), dim3(2048), dim3(256), 0, setup_stream(), m.r.medium, m.r.counts, a);
            TRY_GPU(hipGetLastError());
        }
        if (m.longest > kMediumRow) {
            hipLaunchKernelGGL((permute_long_kernel<1024, kLongestSorted>), dim3(512), dim3(1024), 0, setup_stream(), m.r.large,
                               m.r.counts + 1, a);
            TRY_GPU(hipGetLastError());
        }
    } else {
        unsigned long long *key = nullptr, *sorted = nullptr;
        int32_t *ids = nullptr;
        TRY_GPU(sc.alloc((void **)&ids, sizeof(int32_t) * nnz));
        hipLaunchKernelGGL(iota_kernel, dim3(blocks_for(nnz)), dim3(kThreads), 0, setup_stream(), nnz, ids, (int32_t *)nullptr);
        TRY_GPU(hipGetLastError());
        TRY_GPU(sc.alloc((void **)&key, sizeof(long long) * nnz));
        TRY_GPU(sc.alloc((void **)&sorted, sizeof(long long) * nnz));
        const int bits = key_bits(n);
        hipLaunchKernelGGL(permuted_key_kernel, dim3((unsigned)((nnz + kSlice - 1) / kSlice)), dim3(kThreads), 0, setup_stream(), n, nnz,
                           m.rowptr, m.colidx, d_perm, bits, key);
        TRY_GPU(hipGetLastError());
        TRY_GPU(sort_pairs(key, sorted, reinterpret_cast<const uint32_t *>(ids), reinterpret_cast<uint32_t *>(order), nnz,
                           2 * bits, false, sc));
        hipLaunchKernelGGL(permuted_cols_kernel, dim3(blocks_for(nnz)), dim3(kThreads), 0, setup_stream(), nnz, sorted, bits, ci, flag);
        TRY_GPU(hipGetLastError());
    }
    TRY_GPU(setup_copy(&bad, flag, sizeof(bad), hipMemcpyDeviceToHost));
    if (bad) return kUseHost; // a column twice in a row: their order is the host sort's business
    // (an output in the place of the values is not written before they are read)
    auto in_values = [&](const int32_t *out, int64_t count) {
        return reinterpret_cast<uintptr_t>(out) < reinterpret_cast<uintptr_t>(vals + nnz) &&
               reinterpret_cast<uintptr_t>(vals) < reinterpret_cast<uintptr_t>(out + count);
    };
    if (in_values(out_rowptr, n + 1) || in_values(out_colidx, nnz)) TRY_GPU(values.wait());
    TRY_GPU(copy_to_host(out_rowptr, rp, sizeof(int32_t) * (n + 1)));
    TRY_GPU(copy_to_host(out_colidx, ci, sizeof(int32_t) * nnz));
    TRY_GPU(values.wait());
    hipLaunchKernelGGL(permuted_vals_kernel, dim3(blocks_for(nnz)), dim3(kThreads), 0, setup_stream(), nnz, order, va, va_out);
    TRY_GPU(hipGetLastError());
    TRY_GPU(copy_to_host(out_vals, va_out, sizeof(float) * nnz));
    return PCSR_OK;
}

} // namespace pcsr
