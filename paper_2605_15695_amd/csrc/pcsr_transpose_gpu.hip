// CSR of the transpose from CSR arrays in device memory: a stable sort of the nonzeros by column in two passes of up to 10
// bits each, made for this: the first pass finds the rows itself, the second writes the output arrays, and the
// counts of the second are the output's row pointer.
//
// What bounds it: the ranking in the scatter kernels (a ballot per bit of the digit) and their 32- to 64-byte runs of output.
// 12 M nonzeros, 250,000 columns: 225 us (count 17, scatter 101; count 17, scatter 66; the scans and the rest 24) where
// hipCUB's sort of keys and 8-byte pairs took three passes of 125 us and 515 us in all with the kernels around it; 42 M,
// 1 M columns: both directions in 1.6 ms for 3.7.
#include <hip/hip_runtime.h>
#include <hipcub/hipcub.hpp>

#include <algorithm>

#include "pcsr_build_gpu.h"
#include "pcsr_gpu_util.h"
#include "pcsr_relabel_gpu.h"

namespace pcsr {
namespace {

constexpr int kTurnThreads = 1024, kTurnWaves = kTurnThreads / 64, kTurnItems = 8;
constexpr int kTurnTile = kTurnThreads * kTurnItems; // nonzeros of a workgroup
constexpr int kTurnDigit = 10;                       // bits of a pass at most
// Nonzeros from which it is used: building both directions of 20,000 rows with 20 bits of columns takes 269 us for
// 292 by hipCUB with 262,144 nonzeros, 267 for 245 with half as many; 65,000 x 65,000 with 2^20: 245 for 385.
constexpr int64_t kTurnLeast = int64_t(1) << 18;
constexpr int kRowRounds = 16;                       // rows a tile looks at, kTurnThreads at a time, before it searches instead

struct TurnArgs {
    int64_t nnz, n_rows;
    const int32_t *rowptr, *colidx;
    const float *vals;
    unsigned *mid_key; // between the passes, by the low digit: high digit and row in a word
    float *mid_val;
    int32_t *out_colidx;
    float *out_vals;
    int low_bits, high_bits, row_bits;
    int tiles;
    const int2 *table; // second pass: nonzeros [x, y) of a tile, all of one low digit
    int32_t *counts;   // [digit][tile], then their exclusive sums
};

template <bool SECOND> struct Tile {
    int64_t begin, end;
    int bins, shift;
    __device__ explicit Tile(const TurnArgs &a)
    {
        if constexpr (SECOND) {
            const int2 t = a.table[blockIdx.x];
            begin = t.x;
            end = t.y;
            bins = 1 << a.high_bits;
            shift = a.row_bits;
        } else {
            begin = (int64_t)blockIdx.x * kTurnTile;
            end = begin + kTurnTile < a.nnz ? begin + kTurnTile : a.nnz;
            bins = 1 << a.low_bits;
            shift = 0;
        }
    }
    __device__ unsigned digit(unsigned key) const { return (SECOND ? key >> shift : key) & (unsigned)(bins - 1); }
};

template <bool SECOND> __global__ void __launch_bounds__(kTurnThreads) turn_count_kernel(TurnArgs a)
{
    // kCopies of the counters, on different banks: nonzeros side by side in the second pass often have one digit (rows of a
    // community), and lanes that count on one word take turns (40 us with one copy, 17 so)
    constexpr int kCopies = 8;
    __shared__ int32_t cnt[kCopies * ((1 << kTurnDigit) + 1)];
    const Tile<SECOND> tile(a);
    const int stride = tile.bins + 1;
    for (int d = threadIdx.x; d < kCopies * stride; d += kTurnThreads) cnt[d] = 0;
    __syncthreads();
    unsigned key[kTurnItems];
#pragma unroll
    for (int k = 0; k < kTurnItems; ++k) {
        const int64_t t = tile.begin + k * kTurnThreads + threadIdx.x;
        if (t < tile.end) key[k] = SECOND ? a.mid_key[t] : (unsigned)a.colidx[t];
    }
    int32_t *const own = cnt + (threadIdx.x & (kCopies - 1)) * stride;
#pragma unroll
    for (int k = 0; k < kTurnItems; ++k)
        if (tile.begin + k * kTurnThreads + threadIdx.x < tile.end) atomicAdd(&own[tile.digit(key[k])], 1);
    __syncthreads();
    for (int d = threadIdx.x; d < tile.bins; d += kTurnThreads) {
        int32_t sum = 0;
#pragma unroll
        for (int c = 0; c < kCopies; ++c) sum += cnt[c * stride + d];
        a.counts[(int64_t)d * a.tiles + blockIdx.x] = sum;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) a.counts[(int64_t)tile.bins * a.tiles] = 0;
}

// Tiles of the second pass: every low digit's nonzeros, kTurnTile at a time; first[d]: the first of digit d.
__global__ void __launch_bounds__(1 << kTurnDigit) turn_tiles_kernel(TurnArgs a, const int32_t *offsets, int tiles_before, int2 *table,
                                                                     int32_t *first)
{
    typedef hipcub::BlockScan<int, 1 << kTurnDigit> Scan;
    __shared__ typename Scan::TempStorage tmp;
    const int d = threadIdx.x, bins = 1 << a.low_bits;
    int32_t s = 0, e = 0;
    if (d < bins) {
        s = offsets[(int64_t)d * tiles_before];
        e = offsets[(int64_t)(d + 1) * tiles_before];
    }
    int at;
    const int n = (int)(((int64_t)e - s + kTurnTile - 1) / kTurnTile);
    Scan(tmp).ExclusiveSum(n, at);
    if (d < bins) first[d] = at;
    for (int k = 0; k < n; ++k) {
        const int64_t b = s + (int64_t)k * kTurnTile;
        table[at + k] = {(int)b, (int)(b + kTurnTile < e ? b + kTurnTile : e)};
    }
}

// A wavefront takes 512 nonzeros in a row, 64 at a time: lanes with one digit find each other by a ballot per bit, the first
// of them counts them in the wavefront's own counters, so equal digits stay in their order.  The tile then goes out in
// its new order through LDS (straight from the registers: first pass 159 us for 101, second 101 for 66).  64 registers,
// for two workgroups on a compute unit.
template <bool SECOND>
__global__ void __launch_bounds__(kTurnThreads) __attribute__((amdgpu_waves_per_eu(8))) turn_scatter_kernel(TurnArgs a)
{
    extern __shared__ __align__(16) int32_t lds[]; // counters per wavefront; before them row marks, after them the tile, sorted
    __shared__ int32_t from[1 << kTurnDigit], to[1 << kTurnDigit];
    typedef hipcub::BlockScan<int, kTurnThreads> Scan;
    __shared__ typename Scan::TempStorage tmp;
    __shared__ int s_cnt[kTurnWaves];
    const Tile<SECOND> tile(a);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = (int)(tile.end - tile.begin);
    if (n <= 0) return; // uniform
    const int mine = wave * (64 * kTurnItems) + lane;
    unsigned key[kTurnItems];
    float val[kTurnItems];
#pragma unroll
    for (int k = 0; k < kTurnItems; ++k) {
        const int i = mine + k * 64;
        key[k] = 0;
        val[k] = 0.0f;
        if (i < n) {
            key[k] = SECOND ? a.mid_key[tile.begin + i] : (unsigned)a.colidx[tile.begin + i];
            if constexpr (SECOND) val[k] = a.mid_val[tile.begin + i];
        }
    }
    unsigned row[kTurnItems];
    if constexpr (!SECOND) {
        // the row of the tile's first nonzero, kTurnThreads probes at a time
        int64_t lo = 0, hi = a.n_rows; // rowptr[lo] <= begin < rowptr[hi]
        while (hi - lo > 1) {
            const int64_t step = (hi - lo + kTurnThreads) / (kTurnThreads + 1);
            const int64_t probe = lo + (tid + 1) * step;
            const unsigned long long m = __ballot(probe < hi && a.rowptr[probe < hi ? probe : hi] <= tile.begin);
            if (lane == 0) s_cnt[wave] = __popcll(m);
            __syncthreads();
            int c = 0;
            for (int w = 0; w < kTurnWaves; ++w) c += s_cnt[w];
            __syncthreads();
            lo += c * step;
            hi = hi < lo + step ? hi : lo + step;
        }
        // how many rows start at each nonzero after it, and their sums
        for (int i = tid; i < kTurnTile; i += kTurnThreads) lds[i] = 0;
        __syncthreads();
        bool done = false;
        for (int k = 0; k < kRowRounds && !done; ++k) {
            const int64_t r = lo + 1 + k * kTurnThreads + tid;
            const int64_t at = r < a.n_rows ? (int64_t)a.rowptr[r] - tile.begin : n;
            if (at >= 0 && at < n) atomicAdd(&lds[at], 1);
            done = __syncthreads_or(tid == kTurnThreads - 1 && at >= n);
        }
        if (done) {
            int4 *v = reinterpret_cast<int4 *>(lds) + tid * (kTurnItems / 4);
            int4 x = v[0], y = v[1];
            x.y += x.x;
            x.z += x.y;
            x.w += x.z;
            y.x += x.w;
            y.y += y.x;
            y.z += y.y;
            y.w += y.z;
            int before;
            Scan(tmp).ExclusiveSum(y.w, before);
            v[0] = {x.x + before, x.y + before, x.z + before, x.w + before};
            v[1] = {y.x + before, y.y + before, y.z + before, y.w + before};
            __syncthreads();
        }
#pragma unroll
        for (int k = 0; k < kTurnItems; ++k) {
            const int i = mine + k * 64;
            row[k] = 0;
            if (i < n) row[k] = (unsigned)(done ? lo + lds[i] : row_of_nonzero(a.rowptr, a.n_rows, tile.begin + i));
        }
        __syncthreads(); // the marks are read
    }

    const int bits = SECOND ? a.high_bits : a.low_bits, bins = tile.bins;
    for (int i = tid; i < kTurnWaves * bins; i += kTurnThreads) lds[i] = 0;
    __syncthreads();
    int32_t *const own = lds + wave * bins;
    int rank[kTurnItems];
#pragma unroll
    for (int k = 0; k < kTurnItems; ++k) {
        const bool have = mine + k * 64 < n;
        const unsigned d = tile.digit(key[k]);
        unsigned long long same = __ballot(have);
        for (int b = 0; b < bits; ++b) {
            const bool one = d >> b & 1;
            const unsigned long long ones = __ballot(one);
            same &= one ? ones : ~ones;
        }
        const int leader = same ? __ffsll((unsigned long long)same) - 1 : 0;
        int before = 0;
        if (have && lane == leader) before = atomicAdd(&own[d], (int)__popcll(same));
        before = __shfl(before, leader);
        rank[k] = before + (int)__popcll(same & ((1ull << lane) - 1));
    }
    __syncthreads();
    // per digit: entries of the wavefronts before, of the tile's lower digits, and where the digit's go
    int total = 0;
    if (tid < bins) {
#pragma unroll
        for (int w = 0; w < kTurnWaves; ++w) {
            const int c = lds[w * bins + tid];
            lds[w * bins + tid] = total;
            total += c;
        }
    }
    int start;
    Scan(tmp).ExclusiveSum(total, start);
    if (tid < bins) {
        from[tid] = start;
        to[tid] = a.counts[(int64_t)tid * a.tiles + blockIdx.x] - start;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kTurnItems; ++k) {
        const unsigned d = tile.digit(key[k]);
        rank[k] += own[d] + from[d]; // place in the sorted tile
    }
    // in that order through LDS, one word of a nonzero at a time, so that neighbours go out together
    unsigned *const sorted = reinterpret_cast<unsigned *>(lds);
    auto in_order = [&](auto word, auto take) {
        __syncthreads(); // what was there is read
#pragma unroll
        for (int k = 0; k < kTurnItems; ++k)
            if (mine + k * 64 < n) sorted[rank[k]] = word(k);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kTurnItems; ++k)
            if (tid + k * kTurnThreads < n) take(k, sorted[tid + k * kTurnThreads]);
    };
    int32_t at[kTurnItems];
    unsigned high[kTurnItems];
    in_order([&](int k) { return key[k]; },
             [&](int k, unsigned x) {
                 at[k] = to[tile.digit(x)] + tid + k * kTurnThreads;
                 if constexpr (SECOND)
                     a.out_colidx[at[k]] = (int32_t)(x & ((1u << a.row_bits) - 1));
                 else
                     high[k] = (x >> a.low_bits & ((1u << a.high_bits) - 1)) << a.row_bits;
             });
    if constexpr (!SECOND) {
#pragma unroll
        for (int k = 0; k < kTurnItems; ++k) // (only now: the registers)
            if (mine + k * 64 < n) {
                const int64_t t = tile.begin + mine + k * 64;
                val[k] = a.vals ? a.vals[t] : __int_as_float((int)t);
            }
        in_order([&](int k) { return row[k]; }, [&](int k, unsigned x) { a.mid_key[at[k]] = high[k] | x; });
    }
    in_order([&](int k) { return __float_as_uint(val[k]); },
             [&](int k, unsigned x) { (SECOND ? a.out_vals : a.mid_val)[at[k]] = __uint_as_float(x); });
}

// column c = {high, low digit} starts where the second pass puts the high digit's entries of the first tile of the low one
__global__ void __launch_bounds__(kThreads) turn_rowptr_kernel(int64_t n_cols, int64_t nnz, int low_bits, int tiles,
                                                               const int32_t *offsets, const int32_t *first, int32_t *rowptr)
{
    const int64_t c = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (c > n_cols) return;
    rowptr[c] = c == n_cols ? (int32_t)nnz : offsets[(c >> low_bits) * tiles + first[c & ((1 << low_bits) - 1)]];
}

// t_vals[i] = vals[place i]; its first content are the places.  12 M nonzeros of 500-node communities: 50 us.
__global__ void __launch_bounds__(kThreads) turned_values_kernel(int64_t nnz, const float *vals, float *t_vals)
{
    const int64_t i = ((int64_t)blockIdx.x * kThreads + threadIdx.x) * 4;
    if (i + 4 <= nnz) {
        int4u at = *reinterpret_cast<const int4u *>(t_vals + i);
        float4u v;
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = vals[at[k]];
        *reinterpret_cast<float4u *>(t_vals + i) = v;
    } else {
        for (int64_t k = i; k < nnz; ++k) t_vals[k] = vals[__float_as_int(t_vals[k])];
    }
}

} // namespace

hipError_t turned_values(int64_t nnz, const float *d_vals, float *t_vals)
{
    if (nnz <= 0) return hipSuccess;
    hipLaunchKernelGGL(turned_values_kernel, dim3(blocks_for((nnz + 3) / 4)), dim3(kThreads), 0, setup_stream(), nnz, d_vals, t_vals);
    return hipGetLastError();
}

bool transpose_in_two_passes(int64_t n_rows, int64_t n_cols, int64_t nnz)
{
    const int bits = key_bits(n_cols);
    return nnz >= kTurnLeast && bits >= 2 && bits <= 2 * kTurnDigit && key_bits(n_rows) + (bits + 1) / 2 <= 32;
}

int transpose_two_passes(int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t *d_rowptr, const int32_t *d_colidx,
                         const float *d_vals, int32_t *t_rowptr, int32_t *t_colidx, float *t_vals, int *hip_err)
{
    Scratch sc;
    const int bits = key_bits(n_cols);
    TurnArgs a = {};
    a.nnz = nnz;
    a.n_rows = n_rows;
    a.rowptr = d_rowptr;
    a.colidx = d_colidx;
    a.vals = d_vals;
    a.out_colidx = t_colidx;
    a.out_vals = t_vals;
    a.low_bits = bits / 2;
    a.high_bits = bits - a.low_bits;
    a.row_bits = key_bits(n_rows);
    const int tiles1 = (int)((nnz + kTurnTile - 1) / kTurnTile), tiles2 = tiles1 + (1 << a.low_bits);
    const int64_t n1 = ((int64_t)tiles1 << a.low_bits) + 1, n2 = ((int64_t)tiles2 << a.high_bits) + 1;
    int32_t *counts1, *counts2, *sums1, *sums2, *first;
    int2 *table;
    void *tmp;
    size_t bytes1 = 0, bytes2 = 0;
    HIP_TRY(sc.alloc((void **)&a.mid_key, sizeof(unsigned) * nnz));
    HIP_TRY(sc.alloc((void **)&a.mid_val, sizeof(float) * nnz));
    HIP_TRY(sc.alloc((void **)&counts1, sizeof(int32_t) * n1));
    HIP_TRY(sc.alloc((void **)&counts2, sizeof(int32_t) * n2));
    HIP_TRY(sc.alloc((void **)&sums1, sizeof(int32_t) * n1));
    HIP_TRY(sc.alloc((void **)&sums2, sizeof(int32_t) * n2));
    HIP_TRY(sc.alloc((void **)&first, sizeof(int32_t) << kTurnDigit));
    HIP_TRY(sc.alloc((void **)&table, sizeof(int2) * tiles2));
    HIP_TRY(hipcub::DeviceScan::ExclusiveSum(nullptr, bytes1, counts1, sums1, (int)n1, setup_stream()));
    HIP_TRY(hipcub::DeviceScan::ExclusiveSum(nullptr, bytes2, counts2, sums2, (int)n2, setup_stream()));
    HIP_TRY(sc.alloc(&tmp, bytes1 > bytes2 ? bytes1 : bytes2));
    HIP_TRY(hipMemsetAsync(table, 0, sizeof(int2) * tiles2, setup_stream())); // tiles past the last are empty
    const size_t lds1 = sizeof(int32_t) * std::max(kTurnTile, kTurnWaves << a.low_bits);
    const size_t lds2 = sizeof(int32_t) * std::max(kTurnTile, kTurnWaves << a.high_bits);
    // more than 64 KB of LDS in all has to be allowed
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(&turn_scatter_kernel<false>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, 64 * 1024));
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(&turn_scatter_kernel<true>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, 64 * 1024));
    a.tiles = tiles1;
    a.counts = counts1;
    hipLaunchKernelGGL(turn_count_kernel<false>, dim3(tiles1), dim3(kTurnThreads), 0, setup_stream(), a);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipcub::DeviceScan::ExclusiveSum(tmp, bytes1, counts1, sums1, (int)n1, setup_stream()));
    a.counts = sums1;
    hipLaunchKernelGGL(turn_scatter_kernel<false>, dim3(tiles1), dim3(kTurnThreads), lds1, setup_stream(), a);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(turn_tiles_kernel, dim3(1), dim3(1 << kTurnDigit), 0, setup_stream(), a, sums1, tiles1, table, first);
    HIP_TRY(hipGetLastError());
    a.tiles = tiles2;
    a.table = table;
    a.counts = counts2;
    hipLaunchKernelGGL(turn_count_kernel<true>, dim3(tiles2), dim3(kTurnThreads), 0, setup_stream(), a);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipcub::DeviceScan::ExclusiveSum(tmp, bytes2, counts2, sums2, (int)n2, setup_stream()));
    a.counts = sums2;
    hipLaunchKernelGGL(turn_scatter_kernel<true>, dim3(tiles2), dim3(kTurnThreads), lds2, setup_stream(), a);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(turn_rowptr_kernel, dim3(blocks_for(n_cols + 1)), dim3(kThreads), 0, setup_stream(), n_cols, nnz, a.low_bits, tiles2,
                       sums2, first, t_rowptr);
    HIP_TRY(hipGetLastError());
    HIP_TRY(setup_wait());
    return PCSR_OK;
}

} // namespace pcsr
