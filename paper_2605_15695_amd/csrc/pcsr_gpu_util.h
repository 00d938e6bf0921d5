// What the GPU set-up code shares: launch sizes, scratch memory, the rows of a slice of nonzeros.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "../../include/pcsr.h"
#include "pcsr_pool.h"

namespace pcsr {
namespace {

constexpr int kThreads = 256;

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + kThreads - 1) / kThreads); }
// grid of a kernel that strides over n elements: enough workgroups to fill the chip, few
// enough that one atomic or partial result from each costs nothing
inline unsigned strided_blocks(int64_t n, unsigned most = 2048)
{
    const int64_t b = (n + kThreads - 1) / kThreads;
    return (unsigned)(b < 1 ? 1 : (b > (int64_t)most ? most : b));
}

// bits of the largest key below n
inline int key_bits(int64_t n)
{
    int b = 1;
    while (b < 32 && (int64_t(1) << b) < n) ++b;
    return b;
}

// index of the row that holds nonzero t: the last r with rowptr[r] <= t
__device__ __forceinline__ int64_t row_of_nonzero(const int32_t *rowptr, int64_t n_rows, int64_t t)
{
    int64_t lo = 0, hi = n_rows; // rowptr[lo] <= t < rowptr[hi]
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (rowptr[mid] <= t)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// One step of a search for the first of colidx[lo, hi) that is >= key (lo == hi at the end): three probes at a
// time, since such a chain is bound by its round trips to memory (features of R-MAT scale 20: 77 us for 102 with one).
__device__ __forceinline__ void narrow(const int32_t *colidx, int64_t key, int32_t &lo, int32_t &hi)
{
    const int32_t n = hi - lo;
    if (n <= 0) return;
    const int32_t at[3] = {lo + (n >> 2), lo + (n >> 1), hi - 1 - (n >> 2)};
    const int32_t c[3] = {colidx[at[0]], colidx[at[1]], colidx[at[2]]};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        if (c[k] < key)
            lo = at[k] + 1 > lo ? at[k] + 1 : lo;
        else
            hi = at[k] < hi ? at[k] : hi;
    }
}

// The rows of kSlice consecutive nonzeros, found by a workgroup together: 256-way search for
// the first row (3 dependent loads instead of 20), then the row starts up to the end of the
// slice in LDS, where every thread looks its nonzeros up.  A slice that crosses more rows than
// fit (nearly all of them empty) is searched in memory.
constexpr int kSlice = 1024;
constexpr int kSliceRows = 1536;
struct RowSlice {
    int32_t start[kSliceRows + 1];
    int cnt[kThreads / 64];
    int64_t first; // row of the slice's first nonzero
    int rows;      // row starts held, 0 = too many

    __device__ void find(const int32_t *rowptr, int64_t n_rows, int64_t t0, int64_t t1)
    {
        const int tid = threadIdx.x;
        int64_t lo = 0, hi = n_rows;
        while (hi - lo > 1) {
            const int64_t step = (hi - lo + kThreads) / (kThreads + 1);
            const int64_t probe = lo + (tid + 1) * step;
            const bool below = probe < hi && rowptr[probe] <= t0;
            const unsigned long long m = __ballot(below);
            __syncthreads(); // cnt of the round before is read
            if ((tid & 63) == 0) cnt[tid >> 6] = __popcll(m);
            __syncthreads();
            int c = 0;
            for (int w = 0; w < kThreads / 64; ++w) c += cnt[w];
            lo += c * step;
            hi = hi < lo + step ? hi : lo + step;
        }
        const int64_t r0 = lo;
        int have = 0;
        for (int base = 0; base < kSliceRows; base += kThreads) {
            const int64_t r = r0 + base + tid;
            start[base + tid] = r <= n_rows ? rowptr[r] : INT32_MAX;
            __syncthreads();
            const int32_t lst = start[base + kThreads - 1];
            if (lst >= t1) {
                have = base + kThreads;
                break;
            }
        }
        if (tid == 0) {
            first = r0;
            rows = have;
        }
        __syncthreads();
    }
    __device__ int64_t row(const int32_t *rowptr, int64_t n_rows, int64_t t) const
    {
        if (rows == 0) return row_of_nonzero(rowptr, n_rows, t);
        int lo = 0, hi = rows; // start[lo] <= t
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (start[mid] <= t)
                lo = mid;
            else
                hi = mid;
        }
        return first + lo;
    }
};

// Whether nonzeros start a row, for kSlice consecutive ones, from a table of the row that holds each slice's first one
// (note_slices): the row starts inside the slice are marked in LDS.  A slice that more rows start in than fit is looked
// up in memory.  (Row pointers that do not ascend give wrong answers, never an access out of bounds.)
constexpr int kPerThread = kSlice / kThreads;
typedef int32_t int4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
static_assert(kPerThread == 4, "a thread's nonzeros are one 16-byte access");

struct RowStarts {
    int32_t *starts; // kSlice of LDS: 1 where a row starts
    bool marked;

    __device__ void find(const int32_t *rowptr, int64_t n_rows, int64_t first_row, int64_t t0, int64_t t1)
    {
        const int tid = threadIdx.x;
        const int64_t first = first_row < 0 ? 0 : (first_row < n_rows ? first_row : n_rows - 1);
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) starts[k * kThreads + tid] = 0;
        __syncthreads();
        marked = false;
        for (int base = 0; base < kSliceRows && !marked; base += kThreads) {
            const int64_t r = first + base + tid;
            const int32_t v = r <= n_rows ? rowptr[r] : INT32_MAX;
            if (v >= t0 && v < t1) starts[v - t0] = 1;
            marked = !__syncthreads_or(tid == kThreads - 1 && v < t1);
        }
    }
    __device__ bool starts_row(const int32_t *rowptr, int64_t n_rows, int64_t t0, int64_t t) const
    {
        return marked ? starts[t - t0] != 0 : rowptr[row_of_nonzero(rowptr, n_rows, t)] == t;
    }
};

// For one row of a pass over the row pointer: the slices whose first nonzero it holds.
__device__ __forceinline__ void note_slices(int32_t *table, int64_t row, int64_t s, int64_t e)
{
    for (int64_t k = (s + kSlice - 1) / kSlice; k * kSlice < e; ++k) table[k] = (int32_t)row;
}

struct Scratch { // gives back everything it still owns on scope exit
    void *p[40] = {};
    int n = 0;
    hipError_t alloc(void **out, size_t bytes)
    {
        if (n >= 40) return hipErrorOutOfMemory;
        hipError_t e = pool_alloc(out, bytes);
        if (e == hipSuccess) p[n++] = *out;
        return e;
    }
    void release(void *q)
    {
        for (int i = 0; i < n; ++i)
            if (p[i] == q) p[i] = nullptr;
    }
    ~Scratch()
    {
        // everything here runs on the set-up stream; idle by now unless an error cut it short
        (void)setup_wait();
        for (int i = 0; i < n; ++i) pool_free(p[i]);
    }
};

#define HIP_TRY(expr)                  \
    do {                               \
        hipError_t e_ = (expr);        \
        if (e_ != hipSuccess) {        \
            *hip_err = (int)e_;        \
            (void)hipGetLastError();   \
            return e_ == hipErrorOutOfMemory ? PCSR_E_OOM : PCSR_E_HIP; \
        }                              \
    } while (0)

} // namespace
} // namespace pcsr
