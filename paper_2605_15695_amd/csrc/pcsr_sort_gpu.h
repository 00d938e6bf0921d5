// Stable radix sort of (key, payload) pairs in device memory, for the few hundred thousand to few million
// work items or rows that a set-up call orders.
//
// What bounds it: at these sizes launches.  A pass takes 7 to 10 bits (all of them in as few passes as that
// allows) in three launches: digit counts per tile, for every digit the sums over the tiles (a wavefront each),
// and the scatter, whose workgroups add up the digits and walk their tile in order.
// 250,000 pairs of 20 bits: 46 us of kernels where hipCUB's merge sort took 90 (17 launches); 1 M of 22: 75 for 155.
#pragma once
#include <hip/hip_runtime.h>
#include <hipcub/hipcub.hpp>

#include "pcsr_gpu_util.h"

namespace pcsr {
namespace {

constexpr int kSortTile = 2048;     // pairs a workgroup holds in registers
constexpr int kSortTiles = 512;     // workgroups at most
constexpr int kSortDigit = 10;      // bits of a pass at most
constexpr int kSortRounds = kSortTile / kThreads;
constexpr int64_t kSortLeast = int64_t(1) << 14, kSortMost = int64_t(1) << 21; // pairs this sort is used for

struct SortPass {
    int64_t n, chunk;  // pairs; of them per workgroup, a multiple of kSortTile
    int shift, bits, tiles;
    const uint32_t *kin, *vin;
    uint32_t *kout, *vout;
    int32_t *counts;   // [digit][tile]
    int32_t *totals;   // [digit]
};

__global__ void __launch_bounds__(kThreads) sort_count_kernel(SortPass p)
{
    __shared__ int32_t cnt[1 << kSortDigit];
    const int bins = 1 << p.bits;
    for (int d = threadIdx.x; d < bins; d += kThreads) cnt[d] = 0;
    __syncthreads();
    const int64_t t0 = (int64_t)blockIdx.x * p.chunk, t1 = t0 + p.chunk < p.n ? t0 + p.chunk : p.n;
    for (int64_t t = t0 + threadIdx.x; t < t1; t += kThreads) atomicAdd(&cnt[(p.kin[t] >> p.shift) & (bins - 1)], 1);
    __syncthreads();
    for (int d = threadIdx.x; d < bins; d += kThreads) p.counts[(int64_t)d * p.tiles + blockIdx.x] = cnt[d];
}

// counts of a digit, summed over the tiles before (in place); its total
__global__ void __launch_bounds__(kThreads) sort_tiles_kernel(int bins, int tiles, int32_t *counts, int32_t *totals)
{
    const int lane = threadIdx.x & 63, d = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (d >= bins) return;
    int32_t *row = counts + (int64_t)d * tiles;
    constexpr int N = kSortTiles / 64;
    int32_t v[N], before = 0;
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = k * 64 + lane < tiles ? row[k * 64 + lane] : 0;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        int32_t upto = v[k];
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) {
            const int32_t o = __shfl_up(upto, m);
            if (lane >= m) upto += o;
        }
        if (k * 64 + lane < tiles) row[k * 64 + lane] = before + upto - v[k];
        before += __shfl(upto, 63);
    }
    if (lane == 0) totals[d] = before;
}

// A wavefront ranks 64 pairs at a time by ballots over the digit's bits, in the order they come, and keeps
// its own running counts; the four wavefronts' counts are then added up in order.
__global__ void __launch_bounds__(kThreads) sort_scatter_kernel(SortPass p)
{
    constexpr int W = kThreads / 64;
    __shared__ int32_t cnt[W][1 << kSortDigit];
    __shared__ int32_t next[1 << kSortDigit]; // where the next pair of a digit goes
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int bins = 1 << p.bits;
    const unsigned long long below = (1ull << lane) - 1;
    { // pairs of smaller digits, then those of this one in the tiles before
        constexpr int N = (1 << kSortDigit) / kThreads;
        typedef hipcub::BlockScan<int32_t, kThreads> Scan;
        __shared__ typename Scan::TempStorage tmp;
        int32_t v[N], own = 0, ex;
#pragma unroll
        for (int k = 0; k < N; ++k) own += v[k] = tid * N + k < bins ? p.totals[tid * N + k] : 0;
        Scan(tmp).ExclusiveSum(own, ex);
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const int d = tid * N + k;
            if (d < bins) next[d] = ex + p.counts[(int64_t)d * p.tiles + blockIdx.x];
            ex += v[k];
        }
    }
    const int64_t t0 = (int64_t)blockIdx.x * p.chunk, t1 = t0 + p.chunk < p.n ? t0 + p.chunk : p.n;
    for (int64_t sub = t0; sub < t1; sub += kSortTile) {
        const int64_t at = sub + wave * (kSortTile / W) + lane;
        uint32_t key[kSortRounds], val[kSortRounds];
        int rank[kSortRounds];
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) {
            const int64_t t = at + r * 64;
            key[r] = t < t1 ? p.kin[t] : 0;
            val[r] = t < t1 ? p.vin[t] : 0;
        }
        for (int d = tid; d < bins; d += kThreads)
#pragma unroll
            for (int w = 0; w < W; ++w) cnt[w][d] = 0;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) {
            const bool ok = at + r * 64 < t1;
            const uint32_t digit = (key[r] >> p.shift) & (bins - 1);
            unsigned long long same = __ballot(ok);
            for (int b = 0; b < p.bits; ++b) {
                const bool bit = (digit >> b) & 1;
                const unsigned long long m = __ballot(bit);
                same &= bit ? m : ~m;
            }
            rank[r] = 0;
            if (ok) {
                const int had = cnt[wave][digit];
                rank[r] = had + __popcll(same & below);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); // all have read before the first of them writes
                if ((same & below) == 0) cnt[wave][digit] = had + __popcll(same);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        for (int d = tid; d < bins; d += kThreads) {
            int32_t to = next[d];
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const int32_t c = cnt[w][d];
                cnt[w][d] = to;
                to += c;
            }
            next[d] = to;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) {
            if (at + r * 64 < t1) {
                const int64_t to = cnt[wave][(key[r] >> p.shift) & (bins - 1)] + rank[r];
                p.kout[to] = key[r];
                p.vout[to] = val[r];
            }
        }
        __syncthreads(); // the counts are read
    }
}

// kout / vout: the pairs in ascending order of the keys' lowest `bits` bits, equal keys as they came.  Inputs are
// not written.  On the null stream.  Above 2 M pairs hipCUB's sort moves them once a pass: 116 us at 2 M and 134 at
// 4 M of 20 bits, where this one takes 105 and 160.  Below 1 M it merges blocks, a launch or two per doubling: up to 16 K
// pairs that is 6 to 22 us (this one: 21 to 28), at 20 K 34.
hipError_t sort_pairs_u32(const uint32_t *kin, uint32_t *kout, const uint32_t *vin, uint32_t *vout, int64_t n, int bits,
                          Scratch &sc)
{
    if (n <= 0) return hipSuccess;
    if (n < kSortLeast || n > kSortMost) {
        size_t bytes = 0;
        void *tmp = nullptr;
        hipError_t e = hipcub::DeviceRadixSort::SortPairs(nullptr, bytes, kin, kout, vin, vout, (int)n, 0, bits, setup_stream());
        if (e == hipSuccess) e = sc.alloc(&tmp, bytes);
        return e == hipSuccess ? hipcub::DeviceRadixSort::SortPairs(tmp, bytes, kin, kout, vin, vout, (int)n, 0, bits, setup_stream()) : e;
    }
    SortPass p;
    p.n = n;
    const int64_t subs = (n + kSortTile - 1) / kSortTile;
    const int64_t per = (subs + kSortTiles - 1) / kSortTiles;
    p.chunk = per * kSortTile;
    p.tiles = (int)((n + p.chunk - 1) / p.chunk);
    const int passes = (bits + kSortDigit - 1) / kSortDigit;
    p.bits = (bits + passes - 1) / passes;
    uint32_t *ktmp = nullptr, *vtmp = nullptr;
    hipError_t e = sc.alloc((void **)&p.counts, sizeof(int32_t) * ((int64_t)p.tiles << p.bits));
    if (e == hipSuccess) e = sc.alloc((void **)&p.totals, sizeof(int32_t) << p.bits);
    if (e == hipSuccess && passes > 1) e = sc.alloc((void **)&ktmp, sizeof(uint32_t) * n);
    if (e == hipSuccess && passes > 1) e = sc.alloc((void **)&vtmp, sizeof(uint32_t) * n);
    if (e != hipSuccess) return e;
    for (int i = 0; i < passes; ++i) {
        p.shift = i * p.bits;
        p.kin = i == 0 ? kin : p.kout;
        p.vin = i == 0 ? vin : p.vout;
        const bool last = (passes - 1 - i) % 2 == 0; // passes end in kout / vout
        p.kout = last ? kout : ktmp;
        p.vout = last ? vout : vtmp;
        hipLaunchKernelGGL(sort_count_kernel, dim3(p.tiles), dim3(kThreads), 0, setup_stream(), p);
        hipLaunchKernelGGL(sort_tiles_kernel, dim3(((1 << p.bits) + kThreads / 64 - 1) / (kThreads / 64)), dim3(kThreads), 0,
                           setup_stream(), 1 << p.bits, p.tiles, p.counts, p.totals);
        hipLaunchKernelGGL(sort_scatter_kernel, dim3(p.tiles), dim3(kThreads), 0, setup_stream(), p);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

} // namespace
} // namespace pcsr
