// SpMM computing engine for gfx950 (wave64): the kernel of Algorithm 2 (Section 4.3),
// laid out for 64-lane wavefronts.
//
// Mapping.  A wavefront is cut into G = 64/LPR groups of LPR lanes; each group owns
// one work item (a row panel, or a slice of one when balancing is on).  Lane l of a
// group covers, for r in [0, REP), the VEC consecutive columns starting at
//   kbase + (r*LPR + l)*VEC,      kbase = blockIdx.y * LPR*VEC*REP,
// so every B load of a group is one contiguous LPR*VEC*4-byte segment.  REP plays the
// role of the coarsening factor F, blockDim/64 the role of W, and the V value slots of
// a nonzero vector reuse each fetched B segment V times.
//
// Traversal.  The group reads its colIdx/val range LPR vectors at a time with one
// coalesced load per lane, then broadcasts vector j to all lanes (v_readlane for a
// full-wave group, ds_bpermute otherwise) and gathers B.  Partial sums of one chunk
// are folded into the running sum once per chunk, which keeps fp32 error growth
// logarithmic-ish on rows with 1e5 nonzeros.
#include "pcsr_kernels.h"

#include <array>
#include <mutex>
#include <type_traits>
#include <set>
#include <utility>

// registers of B data a lane keeps in flight per gather step
#define PCSR_INFLIGHT 16
// balanced (power-law) inputs gather scattered lines: twice as deep (see spmm_kernel)
#define PCSR_INFLIGHT_SPLIT 32
// gathers per step at most
#define PCSR_MAXSTEP 8

// Workspace of the entry point that allocates nothing (pcsr_spmm_static).  In host code
// this name is only a handle for hipGetSymbolAddress; kernels get the looked-up address.
static __device__ __align__(256) unsigned char scratch[pcsr::kStaticScratchBytes];

// Read in place of a row of B by the column-window kernel's memory gathers where an entry
// slot past the end of a chunk, or a column past K, has nothing to load (an address select
// instead of a branch around the load).  Indexed by column within the grid.y slice (at most
// 64 lanes * 4 * 4 columns).
static __device__ __align__(16) float g_zero_row[1024];

namespace pcsr {
namespace {

// Vectors of floats in memory.  The hardware takes 8- and 16-byte accesses at any 4-byte
// address, so widths that are no multiple of the vector need no narrower loads.
template <int N> struct Vec;
template <> struct Vec<1> { using type = float; };
template <> struct Vec<2> { typedef float type __attribute__((ext_vector_type(2), aligned(4))); };
template <> struct Vec<4> { typedef float type __attribute__((ext_vector_type(4), aligned(4))); };

template <int VEC> __device__ __forceinline__ void load_vec(const float *p, float (&d)[VEC])
{
    using T = typename Vec<VEC>::type;
    const T t = *reinterpret_cast<const T *>(p);
    if constexpr (VEC == 1) {
        d[0] = t;
    } else {
#pragma unroll
        for (int e = 0; e < VEC; ++e) d[e] = t[e];
    }
}

// The same in LDS, where an access that is not known to be aligned is split into dwords.
template <int N> struct LdsVec {
    typedef float type __attribute__((ext_vector_type(N)));
};
template <int VEC> __device__ __forceinline__ void load_lds(const float *p, float (&d)[VEC])
{
    if constexpr (VEC == 1) {
        d[0] = *p;
    } else {
        const auto t = *reinterpret_cast<const typename LdsVec<VEC>::type *>(p);
#pragma unroll
        for (int e = 0; e < VEC; ++e) d[e] = t[e];
    }
}
// The same by LDS address: an address that is made of a broadcast and a sum takes both in one instruction then.
__device__ __forceinline__ unsigned lds_address(const float *p)
{
    return (unsigned)(uintptr_t)(const __attribute__((address_space(3))) float *)p;
}
template <int VEC> __device__ __forceinline__ void load_lds_at(unsigned at, float (&d)[VEC])
{
    using T = typename std::conditional<VEC == 1, float, typename LdsVec<VEC>::type>::type;
    const T t = *(const __attribute__((address_space(3))) T *)(uintptr_t)at;
    if constexpr (VEC == 1) {
        d[0] = t;
    } else {
#pragma unroll
        for (int e = 0; e < VEC; ++e) d[e] = t[e];
    }
}
template <int VEC> __device__ __forceinline__ void store_lds(float *p, const float (&s)[VEC])
{
    if constexpr (VEC == 1) {
        *p = s[0];
    } else {
        typename LdsVec<VEC>::type t;
#pragma unroll
        for (int e = 0; e < VEC; ++e) t[e] = s[e];
        *reinterpret_cast<typename LdsVec<VEC>::type *>(p) = t;
    }
}

// nontemporal store: C is never read again
template <int VEC> __device__ __forceinline__ void store_vec(float *p, const float (&s)[VEC])
{
    if constexpr (VEC == 1) {
        __builtin_nontemporal_store(s[0], p);
    } else {
        using ext_t = typename Vec<VEC>::type;
        ext_t x;
#pragma unroll
        for (int e = 0; e < VEC; ++e) x[e] = s[e];
        __builtin_nontemporal_store(x, reinterpret_cast<ext_t *>(p));
    }
}

// Elementwise tail of a row of C, columns k .. k + VEC - 1.  self_row and mask_row fetch what it reads of that row; where they
// load it, that is at the point of use (loaded ahead of the bias the mask costs registers also where there is none: road graph of
// 2,000,000 rows with a ReLU, K = 128 402 -> 418 us).
template <int VEC, class Self, class Mask>
__device__ __forceinline__ void finish(const Epilogue &ep, int k, Self self_row, Mask mask_row, float (&v)[VEC])
{
    if (ep.self) {
        const float scale = 1.0f + (ep.self_eps ? *ep.self_eps : 0.0f);
        float t[VEC];
        self_row(t);
#pragma unroll
        for (int e = 0; e < VEC; ++e) v[e] = fmaf(scale, t[e], v[e]);
    }
    if (ep.bias) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) v[e] += ep.bias[k + e];
    }
    if (ep.relu) { // as written NaN stays NaN
#pragma unroll
        for (int e = 0; e < VEC; ++e) v[e] = v[e] <= 0.0f ? 0.0f : v[e];
    }
    if (ep.mask) {
        float t[VEC];
        mask_row(t);
#pragma unroll
        for (int e = 0; e < VEC; ++e) v[e] = t[e] <= 0.0f ? 0.0f : v[e];
    }
}
// One uniform branch for a plain SpMM.
template <int VEC> __device__ __forceinline__ void finish(const Epilogue &ep, long row, int K, int k, float (&v)[VEC])
{
    if (!ep.on) return;
    finish<VEC>(ep, k, [&](float (&t)[VEC]) { load_vec<VEC>(ep.self + row * K + k, t); },
                [&](float (&t)[VEC]) { load_vec<VEC>(ep.mask + row * K + k, t); }, v);
}
// What the tail reads of a row, requested long before the row is there.
template <int VEC> struct TailRow {
    float self[VEC], mask[VEC];
};
template <int VEC> __device__ __forceinline__ void fetch_tail(const Epilogue &ep, long row, int K, int k, TailRow<VEC> &t)
{
    if (ep.self) load_vec<VEC>(ep.self + row * K + k, t.self);
    if (ep.mask) load_vec<VEC>(ep.mask + row * K + k, t.mask);
}
template <int VEC> __device__ __forceinline__ void finish(const Epilogue &ep, int k, const TailRow<VEC> &row, float (&v)[VEC])
{
    auto copy = [](const float (&from)[VEC], float (&t)[VEC]) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) t[e] = from[e];
    };
    finish<VEC>(ep, k, [&](float (&t)[VEC]) { copy(row.self, t); }, [&](float (&t)[VEC]) { copy(row.mask, t); }, v);
}

// cacheable store: workspace partials are read back by the next kernel
template <int VEC> __device__ __forceinline__ void store_vec_cached(float *p, const float (&s)[VEC])
{
    using T = typename Vec<VEC>::type;
    T t;
    if constexpr (VEC == 1) {
        t = s[0];
    } else {
#pragma unroll
        for (int e = 0; e < VEC; ++e) t[e] = s[e];
    }
    *reinterpret_cast<T *>(p) = t;
}

// colIdx / val are read exactly once per SpMM.  (A nontemporal load, meant to keep them
// from displacing B rows in L2, measured no different.)
template <class T> __device__ __forceinline__ T stream_load(const T *p)
{
    return *p;
}

template <int LPR> __device__ __forceinline__ int bcast(int x, int j)
{
    if constexpr (LPR == 64)
        return __builtin_amdgcn_readlane(x, j);
    else
        return __shfl(x, j, LPR);
}
template <int LPR> __device__ __forceinline__ float bcast(float x, int j)
{
    return __int_as_float(bcast<LPR>(__float_as_int(x), j));
}

// Broadcast inside a 16-lane group when the source lane is known at compile time (the
// unrolled step loop): a DPP move, "lane j of every row of 16 to the whole row", which runs
// in the vector ALU instead of going through the LDS crossbar like ds_bpermute.
__device__ __forceinline__ int bcast16_const(int x, int j)
{
#define PCSR_DPP_CASE(J) \
    case J: return __builtin_amdgcn_mov_dpp(x, 0x150 + J, 0xf, 0xf, true)
    switch (j & 15) {
        PCSR_DPP_CASE(0);
        PCSR_DPP_CASE(1);
        PCSR_DPP_CASE(2);
        PCSR_DPP_CASE(3);
        PCSR_DPP_CASE(4);
        PCSR_DPP_CASE(5);
        PCSR_DPP_CASE(6);
        PCSR_DPP_CASE(7);
        PCSR_DPP_CASE(8);
        PCSR_DPP_CASE(9);
        PCSR_DPP_CASE(10);
        PCSR_DPP_CASE(11);
        PCSR_DPP_CASE(12);
        PCSR_DPP_CASE(13);
        PCSR_DPP_CASE(14);
    default: return __builtin_amdgcn_mov_dpp(x, 0x150 + 15, 0xf, 0xf, true);
    }
#undef PCSR_DPP_CASE
}
// whether p holds in every active lane of the wavefront (a uniform branch)
__device__ __forceinline__ bool wave_all(bool p) { return __builtin_amdgcn_ballot_w64(!p) == 0; }

// acc += (lane j of the 16-lane group's a) * b in one instruction: the DPP operand of a
// VOP2 multiply-add does the broadcast, so no separate move is spent on it.
__device__ __forceinline__ void fmac_bcast16_const(float &acc, float a, float b, int j)
{
#define PCSR_FMAC_CASE(J)                                                                             \
    case J:                                                                                           \
        asm("v_fmac_f32_dpp %0, %1, %2 row_newbcast:" #J " row_mask:0xf bank_mask:0xf"                 \
            : "+v"(acc)                                                                               \
            : "v"(a), "v"(b));                                                                        \
        break
    switch (j & 15) {
        PCSR_FMAC_CASE(0);
        PCSR_FMAC_CASE(1);
        PCSR_FMAC_CASE(2);
        PCSR_FMAC_CASE(3);
        PCSR_FMAC_CASE(4);
        PCSR_FMAC_CASE(5);
        PCSR_FMAC_CASE(6);
        PCSR_FMAC_CASE(7);
        PCSR_FMAC_CASE(8);
        PCSR_FMAC_CASE(9);
        PCSR_FMAC_CASE(10);
        PCSR_FMAC_CASE(11);
        PCSR_FMAC_CASE(12);
        PCSR_FMAC_CASE(13);
        PCSR_FMAC_CASE(14);
        PCSR_FMAC_CASE(15);
    }
#undef PCSR_FMAC_CASE
}

template <int LPR, bool CONST_LANE> __device__ __forceinline__ int bcast_any(int x, int j)
{
    if constexpr (LPR == 16 && CONST_LANE)
        return bcast16_const(x, j);
    else
        return bcast<LPR>(x, j);
}
template <int LPR, bool CONST_LANE> __device__ __forceinline__ float bcast_any(float x, int j)
{
    return __int_as_float(bcast_any<LPR, CONST_LANE>(__float_as_int(x), j));
}
// base + the byte offset that lane j of every DPP row holds
__device__ __forceinline__ const float *row_ptr(const float *base, long off, int j)
{
    typedef int i2 __attribute__((ext_vector_type(2)));
    const i2 o = {bcast16_const((int)off, j), bcast16_const((int)(off >> 32), j)};
    return reinterpret_cast<const float *>(reinterpret_cast<const char *>(base) + __builtin_bit_cast(long, o));
}

// Operands of at most kNearBytes: a gather's address is a scalar base and a 32-bit offset, one addition that takes the
// broadcast with it, where 64-bit addresses took five vector instructions.  Where a lane loads one dword, B is a buffer: a
// slot with nothing to load reads past the end, at kPast, which the hardware answers with zeros and no access, and the
// branches around such slots go as well.  (8- and 16-byte loads were 4-6 % slower as buffer loads, at any alignment.)  A
// lane past the last column reads the last one, as its neighbour does: reading anything else, past the end too, it doubled
// the time of a load (16 lanes x dword x 2, K = 22: 131 us for 66).  Cliques of 40, 300,000 rows: K = 16 61 -> 50 us, K = 22
// 77 -> 67, paired rows 45 -> 38 and 61 -> 48; where B comes from memory, R-MAT 2^22, K = 16 1417 -> 1392.  16-byte loads:
// cliques of 24, K = 75 126.6 -> 123.7, paired rows of 40, K = 64 78 -> 76, others as before.
constexpr uint64_t kNearBytes = 0xe0000000u;
constexpr unsigned kPast = 0xf0000000u; // plus a column's bytes (launch_spmm: K is below 2^20) still past the end, and no wrap
__device__ __forceinline__ __amdgpu_buffer_rsrc_t near_operand(const SpmmArgs &a)
{
    // stride 0: num_records in bytes; word 3: 32-bit data
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.B), 0, (int)((unsigned)a.n_cols * ((unsigned)a.K * 4u)),
                                             0x00020000);
}
__device__ __forceinline__ float load_near(__amdgpu_buffer_rsrc_t b, unsigned at)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(b, (int)at, 0, 0));
}
template <int VEC> __device__ __forceinline__ void load_near4(__amdgpu_buffer_rsrc_t b, unsigned at, float (&d)[VEC])
{
    typedef float f4 __attribute__((ext_vector_type(4)));
    const f4 t = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(b, (int)at, 0, 0));
#pragma unroll
    for (int e = 0; e < VEC; ++e) d[e] = t[e & 3];
}

// What an instance of spmm_kernel is for beside the plain product.  Instances of their own: products with short items lost
// 0.5 % to kLongItems' three branches (R-MAT 2^22, K = 16: 1404 -> 1411 us).
constexpr int kAsIs = 0;
constexpr int kLongItems = 1; // balanced handles with long items (SpmmArgs::outer): sums of 32 vectors are added up apart
constexpr int kEarlyTail = 2; // unsplit products whose tail reads the row: the self and mask rows are requested before the traversal
// Single unsplit rows, a band of columns at a time (SpmmArgs::band), one launch each.  Scattered rows of B come from memory, at 57 G
// lines of 128 bytes a second, unless an XCD's L2 holds them, which gives 190 G rows: the band of B that a launch reads is as small
// as that, and the price is C read and written once more by each (uniform columns, 300,000 rows of 134, K = 16: 667 us in one, 542,
// 437, 372, 366 and 446 in 2, 3, 4, 6 and 12).  Sums of 8 vectors are added up to 32 in up to three bands, to 64 in more, before
// they go to the row's, which costs nothing: the rms difference from 64 bits of rows of 44, 60, 90, 134 and 300 ones between 0 and
// 1 is 4.3 to 4.8e-8 of their sum (300: 4.8 to 5.8), 4.7 to 5.1 (5.8) by items of 32 and 5.0 to 7.1 in one sum.  A whole wavefront's
// chunk is 64 vectors: half of it at a time where sums are of 32 (rows of 60, K = 260 4.97 -> 4.19e-8, items of 32 4.18; the time
// is the same).  Over 256 columns it has two tiles of them, in place of the plain kernel, whose sums are of 64 there (rows of 60
// 11.0e-8, of 90 8.8, here 4.45; 1362 us and 1355, 1265 and 1325).
constexpr int kBands = 3;
// One dword a lane, its sums put together more often than the lanes' entries are, and those of 32 added up apart.  Up to 8 columns of
// unsplit rows by 16 lanes (narrow_lanes says why), whose sums are of 4 vectors as those of 4 lanes with wider
// loads are, or of 8 where items are of 22 and more on average: rms difference from 64 bits of rows of 13, 18, 25 and 32 numbers between
// 0 and 1 4.36, 4.53, 4.65 and 4.72e-8 of their sum, by 4 lanes 4.36, 4.53, 4.90 and 5.23, in sums of 16 5.76, 5.73, 5.46 and 5.44.  And
// 17 to 32 columns of single rows by 32 lanes, or 16 with two columns each, in place of 8 with four, in sums of 8 as those have (of 16
// and 32: rows of 30 5.4 and 8.1e-8, of 8 4.7); up to 64 by 32 with two.  Rows of 90, 134 and 300: 4.5, 4.8 and 5.8, in one sum of
// them without those of 32 5.85, 6.6 and 9.6, in sums of 16 5.2, 5.5 and 7.2.
constexpr int kNarrow = 4;

// EPI: with an elementwise tail.  Instances of their own, for the auto launch shapes only: the
// branch alone cost the instance <2, false, 64, 1, 2> 4 %.
// (Seven waves per SIMD are asked for where the compiler would take six for want of a few registers; two is what 512
// threads imply.)
// NEAR: offsets of 32 bits (kNearBytes).
template <int V, bool S, int LPR, int VEC, int REP, bool EPI, int FORM, bool NEAR>
__global__ void __launch_bounds__(512)
__attribute__((amdgpu_waves_per_eu(FORM == kLongItems && V == 2 && LPR == 32 && VEC == 4 && REP == 1 && !EPI ? 7 : 2)))
spmm_kernel(SpmmArgs a)
{
    constexpr bool OUTER = FORM == kLongItems;
    constexpr bool BUFFER = NEAR && VEC == 1;
    constexpr int G = 64 / LPR;
    // vectors gathered per inner step: 16 registers of B data in flight, 32 for balanced
    // handles and for V = 1 with groups of up to 8 lanes (K <= 32: 4-8 % faster on rows of 40
    // and more nonzeros, no different on short rows; with V = 2 it costs road-like inputs
    // 2-7 %, and with wider groups it changes nothing)
    constexpr bool DEEP = S || (V == 1 && LPR <= 8);
    constexpr int U0 = (DEEP ? PCSR_INFLIGHT_SPLIT : PCSR_INFLIGHT) / (REP * VEC);
    constexpr int Uc = U0 < 1 ? 1 : (U0 > PCSR_MAXSTEP ? PCSR_MAXSTEP : U0);
    // Entries per chunk: one per lane, and for groups of more than 16 lanes the same 16 (or twice
    // 16, two per lane) in each of their DPP rows, so that broadcasts stay inside a row.  32 is
    // 5 % faster where rows are long (LPR 32, V = 1: scattered inputs), 16 where paired rows
    // are short (LPR 32, V = 2: road-like and clique inputs, 8-15 %).
    // A whole wavefront on one row broadcasts through scalar registers (v_readlane) instead: its
    // row addresses then cost no vector instruction at all.
    constexpr int CH = LPR == 32 && V == 2 ? 16 : LPR;
    constexpr bool DPP = LPR == 16 || LPR == 32;
    constexpr int NH = DPP ? CH / 16 : 1; // entries per lane
    constexpr int U = Uc > CH ? CH : Uc; // a step never reaches past the chunk
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int waves = blockDim.x >> 6;
    // Consecutive workgroup ids go round-robin over the 8 XCDs.  With xcd_remap each XCD
    // walks its own contiguous range of work items (ranges hold equal work, not equal
    // item counts), so neighbouring rows share one L2.
    long item_l = ((long)blockIdx.x * waves + wave) * G + (lane / LPR);
    int limit = a.M;
    if (a.xcd_remap) {
        const int x = blockIdx.x & 7;
        item_l = a.xb[x] + ((long)(blockIdx.x >> 3) * waves + wave) * G + (lane / LPR);
        limit = a.xb[x + 1];
    }
    const int lg = lane & (LPR - 1);
    if (item_l >= limit) return;

    // Everything the item needs to know about itself, fetched in one round trip: its
    // vector range, the panel it writes to (TRow) and its workspace slot (-1: the only
    // item of its panel).  A column-ordered schedule keeps these as one 16-byte record
    // per launch position.
    int head, tail, panel = (int)item_l, slot = -1;
    if constexpr (S) {
        if (a.sched) {
            const int4 rec = a.sched[item_l];
            head = rec.x;
            tail = rec.x + rec.y;
            panel = rec.z;
            slot = rec.w;
        } else {
            head = a.rowptr[item_l];
            tail = a.rowptr[item_l + 1];
            panel = a.trow[item_l];
            slot = a.item_slot[item_l];
        }
    } else {
        head = a.rowptr[item_l];
        tail = FORM == kBands ? a.trow[item_l] : a.rowptr[item_l + 1];
    }
    if constexpr (LPR == 64) {
        head = __builtin_amdgcn_readfirstlane(head);
        tail = __builtin_amdgcn_readfirstlane(tail);
    }

    const int kbase = blockIdx.y * (LPR * VEC * REP);
    int kc[REP];
    bool kv[REP];
#pragma unroll
    for (int r = 0; r < REP; ++r) {
        kc[r] = kbase + (r * LPR + lg) * VEC;
        kv[r] = kc[r] < a.K;
    }
    // K no multiple of VEC: the last vector of a row is moved back to end with it.  The columns it
    // shares with its neighbour are computed and stored twice, the same bits; the atomic
    // write-back skips them, and bands after the first are launched only where the neighbour is in the same wavefront.
#pragma unroll
    for (int r = 0; r < REP; ++r)
        if (kv[r]) kc[r] = min(kc[r], a.K - VEC);
    // a lane past the last column loads what its neighbour loads and stores nothing
    const int lane_col = kv[0] ? kc[0] : a.K - VEC;
    const float *__restrict__ B_lane = a.B + lane_col;
    int step_col[REP]; // columns from the first load to the r-th
#pragma unroll
    for (int r = 0; r < REP; ++r) step_col[r] = kc[r] - lane_col;

    float acc[V][REP][VEC];
#pragma unroll
    for (int v = 0; v < V; ++v)
#pragma unroll
        for (int r = 0; r < REP; ++r)
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc[v][r][e] = 0.0f;

    const long K = a.K;
    __amdgpu_buffer_rsrc_t Bn;
    unsigned near_col[REP]; // bytes
    if constexpr (BUFFER) Bn = near_operand(a);
    if constexpr (NEAR) {
#pragma unroll
        for (int r = 0; r < REP; ++r) near_col[r] = (unsigned)(kv[r] ? kc[r] : a.K - VEC) * 4u;
    }

    // What the tail reads is requested before the traversal, where it fits the registers: behind it, it is one more round trip
    // to memory for an item that is three of them in all (road graph of 2,000,000 rows with a self term: K = 64 285 -> 275
    // us, K = 128 557 -> 534, with a mask 288 -> 281).  Not where it reads nothing: the registers cost a wavefront per SIMD (with a
    // bias K = 64 235 -> 255, K = 128 449 -> 492).  Items of balanced handles have too many registers in flight for it (R-MAT 2^20,
    // K = 64: 420 -> 447).
    constexpr bool EARLY = FORM == kEarlyTail;
    TailRow<VEC> tail_row[EARLY ? V : 1][EARLY ? REP : 1];
    if constexpr (EARLY) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const long row = (long)panel * V + v;
            if (row < a.n_rows) {
#pragma unroll
                for (int r = 0; r < REP; ++r)
                    if (kv[r]) fetch_tail<VEC>(a.epi, row, a.K, kc[r], tail_row[v][r]);
            }
        }
    }

    // Sums of 32 or 64 vectors are added up here, as OUTER below has it; to what the bands before have left, requested beside the
    // first entries.  (Pairs are local more often than not, and bound by their instructions: none of it there.  20,000 rows of 70 in
    // cliques, K = 16 9.3 and 9.8 us.)  Items of 8 lanes of a dword, up to 8 columns of balanced handles, have sums of 4 where items
    // are short, as the 4 lanes of wide loads had (R-MAT 2^16, K = 4: 3.55e-8 of the sum, of 8 3.74), of 8 where they are of 22 and more
    // on average (30,000 rows of 45 in items of 32: 4.35, of 4 4.65) and at odd widths, which never had 4.
    constexpr bool FOURS = S && LPR == 8 && VEC == 1 && REP == 1;
    constexpr bool APART = FORM == kBands || (FORM == kNarrow && V == 1) || (FOURS && !OUTER);
    float apart[APART ? V : 1][APART ? REP : 1][VEC];
    if constexpr (APART) {
#pragma unroll
        for (int v = 0; v < V; ++v)
#pragma unroll
            for (int r = 0; r < REP; ++r) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) apart[v][r][e] = 0.0f;
                if (FORM == kBands && !(a.band & kBandFirst) && kv[r]) load_vec<VEC>(a.C + (long)panel * K + kc[r], apart[v][r]);
            }
    }

    // one lane's entries of the chunk that starts at `base` (zeros past the end of the range)
    auto load_entry = [&](int base, int (&c)[NH], float (&av)[NH][V]) {
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            const int idx = base + 16 * h + (DPP ? lg & 15 : lg);
            c[h] = 0;
#pragma unroll
            for (int v = 0; v < V; ++v) av[h][v] = 0.0f;
            if (idx < tail) {
                c[h] = stream_load(a.colidx + idx);
                if constexpr (V == 1) {
                    av[h][0] = stream_load(a.val + idx);
                } else {
                    typedef float f2 __attribute__((ext_vector_type(2)));
                    const f2 t = stream_load(reinterpret_cast<const f2 *>(a.val) + idx);
                    av[h][0] = t[0];
                    av[h][1] = t[1];
                }
            }
        }
    };

    // OUTER, as the second pass adds the sums of items of 32 (64 where a whole wavefront takes an item, whose own sums are of
    // 8).  One running sum over a whole row loses more the longer the row.  Rms of the difference from 64 bits, relative to the sum
    // of magnitudes, at K = 8, 32, 64, 256: rows of 300 6.1, 5.9, 6.7 and 6.0e-9 (11.0, 8.1, 7.5 and 8.5e-9 with one running sum,
    // 6.1, 5.9, 6.7 and 6.7e-9 by items of 32), of 1000 4.4, 4.4, 4.7 and 3.9e-9 (9.8, 7.2, 5.8 and 7.4e-9; 4.5, 4.5, 4.8 and
    // 4.8e-9).  The time is the same within 1 % (250,000 rows of 48, K = 16 80 -> 82 us, 128 263, 512 1285).  In LDS, four floats or
    // so per thread, which only that thread uses: four more registers would cost an instance a wavefront per SIMD, and so the
    // slot's address is made anew each time, and the slot holds zeros at first.
    extern __shared__ __align__(16) float lds[];
    const int wave_at = __builtin_amdgcn_readfirstlane(wave) * 64;
    auto outer = [&](auto use) {
        int t; // lane; volatile: not kept in a register across the walk
        asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(t));
#pragma unroll
        for (int v = 0; v < V; ++v)
#pragma unroll
            for (int r = 0; r < REP; ++r) use(acc[v][r], lds + ((v * REP + r) * 64 * waves + wave_at + t) * VEC);
    };
    auto add_outer = [](float (&x)[VEC], const float *at) {
        float t[VEC];
        load_lds<VEC>(at, t);
#pragma unroll
        for (int e = 0; e < VEC; ++e) x[e] += t[e];
    };
    auto keep_apart = [&](float (&x)[VEC], float *at) {
        add_outer(x, at);
        store_lds<VEC>(at, x);
#pragma unroll
        for (int e = 0; e < VEC; ++e) x[e] = 0.0f;
    };
    if constexpr (OUTER) outer([](float (&x)[VEC], float *at) { store_lds<VEC>(at, x); });

    auto put_apart = [&] {
        if constexpr (APART) {
#pragma unroll
            for (int v = 0; v < V; ++v)
#pragma unroll
                for (int r = 0; r < REP; ++r)
#pragma unroll
                    for (int e = 0; e < VEC; ++e) {
                        apart[v][r][e] += acc[v][r][e];
                        acc[v][r][e] = 0.0f;
                    }
        }
    };

    // The next chunk's colIdx/val are requested before the current chunk's gathers, so
    // that a chunk costs one memory round trip, not two.
    int c_next[NH];
    float av_next[NH][V];
    load_entry(head, c_next, av_next);
    constexpr int PERIOD = CH < 32 ? 32 / CH : 1;
    const int band_period = FORM == kBands && (a.band & kBandSums64) ? 64 / CH : PERIOD;
    int until = band_period; // chunks until the next sum is put apart (the same in every lane group)
    for (int base = head; base < tail; base += CH) {
        long off[NH]; // DPP: in bytes, computed once by the lane that holds the entry
        unsigned near_off[NH]; // NEAR: the same
        int c[NH];
        float av[NH][V];
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            c[h] = c_next[h];
            if constexpr (NEAR) {
                const int idx = base + 16 * h + (DPP ? lg & 15 : lg);
                near_off[h] = idx < tail ? (unsigned)c[h] * ((unsigned)a.K * 4u) : kPast;
            } else {
                off[h] = (long)c[h] * (K * 4);
            }
#pragma unroll
            for (int v = 0; v < V; ++v) av[h][v] = av_next[h][v];
        }
        load_entry(base + CH, c_next, av_next);
        const int cnt = min(CH, tail - base);

        float part[V][REP][VEC];
#pragma unroll
        for (int v = 0; v < V; ++v)
#pragma unroll
            for (int r = 0; r < REP; ++r)
#pragma unroll
                for (int e = 0; e < VEC; ++e) part[v][r][e] = 0.0f;

        // Wide instances of balanced handles walk whole rows where these run by community: no sum of more than 8 vectors is kept
        // apart, whatever the chunk.  Rows of 48 against 64 bits, rms of their sum of magnitudes: 1.67e-8, where sums
        // of a chunk of 32 and 64 lanes made it 2.23 and 2.79e-8 (items of 32 in chunks of 16: 1.82e-8).  These kernels wait on
        // memory: the additions cost nothing (250,000 rows, K = 128 262 us, K = 256 577, both as before).
        constexpr bool FOLD = (S && LPR >= 32) || FORM == kBands || FORM == kNarrow;
        static_assert(!FOURS || U == 8);
        const bool even = FOURS && a.K % 2 == 0 && a.mean_item < 22;
        // (Wider groups past the widths they are for: of 8, as 8 lanes' chunks.)
        const bool fours = FORM == kNarrow && REP == 1 && a.mean_item < 22 && (LPR == 16 || (a.K > 16 && a.K <= 32));
        auto fold = [&] {
#pragma unroll
            for (int v = 0; v < V; ++v)
#pragma unroll
                for (int r = 0; r < REP; ++r)
#pragma unroll
                    for (int e = 0; e < VEC; ++e) {
                        acc[v][r][e] += part[v][r][e];
                        part[v][r][e] = 0.0f;
                    }
        };

        // U vectors per step: all gathers first, then the FMAs, so U*REP loads are in flight
        // together.  Slots past the end of the range carry val = 0 (set above) and load
        // nothing.  (Branching around those loads measured 1-3 % faster here than reading a
        // row of zeros through an address select.)  full: no such slots in this step.
        auto step = [&](int j, auto full_step) {
            constexpr bool FULL = decltype(full_step)::value;
            const int h = DPP && NH > 1 ? j >> 4 : 0; // a step stays inside 16 entries
            float b[U][REP][VEC];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                unsigned near_row = 0;
                if constexpr (NEAR) near_row = (unsigned)bcast_any<DPP ? 16 : LPR, DPP>((int)near_off[h], j + u);
                if constexpr (BUFFER) {
#pragma unroll
                    for (int r = 0; r < REP; ++r)
                        b[u][r][0] = load_near(Bn, near_row + near_col[r]);
                    continue;
                }
                const float *at;
                if constexpr (NEAR)
                    at = reinterpret_cast<const float *>(reinterpret_cast<const char *>(a.B) + (near_row + near_col[0]));
                else if constexpr (DPP)
                    at = row_ptr(B_lane, off[h], j + u);
                else if constexpr (LPR == 64)
                    at = a.B + (long)bcast<LPR>(c[h], j + u) * K;
                else
                    at = B_lane + (long)bcast<LPR>(c[h], j + u) * K;
                if (FULL || j + u < cnt) {
                    load_vec<VEC>(LPR == 64 ? at + lane_col : at, b[u][0]);
#pragma unroll
                    for (int r = 1; r < REP; ++r) {
                        if (kv[r]) {
                            load_vec<VEC>(NEAR ? reinterpret_cast<const float *>(reinterpret_cast<const char *>(a.B) +
                                                                                 (near_row + near_col[r]))
                                               : at + (LPR == 64 ? kc[r] : step_col[r]),
                                          b[u][r]);
                        } else {
#pragma unroll
                            for (int e = 0; e < VEC; ++e) b[u][r][e] = 0.0f;
                        }
                    }
                } else {
#pragma unroll
                    for (int r = 0; r < REP; ++r)
#pragma unroll
                        for (int e = 0; e < VEC; ++e) b[u][r][e] = 0.0f;
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    float aj;
                    if constexpr (DPP)
                        aj = __int_as_float(bcast16_const(__float_as_int(av[h][v]), j + u));
                    else
                        aj = bcast<LPR>(av[h][v], j + u);
#pragma unroll
                    for (int r = 0; r < REP; ++r)
#pragma unroll
                        for (int e = 0; e < VEC; ++e) part[v][r][e] = fmaf(aj, b[u][r][e], part[v][r][e]);
                }
                if (FOLD && (j + u) % 8 == 7) fold();
                if (FOURS && (u % 8 == 7 || (u % 4 == 3 && even))) fold();
                if (FORM == kNarrow && (j + u) % 8 == 3 && fours) fold();
                if (FORM == kBands && CH == 64 && (j + u) % 32 == 31 && !(a.band & kBandSums64)) put_apart(); // half a chunk
            }
        };
        if constexpr (DPP) {
            // the steps written out, so every broadcast lane is a constant
#pragma unroll
            for (int j = 0; j < CH; j += U) {
                if (j >= cnt) break;
                if (BUFFER || wave_all(j + U <= cnt))
                    step(j, std::true_type{});
                else
                    step(j, std::false_type{});
            }
        } else {
            for (int j = 0; j < cnt; j += U) {
                if (BUFFER || wave_all(j + U <= cnt))
                    step(j, std::true_type{});
                else
                    step(j, std::false_type{});
            }
        }
        if constexpr (!(FOLD && U % 8 == 0) && !FOURS) // (every step ends with a fold)
#pragma unroll
            for (int v = 0; v < V; ++v)
#pragma unroll
                for (int r = 0; r < REP; ++r)
#pragma unroll
                    for (int e = 0; e < VEC; ++e) acc[v][r][e] += part[v][r][e];
        if constexpr (APART) {
            if (--until == 0) {
                until = band_period;
                put_apart();
            }
        }
        if constexpr (OUTER) {
            if (--until == 0) {
                until = PERIOD;
                const bool more = LPR == 64 ? wave_all(base + CH < tail) : base + CH < tail; // (as one keeps a register free)
                if (more) outer(keep_apart);
            }
        }
    }
    if constexpr (OUTER) outer(add_outer);
    if constexpr (APART && FORM != kBands) {
#pragma unroll
        for (int v = 0; v < V; ++v)
#pragma unroll
            for (int r = 0; r < REP; ++r)
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc[v][r][e] = apart[v][r][e] + acc[v][r][e];
    }

    // write-back (Algorithm 2, last block): plain store for an item that is the only one
    // of its panel.  An item of a panel that was split (TRow names the panel) either
    // leaves its partial rows in the workspace slot that belongs to it, for the second
    // pass to add in item order, or, without a workspace, accumulates with atomics.
    if constexpr (FORM == kBands) {
        static_assert(V == 1 && !S);
        if (tail == head && !(a.band & kBandFirst) && !(EPI && (a.band & kBandLast))) return; // C is as it was
#pragma unroll
        for (int r = 0; r < REP; ++r) {
            if (!kv[r]) continue;
            float *const at = a.C + (long)panel * K + kc[r];
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc[0][r][e] = apart[0][r][e] + acc[0][r][e];
            if (a.band & kBandLast) {
                if constexpr (EPI) finish<VEC>(a.epi, (long)panel, a.K, kc[r], acc[0][r]);
                store_vec<VEC>(at, acc[0][r]);
            } else {
                store_vec_cached<VEC>(at, acc[0][r]);
            }
        }
        return;
    }
    const bool sole = slot < 0;
    float *wrow = nullptr;
    if constexpr (S) {
        if (!sole && a.ws) wrow = a.ws + (long)slot * V * K;
    }
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const long row = (long)panel * V + v;
        if (row < a.n_rows) {
            float *crow = wrow ? wrow + v * K : a.C + row * K;
#pragma unroll
            for (int r = 0; r < REP; ++r) {
                if (kv[r]) {
                    if (sole) {
                        if constexpr (EARLY)
                            finish<VEC>(a.epi, kc[r], tail_row[v][r], acc[v][r]);
                        else if constexpr (EPI)
                            finish<VEC>(a.epi, row, a.K, kc[r], acc[v][r]);
                        store_vec<VEC>(crow + kc[r], acc[v][r]);
                    } else if (wrow) {
                        store_vec_cached<VEC>(crow + kc[r], acc[v][r]);
                    } else {
#pragma unroll
                        for (int e = 0; e < VEC; ++e)
                            if (kc[r] + e >= kbase + (r * LPR + lg) * VEC) atomicAdd(crow + kc[r] + e, acc[v][r][e]);
                    }
                }
            }
        }
    }
}

// Batched walk for matrices of short rows (no balancing): one lane group owns IPG
// consecutive work items and walks their joint colIdx/val range as one stream, so the
// gathers of several rows are in flight together.  Every entry carries the index of the
// item it belongs to and only that item's accumulator takes the multiply-add (a select,
// not a multiplication by zero: a non-finite B row must not leak into rows that do not
// reference it).  IPG-fold ALU work, irrelevant next to the memory time of short rows.
template <int V, int LPR, int VEC, int REP, int IPG>
__global__ void __launch_bounds__(512) spmm_batched_kernel(SpmmArgs a)
{
    static_assert(IPG < LPR, "item boundaries are broadcast from the group's own lanes");
    constexpr int G = 64 / LPR;
    constexpr int U0 = PCSR_INFLIGHT / (REP * VEC);
    constexpr int Uc = U0 < 1 ? 1 : (U0 > 8 ? 8 : U0);
    constexpr int U = Uc > LPR ? LPR : Uc; // a step never reaches past the group's chunk
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int waves = blockDim.x >> 6;
    long item0_l = (((long)blockIdx.x * waves + wave) * G + (lane / LPR)) * IPG;
    int limit = a.M;
    if (a.xcd_remap) { // work-balanced contiguous item range per XCD, as in spmm_kernel
        const int x = blockIdx.x & 7;
        item0_l = a.xb[x] + (((long)(blockIdx.x >> 3) * waves + wave) * G + (lane / LPR)) * IPG;
        limit = a.xb[x + 1];
    }
    const int lg = lane & (LPR - 1);
    if (item0_l >= limit) return;
    const int item0 = (int)item0_l;

    const int kbase = blockIdx.y * (LPR * VEC * REP);
    int kc[REP];
    bool kv[REP];
#pragma unroll
    for (int r = 0; r < REP; ++r) {
        kc[r] = kbase + (r * LPR + lg) * VEC;
        kv[r] = kc[r] < a.K;
    }

    // item boundaries: lane i of the group fetches rowPtr[item0 + i], i <= IPG
    const int bsel = item0 + (lg < IPG ? lg : IPG);
    const int my_rp = a.rowptr[bsel < limit ? bsel : limit];
    int rp[IPG + 1];
#pragma unroll
    for (int i = 0; i <= IPG; ++i) rp[i] = bcast<LPR>(my_rp, i);
    const int head = rp[0], tail = rp[IPG];

    float acc[IPG][V][REP][VEC];
#pragma unroll
    for (int i = 0; i < IPG; ++i)
#pragma unroll
        for (int v = 0; v < V; ++v)
#pragma unroll
            for (int r = 0; r < REP; ++r)
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc[i][v][r][e] = 0.0f;

    const float *__restrict__ B = a.B;
    const long K = a.K;

    for (int base = head; base < tail; base += LPR) {
        const int idx = base + lg;
        int c = 0, tag = 0;
        float av[V];
#pragma unroll
        for (int v = 0; v < V; ++v) av[v] = 0.0f;
        if (idx < tail) {
            c = stream_load(a.colidx + idx);
            if constexpr (V == 1) {
                av[0] = stream_load(a.val + idx);
            } else {
                typedef float f2 __attribute__((ext_vector_type(2)));
                const f2 t = stream_load(reinterpret_cast<const f2 *>(a.val) + idx);
                av[0] = t[0];
                av[1] = t[1];
            }
#pragma unroll
            for (int i = 1; i < IPG; ++i) tag += (idx >= rp[i]);
        }
        const int cnt = min(LPR, tail - base);
        for (int j = 0; j < cnt; j += U) {
            int cj[U], tj[U];
            float aj[U][V];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                cj[u] = bcast<LPR>(c, j + u);
                tj[u] = bcast<LPR>(tag, j + u);
#pragma unroll
                for (int v = 0; v < V; ++v) aj[u][v] = bcast<LPR>(av[v], j + u);
            }
            float b[U][REP][VEC];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float *brow = B + (long)cj[u] * K;
                const bool ok = j + u < cnt;
#pragma unroll
                for (int r = 0; r < REP; ++r) {
                    if (ok && kv[r]) {
                        load_vec<VEC>(brow + kc[r], b[u][r]);
                    } else {
#pragma unroll
                        for (int e = 0; e < VEC; ++e) b[u][r][e] = 0.0f;
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int i = 0; i < IPG; ++i)
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        const bool mine = tj[u] == i;
#pragma unroll
                        for (int r = 0; r < REP; ++r)
#pragma unroll
                            for (int e = 0; e < VEC; ++e) {
                                const float t = fmaf(aj[u][v], b[u][r][e], acc[i][v][r][e]);
                                acc[i][v][r][e] = mine ? t : acc[i][v][r][e];
                            }
                    }
        }
    }

#pragma unroll
    for (int i = 0; i < IPG; ++i) {
        const long item = (long)item0 + i;
        if (item < limit) {
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const long row = item * V + v;
                if (row < a.n_rows) {
                    float *crow = a.C + row * K;
#pragma unroll
                    for (int r = 0; r < REP; ++r)
                        if (kv[r]) {
                            finish<VEC>(a.epi, row, a.K, kc[r], acc[i][v][r]);
                            store_vec<VEC>(crow + kc[r], acc[i][v][r]);
                        }
                }
            }
        }
    }
}

// Column-window kernel (no balancing): one workgroup owns a block of consecutive work items
// (cut at build time where the rows move on to other columns) and one grid.y column slice.  It first copies rows [c0, c0 + win_cols) of
// that B slice into LDS (c0 chosen at build time as the densest window of the block's
// columns), then walks its items like spmm_kernel, taking each B segment from LDS when
// the column falls inside the window and from memory otherwise.  On clustered matrices
// most gathers then cost LDS bandwidth instead of L2 round trips: a compute unit can only
// keep a few hundred cache lines in flight, which caps L2-resident gathers near 23 TB/s
// on the whole chip, while its LDS delivers 128 bytes per clock.
// Everything that would put a memory round trip into the walk is requested one step ahead:
// the next item's vector range while the current item is processed, the next chunk of
// colIdx/val while the current chunk's rows are read.
// ROWS: windows of communities (SpmmArgs::rows): the window of a block is the rows of B with the numbers of its own
// items, found through a list, and the vectors inside come first in each item.
// LONG: for long items (SpmmArgs::outer), see the sums below.
// NEAR: gathers read B as a buffer (near_operand), with slots past the end of a run past its end.
template <int V, int LPR, int VEC, int REP, bool ROWS, bool LONG, bool NEAR>
__global__ void __launch_bounds__(1024) spmm_window_kernel(SpmmArgs a)
{
    extern __shared__ __align__(16) float lds[];
    constexpr int G = 64 / LPR;
    constexpr int TW = LPR * VEC * REP; // columns per slice
    constexpr int LW = TW + 4;          // floats per staged row, padded so rows start on different banks
    // Vectors per step.  The LDS window caps a compute unit at one or two workgroups, so a
    // wavefront may use many registers: memory gathers go 64 registers deep (the few
    // out-of-window vectors of an item then cost one round trip), LDS reads 32.
    constexpr int UG0 = 64 / (REP * VEC), UL0 = 32 / (REP * VEC);
    constexpr int UGc = UG0 < 1 ? 1 : (UG0 > 16 ? 16 : UG0), ULc = UL0 < 1 ? 1 : (UL0 > 16 ? 16 : UL0);
    constexpr int UG = UGc > LPR ? LPR : UGc; // a step never reaches past the group's chunk
    constexpr int UL = ULc > LPR ? LPR : ULc;
    // out-of-window vectors of an item whose gathers are issued before its LDS walk and used
    // after it (32 registers held across the walk)
    constexpr int UP = UL;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int waves = blockDim.x >> 6;
    // Each XCD takes one contiguous range of (block, slice) pairs, slices fastest: the slices of a block run side by
    // side on one XCD and its colIdx/val stream comes from that L2 for all but the first (one block after another per
    // slice read it from memory each time: sbm, 250,000 rows of 48, K = 256: 17.5 M lines from memory for 14.7 M now,
    // 395 us for 380).  Workgroups go round-robin over the XCDs in the order of their linear index.
    // The pairs past a.win_whole, fewer than the XCD's compute units hold at once, are cut into a.win_parts each
    // (window_tail says when).
    int bid = blockIdx.x, slice = blockIdx.y, part = 0, parts = 1;
    if (a.xcd_remap) {
        const unsigned id = blockIdx.y * gridDim.x + blockIdx.x, total = (unsigned)a.nblk * a.n_slices;
        const unsigned x = id & 7, q = total >> 3, r = total & 7;
        unsigned pair = id >> 3;
        if (pair >= (unsigned)a.win_whole) {
            const unsigned t = pair - a.win_whole;
            parts = a.win_parts;
            pair = a.win_whole + t / parts;
            part = t % parts;
            if (pair >= q + (x < r)) return; // an XCD of one pair less than the others
        }
        pair += x * q + (x < r ? x : r);
        bid = pair / a.n_slices;
        slice = pair - bid * a.n_slices;
    }
    const int lg = lane & (LPR - 1);
    const int kbase = slice * TW;
    const float *__restrict__ B = a.B;
    const long K = a.K;

    int item_begin = a.win_ptr[bid];
    int item_end = a.win_ptr[bid + 1];
    const int c0 = ROWS ? item_begin : a.win_start[bid];
    const int staged = ROWS ? item_end - item_begin : a.win_cols; // rows of B in LDS
    if (parts > 1) {
        const int n = item_end - item_begin;
        item_end = item_begin + (int)((long)n * (part + 1) / parts);
        item_begin += (int)((long)n * part / parts);
        if (item_begin == item_end) return;
    }
    const int stride = waves * G;
    int item = item_begin + wave * G + lane / LPR;
    // the first item's ranges are requested before the window is staged
    int head = 0, tail = 0, lo = 0, hi = 0, row = 0;
    if (item < item_end) {
        head = a.rowptr[item];
        tail = a.rowptr[item + 1];
        lo = a.win_lo[item];
        hi = a.win_hi[item];
        if constexpr (ROWS) row = a.rows[item];
    }

    if (c0 >= 0) { // uniform over the workgroup
        // A compute unit holds one workgroup (139 of 160 KB), so nothing runs beside the staging: all of a thread's
        // loads (8 of 16 bytes) are requested before the first is written.  One after the other they were nine
        // round trips per workgroup: sbm, K = 256: 380 us for 365 now.
        constexpr int VPR = TW / VEC;  // vector loads per staged row
        constexpr int PASS = 32 / VEC; // loads in flight per thread
        const int total = staged * VPR;
        for (int q0 = tid; q0 < total; q0 += PASS * blockDim.x) {
            float t[PASS][VEC];
            int cols[PASS];
#pragma unroll
            for (int i = 0; i < PASS; ++i) {
                const int q = q0 + i * blockDim.x;
                cols[i] = c0 + q / VPR;
                if constexpr (ROWS) cols[i] = a.rows[q < total ? cols[i] : c0];
            }
#pragma unroll
            for (int i = 0; i < PASS; ++i) {
                const int q = q0 + i * blockDim.x;
                const int col = cols[i], e = q % VPR * VEC;
                const bool ok = q < total && col < a.n_cols && kbase + e < a.K;
                load_vec<VEC>(ok ? B + (long)col * K + kbase + e : g_zero_row, t[i]);
            }
#pragma unroll
            for (int i = 0; i < PASS; ++i) {
                const int q = q0 + i * blockDim.x;
                if (q < total) store_lds<VEC>(lds + q / VPR * LW + q % VPR * VEC, t[i]);
            }
        }
        for (int e = tid; e < LW; e += blockDim.x) lds[a.win_cols * LW + e] = 0.0f; // the row of zeros
    }

    int kl[REP]; // column offset inside the slice
    unsigned lds_col[REP]; // its LDS address in a row at 0
    bool kv[REP];
#pragma unroll
    for (int r = 0; r < REP; ++r) {
        kl[r] = (r * LPR + lg) * VEC;
        lds_col[r] = lds_address(lds) + (unsigned)kl[r] * 4u;
        kv[r] = kbase + kl[r] < a.K;
    }
    [[maybe_unused]] __amdgpu_buffer_rsrc_t Bn;
    unsigned near_col = 0; // bytes
    if constexpr (NEAR) {
        static_assert(VEC == 4 && REP == 1);
        Bn = near_operand(a);
        near_col = (unsigned)min(kbase + kl[0], a.K - VEC) * 4u;
    }
    const unsigned row_bytes = (unsigned)K * 4u;

    // This lane's entry of the chunk that starts at member i0 of a walk: the walk's i-th
    // member is vector first + i (i < n1) or second + (i - n1); zeros past its n members.
    auto load_entry = [&](int first, int n1, int second, int n, int i0, int &c, float (&av)[V]) {
        const int i = i0 + lg;
        c = 0;
#pragma unroll
        for (int v = 0; v < V; ++v) av[v] = 0.0f;
        if (i < n) {
            const int idx = i < n1 ? first + i : second + (i - n1);
            c = stream_load(a.colidx + idx);
            if constexpr (V == 1) {
                av[0] = stream_load(a.val + idx);
            } else {
                typedef float f2 __attribute__((ext_vector_type(2)));
                const f2 t = stream_load(reinterpret_cast<const f2 *>(a.val) + idx);
                av[0] = t[0];
                av[1] = t[1];
            }
        }
    };
    // first chunk of both walks of the current item, requested while the previous item was
    // still being processed (here: before the window is complete)
    int cg0, cl0;
    float avg0[V], avl0[V];
    load_entry(head, lo - head, hi, (lo - head) + (tail - hi), 0, cg0, avg0);
    load_entry(lo, hi - lo, lo, hi - lo, 0, cl0, avl0);
    if (c0 >= 0) __syncthreads(); // the staged window is complete (uniform over the workgroup)

    while (item < item_end) {
        // ranges of the item this group takes next
        const int item_next = item + stride;
        int head_next = 0, tail_next = 0, lo_next = 0, hi_next = 0, row_next = 0;
        if (item_next < item_end) {
            head_next = a.rowptr[item_next];
            tail_next = a.rowptr[item_next + 1];
            lo_next = a.win_lo[item_next];
            hi_next = a.win_hi[item_next];
            if constexpr (ROWS) row_next = a.rows[item_next];
        }

        // Sums of 8 vectors (16 where a step has as many), which one running sum adds up: it loses more the longer the row.  LONG
        // therefore adds up sums of 32 apart with ROWS, whose rows were items of 32 vectors and a second pass without the windows,
        // and makes the sums 16 vectors elsewhere, which costs no registers.  Rms of the difference from 64 bits, relative to
        // the sum of magnitudes, equal values: ROWS at rows of 48, 100 and 300 1.25, 1.03 and 0.85e-8, with LONG 1.16, 0.88 and
        // 0.60e-8, items of 32 1.30, 0.99 and 0.67e-8; column windows at rows of 200 and 400 0.90 and 0.81e-8, with
        // LONG 0.83 and 0.70e-8, gathered from memory 0.82 and 0.68e-8.  (A third level for all of them: 250,000 rows of 48,
        // K = 256 366 -> 371 us; paired rows, whose instances spill, 532 -> 660.)
        constexpr bool OUTER = LONG && ROWS;
        constexpr int PART = LONG && !ROWS ? 16 : 8; // vectors of a sum, in whole steps and within a chunk
        float acc[V][REP][VEC], outer[OUTER ? V : 1][OUTER ? REP : 1][VEC];
        auto add_to = [](auto &sum, float (&x)[V][REP][VEC]) { // sum += x, x = 0
#pragma unroll
            for (int v = 0; v < V; ++v)
#pragma unroll
                for (int r = 0; r < REP; ++r)
#pragma unroll
                    for (int e = 0; e < VEC; ++e) {
                        sum[v][r][e] += x[v][r][e];
                        x[v][r][e] = 0.0f;
                    }
        };
#pragma unroll
        for (int v = 0; v < V; ++v)
#pragma unroll
            for (int r = 0; r < REP; ++r)
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    acc[v][r][e] = 0.0f;
                    if constexpr (OUTER) outer[v][r][e] = 0.0f;
                }

        // Walks the n vectors whose i-th member is vector first + i (i < n1) or
        // second + (i - n1): one contiguous run, or two runs taken as one.  The columns of an
        // item ascend, so the vectors inside the window are one run [lo, hi) and the others
        // the two runs around it; each kind is walked on its own, the memory gathers with
        // several loads in flight and no LDS access in between, the LDS reads with no memory
        // round trip in between.
        auto walk = [&](int first, int n1, int second, int n, int i_start, int c_first,
                        const float (&av_first)[V], auto from_lds) {
            constexpr bool LDS = decltype(from_lds)::value;
            constexpr int U = LDS ? UL : UG;
            int c_next = c_first;
            float av_next[V];
#pragma unroll
            for (int v = 0; v < V; ++v) av_next[v] = av_first[v];
            for (int base = i_start; base < n; base += LPR) {
                const int c = c_next;
                float av[V];
#pragma unroll
                for (int v = 0; v < V; ++v) av[v] = av_next[v];
                load_entry(first, n1, second, n, base + LPR, c_next, av_next);
                const int cnt = min(LPR, n - base);
                // where this lane's entry sits in the staged window (bytes from lds); a slot
                // past the end of the run reads the row of zeros staged after the window.  NEAR: in B
                const int loff = LDS ? (base + lg < n ? c - c0 : a.win_cols) * (LW * 4)
                                     : (NEAR && base + lg < n ? (int)((unsigned)c * row_bytes) : (int)kPast);
                float part[V][REP][VEC];
#pragma unroll
                for (int v = 0; v < V; ++v)
#pragma unroll
                    for (int r = 0; r < REP; ++r)
#pragma unroll
                        for (int e = 0; e < VEC; ++e) part[v][r][e] = 0.0f;
                auto step = [&](int j, auto const_lane) {
                    constexpr bool CL = decltype(const_lane)::value;
                    // LDS reads of a 16-lane group with constant source lanes: the broadcast of
                    // the value rides on the multiply-add, and the row's LDS offset was
                    // computed once by the lane that holds the entry
                    constexpr bool FUSED = LDS && CL && LPR == 16;
                    int cj[U];
                    float aj[U][V];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        if constexpr (LDS && REP == 1)
                            cj[u] = (int)((unsigned)bcast_any<LPR, CL>(loff, j + u) + lds_col[0]);
                        else
                            cj[u] = bcast_any<LPR, CL>(LDS || NEAR ? loff : c, j + u);
                        if constexpr (!FUSED) {
#pragma unroll
                            for (int v = 0; v < V; ++v) aj[u][v] = bcast_any<LPR, CL>(av[v], j + u);
                        }
                    }
                    float b[U][REP][VEC];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
#pragma unroll
                        for (int r = 0; r < REP; ++r) {
                            if constexpr (LDS) {
                                // one ds_read of VEC floats, never predicated: slots past the
                                // end point at the zero row, columns past K were staged as zeros
                                load_lds_at<VEC>((unsigned)cj[u] + (REP == 1 ? 0u : lds_col[r]), b[u][r]);
                            } else if constexpr (NEAR) {
                                load_near4(Bn, (unsigned)cj[u] + near_col, b[u][r]);
                            } else {
                                const bool ok = j + u < cnt;
                                const float *src = (ok && kv[r]) ? B + (long)cj[u] * K + kbase + kl[r]
                                                                 : g_zero_row + kl[r];
                                load_vec<VEC>(src, b[u][r]);
                            }
                        }
                    }
                    if constexpr (FUSED && V == 1) __builtin_amdgcn_sched_barrier(0); // a step's reads in flight together
#pragma unroll
                    for (int u = 0; u < U; ++u)
#pragma unroll
                        for (int r = 0; r < REP; ++r)
#pragma unroll
                            for (int v = 0; v < V; ++v)
#pragma unroll
                                for (int e = 0; e < VEC; ++e) {
                                    if constexpr (FUSED)
                                        fmac_bcast16_const(part[v][r][e], av[v], b[u][r][e], j + u);
                                    else
                                        part[v][r][e] = fmaf(aj[u][v], b[u][r][e], part[v][r][e]);
                                }
                    if (U >= PART || ((j + U) & (PART - 1)) == 0) add_to(acc, part);
                };
                if constexpr (LPR == 16) {
#pragma unroll
                    for (int j = 0; j < LPR; j += U)
                        if (j < cnt) step(j, std::true_type{});
                } else {
                    for (int j = 0; j < cnt; j += U) step(j, std::false_type{});
                }
                if constexpr (U < PART) add_to(acc, part);
                if constexpr (OUTER)
                    if (((base - i_start + LPR) & 31) == 0 && base + LPR < n) add_to(outer, acc);
            }
        };
        // Outside the window: memory gathers.  Those of the first UP such vectors are only
        // issued here; the LDS walk below runs while they are in flight, then they are added.
        const int n_out = (lo - head) + (tail - hi);
        float gb[UP][REP][VEC];
        [[maybe_unused]] const int goff = NEAR && lg < n_out ? (int)((unsigned)cg0 * row_bytes) : (int)kPast;
#pragma unroll
        for (int u = 0; u < UP; ++u) {
            if constexpr (NEAR) {
                load_near4(Bn, (unsigned)bcast_any<LPR, true>(goff, u) + near_col, gb[u][0]);
                continue;
            }
            const int cu = bcast_any<LPR, true>(cg0, u);
#pragma unroll
            for (int r = 0; r < REP; ++r) {
                const float *src = (u < n_out && kv[r]) ? B + (long)cu * K + kbase + kl[r] : g_zero_row + kl[r];
                load_vec<VEC>(src, gb[u][r]);
            }
        }
        // the next item's first chunks: its ranges have arrived by now, and the LDS walk
        // below covers the latency of these loads
        int cg0_next, cl0_next;
        float avg0_next[V], avl0_next[V];
        load_entry(head_next, lo_next - head_next, hi_next, (lo_next - head_next) + (tail_next - hi_next), 0,
                   cg0_next, avg0_next);
        load_entry(lo_next, hi_next - lo_next, lo_next, hi_next - lo_next, 0, cl0_next, avl0_next);
        // inside the window: LDS reads
        walk(lo, hi - lo, lo, hi - lo, 0, cl0, avl0, std::true_type{});
        // The gathers issued above, as a sum of their own like every step of the walk: rows of 48 then differ from 64 bits by
        // rms 1.69e-8 of their sum of magnitudes (plain kernel 1.84e-8).  Added to the item's sum one by one, and with
        // chunks of 16 in the walk, it was 2.10e-8; the additional instructions cost 1 % (sbm, K = 256: 359 us for 364).
        float part[V][REP][VEC];
#pragma unroll
        for (int v = 0; v < V; ++v)
#pragma unroll
            for (int r = 0; r < REP; ++r)
#pragma unroll
                for (int e = 0; e < VEC; ++e) part[v][r][e] = 0.0f;
#pragma unroll
        for (int u = 0; u < UP; ++u)
#pragma unroll
            for (int r = 0; r < REP; ++r)
#pragma unroll
                for (int v = 0; v < V; ++v)
#pragma unroll
                    for (int e = 0; e < VEC; ++e) {
                        if constexpr (LPR == 16)
                            fmac_bcast16_const(part[v][r][e], avg0[v], gb[u][r][e], u);
                        else
                            part[v][r][e] = fmaf(bcast<LPR>(avg0[v], u), gb[u][r][e], part[v][r][e]);
                    }
        add_to(acc, part);
        // the rare item with more out-of-window vectors than that: the rest, one step at a time
        if (n_out > UP) {
            int cg;
            float avg[V];
            load_entry(head, lo - head, hi, n_out, UP, cg, avg);
            walk(head, lo - head, hi, n_out, UP, cg, avg, std::false_type{});
        }
        if constexpr (OUTER) add_to(acc, outer);

#pragma unroll
        for (int v = 0; v < V; ++v) {
            const long at = ROWS ? (long)row : (long)item * V + v;
            if (at < a.n_rows) {
                float *crow = a.C + at * K + kbase;
#pragma unroll
                for (int r = 0; r < REP; ++r)
                    if (kv[r]) {
                        finish<VEC>(a.epi, at, a.K, kbase + kl[r], acc[v][r]);
                        store_vec<VEC>(crow + kl[r], acc[v][r]);
                    }
            }
        }
        item = item_next;
        row = row_next;
        head = head_next;
        tail = tail_next;
        lo = lo_next;
        hi = hi_next;
        cg0 = cg0_next;
        cl0 = cl0_next;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            avg0[v] = avg0_next[v];
            avl0[v] = avl0_next[v];
        }
    }
}

__global__ void __launch_bounds__(256) zero_panels_kernel(const int32_t *__restrict__ panels,
                                                          long n_panels, int V, float *C,
                                                          int n_rows, int K)
{
    // one thread per fp32 element of the listed rows
    const long total = n_panels * V * (long)K;
    for (long t = (long)blockIdx.x * blockDim.x + threadIdx.x; t < total;
         t += (long)gridDim.x * blockDim.x) {
        const long r = t / K;
        const int k = (int)(t - r * K);
        const long row = (long)panels[r / V] * V + (r % V);
        if (row < n_rows) C[row * K + k] = 0.0f;
    }
}

struct ReduceArgs {
    const int32_t *split_panels, *split_slot, *long_panels;
    int64_t n_split;
    int32_t long_blocks, long_chunks; // workgroups of the long panels; per row of one
    int32_t lanes_log2, chunks;       // of the others: lanes to a row (in vectors), workgroups that share its width
    int32_t V, n_rows, K;
    const float *ws;
    float *C;
    Epilogue epi;
};

// Second pass of the balanced write-back.  Long panels (a hub row of a power-law graph is cut into thousands of items)
// take the first workgroups: one per (row, 16 vectors of C), 16 threads per vector.  Thread j of a vector adds slots j, j+16,
// j+32, ... in ascending order, then the 16 partial sums are added in ascending j.  Of the other split panels a thread takes
// VEC consecutive elements of a row and adds its slots in item order.  Both orders depend on the slot numbers alone, so the
// balanced result is the same bits on every run and for every schedule.
// One launch for both, so that the long panels' serial sums run beside the others' traffic: R-MAT 2^22, K = 16 34 + 25 us as
// two, 39 as one; 2^20, K = 64 18 + 9, 18.  At K = 512 (8.8 GB, 5.1 TB/s) it is 1.72 ms either way.
template <int VEC> __global__ void __launch_bounds__(256) reduce_kernel(ReduceArgs a)
{
    __shared__ float part[kLongReduceLanes][16][VEC];
    const int vectors = (a.K + VEC - 1) / VEC; // per row, the last one moved back to end with it
    const long stride = (long)a.V * a.K;
    float sum[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) sum[e] = 0.0f;

    if ((int)blockIdx.x < a.long_blocks) { // uniform
        const int c = threadIdx.x % 16, j = threadIdx.x / 16;
        const int r = blockIdx.x / a.long_chunks, at = (blockIdx.x - r * a.long_chunks) * 16 + c;
        const int q = a.long_panels[r / a.V], v = r % a.V;
        const long row = (long)a.split_panels[q] * a.V + v;
        if (row >= a.n_rows) return; // the whole workgroup leaves: no barrier is skipped by a part of it
        const bool live = at < vectors;
        const int k = min(at * VEC, a.K - VEC);
        const long s0 = a.split_slot[q], s1 = a.split_slot[q + 1];
        const long step = kLongReduceLanes * stride;
        if (live) {
            long jj = s0 + j;
            const float *w = a.ws + (jj * a.V + v) * (long)a.K + k;
            for (; jj + 3 * kLongReduceLanes < s1; jj += 4 * kLongReduceLanes, w += 4 * step) {
                float t4[4][VEC];
#pragma unroll
                for (int u = 0; u < 4; ++u) load_vec<VEC>(w + u * step, t4[u]);
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int e = 0; e < VEC; ++e) sum[e] += t4[u][e];
            }
            for (; jj < s1; jj += kLongReduceLanes, w += step) {
                float t1[VEC];
                load_vec<VEC>(w, t1);
#pragma unroll
                for (int e = 0; e < VEC; ++e) sum[e] += t1[e];
            }
        }
#pragma unroll
        for (int e = 0; e < VEC; ++e) part[j][c][e] = sum[e];
        __syncthreads();
        if (j == 0 && live) {
            for (int jj = 1; jj < kLongReduceLanes; ++jj)
#pragma unroll
                for (int e = 0; e < VEC; ++e) sum[e] += part[jj][c][e];
            finish<VEC>(a.epi, row, a.K, k, sum);
            store_vec<VEC>(a.C + row * a.K + k, sum);
        }
        return;
    }

    const int b = blockIdx.x - a.long_blocks, group = b / a.chunks; // uniform
    const int at = ((b - group * a.chunks) << a.lanes_log2) + (threadIdx.x & ((1 << a.lanes_log2) - 1));
    const long r = ((long)group << (8 - a.lanes_log2)) + (threadIdx.x >> a.lanes_log2);
    const long q = a.V == 1 ? r : r >> 1;
    const int v = a.V == 1 ? 0 : (int)(r & 1);
    if (q >= a.n_split || at >= vectors) return;
    const int k = min(at * VEC, a.K - VEC);
    const long row = (long)a.split_panels[q] * a.V + v;
    const long s0 = a.split_slot[q], s1 = a.split_slot[q + 1];
    if (row >= a.n_rows || (a.long_blocks && s1 - s0 > kLongPanelSlots)) return;
    const float *w = a.ws + (s0 * a.V + v) * (long)a.K + k;
    long j = s0;
    for (; j + 4 <= s1; j += 4, w += 4 * stride) { // four loads in flight, adds in item order
        float t4[4][VEC];
#pragma unroll
        for (int u = 0; u < 4; ++u) load_vec<VEC>(w + u * stride, t4[u]);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int e = 0; e < VEC; ++e) sum[e] += t4[u][e];
    }
    for (; j < s1; ++j, w += stride) {
        float t1[VEC];
        load_vec<VEC>(w, t1);
#pragma unroll
        for (int e = 0; e < VEC; ++e) sum[e] += t1[e];
    }
    finish<VEC>(a.epi, row, a.K, k, sum);
    store_vec<VEC>(a.C + row * a.K + k, sum);
}

using KernelFn = void (*)(SpmmArgs);

template <int V, bool S, int LPR, int VEC, int REP, bool EPI, int FORM> KernelFn instance(bool near)
{
    if constexpr (FORM == kLongItems && !(S && (V == 1 || LPR >= 32))) // (spmm_enqueue says which)
        return nullptr;
    else if constexpr (FORM == kEarlyTail && (S || V * REP * VEC > 8))
        return nullptr;
    else if constexpr (FORM == kBands && (S || V != 1 || LPR < 8 || (VEC == 1 && LPR > 32) || (VEC == 2 && LPR != 32) || (REP != 1 && !(REP == 2 && VEC == 4 && LPR == 64))))
        return nullptr;
    else if constexpr (FORM == kNarrow && (S || VEC != 1 || !((LPR == 16 && REP == 1) || (V == 1 && LPR >= 16 && LPR <= 32 && LPR * REP >= 32 && REP <= 2))))
        return nullptr;
    else {
        // A whole wavefront to a row has its addresses in scalar registers; more repeats than these are taken only where asked for.
        if constexpr (LPR < 64 && REP <= 2)
            if (near) return &spmm_kernel<V, S, LPR, VEC, REP, EPI, FORM, true>;
        return &spmm_kernel<V, S, LPR, VEC, REP, EPI, FORM, false>;
    }
}
template <int V, bool S, int LPR, int VEC, bool EPI, int FORM> KernelFn pick_rep(int rep, bool near)
{
    if constexpr (!EPI) {
        switch (rep) {
        case 1: return instance<V, S, LPR, VEC, 1, EPI, FORM>(near);
        case 2: return instance<V, S, LPR, VEC, 2, EPI, FORM>(near);
        case 4: return instance<V, S, LPR, VEC, 4, EPI, FORM>(near);
        }
    } else { // the shapes resolve_launch arrives at when everything is left to it
        if (rep == 1) return instance<V, S, LPR, VEC, 1, EPI, FORM>(near);
        if constexpr (FORM == kNarrow)
            if (rep == 2) return instance<V, S, LPR, VEC, 2, EPI, FORM>(near);
        if constexpr (LPR == 64) {
            if (rep == 2) return instance<V, S, LPR, VEC, 2, EPI, FORM>(near);
            if constexpr (!S)
                if (rep == 4) return instance<V, S, LPR, VEC, 4, EPI, FORM>(near);
        }
    }
    return nullptr;
}
template <int V, bool S, int LPR, bool EPI, int FORM> KernelFn pick_vec(int vec, int rep, bool near)
{
    switch (vec) {
    case 1: return pick_rep<V, S, LPR, 1, EPI, FORM>(rep, near);
    case 2: return pick_rep<V, S, LPR, 2, EPI, FORM>(rep, near);
    case 4: return pick_rep<V, S, LPR, 4, EPI, FORM>(rep, near);
    }
    return nullptr;
}
template <int V, bool S, bool EPI, int FORM> KernelFn pick_lpr(int lpr, int vec, int rep, bool near)
{
    switch (lpr) {
    case 4: return pick_vec<V, S, 4, EPI, FORM>(vec, rep, near);
    case 8: return pick_vec<V, S, 8, EPI, FORM>(vec, rep, near);
    case 16: return pick_vec<V, S, 16, EPI, FORM>(vec, rep, near);
    case 32: return pick_vec<V, S, 32, EPI, FORM>(vec, rep, near);
    case 64: return pick_vec<V, S, 64, EPI, FORM>(vec, rep, near);
    }
    return nullptr;
}
template <bool EPI, int FORM = kAsIs> KernelFn pick(int V, int S, int lpr, int vec, int rep, bool near = false)
{
    if (V == 1) return S ? pick_lpr<1, true, EPI, FORM>(lpr, vec, rep, near) : pick_lpr<1, false, EPI, FORM>(lpr, vec, rep, near);
    if (V == 2) return S ? pick_lpr<2, true, EPI, FORM>(lpr, vec, rep, near) : pick_lpr<2, false, EPI, FORM>(lpr, vec, rep, near);
    return nullptr;
}

// batched instances exist where the accumulators stay within 32 registers
template <int V, int LPR, int VEC, int REP> KernelFn pickb_ipg(int ipg)
{
    if constexpr (2 < LPR && V * VEC * REP * 2 <= 32)
        if (ipg == 2) return &spmm_batched_kernel<V, LPR, VEC, REP, 2>;
    if constexpr (4 < LPR && V * VEC * REP * 4 <= 32)
        if (ipg == 4) return &spmm_batched_kernel<V, LPR, VEC, REP, 4>;
    return nullptr;
}
template <int V, int LPR, int VEC> KernelFn pickb_rep(int rep, int ipg)
{
    switch (rep) {
    case 1: return pickb_ipg<V, LPR, VEC, 1>(ipg);
    case 2: return pickb_ipg<V, LPR, VEC, 2>(ipg);
    case 4: return pickb_ipg<V, LPR, VEC, 4>(ipg);
    }
    return nullptr;
}
template <int V, int LPR> KernelFn pickb_vec(int vec, int rep, int ipg)
{
    switch (vec) {
    case 1: return pickb_rep<V, LPR, 1>(rep, ipg);
    case 2: return pickb_rep<V, LPR, 2>(rep, ipg);
    case 4: return pickb_rep<V, LPR, 4>(rep, ipg);
    }
    return nullptr;
}
template <int V> KernelFn pickb_lpr(int lpr, int vec, int rep, int ipg)
{
    switch (lpr) {
    case 4: return pickb_vec<V, 4>(vec, rep, ipg);
    case 8: return pickb_vec<V, 8>(vec, rep, ipg);
    case 16: return pickb_vec<V, 16>(vec, rep, ipg);
    case 32: return pickb_vec<V, 32>(vec, rep, ipg);
    case 64: return pickb_vec<V, 64>(vec, rep, ipg);
    }
    return nullptr;
}
KernelFn pick_any(int V, int S, int lpr, int vec, int rep, int ipg, bool near = false)
{
    if (ipg <= 1) return pick<false>(V, S, lpr, vec, rep, near);
    if (S) return nullptr;
    if (V == 1) return pickb_lpr<1>(lpr, vec, rep, ipg);
    if (V == 2) return pickb_lpr<2>(lpr, vec, rep, ipg);
    return nullptr;
}

template <int V, int LPR, int VEC> KernelFn pickw_rep(int rep, bool long_items, bool near)
{
    if constexpr (LPR == 16 && VEC == 4) // the shape that is taken unasked
        if (rep == 1 && near)
            return long_items ? &spmm_window_kernel<V, LPR, VEC, 1, false, true, true>
                              : &spmm_window_kernel<V, LPR, VEC, 1, false, false, true>;
    if constexpr (LPR >= 16 && VEC == 4) // steps of 8 in chunks of more, of the shapes that are taken unasked
        if (rep == 1 && long_items) return &spmm_window_kernel<V, LPR, VEC, 1, false, true, false>;
    switch (rep) {
    case 1: return &spmm_window_kernel<V, LPR, VEC, 1, false, false, false>;
    case 2: return &spmm_window_kernel<V, LPR, VEC, 2, false, false, false>;
    case 4: return &spmm_window_kernel<V, LPR, VEC, 4, false, false, false>;
    }
    return nullptr;
}
template <int V, int LPR> KernelFn pickw_vec(int vec, int rep, bool long_items, bool near)
{
    switch (vec) {
    case 1: return pickw_rep<V, LPR, 1>(rep, long_items, near);
    case 2: return pickw_rep<V, LPR, 2>(rep, long_items, near);
    case 4: return pickw_rep<V, LPR, 4>(rep, long_items, near);
    }
    return nullptr;
}
template <int V> KernelFn pickw_lpr(int lpr, int vec, int rep, bool long_items, bool near)
{
    switch (lpr) {
    case 4: return pickw_vec<V, 4>(vec, rep, long_items, near);
    case 8: return pickw_vec<V, 8>(vec, rep, long_items, near);
    case 16: return pickw_vec<V, 16>(vec, rep, long_items, near);
    case 32: return pickw_vec<V, 32>(vec, rep, long_items, near);
    case 64: return pickw_vec<V, 64>(vec, rep, long_items, near);
    }
    return nullptr;
}
KernelFn pick_window(int V, int lpr, int vec, int rep, bool long_items, bool near)
{
    if (V == 1) return pickw_lpr<1>(lpr, vec, rep, long_items, near);
    if (V == 2) return pickw_lpr<2>(lpr, vec, rep, long_items, near);
    return nullptr;
}
KernelFn pick_row_window(bool long_items, bool near)
{
    if (near)
        return long_items ? &spmm_window_kernel<1, kRowsLanes, kRowsVec, 1, true, true, true>
                          : &spmm_window_kernel<1, kRowsLanes, kRowsVec, 1, true, false, true>;
    return long_items ? &spmm_window_kernel<1, kRowsLanes, kRowsVec, 1, true, true, false>
                      : &spmm_window_kernel<1, kRowsLanes, kRowsVec, 1, true, false, false>;
}

} // namespace

// More than 64 KiB of dynamic LDS has to be allowed per kernel function: raised to
// the 160 KiB of the CU once per function and device, not on every launch (the
// call is host work and is not capturable in a HIP graph).
// all: the forms of an instance, raised together, so that a handle whose products run another one finds it done.
using WindowForms = std::array<KernelFn, 4>;
static hipError_t allow_window_lds(const WindowForms &all)
{
    static std::mutex mu;
    static std::set<std::pair<int, const void *>> raised;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(mu);
    if (!raised.count(std::make_pair(dev, reinterpret_cast<const void *>(all[0])))) {
        for (KernelFn f : all) {
            e = hipFuncSetAttribute(reinterpret_cast<const void *>(f),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
            if (e != hipSuccess) return e;
        }
        try {
            raised.insert(std::make_pair(dev, reinterpret_cast<const void *>(all[0])));
        } catch (...) { // no memory to note it: raised again next time
        }
    }
    return hipSuccess;
}

// form 2 * near + long_items
template <class Pick> static WindowForms window_forms(Pick pick)
{
    return {pick(false, false), pick(true, false), pick(false, true), pick(true, true)};
}

hipError_t prepare_row_windows() { return allow_window_lds(window_forms(pick_row_window)); }

bool window_kernel_exists(int V, int lpr, int vec, int rep)
{
    return pick_window(V, lpr, vec, rep, false, false) != nullptr;
}

bool kernel_exists(int V, int S, int lpr, int vec, int rep, int ipg)
{
    return pick_any(V, S, lpr, vec, rep, ipg) != nullptr;
}

bool band_kernel_exists(int lpr, int vec, int rep, bool epilogue)
{
    return (epilogue ? pick<true, kBands>(1, 0, lpr, vec, rep) : pick<false, kBands>(1, 0, lpr, vec, rep)) != nullptr;
}

bool epilogue_kernel_exists(int V, int S, int lpr, int vec, int rep)
{
    return pick<true>(V, S, lpr, vec, rep) != nullptr || pick<true, kNarrow>(V, S, lpr, vec, rep) != nullptr;
}

static bool near_enough(const SpmmArgs &a)
{
    return !a.far && (uint64_t)a.n_cols * (uint64_t)a.K * 4u <= kNearBytes && a.K < (1 << 20);
}

hipError_t launch_spmm(int V, int S, const LaunchShape &ls, const SpmmArgs &args, hipStream_t stream)
{
    if (ls.grid_x <= 0 || ls.grid_y <= 0) return hipSuccess; // nothing to do
    if (ls.window) {
        const WindowForms all = window_forms([&](bool long_items, bool near) -> KernelFn {
            if (args.rows) return pick_row_window(long_items, near);
            return S ? nullptr : pick_window(V, ls.lpr, ls.vec, ls.rep, long_items, near);
        });
        KernelFn fn = all[2 * near_enough(args) + (args.outer != 0)];
        if (!fn) return hipErrorInvalidValue;
        const hipError_t e = allow_window_lds(all);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(fn, dim3(ls.k_grid_x, ls.k_grid_y), dim3(64 * ls.waves), ls.lds_bytes, stream, args);
        return hipGetLastError();
    }
    const bool epi = args.epi.on && ls.ipg <= 1;
    // Unsplit items of less than a chunk.  4 and 8 lanes: 32-bit offsets save little beside the slots and lanes that have nothing to
    // load and now read all the same (time with them over without, rows of 3 to 14, the shapes that are taken unasked: 300,000 rows
    // 0.97-1.05, 1,500,000 0.96-1.10 but for one 0.82; items of 16 to 24 0.96-1.05).  Paired items of one dword a lane, plain: B of
    // 72 and 96 MB 1.00-1.11 with 10 and 14 vectors, 0.96-1.05 with 17 and 20; of 14 and 19 MB, which L2 holds, 0.93-0.96 at any
    // length.  Single ones gain (8 to 18 vectors 0.84-1.00, uniform columns 0.98-1.00), and so do tails (pairs 0.87-1.03, mostly
    // below 0.95) and wide loads of 16 lanes and more (0.93-1.02).
    const bool past_l2 = (double)args.n_cols * args.K * 4.0 > 32.0 * 1048576.0;
    const bool short_items = !S && args.mean_item < 16 && (ls.k_lpr < 16 || (V == 2 && ls.k_vec == 1 && !epi && past_l2));
    const bool near = near_enough(args) && !short_items;
    // Plain products in these shapes at any width: pcsr_select gives them to handles that had sums of 4 to 8 vectors in wide loads
    // (20,000 rows of 22, a handle for K = 8 at K = 64: rms 4.7e-8 of the sum, 5.6 in sums of 16, 4.7 now), and the additions show
    // nowhere (K = 9 to 16, rows of 9 to 80: 0.99-1.02 of the time).  But pairs of over 8 columns have sums of 16 as before, where they are
    // of 22 and more on average (100,000 rows of 80 in cliques 5.4, of 8 6.3) or of 9 to 16 columns, and so have tails of 9 to 16, which come
    // in auto shapes and ask for their rows early.
    const bool at_width = V == 1 ? !epi || args.K <= 8 || args.K > 16 : args.K <= 8 || (args.K > 16 && args.mean_item < 22);
    const bool narrow = !S && ls.k_vec == 1 && ls.ipg <= 1 && at_width &&
                        ((ls.k_lpr == 16 && ls.k_rep == 1) ||
                         (V == 1 && ls.k_lpr >= 16 && ls.k_lpr <= 32 && ls.k_rep <= 2 && ls.k_lpr * ls.k_rep >= 32));
    KernelFn fn;
    size_t lds = 0;
    if (args.band) {
        fn = epi ? pick<true, kBands>(V, S, ls.k_lpr, ls.k_vec, ls.k_rep, near_enough(args))
                 : pick<false, kBands>(V, S, ls.k_lpr, ls.k_vec, ls.k_rep, near_enough(args));
    } else if (narrow) {
        fn = epi ? pick<true, kNarrow>(V, S, ls.k_lpr, 1, ls.k_rep, near) : pick<false, kNarrow>(V, S, ls.k_lpr, 1, ls.k_rep, near);
    } else if (args.outer) {
        fn = epi ? pick<true, kLongItems>(V, S, ls.k_lpr, ls.k_vec, ls.k_rep, near)
                 : pick<false, kLongItems>(V, S, ls.k_lpr, ls.k_vec, ls.k_rep, near);
        lds = sizeof(float) * 64 * ls.waves * V * ls.k_rep * ls.k_vec; // 64 KB at most
    } else {
        fn = epi && (args.epi.self || args.epi.mask) ? pick<true, kEarlyTail>(V, S, ls.k_lpr, ls.k_vec, ls.k_rep, near) : nullptr;
        if (!fn) fn = epi ? pick<true>(V, S, ls.k_lpr, ls.k_vec, ls.k_rep, near) : pick_any(V, S, ls.k_lpr, ls.k_vec, ls.k_rep, ls.ipg, near);
    }
    if (!fn) return hipErrorInvalidValue;
    hipLaunchKernelGGL(fn, dim3(ls.k_grid_x, ls.k_grid_y), dim3(64 * ls.waves), lds, stream, args);
    return hipGetLastError();
}

hipError_t launch_zero_panels(const int32_t *panels, int64_t n_panels, int V, float *C,
                              int32_t n_rows, int32_t K, hipStream_t stream)
{
    if (n_panels <= 0) return hipSuccess;
    const long total = n_panels * V * (long)K;
    long blocks = (total + 255) / 256;
    if (blocks > 256 * 64) blocks = 256 * 64;
    hipLaunchKernelGGL(zero_panels_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, panels,
                       (long)n_panels, V, C, n_rows, K);
    return hipGetLastError();
}

hipError_t static_scratch(void **ptr)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void *addr[kMaxDevices] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        // every GPU holds its own copy of the array at its own address
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return hipSuccess;
}

hipError_t launch_reduce_split(const int32_t *split_panels, const int32_t *split_slot, int64_t n_split,
                               const int32_t *long_panels, int64_t n_long, int V, const float *ws, float *C,
                               int32_t n_rows, int32_t K, const Epilogue &epi, hipStream_t stream)
{
    if (n_split <= 0) return hipSuccess;
    const int vec = K >= 4 ? 4 : 1, vectors = (K + vec - 1) / vec;
    ReduceArgs a;
    a.split_panels = split_panels;
    a.split_slot = split_slot;
    a.long_panels = long_panels;
    a.n_split = n_split;
    a.long_chunks = (vectors + 15) / 16;
    a.lanes_log2 = 0;
    while (a.lanes_log2 < 6 && (1 << a.lanes_log2) < vectors) ++a.lanes_log2;
    a.chunks = (vectors + (1 << a.lanes_log2) - 1) >> a.lanes_log2;
    a.V = V;
    a.n_rows = n_rows;
    a.K = K;
    a.ws = ws;
    a.C = C;
    a.epi = epi;
    const int rows = 256 >> a.lanes_log2; // of a workgroup
    const int64_t long_blocks = n_long > 0 ? n_long * V * a.long_chunks : 0;
    const int64_t blocks = long_blocks + (n_split * V + rows - 1) / rows * a.chunks;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    a.long_blocks = (int32_t)long_blocks;
    if (vec == 4)
        hipLaunchKernelGGL(reduce_kernel<4>, dim3((unsigned)blocks), dim3(256), 0, stream, a);
    else
        hipLaunchKernelGGL(reduce_kernel<1>, dim3((unsigned)blocks), dim3(256), 0, stream, a);
    return hipGetLastError();
}

} // namespace pcsr
