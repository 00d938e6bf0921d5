// Launchers of the HIP SpMM kernel family (internal to the library).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace pcsr {

// What the write-back does to an element before it is stored (a GNN layer's elementwise tail,
// see pcsr_gnn.h); off for a plain SpMM.
struct Epilogue {
    int32_t on = 0;
    int32_t relu = 0;
    const float *bias = nullptr;     // K
    const float *self = nullptr;     // n_rows x K
    const float *self_eps = nullptr; // one value
    const float *mask = nullptr;     // n_rows x K
};

// the first band, the last one, and: its vectors are added up in sums of 64, not 32
constexpr int32_t kBandOn = 1, kBandFirst = 2, kBandLast = 4, kBandSums64 = 8;

struct SpmmArgs {
    const int32_t *rowptr; // M+1, device
    const int32_t *colidx; // nnz_v, device
    const float *val;      // nnz_v * V, device
    const int32_t *trow;   // M, device: S: the items' panels; in bands: where the rows' vectors of this band end
    const float *B;
    float *C;
    int32_t M;      // work items
    int32_t n_rows; // rows of C
    int32_t K;
    int32_t nblk;      // grid.x
    int32_t xcd_remap; // 1: one contiguous, work-balanced item range per XCD
    int32_t xb[9];     // item range [xb[x], xb[x+1]) of XCD x (xcd_remap only)
    // Balanced handles, deterministic write-back: an item of a panel that was split over
    // several items stores its partial rows in `ws` (slot-major: (slot*V + v)*K + k) and
    // reduce_kernel adds them in item order.  ws == nullptr selects the atomic write-back.
    float *ws;
    const int32_t *item_slot; // M (S only): workspace slot of an item of a split panel, -1 for
                              // an item that is the only one of its panel
    // Column-ordered schedule (S only, may be null): for launch position i the record
    // {first vector, vector count, panel (TRow), workspace slot or -1} of the work item
    // that runs there.  xb then bounds positions, not items.
    const int4 *sched;
    int32_t outer; // long items: sums of 32 vectors are added up apart (plain walk with S), or as the window kernel says
    int32_t mean_item; // vectors of a work item on average
    int32_t far; // 1: no 32-bit offsets into B
    // One band of columns (0: all of them): row i's vectors in it are [rowptr[i], trow[i]), and their sum is added to what the bands
    // before left in C.
    int32_t band; // kBand* bits
    // column-window blocking (window kernel only)
    const int32_t *win_ptr;   // item range [win_ptr[b], win_ptr[b+1]) of block b (= workgroup b)
    const int32_t *win_start; // per item block: first column of the staged window or -1
    const int32_t *win_lo;    // per item: its vectors [win_lo, win_hi) lie inside the block's
    const int32_t *win_hi;    // window (an empty range when the block has none)
    int32_t win_cols;         // rows of B staged in LDS
    int32_t n_cols;
    int32_t n_slices;  // column slices of a block (window kernel only)
    int32_t win_whole; // (block, slice) pairs an XCD takes whole; the rest run as win_parts workgroups each
    int32_t win_parts;
    // Windows of communities (cluster_windows; null: column windows): item i is row rows[i] of C, the window of a block
    // its own rows of B, and colIdx holds an item's vectors inside the window first, as items, the others as columns.
    const int32_t *rows;
    Epilogue epi;
};

// Resolved launch shape.
struct LaunchShape {
    int32_t lpr, vec, rep, waves;
    int32_t ipg; // work items per lane group (1 = one item per group)
    int32_t window; // 1: column-window kernel (one workgroup per item block, B window in LDS)
    int32_t lds_bytes;
    int32_t grid_x, grid_y;
    // What is launched in place of that shape where it reads rows badly: wide loads at 4-byte
    // addresses (see resolve_launch).  The same shape everywhere else.
    int32_t k_lpr, k_vec, k_rep, k_grid_x, k_grid_y;
    int32_t win_whole, win_parts; // as SpmmArgs (window only)
};

bool kernel_exists(int V, int S, int lpr, int vec, int rep, int ipg);
// with an epilogue (plain walk; the batched and window kernels take one at any shape)
bool epilogue_kernel_exists(int V, int S, int lpr, int vec, int rep);
// for a band of columns
bool band_kernel_exists(int lpr, int vec, int rep, bool epilogue);
bool window_kernel_exists(int V, int lpr, int vec, int rep);
// The one shape of the kernel for windows of communities; what its first launch on a device needs done outside a capture.
constexpr int kRowsLanes = 16, kRowsVec = 4, kRowsMost = 512;
hipError_t prepare_row_windows();

// Enqueues the SpMM kernel <V,S,lpr,vec,rep> with `waves` wavefronts per workgroup.
hipError_t launch_spmm(int V, int S, const LaunchShape &ls, const SpmmArgs &args,
                       hipStream_t stream);

// Clears the C rows of the listed panels (rows panel*V .. panel*V+V-1, K floats each).
hipError_t launch_zero_panels(const int32_t *panels, int64_t n_panels, int V, float *C,
                              int32_t n_rows, int32_t K, hipStream_t stream);

// Second pass of the deterministic balanced write-back: for every split panel q and
// v < V, C[panel*V + v][:] = sum over its items of the partial rows the SpMM kernel left
// in ws.  Panels with at most kLongPanelSlots items are added in item order by one thread
// per vector of C; the others (indices into the split tables listed in long_panels,
// n_long of them) by kLongReduceLanes threads per vector, thread j taking items j,
// j + kLongReduceLanes, ... in order, the partial sums then added in ascending j.
constexpr int kLongPanelSlots = 64;
constexpr int kLongReduceLanes = 16;
hipError_t launch_reduce_split(const int32_t *split_panels, const int32_t *split_slot, int64_t n_split,
                               const int32_t *long_panels, int64_t n_long, int V, const float *ws, float *C,
                               int32_t n_rows, int32_t K, const Epilogue &epi, hipStream_t stream);

// Fixed workspace for callers that cannot allocate: one block of kStaticScratchBytes
// bytes per GPU, part of the library's device image and held until the process ends.
// static_scratch returns its address on the current device (looked up once per device).
constexpr size_t kStaticScratchBytes = size_t(64) << 20;
hipError_t static_scratch(void **ptr);

} // namespace pcsr
