// C ABI of the PCSR SpMM library (see include/pcsr.h for the contract of each call).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <thread>
#include <vector>

#include "../../include/pcsr.h"
#include "pcsr_build_gpu.h"
#include "pcsr_gnn.h"
#include "pcsr_host.h"
#include "pcsr_kernels.h"
#include "pcsr_pool.h"
#include "pcsr_relabel_gpu.h"

namespace {

// Columns from which a handle with windows of communities uses them (250,000 rows of 48: K = 64 146 -> 110 us, 128 262 -> 183).
constexpr int kRowsLeast = 64;
constexpr uint32_t kMagic = 0x50435352u; // "PCSR"

// Bits of pcsr_params_t.flags in which pcsr_select passes a shape to launch in place of the one in
// lanes_per_row, vec and rep (see resolve_launch): 4 (kWidePair: 2) floats per load, one (kWideTwice:
// two) loads per lane, lanes per row 4 << (code - 1) for codes 1 to 5; above them the shape that it
// stands in for (stands_for), without which the bits say nothing; kWideBeyond: only for rows wider than
// that one's tile; kAutoNarrow: up to kAutoNarrowMost columns the auto shapes instead, of a handle whose own
// has that stands_for.  Cleared by pcsr_set_kernel_params.
constexpr int kWideShift = 16;
constexpr int32_t kWideShape = 7 << kWideShift;
constexpr int32_t kWidePair = 8 << kWideShift;
constexpr int32_t kWideTwice = 16 << kWideShift;
constexpr int kWideForShift = 21;
constexpr int32_t kWideFor = 127 << kWideForShift;
constexpr int32_t kWideBeyond = 1 << 29;
constexpr int32_t kAutoNarrow = 1 << 30;
constexpr int32_t kAutoNarrowMost = 32;
constexpr int32_t kWideBits = kWideShape | kWidePair | kWideTwice | kWideFor | kWideBeyond | kAutoNarrow;

// Set by pcsr_operator_build, whose handles run auto shapes, where it picked the parameters: the columns are scattered.
constexpr int32_t kScattered = 1 << 15;

// No more nonzeros near the diagonal than four times what uniform columns would put there.
bool scattered_columns(const double *f) { return f[16] < 4.0 * 1025.0 / (f[0] > 1.0 ? f[0] : 1.0); }

int32_t stands_for(int lanes, int vec, int rep)
{
    auto bits = [](int x) { return x > 0 ? 31 - __builtin_clz((unsigned)x) : 0; };
    return (bits(lanes) | bits(vec) << 3 | bits(rep) << 5) << kWideForShift;
}

// The flags of a handle: a caller who changed the shape that pcsr_select returned gets that shape,
// and bits that pcsr_select never sets do nothing.
int32_t checked_flags(const pcsr_params_t &p)
{
    const int code = (p.flags & kWideShape) >> kWideShift;
    const bool own = p.lanes_per_row && p.vec && p.rep;
    if (own && (code >= 1 || (p.flags & kAutoNarrow)) && code <= 5 && (p.flags & kWideFor) == stands_for(p.lanes_per_row, p.vec, p.rep)) return p.flags;
    return p.flags & ~kWideBits;
}

// Lanes of one dword for a row of up to 8 columns: more than it has, as a group of 16 runs to the end of its own row, not of four,
// and broadcasts by DPP where 4 lanes shuffle.  Time of 8 and 16 lanes over 4 of the widest loads: rows of 16 to 134 that are not
// split, K = 2, 4 and 8 0.65-0.97 and 0.48-0.94 (300,000 rows of 134, K = 4 553 us, 387 and 333; 250,000 of 48 in communities, K = 8
// 84, 57 and 52), pairs 0.72-1.00 and 0.62-0.92; items of balanced handles 0.72-0.85 and 0.72-0.90, which take 8 (R-MAT 2^22, K = 8: 1731
// us, 1280 and 1308).  Rows of 6 to 14 with local columns 0.96-1.7.
int narrow_lanes(int S) { return S ? 8 : 16; }

// The narrowest tile of 16-byte loads that covers a row of K columns.
void wide_shape(int32_t K, int cap, int *lanes, int *rep)
{
    *lanes = 4;
    while (*lanes * 4 < K && *lanes < cap) *lanes <<= 1;
    *rep = *lanes == 64 && K > 256 ? 2 : 1;
}

thread_local int g_last_hip = 0;

inline bool hip_ok(hipError_t e)
{
    if (e == hipSuccess) return true;
    g_last_hip = (int)e;
    (void)hipGetLastError(); // clear the sticky error so later calls are not blamed
    return false;
}

inline bool is_pow2(int x) { return x > 0 && (x & (x - 1)) == 0; }

int check_kernel_params(int lpr, int vec, int rep, int waves, int ipg)
{
    if (ipg != 0 && ipg != 1 && ipg != 2 && ipg != 4) return PCSR_E_UNSUPPORTED;
    if (lpr != 0 && !(is_pow2(lpr) && lpr >= 4 && lpr <= 64)) return PCSR_E_UNSUPPORTED;
    if (vec != 0 && vec != 1 && vec != 2 && vec != 4) return PCSR_E_UNSUPPORTED;
    if (rep != 0 && rep != 1 && rep != 2 && rep != 4) return PCSR_E_UNSUPPORTED;
    if (waves != 0 && waves != 1 && waves != 2 && waves != 4 && waves != 8 && waves != 16)
        return PCSR_E_UNSUPPORTED;
    return PCSR_OK;
}

} // namespace

struct pcsr_handle_s {
    uint32_t magic = kMagic;
    pcsr::HostPcsr host; // arrays kept only for host-only handles; scalars always valid
    bool host_only = false;
    int device = -1;
    int32_t *d_rowptr = nullptr;
    int32_t *d_colidx = nullptr;
    float *d_val = nullptr;
    int32_t *d_trow = nullptr;
    int32_t *d_split = nullptr;       // panels that own more than one item, ascending
    int32_t *d_item_slot = nullptr;   // per item: workspace slot, -1 for a sole item (S only)
    int32_t *d_sched = nullptr;       // column-ordered schedule: 4 int32 per launch position
    int32_t *d_split_slot = nullptr;  // their first workspace slots (n_split + 1 entries)
    bool dropped = false;             // built without an array that did not fit (DeviceBuild::dropped)
    int32_t *d_bands = nullptr;       // PCSR_FLAG_COLUMN_BANDS: where the rows' columns pass into each band but the first
    int32_t *d_long = nullptr;        // positions in d_split of panels with more than kLongPanelSlots items
    int64_t n_long = 0;
    int32_t *d_win = nullptr;     // window start per item block
    int32_t *d_win_ptr = nullptr; // item range per item block
    int32_t *d_win_lo = nullptr;  // per item: run of vectors inside the block's window
    int32_t *d_win_hi = nullptr;
    int64_t n_win_blocks = 0;
    bool clustered = false; // scheduled community by community (PCSR_FLAG_CLUSTER_IF_USEFUL)
    int32_t asked_vec = 0;  // of such a handle: the load width of the shape that the order replaced (0: none given)
    decltype(pcsr::DeviceBuild::win) win; // of such a handle: windows of communities (blocks 0: none)
    int64_t n_split = 0;
    int64_t n_split_items = 0; // workspace slots: items that belong to split panels
    float *d_ws = nullptr;     // partial rows of those items, grown on demand
    size_t ws_bytes = 0;
    int32_t lpr = 0, vec = 0, rep = 0, waves = 0, ipg = 0, flags = 0;
};

namespace {

inline bool valid(pcsr_handle_t h) { return h && h->magic == kMagic; }

void release_device(pcsr_handle_t h)
{
    void *const all[] = {h->d_rowptr, h->d_colidx,     h->d_val,  h->d_trow, h->d_split,   h->d_item_slot, h->d_sched,
                         h->d_split_slot, h->d_long, h->d_win,  h->d_win_ptr, h->d_win_lo, h->d_win_hi, h->d_ws,
                         h->win.rowptr, h->win.colidx, h->win.val, h->win.rows, h->win.ptr, h->win.hi, h->d_bands};
    // the blocks are handed out again at once, so nothing may still be using them
    const bool idle = h->device >= 0 && pcsr::pool_quiesce(h->device);
    for (void *p : all) idle ? pcsr::pool_free(p) : pcsr::pool_release(p);
    h->d_rowptr = h->d_colidx = h->d_trow = h->d_split = h->d_win = nullptr;
    h->d_item_slot = h->d_sched = h->d_split_slot = h->d_long = h->d_win_ptr = nullptr;
    h->d_win_lo = h->d_win_hi = nullptr;
    h->d_val = h->d_ws = nullptr;
    h->d_bands = nullptr;
    h->ws_bytes = 0;
    h->win = {};
}

template <class T> int upload(const std::vector<T> &src, T **dst)
{
    *dst = nullptr;
    // one spare element so empty arrays still have a valid device address
    size_t bytes = (src.size() + 1) * sizeof(T);
    hipError_t e = pcsr::pool_alloc((void **)dst, bytes);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        return PCSR_E_OOM;
    }
    if (!hip_ok(e)) return PCSR_E_HIP;
    if (!src.empty() && !hip_ok(hipMemcpy(*dst, src.data(), src.size() * sizeof(T), hipMemcpyHostToDevice)))
        return PCSR_E_HIP;
    return PCSR_OK;
}

// PCSR_FLAG_WINDOW_IF_USEFUL: without structure for the window kernel to use, an ordinary handle.
void drop_poor_windows(pcsr_handle_t h)
{
    if (!h->host.win_cols || !(h->flags & PCSR_FLAG_WINDOW_IF_USEFUL)) return;
    if (h->host.win_hit >= 0.5 && h->host.M >= 128 * h->n_win_blocks) return;
    h->host.win_cols = 0;
    h->host.win_hit = 0.0;
    h->n_win_blocks = 0;
    std::vector<int32_t>().swap(h->host.win_start);
    std::vector<int32_t>().swap(h->host.win_ptr);
    std::vector<int32_t>().swap(h->host.win_lo);
    std::vector<int32_t>().swap(h->host.win_hi);
    for (int32_t **p : {&h->d_win, &h->d_win_ptr, &h->d_win_lo, &h->d_win_hi}) {
        pcsr::pool_free(*p); // built a moment ago, nothing reads them
        *p = nullptr;
    }
    h->lpr = h->vec = h->rep = h->waves = h->ipg = 0;
}

// Lists the split panels (by position in the split tables) with more than
// pcsr::kLongPanelSlots items and puts the list in device memory: the second pass of the
// balanced write-back gives those panels a workgroup each.  split_slot: n_split + 1 entries
// in host memory.
static int upload_long_panels(pcsr_handle_s *h, const int32_t *split_slot)
{
    std::vector<int32_t> list;
    for (int64_t q = 0; q < h->n_split; ++q)
        if (split_slot[q + 1] - split_slot[q] > pcsr::kLongPanelSlots) list.push_back((int32_t)q);
    h->n_long = (int64_t)list.size();
    if (list.empty()) return PCSR_OK;
    return upload(list, &h->d_long);
}

// Workgroups of `waves` wavefronts of 64/lpr groups, each taking ipg items, for all items.
int64_t grid_for(pcsr_handle_t h, int waves, int lpr, int ipg)
{
    const int64_t items_per_wg = (int64_t)waves * (64 / lpr) * ipg;
    if (h->flags & PCSR_FLAG_NO_XCD_REMAP) return (h->host.M + items_per_wg - 1) / items_per_wg;
    // every XCD walks its own item range: 8 x the workgroups of the longest range
    int64_t longest = 0;
    for (int x = 0; x < 8; ++x)
        longest = std::max<int64_t>(longest, h->host.xcd_bounds[x + 1] - h->host.xcd_bounds[x]);
    return 8 * ((longest + items_per_wg - 1) / items_per_wg);
}

// Column-window launches: a compute unit holds one or two workgroups, each of a whole (block, slice) pair, so the
// last round of them leaves most of the chip idle (1056 pairs on 256 compute units: 4 rounds and an eighth).  Its
// pairs are cut into `parts` workgroups of as many items less, each staging the window again: a part costs 1/parts
// of a whole one and 0.15 for the staging, and the cheapest number of rounds is taken, if it beats one whole round.
// Communities of 500 rows of 48, us whole / cut: 250,000 rows K = 64 120 / 96, 128 181 / 173, 256 352 / 341, 512
// 730 / 720; 60,000 rows K = 64 44 / 28, 192 85 / 69.  Where the last round is nearly full no cut pays (60,000 rows,
// K = 512: 171 whole, 172 in 2, 190 in 8) and the rule takes none.  Not for blocks of fewer items than a
// workgroup's 64 lane groups, which a part would leave idle.
void window_tail(pcsr_handle_t h, pcsr::LaunchShape *ls)
{
    ls->win_whole = 0x7fffffff;
    ls->win_parts = 1;
    const int64_t pairs = (int64_t)ls->grid_x * ls->grid_y;
    if ((h->flags & PCSR_FLAG_NO_XCD_REMAP) || pairs == 0 || pairs > (1 << 20)) return;
    const int64_t at_once = 32 * std::max(1, std::min(160 * 1024 / ls->lds_bytes, 16 / ls->waves)); // of an XCD
    const int64_t most = (pairs + 7) / 8, rest = most % at_once;
    int parts = 1;
    double best = 1.15;
    for (int p = 2; rest && p <= 8; ++p) {
        const double cost = (double)((rest * p + at_once - 1) / at_once) * (1.0 / p + 0.15);
        if (cost < best - 0.05) {
            best = cost;
            parts = p;
        }
    }
    if (parts == 1 || h->host.M < pairs / ls->grid_y * 64) return;
    ls->win_whole = (int32_t)(most - rest);
    ls->win_parts = parts;
    ls->k_grid_x = (int32_t)(8 * (most - rest + rest * parts));
    ls->k_grid_y = 1;
}

// Auto shapes' slices of rows of over 64 columns are in parts of 20 and more, as the tiles of whole rows were that they have taken the
// place of (100,000 rows of 60, K = 128: rms 4.66e-8 of the sum in 6 bands, 4.38 in 3; 296 us and 315, 373 in those tiles).
constexpr double kSlicedPart = 20.0;
constexpr int32_t kSlicedMost = 1 << 20; // (more slices than a grid has otherwise)

// How many bands of columns a product of scattered rows is best walked in (a divisor of kColumnBands), and the us that they save.  A
// band of B that an XCD's L2 holds is gathered from there; each band of several costs a launch, a look at every row and a pass over
// C.  The rates are those that fit 1,200 measured times best (uniform columns, 14 to 300 a row, 40,000 to 1,000,000 rows, 6 to 256
// columns, 1 to 12 bands): the number picked is 0.9 % off the best of them on average and 14 % at most, and never over 1.3 % off
// one band.  Us in one band and in those picked: rows of 134, 300,000 of them, K = 16 667 and 366 (6 bands), K = 32 706 and 527 (6),
// K = 64 1459 and 1197 (6); of 60, 150,000, K = 16 118 and 76 (3), K = 48 291 and 211 (6); of 60, 400,000, K = 10 462 and 235 (4),
// K = 64 908 in one; of 30, 400,000, K = 9 202 and 145 (3), K = 16 193 in one; of 300, 100,000, K = 32 385 and 224 (4).
// least_part: vectors of a row in a band, at least.
int band_count(double n_rows, double n_cols, double nnz, int32_t K, int lanes, int32_t tile, double *saved, double least_part = 0.0)
{
    const double slices = (K + tile - 1) / tile, row = 4.0 * K / slices;
    const double grain = (double)std::min(128, (4 * K) & -(4 * K)); // rows of B begin at multiples of it
    const double miss = std::ceil((row + 128.0 - grain) / 32.0) / 4.0 / 39e3, hit = std::max(1.0 / 140e3, row / 31e6);
    auto us = [&](int m) {
        const double near = std::cbrt(std::min(1.0, 3.5e6 * m / std::max(n_cols * row, 1.0)));
        const double passes = m * (1.7 + n_rows * 1e-3 * (slices * (0.006 + 0.00106 * lanes) + 0.00133 * K));
        return slices * nnz * (near * hit + (1.0 - near) * miss) + (m > 1 ? passes : 0.0);
    };
    int best = 1;
    // Rows of less than 256 are better added up in fewer than 12 parts, and in tiles of whole rows by whole and half wavefronts, whose
    // sums were of 8 before, in parts of 20 and more.
    const double least = tile >= 128 || (K > 64 && K % 32 != 0) ? 20.0 : least_part;
    for (const int m : {2, 3, 4, 6, 12})
        if (nnz >= std::max(m < 12 ? 0.0 : 256.0, least * m) * n_rows && us(m) < (best > 1 ? 0.98 : 1.0) * us(best)) best = m;
    *saved = us(1) - us(best);
    // (Tiles of 512 columns, which those times do not have, save 0.05 to 0.15 less than that: K = 260 to 500, 100,000 rows of 134
    // 0.88-0.99 of the time in 6 where 0.81-0.87 was expected, 200,000 of 100 1.02-1.06 for 0.95, 300,000 of 90 1.05 for 0.96.)
    return *saved > (tile > 256 ? 0.1 : 0.03) * us(1) ? best : 1;
}

// Launch shape for width K under the handle's kernel parameters ("0 = auto" resolved).
// epilogue: for pcsr_spmm_epilogue, whose kernels exist for the auto shapes only; a handle with
// another shape of its own uses those.
int resolve_launch(pcsr_handle_t h, int32_t K, pcsr::LaunchShape *ls, bool epilogue = false)
{
    if (K <= 0) return PCSR_E_UNSUPPORTED;
    if (h->win.blocks && K >= kRowsLeast && K % 4 == 0 && !(h->lpr || h->vec || h->rep || h->waves || h->ipg)) {
        const int tile = pcsr::kRowsLanes * pcsr::kRowsVec, gy = (K + tile - 1) / tile;
        if (gy > 65535) return PCSR_E_TOO_LARGE;
        ls->lpr = ls->k_lpr = pcsr::kRowsLanes;
        ls->vec = ls->k_vec = pcsr::kRowsVec;
        ls->rep = ls->k_rep = ls->ipg = 1;
        ls->waves = 16;
        ls->window = 1;
        ls->lds_bytes = (pcsr::kRowsMost + 1) * (tile + 4) * 4;
        ls->grid_x = ls->k_grid_x = (int32_t)h->win.blocks;
        ls->grid_y = ls->k_grid_y = gy;
        window_tail(h, ls);
        return PCSR_OK;
    }
    const bool plain = h->host.win_cols == 0 && h->ipg <= 1;
    const bool own = !(epilogue && plain && (h->lpr || h->vec || h->rep)) && !((h->flags & kAutoNarrow) && K <= kAutoNarrowMost);
    const int h_lpr = own ? h->lpr : 0, h_vec = own ? h->vec : 0, h_rep = own ? h->rep : 0;
    int vec = h_vec ? h_vec : (K % 4 == 0 ? 4 : (K % 2 == 0 ? 2 : 1));
    // as pcsr_select: K of 9..16 is served by 16 lanes of one dword unless rows are very short
    if (!h_vec && !h_lpr && K > 8 && K <= 16 && h->host.win_cols == 0 &&
        h->host.nnz_v >= 8 * std::max<int64_t>(h->host.P, 1))
        vec = 1;
    // and K of up to 8, rows of 32 and more (single rows of 18 and 27 that share their neighbours' columns 0.86-1.58 of 4 lanes' time)
    const bool narrow = !h_vec && !h_lpr && !h_rep && K <= 8 && h->host.win_cols == 0 && h->ipg <= 1 &&
                        h->host.nnz_v >= 32 * std::max<int64_t>(h->host.P, 1);
    // and K of 17 to 32, single rows of 32 and more, for which pcsr_select has these shapes, too: half as many rows a wavefront as
    // with 8 lanes of 16 bytes take 0.62-0.92 of the time in half wavefronts, scattered and in bands, 0.84-0.92 otherwise, tails
    // 0.63-0.94 (150,000 scattered rows of 60, K = 24 209 us and 126; 250,000 of 48 in shuffled communities, K = 32 236 and 198;
    // 100,000 of 85 in cliques 64 and 57; of less than 32 1.00).  Up to 64 columns likewise, two to a lane of a half wavefront, in
    // place of 16 lanes of 16 bytes: 0.90-0.97 (100,000 rows of 85 in cliques, K = 64 110 us and 99), but not in bands (100,000 of
    // 48, K = 48 107 us and 137), nor long rows of scattered columns where an XCD's L2 holds some of B and the memory-side cache
    // the rest: operators of 16,000 to 80,000 rows of 60 and more, K = 52 to 64 1.01-1.18 (30,000 of 134 64 us and 73, of 300 125
    // and 148; 0.91-1.00 below, 0.97-1.00 above; with a tail, whose rows that form asks for late, 1.01-1.19 from 2.5 MB on), K = 36
    // to 48 0.96-1.06, of 134 1.02-1.06 from 7 MB on.  (Rows of 36 0.95-1.06, and more exact.)
    const double b_bytes = 4.0 * (double)h->host.n_cols * K;
    const int64_t panels = std::max<int64_t>(h->host.P, 1);
    const bool between = (h->flags & kScattered) && b_bytes < 18e6 && h->host.nnz_v >= 56 * panels &&
                         (K > 48 ? b_bytes > (epilogue ? 2.5e6 : 3.8e6) : b_bytes > 7e6 && h->host.nnz_v >= 100 * panels);
    const bool dwords = !h_vec && !h_lpr && !h_rep && K > 16 && (K <= 32 || (K <= 64 && K % 4 == 0 && !h->d_bands && !between)) &&
                        h->host.win_cols == 0 && h->ipg <= 1 && h->host.V == 1 && !h->host.S &&
                        h->host.nnz_v >= 32 * std::max<int64_t>(h->host.P, 1);
    // Rows of over 64 columns of a handle with bands go in slices, as pcsr_select has them: of 64 columns in 16 lanes where there
    // are several bands, else half a wavefront to 64 columns.  Us of such slices, of a tile of the whole row and of items of 32 in
    // column order: rows of 90, 100,000 of them, K = 128 392, 471 and 483, K = 256 775, 1182 and 965, K = 512 1549, 2512 and 1941;
    // of 134, 300,000, K = 256 4781, 5774 and 5356; of 44, 500,000 (one band), K = 256 3028, 3113 and 3796.  Rows that are no
    // multiple of 128 bytes long have lines that two slices would read: in such a tile K = 200 959, and 1065 in items, K = 300 1544 and
    // 1667 (in slices, of another session, 1.04 and 1.14 of the tile).
    double saved;
    const bool sliced = !h_vec && !h_lpr && !h_rep && h->d_bands && h->ipg <= 1 && K > 64 && K % 32 == 0 && K <= kSlicedMost;
    const bool in_bands =
        sliced && band_count((double)h->host.n_rows, (double)h->host.n_cols, (double)h->host.nnz, K, 16, 64, &saved, kSlicedPart) > 1;
    if (narrow || dwords) vec = 1;
    if (sliced) vec = in_bands ? 4 : 2;
    if (K % vec != 0) return PCSR_E_UNSUPPORTED;
    int lpr = h_lpr;
    if (narrow) lpr = narrow_lanes(h->host.S);
    if (dwords) lpr = h->d_bands || K > 32 ? 32 : 16;
    if (sliced) lpr = in_bands ? 16 : 32;
    if (!lpr) {
        int need = (K + vec - 1) / vec;
        if (h->host.win_cols > 0) {
            // column window: the staged slice (win_cols rows of lanes*vec columns) gets 128 KiB
            const int fit = (128 * 1024 / 4 / h->host.win_cols - 4) / vec;
            if (need > fit) need = fit;
        }
        // balanced (power-law) handles: four items per wavefront, as pcsr_select picks.  Rows run community by
        // community gather from L2, and whole rows of B then beat slices of 64 columns (250,000 rows of 48:
        // K = 128 262 us for 296, K = 256 578 for 680, K = 300 879 for 1032).
        const int cap = h->host.S && !h->clustered ? 16 : 64;
        lpr = 4;
        while (lpr < need && lpr < cap) lpr <<= 1;
    }
    int rep = h_rep;
    if (!rep) {
        int need = (K + lpr * vec - 1) / (lpr * vec);
        rep = 1;
        const int most = sliced ? 1 : h->d_bands ? 2 : !h->host.S ? 4 : (h->clustered ? 2 : 1); // (the band kernel's)
        if (h->host.win_cols == 0)
            while (rep < need && rep < most) rep <<= 1;
    }
    int waves = h->waves ? h->waves : 4;
    int ipg = h->ipg ? h->ipg : 1;
    if (ipg > 1) {
        // the batched walk accumulates each item sequentially and has no atomic write-back
        if (h->host.S || h->host.max_item_len > 1024) return PCSR_E_UNSUPPORTED;
    }
    const int64_t tile = (int64_t)lpr * vec * rep;
    ls->window = 0;
    ls->lds_bytes = 0;
    int64_t gx;
    if (h->host.win_cols > 0) {
        // column-window kernel: one workgroup per item block
        if (h->host.S || ipg > 1) return PCSR_E_UNSUPPORTED;
        if (!pcsr::window_kernel_exists(h->host.V, lpr, vec, rep)) return PCSR_E_UNSUPPORTED;
        // win_cols rows of B and one row of zeros, each padded by 4 floats
        const int64_t lds = ((int64_t)h->host.win_cols + 1) * (tile + 4) * 4;
        if (lds > 160 * 1024) return PCSR_E_UNSUPPORTED;
        if (!h->waves) waves = 16;
        ls->window = 1;
        ls->lds_bytes = (int32_t)lds;
        gx = h->n_win_blocks;
    } else {
        if (waves > 8) return PCSR_E_UNSUPPORTED;
        if (!(epilogue && ipg == 1 ? pcsr::epilogue_kernel_exists(h->host.V, h->host.S, lpr, vec, rep)
                                   : pcsr::kernel_exists(h->host.V, h->host.S, lpr, vec, rep, ipg)))
            return PCSR_E_UNSUPPORTED;
        gx = grid_for(h, waves, lpr, ipg);
    }
    const int64_t gy = (K + tile - 1) / tile;
    if (gx > 0x7fffffffLL || gy > 65535) return PCSR_E_TOO_LARGE;
    ls->lpr = lpr;
    ls->vec = vec;
    ls->rep = rep;
    ls->waves = waves;
    ls->ipg = ipg;
    ls->grid_x = (int32_t)gx;
    ls->grid_y = (int32_t)gy;
    ls->k_lpr = lpr;
    ls->k_vec = vec;
    ls->k_rep = rep;
    ls->k_grid_x = ls->grid_x;
    ls->k_grid_y = ls->grid_y;
    if (ls->window) window_tail(h, ls);
    // Where the shape above reads rows badly another one is launched in its place, with wide loads
    // at 4-byte addresses (pcsr_select's, carried in the flags, or this function's own pick for an
    // auto shape; never where the caller asked for lanes or vectors): widths that are no
    // multiple of 4, and 64-column slices of rows that are no multiple of 128 bytes long, of which
    // every slice touches a line more than it needs.
    const bool beyond = (h_lpr || h_vec || h_rep) && (h->flags & kWideBeyond);
    if (!ls->window && ipg == 1 && K > (beyond ? tile : 16)) {
        int wide = 0, wide_vec = 4, wide_rep = 1;
        if (h_lpr || h_vec || h_rep) {
            if (h->flags & kWideShape) wide = 4 << ((h->flags & kWideShape) >> kWideShift) >> 1;
            if (h->flags & kWidePair) wide_vec = 2;
            if (h->flags & kWideTwice) wide_rep = 2;
            // In bands, slices that share columns take one (band_passes): at other widths than the one that the shape came with a
            // row in one tile instead (300,000 rows of 134, selected at K = 50, us at K = 66 2777 and 1597; 100,000 of 90 509 and 248).
            if (wide && h->d_bands && K % wide_vec != 0 && wide * wide_vec * wide_rep < K) {
                wide_vec = 4;
                wide_shape(K, 64, &wide, &wide_rep);
            }
        } else if (!dwords && (K % 4 != 0 || (h->host.S && K > 64 && K % 32 != 0))) {
            wide_shape(K, h->host.S && K <= 64 ? 16 : 64, &wide, &wide_rep);
        }
        const int64_t wt = (int64_t)wide * wide_vec * wide_rep;
        if (wide) {
            const int64_t wx = grid_for(h, waves, wide, 1), wy = (K + wt - 1) / wt;
            if (wx <= 0x7fffffffLL && wy <= 65535) {
                ls->k_lpr = wide;
                ls->k_vec = wide_vec;
                ls->k_rep = wide_rep;
                ls->k_grid_x = (int32_t)wx;
                ls->k_grid_y = (int32_t)wy;
            }
        }
    }
    return PCSR_OK;
}

// Host CSR arrays in device memory for the length of a call.  The values follow beside the work on the pattern:
// their half of the upload (48 MB: 1 ms) is under way when put() returns.
struct UploadedCsr {
    int32_t *rowptr = nullptr, *colidx = nullptr;
    float *vals = nullptr;
    pcsr::Upload values;
    int put(int64_t n_rows, int64_t nnz, const int32_t *h_rowptr, const int32_t *h_colidx, const float *h_vals)
    {
        auto one = [](void **d, const void *src, size_t bytes) {
            hipError_t e = pcsr::pool_alloc(d, bytes + 4);
            if (e == hipSuccess && bytes && src) e = pcsr::copy_to_device(*d, src, bytes);
            return e;
        };
        hipError_t e = one((void **)&rowptr, h_rowptr, sizeof(int32_t) * (n_rows + 1));
        if (e == hipSuccess) e = one((void **)&vals, nullptr, sizeof(float) * nnz);
        if (e == hipSuccess) e = one((void **)&colidx, h_colidx, sizeof(int32_t) * nnz);
        if (e == hipErrorOutOfMemory) {
            (void)hipGetLastError();
            return PCSR_E_OOM;
        }
        if (!hip_ok(e)) return PCSR_E_HIP;
        values.start(vals, h_vals, sizeof(float) * nnz);
        return PCSR_OK;
    }
    ~UploadedCsr()
    {
        (void)values.wait();
        if (!rowptr) return;
        (void)pcsr::setup_wait();
        pcsr::pool_free(rowptr);
        pcsr::pool_free(colidx);
        pcsr::pool_free(vals);
    }
};

// A handle in the making, given up if the scope is left without keep().
struct Draft {
    pcsr_handle_t h;
    pcsr_handle_t keep()
    {
        pcsr_handle_t made = h;
        h = nullptr;
        return made;
    }
    ~Draft()
    {
        if (!h) return;
        release_device(h);
        delete h;
    }
};

// Returned by handle_from_device where the windows have to be chosen on the host.
constexpr int kWindowsOnHost = 1;

// Nonzeros and rows below which pcsr_operator_build stays on the host.
constexpr int64_t kHostOperator = 10000; // 0.5 ms there, 0.65 ms on the GPU at any size up to here

// A handle from CSR arrays in device memory, everything built there.  late: the copy that fills vals, if it is still
// under way; known: see build_device.
int handle_from_device(int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t *rowptr, const int32_t *colidx,
                       const float *vals, const pcsr_params_t &prm, const pcsr::RowStats *known, pcsr::Late *late,
                       pcsr_handle_s **out)
{
    const bool column_order = (prm.flags & PCSR_FLAG_COLUMN_ORDER) != 0;
    pcsr_handle_s *h = new (std::nothrow) pcsr_handle_s();
    if (!h) return PCSR_E_OOM;
    if (!hip_ok(hipGetDevice(&h->device))) {
        delete h;
        return PCSR_E_HIP;
    }
    pcsr::DeviceBuild db;
    int herr = 0;
    int rc = pcsr::build_device(n_rows, n_cols, nnz, rowptr, colidx, vals, prm.V, prm.S, prm.SG, prm.omega,
                                !(prm.flags & PCSR_FLAG_NO_VALIDATE), column_order,
                                (prm.flags & PCSR_FLAG_CLUSTER_IF_USEFUL) && !prm.col_window,
                                (prm.flags & PCSR_FLAG_CLUSTER_WINDOWS) != 0,
                                (prm.flags & PCSR_FLAG_COLUMN_BANDS) && !prm.col_window, known, late, &db, &herr);
    h->host.n_rows = n_rows;
    h->host.n_cols = n_cols;
    h->host.nnz = nnz;
    h->host.V = prm.V;
    h->host.S = rc == PCSR_OK ? db.S : prm.S;
    h->host.P = db.P;
    h->host.M = db.M;
    h->host.nnz_v = db.nnz_v;
    h->host.SG = db.SG;
    h->host.max_item_len = db.max_item_len;
    for (int x = 0; x < 9; ++x) h->host.xcd_bounds[x] = db.xcd_bounds[x];
    h->d_rowptr = db.rowptr;
    h->d_colidx = db.colidx;
    h->d_val = db.val;
    h->d_trow = db.trow;
    h->d_split = db.split;
    h->d_item_slot = db.item_slot;
    h->d_sched = db.sched;
    h->d_split_slot = db.split_slot;
    h->d_long = db.long_list;
    h->d_bands = db.bands;
    h->dropped = db.dropped;
    h->n_split = db.n_split;
    h->n_split_items = db.n_split_items;
    h->n_long = db.n_long;
    h->win = db.win;
    h->lpr = prm.lanes_per_row;
    h->vec = prm.vec;
    h->rep = prm.rep;
    h->waves = prm.waves_per_wg;
    h->ipg = prm.items_per_group;
    h->flags = checked_flags(prm);
    if (rc == PCSR_OK && db.clustered) { // the caller's shape was for the order it would have had otherwise
        h->clustered = true;
        h->asked_vec = h->vec;
        h->lpr = h->vec = h->rep = h->waves = h->ipg = 0;
        h->flags &= ~kWideBits;
    }
    if (rc == PCSR_OK && prm.col_window) {
        pcsr::DeviceWindows w;
        rc = pcsr::windows_device(db.M, n_cols, prm.col_window, db.rowptr, db.colidx, &w, &herr);
        if (rc == PCSR_E_UNSUPPORTED) rc = kWindowsOnHost;
        if (rc == PCSR_OK) {
            h->d_win = w.start;
            h->d_win_ptr = w.ptr;
            h->d_win_lo = w.lo;
            h->d_win_hi = w.hi;
            h->host.win_cols = prm.col_window;
            h->host.win_hit = db.nnz_v ? double(w.hits) / double(db.nnz_v) : 0.0;
            h->n_win_blocks = w.blocks;
            drop_poor_windows(h);
        }
    }
    if (rc == PCSR_OK && db.vals_due) {
        hipError_t e = late->wait();
        if (e == hipSuccess && nnz > 0)
            e = hipMemcpyAsync(h->d_val, vals, sizeof(float) * nnz, hipMemcpyDeviceToDevice, pcsr::setup_stream());
        if (e == hipSuccess) e = pcsr::setup_wait();
        if (e != hipSuccess) {
            herr = (int)e;
            (void)hipGetLastError();
            rc = PCSR_E_HIP;
        }
    }
    if (rc != PCSR_OK) {
        if (rc == PCSR_E_HIP) g_last_hip = herr;
        release_device(h);
        delete h;
        return rc;
    }
    *out = h;
    return PCSR_OK;
}

} // namespace

extern "C" {

// pcsr_build; known: see build_device; late: the copy that fills vals (device memory), if it is still under way.
static int build_from(int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t *rowptr, const int32_t *colidx,
                      const float *vals, const pcsr_params_t *p, const pcsr::RowStats *known, pcsr::Late *late, pcsr_handle_t *out)
{
    if (!out || !rowptr || n_rows < 0 || n_cols < 0 || nnz < 0) return PCSR_E_INVALID_ARG;
    if (nnz > 0 && (!colidx || !vals)) return PCSR_E_INVALID_ARG;
    pcsr_params_t prm;
    std::memset(&prm, 0, sizeof(prm));
    if (p) prm = *p;
    if (prm.V == 0) prm.V = 1;
    if (prm.V != 1 && prm.V != 2) return PCSR_E_UNSUPPORTED;
    if (prm.S != 0 && prm.S != 1) return PCSR_E_UNSUPPORTED;
    if (prm.SG < 0 || prm.omega < 0) return PCSR_E_INVALID_ARG;
    if (prm.reserved[0]) return PCSR_E_INVALID_ARG;
    if (prm.col_window != 0 && prm.col_window != 256 && prm.col_window != 512 && prm.col_window != 1024 &&
        prm.col_window != 2048)
        return PCSR_E_UNSUPPORTED;
    if (prm.col_window && prm.S) return PCSR_E_UNSUPPORTED;
    if (nnz >= (int64_t(1) << 31) || n_rows >= (int64_t(1) << 31) - 1 || n_cols >= (int64_t(1) << 31))
        return PCSR_E_TOO_LARGE;
    int rc = check_kernel_params(prm.lanes_per_row, prm.vec, prm.rep, prm.waves_per_wg, prm.items_per_group);
    if (rc != PCSR_OK) return rc;
    const bool host_only = (prm.flags & PCSR_FLAG_HOST_ONLY) != 0;
    if (host_only && (prm.flags & PCSR_FLAG_DEVICE_CSR)) return PCSR_E_INVALID_ARG;

    const bool device_csr = (prm.flags & PCSR_FLAG_DEVICE_CSR) != 0;
    const bool column_order = (prm.flags & PCSR_FLAG_COLUMN_ORDER) != 0;
    if (column_order && (!prm.S || prm.col_window)) return PCSR_E_UNSUPPORTED;
    if (host_only && (prm.flags & PCSR_FLAG_GPU_BUILD) && !prm.col_window) return PCSR_E_INVALID_ARG;
    // On the GPU wherever the arrays are there already, the caller asks for it, or the upload and
    // the launches cost less than the host threads take (12 M nonzeros: 6 ms against 25-60).  Nobody
    // asked in the last case, so if the scratch does not fit the host builder, which needs none, does it.
    const bool asked = device_csr || ((prm.flags & PCSR_FLAG_GPU_BUILD) && !prm.col_window);
    if (!host_only && (asked || pcsr::relabel_on_gpu(nnz))) {
        UploadedCsr up;
        const int32_t *d_rowptr = rowptr, *d_colidx = colidx;
        const float *d_vals = vals;
        if (!device_csr) {
            rc = up.put(n_rows, nnz, rowptr, colidx, vals);
            d_rowptr = up.rowptr;
            d_colidx = up.colidx;
            d_vals = up.vals;
        }
        pcsr_handle_s *h = nullptr;
        if (rc == PCSR_OK)
            rc = handle_from_device(n_rows, n_cols, nnz, d_rowptr, d_colidx, d_vals, prm, known,
                                    device_csr ? late : static_cast<pcsr::Late *>(&up.values), &h);
        if (rc == PCSR_OK) *out = h;
        if (rc != kWindowsOnHost && !(rc == PCSR_E_OOM && !asked)) return rc;
    }

    try {
        // The host builder: handles without a GPU, small matrices, and column windows over rows
        // too long for the GPU's (CSR arrays in device memory are copied here for those).
        std::vector<int32_t> s_rowptr, s_colidx;
        std::vector<float> s_vals;
        if (device_csr) {
            if (late && !hip_ok(late->wait())) return PCSR_E_HIP;
            s_rowptr.resize(n_rows + 1);
            s_colidx.resize(nnz);
            s_vals.resize(nnz);
            if (!hip_ok(hipMemcpy(s_rowptr.data(), rowptr, sizeof(int32_t) * (n_rows + 1), hipMemcpyDeviceToHost)))
                return PCSR_E_HIP;
            if (nnz > 0 &&
                (!hip_ok(hipMemcpy(s_colidx.data(), colidx, sizeof(int32_t) * nnz, hipMemcpyDeviceToHost)) ||
                 !hip_ok(hipMemcpy(s_vals.data(), vals, sizeof(float) * nnz, hipMemcpyDeviceToHost))))
                return PCSR_E_HIP;
            rowptr = s_rowptr.data();
            colidx = s_colidx.data();
            vals = s_vals.data();
        }
        if (!(prm.flags & PCSR_FLAG_NO_VALIDATE)) {
            rc = pcsr::validate_csr(n_rows, n_cols, nnz, rowptr, colidx);
            if (rc != PCSR_OK) return rc;
        } else if (rowptr[0] != 0 || rowptr[n_rows] != nnz) {
            return PCSR_E_BAD_CSR;
        }

        Draft draft{new pcsr_handle_s()};
        pcsr_handle_s *const h = draft.h;
        rc = pcsr::build_host(n_rows, n_cols, nnz, rowptr, colidx, vals, prm.V, prm.S, prm.SG,
                              prm.omega, &h->host);
        if (rc != PCSR_OK) return rc;
        if (column_order) {
            rc = pcsr::schedule_by_column(&h->host);
            if (rc != PCSR_OK) return rc;
        }
        if (prm.col_window) {
            rc = pcsr::choose_windows(&h->host, prm.col_window);
            if (rc != PCSR_OK) return rc;
        }
        h->n_win_blocks = (int64_t)h->host.win_start.size();
        h->host_only = host_only;
        h->lpr = prm.lanes_per_row;
        h->vec = prm.vec;
        h->rep = prm.rep;
        h->waves = prm.waves_per_wg;
        h->ipg = prm.items_per_group;
        h->flags = checked_flags(prm);
        drop_poor_windows(h);
        h->n_split = (int64_t)h->host.split_panels.size();
        h->n_split_items = h->host.split_slot.empty() ? 0 : h->host.split_slot.back();
        if (!host_only) {
            if (!hip_ok(hipGetDevice(&h->device))) return PCSR_E_HIP;
            rc = upload(h->host.rowptr, &h->d_rowptr);
            if (rc == PCSR_OK) rc = upload(h->host.colidx, &h->d_colidx);
            if (rc == PCSR_OK) rc = upload(h->host.val, &h->d_val);
            if (rc == PCSR_OK && h->host.S) rc = upload(h->host.trow, &h->d_trow);
            if (rc == PCSR_OK && h->n_split) rc = upload(h->host.split_panels, &h->d_split);
            if (rc == PCSR_OK && h->host.S) rc = upload(h->host.item_slot, &h->d_item_slot);
            if (rc == PCSR_OK && !h->host.sched.empty()) rc = upload(h->host.sched, &h->d_sched);
            if (rc == PCSR_OK && h->n_split) rc = upload(h->host.split_slot, &h->d_split_slot);
            if (rc == PCSR_OK && h->n_split) rc = upload_long_panels(h, h->host.split_slot.data());
            if (rc == PCSR_OK && h->host.win_cols) rc = upload(h->host.win_start, &h->d_win);
            if (rc == PCSR_OK && h->host.win_cols) rc = upload(h->host.win_ptr, &h->d_win_ptr);
            if (rc == PCSR_OK && h->host.win_cols) rc = upload(h->host.win_lo, &h->d_win_lo);
            if (rc == PCSR_OK && h->host.win_cols) rc = upload(h->host.win_hi, &h->d_win_hi);
            if (rc != PCSR_OK) return rc;
            // the device copies are the product; drop the host staging arrays
            std::vector<int32_t>().swap(h->host.rowptr);
            std::vector<int32_t>().swap(h->host.colidx);
            std::vector<float>().swap(h->host.val);
            std::vector<int32_t>().swap(h->host.trow);
            std::vector<int32_t>().swap(h->host.split_panels);
            std::vector<int32_t>().swap(h->host.item_slot);
            std::vector<int32_t>().swap(h->host.sched);
            std::vector<int32_t>().swap(h->host.split_slot);
            std::vector<int32_t>().swap(h->host.win_start);
            std::vector<int32_t>().swap(h->host.win_ptr);
            std::vector<int32_t>().swap(h->host.win_lo);
            std::vector<int32_t>().swap(h->host.win_hi);
        }
        *out = draft.keep();
        return PCSR_OK;
    } catch (const std::bad_alloc &) {
        return PCSR_E_OOM;
    }
}

int pcsr_build(int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t *rowptr, const int32_t *colidx,
               const float *vals, const pcsr_params_t *p, pcsr_handle_t *out)
{
    return build_from(n_rows, n_cols, nnz, rowptr, colidx, vals, p, nullptr, nullptr, out);
}

// pcsr_operator_build's parameters for one direction: the caller's, or what pcsr_select picks for
// these features, its launch shape left on auto so that one handle serves every layer width.
static int operator_params(const pcsr_params_t *p, bool pick, const double *f, int32_t K, pcsr_params_t *prm)
{
    if (!pick) {
        *prm = *p;
        return PCSR_OK;
    }
    const int rc = pcsr_select(f, K, prm);
    if (rc == PCSR_OK) prm->lanes_per_row = prm->vec = prm->rep = 0;
    if (rc == PCSR_OK && scattered_columns(f)) prm->flags |= kScattered;
    return rc;
}

// Both directions from arrays in host memory with what needs no scratch on the GPU.
static int operator_on_host(int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t *rowptr, const int32_t *colidx,
                            const float *vals, const pcsr_params_t *p, bool pick, int32_t K, bool with_transpose,
                            pcsr_handle_t made[2])
{
    auto direction = [&](int64_t nr, int64_t nc, const int32_t *rp, const int32_t *ci, const float *va,
                         pcsr_handle_t *h) -> int {
        pcsr_params_t prm;
        double f[PCSR_N_FEATURES];
        int rc = pick ? pcsr_features(nr, nc, nnz, rp, ci, 0, f, PCSR_N_FEATURES) : PCSR_OK;
        if (rc == PCSR_OK) rc = operator_params(p, pick, f, K, &prm);
        return rc == PCSR_OK ? pcsr_build(nr, nc, nnz, rp, ci, va, &prm, h) : rc;
    };
    int rc = direction(n_rows, n_cols, rowptr, colidx, vals, &made[0]);
    try {
        if (rc == PCSR_OK && with_transpose) {
            std::vector<int32_t> rp(n_cols + 1), ci(nnz);
            std::vector<float> va(nnz);
            rc = pcsr_transpose_csr(n_rows, n_cols, rowptr, colidx, vals, rp.data(), ci.data(), va.data());
            if (rc == PCSR_OK) rc = direction(n_cols, n_rows, rp.data(), ci.data(), va.data(), &made[1]);
        }
    } catch (const std::bad_alloc &) {
        rc = PCSR_E_OOM;
    }
    return rc;
}

// Values of the transpose, whose pattern was there before them.
struct TurnedValues final : pcsr::Late {
    pcsr::Upload *up;
    const float *vals;
    float *t_vals;
    int64_t nnz;
    bool due;
    hipError_t wait() noexcept override
    {
        hipError_t e = up->wait();
        if (e != hipSuccess || !due) return e;
        due = false;
        e = pcsr::turned_values(nnz, vals, t_vals);
        return e == hipSuccess ? pcsr::setup_wait() : e;
    }
};

// Both directions set up on the GPU, from one upload where the arrays are in host memory.  at_once: each on a thread and stream of
// its own, the transpose from the pattern alone while the values are still on their way.  A direction is a chain of small kernels and
// waits, and a GPU that runs one of them is mostly idle: 250,000 rows of 48 in communities, not symmetric 3.57 -> 2.95 ms with the first
// product each way (upload 2 of them), 4656 rows of 3 600 -> 460 us.
static int operator_on_gpu(int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t *rowptr, const int32_t *colidx,
                           const float *vals, const pcsr_params_t *p, bool pick, int32_t K, bool with_transpose,
                           bool device_csr, bool at_once, pcsr_handle_t made[2])
{
    UploadedCsr up;
    int herr = 0, rc = PCSR_OK;
    if (!device_csr) {
        rc = up.put(n_rows, nnz, rowptr, colidx, vals);
        if (rc != PCSR_OK) return rc;
        rowptr = up.rowptr;
        colidx = up.colidx;
        vals = up.vals;
    }
    auto failed = [](int code, int hip) {
        if (code == PCSR_E_HIP && hip) g_last_hip = hip;
        return code;
    };
    rc = pcsr::validate_device(n_rows, n_cols, nnz, rowptr, colidx, &herr);
    if (rc != PCSR_OK) return failed(rc, herr);
    auto direction = [&](int64_t nr, int64_t nc, const int32_t *rp, const int32_t *ci, const float *va, pcsr::Late *late,
                         pcsr_handle_t *h) -> int {
        pcsr_params_t prm;
        double f[PCSR_N_FEATURES];
        int hip = 0, r = pick ? pcsr::features_device(nr, nc, nnz, rp, ci, 0, f, &hip) : PCSR_OK;
        if (r == PCSR_OK) r = operator_params(p, pick, f, K, &prm);
        if (r != PCSR_OK) return failed(r, hip);
        prm.flags |= PCSR_FLAG_DEVICE_CSR | PCSR_FLAG_NO_VALIDATE;
        const pcsr::RowStats known = {(int64_t)f[6], (int64_t)f[1]};
        return build_from(nr, nc, nnz, rp, ci, va, &prm, pick ? &known : nullptr, late, h);
    };
    pcsr::Late *const late = device_csr ? nullptr : &up.values;
    auto forward = [&] { return direction(n_rows, n_cols, rowptr, colidx, vals, late, &made[0]); };
    auto backward = [&]() -> int {
        UploadedCsr t;
        const bool due = !device_csr && up.values.beside() && pcsr::transpose_in_two_passes(n_rows, n_cols, nnz);
        if (!due && !hip_ok(up.values.wait())) return PCSR_E_HIP;
        int hip = 0;
        const int r = pcsr::transpose_device(n_rows, n_cols, nnz, rowptr, colidx, due ? nullptr : vals, &t.rowptr, &t.colidx,
                                             &t.vals, &hip);
        if (r != PCSR_OK) return failed(r, hip);
        TurnedValues turned;
        turned.up = &up.values;
        turned.vals = vals;
        turned.t_vals = t.vals;
        turned.nnz = nnz;
        turned.due = due;
        return direction(n_cols, n_rows, t.rowptr, t.colidx, t.vals, due ? &turned : nullptr, &made[1]);
    };
    if (with_transpose && at_once) {
        int dev = -1;
        const pcsr::SideStream side;
        if (side.get() && hip_ok(hipGetDevice(&dev))) {
            int rc2 = PCSR_OK, hip2 = 0;
            std::thread beside;
            try {
                beside = std::thread([&] {
                    const pcsr::SetupOn on(side.get());
                    g_last_hip = 0;
                    try {
                        rc2 = hip_ok(hipSetDevice(dev)) ? backward() : PCSR_E_HIP;
                    } catch (...) { // no host memory
                        rc2 = PCSR_E_OOM;
                    }
                    (void)hipStreamSynchronize(side.get());
                    hip2 = g_last_hip;
                });
            } catch (...) { // no thread
            }
            if (beside.joinable()) {
                try {
                    rc = forward();
                } catch (...) {
                    rc = PCSR_E_OOM;
                }
                beside.join();
                if (rc == PCSR_OK) rc = failed(rc2, hip2);
                // What the one had no room for beside the other's scratch may fit when it is alone: the same memory, the same handles.
                if (rc == PCSR_OK && (made[0]->dropped || made[1]->dropped)) rc = PCSR_E_OOM;
                return rc;
            }
        }
    }
    rc = forward();
    return rc == PCSR_OK && with_transpose ? backward() : rc;
}

int pcsr_operator_build(int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t *rowptr, const int32_t *colidx,
                        const float *vals, const pcsr_params_t *p, int32_t K, int32_t with_transpose,
                        pcsr_handle_t out[2])
{
    if (!out || !rowptr || n_rows < 0 || n_cols < 0 || nnz < 0 || (nnz > 0 && (!colidx || !vals)))
        return PCSR_E_INVALID_ARG;
    if (nnz >= (int64_t(1) << 31) || n_rows >= (int64_t(1) << 31) - 1 || n_cols >= (int64_t(1) << 31) - 1)
        return PCSR_E_TOO_LARGE;
    const bool device_csr = p && (p->flags & PCSR_FLAG_DEVICE_CSR);
    const bool pick = !p || p->reserved[0] == PCSR_OPERATOR_SELECT;
    // small: the host is done before the GPU's launches and waits would be
    const bool small = !device_csr && nnz < kHostOperator && n_rows < kHostOperator && n_cols < kHostOperator;
    pcsr_handle_t made[2] = {nullptr, nullptr};
    auto give_back = [&] {
        (void)pcsr_free(made[0]);
        (void)pcsr_free(made[1]);
        made[0] = made[1] = nullptr;
    };
    int rc = PCSR_E_OOM;
    if (!small) {
        for (const bool at_once : {true, false}) { // one after the other where the scratch of both does not fit
            rc = operator_on_gpu(n_rows, n_cols, nnz, rowptr, colidx, vals, p, pick, K, with_transpose, device_csr, at_once, made);
            if (rc != PCSR_OK) give_back();
            if (rc != PCSR_E_OOM || !with_transpose) break;
        }
    }
    // the scratch did not fit: the host needs none
    if (rc == PCSR_E_OOM && !device_csr) {
        rc = operator_on_host(n_rows, n_cols, nnz, rowptr, colidx, vals, p, pick, K, with_transpose, made);
        if (rc != PCSR_OK) give_back();
    }
    if (rc != PCSR_OK) return rc;
    out[0] = made[0];
    out[1] = made[1];
    return PCSR_OK;
}

// Bytes of workspace one SpMM of width K needs: V*K floats per item of a split panel
// (deterministic balanced write-back only).
static int64_t workspace_need(pcsr_handle_t h, int32_t K)
{
    if (!h->host.S || (h->flags & PCSR_FLAG_ATOMIC_SPLIT)) return 0;
    return h->n_split_items * (int64_t)h->host.V * (int64_t)K * (int64_t)sizeof(float);
}

// Bytes that the operands have to be aligned to: those of the load width that the parameters mean, not of what is launched
// (whose loads are at 4-byte addresses anyway).  An order that the build found does not ask for more, nor do auto shapes in place of
// the handle's own.
static uintptr_t operand_align(pcsr_handle_t h, const pcsr::LaunchShape &ls)
{
    const int asked = h->asked_vec ? h->asked_vec : h->flags & kAutoNarrow ? h->vec : 0;
    return 4u * (unsigned)(asked ? std::min(asked, ls.vec) : ls.vec);
}

// Checks shared by the SpMM entry points; resolves the launch shape.
static int spmm_check(pcsr_handle_t h, const float *B, float *C, int32_t K, pcsr::LaunchShape *ls,
                      bool epilogue = false)
{
    if (!valid(h)) return PCSR_E_INVALID_ARG;
    if (h->host_only) return PCSR_E_UNSUPPORTED;
    if (K <= 0) return PCSR_E_UNSUPPORTED;
    if (!C && h->host.n_rows > 0) return PCSR_E_INVALID_ARG;
    if (!B && h->host.n_cols > 0 && h->host.nnz_v > 0) return PCSR_E_INVALID_ARG;
    int rc = resolve_launch(h, K, ls, epilogue);
    if (rc != PCSR_OK) return rc;
    const uintptr_t align = operand_align(h, *ls);
    if ((reinterpret_cast<uintptr_t>(B) % align) || (reinterpret_cast<uintptr_t>(C) % align))
        return PCSR_E_INVALID_ARG;
    if (h->host.n_rows == 0) return PCSR_OK;
    // B and C may not overlap: the kernel reads B while other workgroups write C
    const uintptr_t b0 = reinterpret_cast<uintptr_t>(B), c0 = reinterpret_cast<uintptr_t>(C);
    const uintptr_t b1 = b0 + (uintptr_t)h->host.n_cols * (uintptr_t)K * 4u;
    const uintptr_t c1 = c0 + (uintptr_t)h->host.n_rows * (uintptr_t)K * 4u;
    if (b0 < c1 && c0 < b1 && h->host.n_cols > 0) return PCSR_E_INVALID_ARG;
    // the handle's arrays live on the device that was current at pcsr_build
    int dev = -1;
    if (!hip_ok(hipGetDevice(&dev))) return PCSR_E_HIP;
    if (dev != h->device) return PCSR_E_INVALID_ARG;
    return PCSR_OK;
}

// Bands add to what is in C.  Where a shape's loads do not divide K, the last lane of a row also computes columns of the lane before it:
// harmless in one wavefront, which reads all of them before it writes any, and while all write the same bits; but the lane before the
// last slice's is in another workgroup, whose sum of this band may be there already.  (The first band reads nothing.)
static bool slices_share_columns(int32_t K, const pcsr::LaunchShape &ls) { return K % ls.k_vec != 0 && ls.k_grid_y > 1; }

// Bands leave their sums in C, where the tail of one pass has its rows read before they are written.
static bool tail_reads_c(const pcsr::Epilogue &e, const float *C, int64_t n_rows, int32_t K)
{
    auto meets = [&](const float *p, int64_t count) {
        const uintptr_t a = reinterpret_cast<uintptr_t>(p), c = reinterpret_cast<uintptr_t>(C);
        return p && a < c + 4u * (uintptr_t)n_rows * (uintptr_t)K && c < a + 4u * (uintptr_t)count;
    };
    return e.on && (meets(e.self, n_rows * K) || meets(e.mask, n_rows * K) || meets(e.bias, K) || meets(e.self_eps, 1));
}

// 0: the kernel for bands does not have the shape.  (A product in one band is that kernel's, too: it adds up long rows more exactly.)
static int band_passes(pcsr_handle_t h, int32_t K, const pcsr::LaunchShape &ls, const pcsr::Epilogue &epi, const float *C)
{
    double saved;
    if (ls.window || ls.ipg > 1 || !pcsr::band_kernel_exists(ls.k_lpr, ls.k_vec, ls.k_rep, epi.on)) return 0;
    if (slices_share_columns(K, ls) || tail_reads_c(epi, C, h->host.n_rows, K)) return 1;
    return band_count((double)h->host.n_rows, (double)h->host.n_cols, (double)h->host.nnz, K, ls.k_lpr, ls.k_lpr * ls.k_vec * ls.k_rep,
                      &saved, !(h->lpr || h->vec || h->rep) && K > 64 ? kSlicedPart : 0.0);
}

// Enqueues the kernels of one SpMM.  ws: workspace of at least workspace_need(h, K) bytes
// (ignored when that is 0).
static int spmm_enqueue(pcsr_handle_t h, const float *B, float *C, int32_t K, const pcsr::LaunchShape &ls,
                        float *ws, hipStream_t s, const pcsr::Epilogue &epi = pcsr::Epilogue())
{
    const bool two_pass = workspace_need(h, K) > 0;
    if (h->host.S && h->n_split > 0 && !two_pass) {
        if (!hip_ok(pcsr::launch_zero_panels(h->d_split, h->n_split, h->host.V, C,
                                             (int32_t)h->host.n_rows, K, s)))
            return PCSR_E_HIP;
    }
    pcsr::SpmmArgs a;
    a.rowptr = h->d_rowptr;
    a.colidx = h->d_colidx;
    a.val = h->d_val;
    a.trow = h->d_trow;
    a.B = B;
    a.C = C;
    a.M = (int32_t)h->host.M;
    a.mean_item = (int32_t)(h->host.nnz_v / std::max<int64_t>(h->host.M, 1));
    a.far = (h->flags & PCSR_FLAG_FAR_OFFSETS) != 0;
    a.n_rows = (int32_t)h->host.n_rows;
    a.K = K;
    a.nblk = ls.grid_x;
    a.xcd_remap = (h->flags & PCSR_FLAG_NO_XCD_REMAP) ? 0 : 1;
    for (int x = 0; x < 9; ++x) a.xb[x] = h->host.xcd_bounds[x];
    a.ws = two_pass ? ws : nullptr;
    a.item_slot = h->d_item_slot;
    a.sched = reinterpret_cast<const int4 *>(h->d_sched);
    // Where an item's sum would be less exact than that of items of 32 vectors: in the order by community, whose items
    // are whole rows, past 32, or 88 from their windows (sums of 8 there: rows of 80 1.36e-8 against 1.39e-8, of 100 1.30 against
    // 1.28); elsewhere, where 32 lanes and more keep sums of 8 apart in place of a chunk's, past 64.  Column windows: sums
    // of 16 in place of 8 where the longest row (or pair) has over 256.  They are better for rows of 130 and more (200: 0.83 against
    // 0.90e-8), worse for shorter ones (90: by 4 %), which such a handle may hold as well.
    const int64_t exact = h->host.win_cols ? 256 : ls.window ? 88 : h->clustered ? 32 : h->host.S && ls.k_lpr >= 32 ? 64 : INT32_MAX;
    a.outer = h->host.max_item_len > exact;
    a.win_start = h->d_win;
    a.win_cols = h->host.win_cols;
    a.win_ptr = h->d_win_ptr;
    a.win_lo = h->d_win_lo;
    a.win_hi = h->d_win_hi;
    a.n_cols = (int32_t)h->host.n_cols;
    a.n_slices = ls.grid_y;
    a.win_whole = ls.win_whole;
    a.win_parts = ls.win_parts;
    a.rows = nullptr;
    if (ls.window && h->win.blocks) {
        a.rowptr = a.win_lo = h->win.rowptr;
        a.colidx = h->win.colidx;
        a.val = h->win.val;
        a.win_ptr = h->win.ptr;
        a.win_hi = h->win.hi;
        a.win_cols = pcsr::kRowsMost;
        a.rows = h->win.rows;
    }
    a.epi = epi;
    a.band = 0;
    const int passes = h->d_bands ? band_passes(h, K, ls, epi, C) : 0;
    if (passes > 0) {
        const int step = pcsr::kColumnBands / passes;
        const int64_t n = h->host.n_rows;
        for (int p = 0; p < passes; ++p) {
            const bool first = p == 0, last = p == passes - 1;
            a.band = pcsr::kBandOn | (first ? pcsr::kBandFirst : 0) | (last ? pcsr::kBandLast : 0) | (passes > 3 ? pcsr::kBandSums64 : 0);
            a.rowptr = first ? h->d_rowptr : h->d_bands + (p * step - 1) * n;
            a.trow = last ? h->d_rowptr + 1 : h->d_bands + ((p + 1) * step - 1) * n;
            a.epi = last ? epi : pcsr::Epilogue();
            if (!hip_ok(pcsr::launch_spmm(h->host.V, h->host.S, ls, a, s))) return PCSR_E_HIP;
        }
        return PCSR_OK;
    }
    if (!hip_ok(pcsr::launch_spmm(h->host.V, h->host.S, ls, a, s))) return PCSR_E_HIP;
    if (two_pass) {
        if (!hip_ok(pcsr::launch_reduce_split(h->d_split, h->d_split_slot, h->n_split, h->d_long, h->n_long, h->host.V, ws, C,
                                              (int32_t)h->host.n_rows, K, epi, s)))
            return PCSR_E_HIP;
    }
    return PCSR_OK;
}

// Makes the handle's own workspace at least `need` bytes.  Allocates, so not for use
// under stream capture.
static int grow_workspace(pcsr_handle_t h, int64_t need)
{
    if (need <= (int64_t)h->ws_bytes) return PCSR_OK;
    if (h->d_ws) {
        // an earlier SpMM may still use the old block
        if (!hip_ok(hipDeviceSynchronize())) return PCSR_E_HIP;
        pcsr::pool_free(h->d_ws);
        h->d_ws = nullptr;
        h->ws_bytes = 0;
    }
    hipError_t e = pcsr::pool_alloc((void **)&h->d_ws, (size_t)need);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        h->d_ws = nullptr;
        return PCSR_E_OOM;
    }
    if (!hip_ok(e)) {
        h->d_ws = nullptr;
        return PCSR_E_HIP;
    }
    h->ws_bytes = (size_t)need;
    return PCSR_OK;
}

int pcsr_spmm(pcsr_handle_t h, const float *B, float *C, int32_t K, void *stream)
{
    pcsr::LaunchShape ls;
    int rc = spmm_check(h, B, C, K, &ls);
    if (rc != PCSR_OK) return rc;
    if (h->host.n_rows == 0) return PCSR_OK;
    rc = grow_workspace(h, workspace_need(h, K));
    if (rc != PCSR_OK) return rc;
    return spmm_enqueue(h, B, C, K, ls, h->d_ws, static_cast<hipStream_t>(stream));
}

int pcsr_spmm_epilogue(pcsr_handle_t h, const float *B, float *C, int32_t K, const pcsr_epilogue_t *epi,
                       void *stream)
{
    if (!epi) return PCSR_E_INVALID_ARG;
    pcsr::LaunchShape ls;
    int rc = spmm_check(h, B, C, K, &ls, true);
    if (rc != PCSR_OK) return rc;
    const uintptr_t align = operand_align(h, ls);
    if (reinterpret_cast<uintptr_t>(epi->self) % align || reinterpret_cast<uintptr_t>(epi->mask) % align)
        return PCSR_E_INVALID_ARG;
    if (h->n_split > 0 && (h->flags & PCSR_FLAG_ATOMIC_SPLIT)) return PCSR_E_UNSUPPORTED;
    if (h->host.n_rows == 0) return PCSR_OK;
    rc = grow_workspace(h, workspace_need(h, K));
    if (rc != PCSR_OK) return rc;
    pcsr::Epilogue e;
    e.on = 1;
    e.relu = epi->relu;
    e.bias = epi->bias;
    e.self = epi->self;
    e.self_eps = epi->self_eps;
    e.mask = epi->mask;
    return spmm_enqueue(h, B, C, K, ls, h->d_ws, static_cast<hipStream_t>(stream), e);
}

int pcsr_spmm_static(pcsr_handle_t h, const float *B, float *C, int32_t K, void *stream)
{
    pcsr::LaunchShape ls;
    int rc = spmm_check(h, B, C, K, &ls);
    if (rc != PCSR_OK) return rc;
    if (h->host.n_rows == 0) return PCSR_OK;
    if (workspace_need(h, K) > (int64_t)pcsr::kStaticScratchBytes) return PCSR_E_TOO_LARGE;
    void *ws = nullptr;
    if (!hip_ok(pcsr::static_scratch(&ws))) return PCSR_E_HIP;
    return spmm_enqueue(h, B, C, K, ls, static_cast<float *>(ws), static_cast<hipStream_t>(stream));
}

int64_t pcsr_static_scratch_bytes(void) { return (int64_t)pcsr::kStaticScratchBytes; }

int pcsr_workspace_bytes(pcsr_handle_t h, int32_t K, int64_t *bytes)
{
    if (!valid(h) || !bytes) return PCSR_E_INVALID_ARG;
    if (K <= 0) return PCSR_E_UNSUPPORTED;
    *bytes = workspace_need(h, K);
    return PCSR_OK;
}

int pcsr_reserve_workspace(pcsr_handle_t h, int32_t K)
{
    if (!valid(h)) return PCSR_E_INVALID_ARG;
    if (h->host_only || K <= 0) return PCSR_E_UNSUPPORTED;
    int dev = -1;
    if (!hip_ok(hipGetDevice(&dev))) return PCSR_E_HIP;
    if (dev != h->device) return PCSR_E_INVALID_ARG;
    return grow_workspace(h, workspace_need(h, K));
}

int pcsr_free(pcsr_handle_t h)
{
    if (!h) return PCSR_OK;
    if (!valid(h)) return PCSR_E_INVALID_ARG;
    release_device(h);
    h->magic = 0;
    delete h;
    return PCSR_OK;
}

int pcsr_release_cached(int64_t *bytes)
{
    size_t n = 0;
    if (!hip_ok(pcsr::pool_give_back(&n))) return PCSR_E_HIP;
    if (bytes) *bytes = (int64_t)n;
    return PCSR_OK;
}

int pcsr_set_kernel_params(pcsr_handle_t h, int32_t lanes_per_row, int32_t vec, int32_t rep,
                           int32_t waves_per_wg, int32_t items_per_group, int32_t flags)
{
    if (!valid(h)) return PCSR_E_INVALID_ARG;
    int rc = check_kernel_params(lanes_per_row, vec, rep, waves_per_wg, items_per_group);
    if (rc != PCSR_OK) return rc;
    h->lpr = lanes_per_row;
    h->vec = vec;
    h->asked_vec = 0;
    h->rep = rep;
    h->waves = waves_per_wg;
    h->ipg = items_per_group;
    constexpr int32_t kLaunchFlags = PCSR_FLAG_NO_XCD_REMAP | PCSR_FLAG_ATOMIC_SPLIT | PCSR_FLAG_FAR_OFFSETS;
    h->flags = (h->flags & ~(kLaunchFlags | kWideBits)) | (flags & kLaunchFlags);
    return PCSR_OK;
}

int pcsr_query_launch(pcsr_handle_t h, int32_t K, int32_t out[8])
{
    if (!valid(h) || !out) return PCSR_E_INVALID_ARG;
    pcsr::LaunchShape ls;
    int rc = resolve_launch(h, K, &ls);
    if (rc != PCSR_OK) return rc;
    out[0] = ls.lpr;
    out[1] = ls.vec;
    out[2] = ls.rep;
    out[3] = ls.waves;
    out[4] = ls.grid_x;
    out[5] = ls.grid_y;
    out[6] = ls.ipg;
    out[7] = ls.lds_bytes;
    return PCSR_OK;
}

int pcsr_query_kernel(pcsr_handle_t h, int32_t K, int32_t out[8])
{
    if (!valid(h) || !out) return PCSR_E_INVALID_ARG;
    pcsr::LaunchShape ls;
    int rc = resolve_launch(h, K, &ls);
    if (rc != PCSR_OK) return rc;
    out[0] = ls.k_lpr;
    out[1] = ls.k_vec;
    out[2] = ls.k_rep;
    out[3] = ls.waves;
    out[4] = ls.k_grid_x;
    out[5] = ls.k_grid_y;
    out[6] = ls.ipg;
    out[7] = ls.lds_bytes;
    return PCSR_OK;
}

int pcsr_window_stats(pcsr_handle_t h, double out[3])
{
    if (!valid(h) || !out) return PCSR_E_INVALID_ARG;
    out[0] = (double)h->host.win_cols;
    out[1] = h->n_win_blocks ? (double)h->host.M / (double)h->n_win_blocks : 0.0;
    out[2] = h->host.win_hit;
    return PCSR_OK;
}

int pcsr_export(pcsr_handle_t h, int64_t sizes[6], int32_t *rowptr, int32_t *colidx, float *val,
                int32_t *trow)
{
    if (!valid(h)) return PCSR_E_INVALID_ARG;
    const pcsr::HostPcsr &m = h->host;
    if (sizes) {
        sizes[0] = m.P;
        sizes[1] = m.M;
        sizes[2] = m.nnz_v;
        sizes[3] = m.V;
        sizes[4] = m.SG;
        sizes[5] = m.S ? 1 : 0;
    }
    auto fetch = [&](void *dst, const void *host_src, const void *dev_src, size_t bytes) -> int {
        if (!dst || bytes == 0) return PCSR_OK;
        if (h->host_only) {
            std::memcpy(dst, host_src, bytes);
            return PCSR_OK;
        }
        return hip_ok(hipMemcpy(dst, dev_src, bytes, hipMemcpyDeviceToHost)) ? PCSR_OK : PCSR_E_HIP;
    };
    int rc = fetch(rowptr, m.rowptr.data(), h->d_rowptr, sizeof(int32_t) * (m.M + 1));
    if (rc == PCSR_OK) rc = fetch(colidx, m.colidx.data(), h->d_colidx, sizeof(int32_t) * m.nnz_v);
    if (rc == PCSR_OK) rc = fetch(val, m.val.data(), h->d_val, sizeof(float) * m.nnz_v * m.V);
    if (rc == PCSR_OK && m.S) rc = fetch(trow, m.trow.data(), h->d_trow, sizeof(int32_t) * m.M);
    return rc;
}

int pcsr_export_schedule(pcsr_handle_t h, int64_t *n_positions, int32_t *sched, int32_t xcd_bounds[9])
{
    if (!valid(h)) return PCSR_E_INVALID_ARG;
    const bool has = h->host_only ? !h->host.sched.empty() : h->d_sched != nullptr;
    if (n_positions) *n_positions = has ? h->host.M : 0;
    if (xcd_bounds)
        for (int x = 0; x < 9; ++x) xcd_bounds[x] = h->host.xcd_bounds[x];
    if (!sched || !has || h->host.M == 0) return PCSR_OK;
    const size_t bytes = sizeof(int32_t) * 4 * (size_t)h->host.M;
    if (h->host_only) {
        std::memcpy(sched, h->host.sched.data(), bytes);
        return PCSR_OK;
    }
    return hip_ok(hipMemcpy(sched, h->d_sched, bytes, hipMemcpyDeviceToHost)) ? PCSR_OK : PCSR_E_HIP;
}

int pcsr_features(int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t *rowptr,
                  const int32_t *colidx, int32_t omega, double *out, int32_t n_out)
{
    if (!out || n_out < PCSR_N_FEATURES || !rowptr || omega < 0) return PCSR_E_INVALID_ARG;
    int rc = pcsr::validate_csr(n_rows, n_cols, nnz, rowptr, colidx);
    if (rc != PCSR_OK) return rc;
    try {
        return pcsr::features_host(n_rows, n_cols, nnz, rowptr, colidx, omega, out);
    } catch (const std::bad_alloc &) {
        return PCSR_E_OOM;
    }
}

int pcsr_features_device(int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t *rowptr,
                         const int32_t *colidx, int32_t omega, double *out, int32_t n_out)
{
    if (!out || n_out < PCSR_N_FEATURES || !rowptr || omega < 0 || n_rows < 0 || n_cols < 0 || nnz < 0)
        return PCSR_E_INVALID_ARG;
    if (nnz > 0 && !colidx) return PCSR_E_INVALID_ARG;
    if (nnz >= (int64_t(1) << 31) || n_rows >= (int64_t(1) << 31) - 1) return PCSR_E_TOO_LARGE;
    int herr = 0;
    int rc = pcsr::features_device(n_rows, n_cols, nnz, rowptr, colidx, omega, out, &herr);
    if (rc == PCSR_E_HIP) g_last_hip = herr;
    return rc;
}

int pcsr_select(const double *f, int32_t K, pcsr_params_t *out)
{
    if (!f || !out) return PCSR_E_INVALID_ARG;
    if (K <= 0) return PCSR_E_UNSUPPORTED;
    pcsr_params_t p;
    std::memset(&p, 0, sizeof(p));
    const double d_hat = f[5], d_max = f[6], cv = f[7], pr2 = f[15];

    // Balancing (Section 3.2) pays when a few rows dwarf the average one.  On MI355X the
    // recorded sweeps then prefer short items (32 or 64 vectors, see SG below) run in column
    // order: the items of the long rows, sorted by first column, make the wavefronts of an XCD gather the same B
    // rows at about the same time (R-MAT scale 22: 1.6-2x over the best index-order tuple at
    // every width from 16 to 512; neutral on small or uniform inputs).
    const bool skewed = cv > 1.5 && d_max > 256.0;
    // Loads per lane: the widest vector that divides K, except where fewer rows per
    // wavefront pay more than wide loads.  A wavefront runs until the longest of its work
    // items ends, so with rows of varying length every further item per wavefront costs
    // lane time.  K of 9..16: one dword per lane, 16 lanes per row (4 items per wavefront
    // instead of 16: 11-18 % faster on every input but road-like ones, whose rows of 3 want
    // many rows per wavefront).
    int vec = K % 4 == 0 ? 4 : (K % 2 == 0 ? 2 : 1);
    if (K > 8 && K <= 16 && d_hat >= 8.0) vec = 1;
    const double n = f[0];
    const bool scattered = scattered_columns(f); // (see below)
    // Up to 8 the same (narrow_lanes); of scattered rows from 8 on, which wait on memory (1,000,000 rows of 9, K = 8: 160 -> 150
    // us).  Odd widths had one dword a lane before: local rows of 15 0.95-1.05, one column of 9 to 21 a row 1.16-1.30.
    // Two to four columns of under 12 that L2 holds but L1 does not: their wide loads are faster (300,000 rows of 8.5, K = 2 17.5 us
    // and 20.9, K = 3 20.7 and 22.6; 1.02-1.20 from 1.7 MB, 1.1 of three columns, up to 5, 0.94-1.01 from there on; rows of 10
    // 0.97-1.09, of 12 0.84-1.02; four columns 1.03-1.04, but 0.99 with 9 a row).  Five 1.02-1.10, but a dword in 8 lanes has sums of
    // 8 there: rms 4.44e-8 of the sum for 4.04.
    const double b_few = n * (double)K * 4.0;
    const bool few = K >= 2 && K <= 4 && b_few > (K == 3 ? 1.1e6 : 1.7e6) && b_few < 5e6;
    const double least_few = !few ? 8.0 : K == 4 ? 8.8 : 11.5;
    const double least_narrow = K == 1 ? 32.0 : scattered && !skewed ? least_few : K % 2 ? 20.0 : 16.0;
    const bool narrow = K <= 8 && d_hat >= least_narrow && !(skewed && K % 2);
    if (narrow) vec = 1;
    // Rows that gather from a neighbourhood of their own index are served from LDS instead
    // (see the column window below), from K = 64 (at 32 it ties with the plain kernel) and if
    // the product is large enough to give every compute unit a few window blocks: a block
    // occupies a whole compute unit, and with too few rounds of blocks the last one leaves
    // most of the chip idle (90,000 rows in communities of 300: 0.55x of the plain kernel
    // at K = 32, 0.81x at K = 128; 200,000 rows at K = 64: 1.1x).
    // Rows that share most columns with their neighbour (padding below 30 %) do better
    // paired, V = 2, than from LDS (cliques of 48, K = 128: 0.98 against 0.82 of the best).
    const bool windowed = !skewed && f[16] >= 0.6 && d_hat >= 40.0 && vec == 4 && pr2 >= 0.3 && K >= 64 &&
                          n * (double)((K + 63) / 64) >= 200000.0;
    // Uniformly long rows with scattered columns (mean length 40 or more, no more nonzeros near the diagonal than four times what
    // uniform columns would put there).  From K = 64 the same column-ordered schedule, with items of 32, turns the split into a
    // column partition of A, each XCD gathering from its own range of B rows (uniform random columns, 96 per row, K = 128: 1.5x; 48
    // per row, K = 256: 1.13x; at 32 per row the second items are too short and it loses 15 %).  Narrower rows of B are walked in
    // bands of columns, or paired (below).  Rows with local columns lose up to half their speed under the column order (it gives up
    // the reuse between neighbouring rows).  Such rows walked in bands of columns: where one product saves what the handle's table
    // of them costs its build (300,000 rows of 134: 183 -> 263 us, 60,000 of 140: 78 -> 99, 1,000,000 of 44: 187 -> 336), or where
    // the other choice is the far dearer build of pairs.
    const int band_lanes = K <= 16 || (K > 32 && K <= 64) || (K > 64 && K % 32 == 0) ? 16 : K <= 128 ? 32 : 64;
    const int band_tile = K <= 32 ? band_lanes : 4 * band_lanes;
    double saved = 0.0;
    const bool fills_paired = n * (double)(K < 32 ? 4 : 8) / 128.0 >= 3500.0;
    const bool paired_else =
        d_hat >= 40.0 && fills_paired && K > 16 && K < 64 && (K > 32 || n * (double)K * 4.0 <= 16.0 * 1048576.0);
    const bool banded = !skewed && !windowed && scattered && d_hat >= 12.0 && K > 2 &&
                        band_count(n, n, f[2], K, band_lanes, band_tile, &saved) > 1 &&
                        (paired_else || saved > 12.0 + 1e-6 * f[2] + 1e-4 * n);
    // K of 17..32 with scattered columns: one dword per lane again, a row per half wavefront (uniform random columns, 16 to 64 per
    // row, 150,000 rows or more: 7-24 % faster than the best 16-byte shape; slower when the columns are local.  In bands: 300,000
    // rows of 134, K = 32: 527 us, 8 lanes of 16 bytes 580.  A B of less than 16 MB: over 8 lanes of 16 bytes and 16 of two dwords
    // 0.73-0.98, rows of 14 to 140, 4,000 to 200,000 of them, but 1.03 with 13 a row and K = 17).  Rows that are paired otherwise
    // stay so.
    const bool wide_scatter = !skewed && scattered && d_hat >= 12.0 && K > 16 && K <= 32 &&
                              (banded || n * (double)K * 4.0 > 16.0 * 1048576.0 ||
                               ((d_hat < 40.0 || !fills_paired) && (d_hat >= 16.0 || K % 4 == 0)));
    if (wide_scatter) vec = 1;
    const bool long_uniform = !skewed && !windowed && !wide_scatter && d_hat >= 40.0 && scattered;
    // But not where a slice of B is over 20 MB, 2.5 times what the L2s hold together: the order then saves less than the parts'
    // sums cost, and unsplit rows, in bands or not, take 0.77-0.95 of the time (rows of 44 to 300, 100,000 to 1,000,000 of them, K
    // = 64 to 256; rows of 90, 100,000 of them, K = 128: 485 -> 350 us, of 44, 1,000,000: 3937 -> 3087; slices of 15 MB 0.92-1.10,
    // of 10 MB 0.95-1.15).  Rows over kClusterItem stay split, as communities among them would have to be, and so do widths over 256
    // that are no multiple of 32, whose tile no band kernel has.
    const bool split_pays =
        n * 4.0 * std::min(K, band_tile) <= 20e6 || d_max > pcsr::kClusterItem || (K > 256 && K % 32 != 0);
    const bool long_uniform_wide = long_uniform && K >= 64 && split_pays;
    p.S = (skewed || long_uniform_wide) ? 1 : 0;
    // Items of 32 vectors where uniform rows are split (of 64: 2-31 % slower on rows of 70 and more,
    // 9-12 % faster on uniform rows of 48).  Of 64 for power-law
    // inputs, at half the workspace, with two exceptions.  Small products end with few items in
    // flight: R-MAT graphs of under 15 M nonzeros (2^16 to 2^20 nodes, 8 to 60 per row) are 0-13 % faster
    // with items of 32 up to K = 48, on a par or slower from K = 64; from 15 M on items of 64 are 1-15 % faster from
    // K = 32 (below, between 7 % slower and 7 % faster).  And where a B of 1 GB or more is gathered in
    // an order that has its hubs side by side (natural R-MAT ids, scale 22 from K = 64) items of 32
    // are 1-5 % faster.
    const bool short_items = !skewed || (f[2] < 15e6 && K <= 48) || (!scattered && K >= 64 && n * (double)K * 4.0 >= 1e9);
    p.SG = p.S ? (short_items ? 32 : 64) : 0;
    p.omega = 64;
    if (p.S) p.flags |= PCSR_FLAG_COLUMN_ORDER;
    // Vector size 2 (Section 3.1) when adjacent rows share columns, and for short rows, where
    // pairing rows doubles the gathers a lane group keeps in flight.  The paper's A6000 data
    // puts the break-even near 30 % padding; on MI355X clique-like inputs win at 11 %
    // padding (1.23x at K=128) and lose at 27 %, because adjacent rows of one wavefront
    // already share their B lines in L1.  Power-law inputs: V = 2 ties or loses in the sweeps.
    // Long scattered rows of a B that needs no bands: paired as well below K = 64, which doubles the gathers a lane group has in
    // flight, unless the matrix is so small that halving the number of work items leaves wavefront slots empty (30,000 rows of
    // 160, K = 32: V = 2 runs at 0.55 of V = 1), and not up to K = 16 or with a B beyond 16 MB: there V = 2 takes 0.98-1.18 of the time
    // and 5 to 9 times the build (1,000,000 rows of 44, K = 48: 1649 us for 1534, 1646 to build for 187).
    const bool pairs = long_uniform && K < 64 && fills_paired;
    const bool pair_long = pairs && !banded && K > 16 && n * (double)K * 4.0 <= 16.0 * 1048576.0;
    // Rows of C of 48 or 64 bytes are written one by one by a pair's lanes, part lines each, where single rows' lane groups
    // fill lines together: V = 1 takes 0.59-0.99 of V = 2 (with a self term 0.50-1.03, and a mask 0.58-0.99) on road-like graphs of 2 to 7
    // a row and uniform ones of 3 to 6, 300,000 and 2,000,000 rows.  C below 8 MB (120,000 rows) 0.85-1.01, products of under 10 us.
    // A handle has one V, so an operator made for these widths runs its others so too: training with hidden 12 and 16 and 8, 16 or 32
    // features takes 0.80-1.02 of V = 2 on graphs of 3 to 7 a row (but 1.05 in a GCN of two layers from 8 features on 2,000,000 rows of 3).
    // Its plain products of 8 columns 0.81-1.15, of 20 to 32 0.87-1.30, the slowest where rows are local: which is why those
    // widths stay paired where they are what the handle is made for.
    const bool part_lines = K > 8 && K <= 16 && K % 4 == 0 && d_hat < 8.0 && pr2 >= 0.20 && n * (double)K * 4.0 >= 8e6;
    p.V = (!p.S && !part_lines && (d_hat < 6.0 || (d_hat < 12.0 && pr2 < 0.45) || pr2 < 0.20 || pair_long)) ? 2 : 1;

    // Scattered rows may belong to communities whose ids were shuffled.  Looking for them and ordering the schedule by
    // them costs the build some 0.15 ms and 0.6 ns a row; run side by side the rows of a community gather from L2 and the
    // product takes 0.3 ps per nonzero and column less (250,000 rows of 48: K = 64 377 -> 145 us, K = 128
    // 747 -> 262, K = 256 1485 -> 578; rows of 12, K = 256: 919 -> 508).  Asked for where one product pays for it, and not
    // where it would split a row of a handle that is not split otherwise: products on that one need no workspace, so
    // the first of all may be captured in a graph.
    if (!skewed && !windowed && scattered && p.V == 1 && (p.S || d_max <= pcsr::kClusterItem) && d_hat >= 12.0 &&
        3e-7 * f[2] * (double)K >= 150.0 + 6e-4 * n)
        p.flags |= PCSR_FLAG_CLUSTER_IF_USEFUL;
    // And, for wide rows, windows of those communities in LDS (cluster_windows): 0.1 ms and 0.25 ns a row of build for
    // 0.06 ps per nonzero and column (250,000 rows of 48 in communities of 500: K = 256 577 -> 378 us, build 414 -> 586;
    // of 30: 379 -> 279, 382 -> 525; 500,000 of 24: K = 512 1550 -> 1150, 529 -> 726).  Fewer vectors a row do not
    // pay for the staging (250,000 rows of 14: 205 -> 225).  Where one product pays for it, too.
    if ((p.flags & PCSR_FLAG_CLUSTER_IF_USEFUL) && d_hat >= 22.0 && K >= 192 && K % 4 == 0 &&
        6e-8 * f[2] * (double)K >= 100.0 + 2.5e-4 * n)
        p.flags |= PCSR_FLAG_CLUSTER_WINDOWS;

    // Launch shape: the widest vector load that divides K, one lane group spanning the
    // whole row of C when it fits a wavefront, repeats beyond that.
    // Balanced power-law inputs do best without repeats and, once B outgrows the 256 MB
    // memory-side cache, with 64-column slices (four items per wavefront; grid.y covers
    // wider rows), which shrinks the bytes a cached B row occupies; a smaller B is gathered
    // in 128-column slices.
    const double b_bytes = f[0] * (double)K * 4.0;
    const int lpr_cap = p.S ? ((long_uniform_wide || b_bytes > 192.0 * 1048576.0) ? 16 : 32) : 64;
    int lpr = 4;
    while (lpr * vec < K && lpr < lpr_cap) lpr <<= 1;
    int rep = 1;
    while (!p.S && lpr * vec * rep < K && rep < 4) rep <<= 1;
    if (!p.S && p.V == 1 && d_hat < 8.0 && lpr >= 32 && rep == 1) {
        lpr >>= 1; // short rows: more rows per wavefront, two loads per lane
        rep = 2;
    }
    // Scattered columns, rows of 8 to 40, K from 64: a 64-column slice per half wavefront
    // with dwordx2 loads (uniform random columns, 8 to 32 per row, K = 64 and 128: 3-7 %
    // over the best 16-byte shape; local columns keep the 16-byte shapes).
    // But 16 bytes a lane where B is so small that L2 holds it: K = 128 and 192, 2 to 16 MB 0.79-0.98 (8,000 rows of 22, K = 128 9.9 us
    // and 7.8; 25 MB and more 0.99-1.08), and in bands.  That shape only stands in (below): the handle takes every even width and
    // operands at 8-byte addresses.
    bool quads = false;
    if (!skewed && !windowed && !p.S && (!banded || d_hat < 40.0) && scattered && d_hat >= 8.0 && K >= 64 && K % 2 == 0) {
        const bool in_l2 = b_bytes > 2e6 && b_bytes < 16e6 && K >= 96;
        lpr = 32;
        vec = 2;
        rep = 1;
        quads = (in_l2 || banded) && K % 32 == 0;
    }
    // Single long rows of 33 to 64 columns: a dword a lane and two columns of it, as resolve_launch has it for auto shapes; and
    // scattered ones of 12 and more, K = 64, that L2 holds: 0.77-0.95 of 32 lanes of two floats (20,000 rows of 34 15.7 us and
    // 12.4; at 13 MB 0.98-1.00).
    if (!p.S && p.V == 1 && !windowed && !banded && K > 32 && K <= 64 && K % 4 == 0 &&
        (scattered ? K == 64 && d_hat >= 12.0 && b_bytes < 10e6 : d_hat >= 32.0)) {
        lpr = 32;
        vec = 1;
        rep = 2;
    }
    if (narrow) {
        lpr = narrow_lanes(p.S);
        rep = 1;
    }
    if (banded && K >= 64 && (d_hat >= 40.0 || K % 2)) { // (300,000 rows of 134 in bands, K = 128: 2212 us, halves of two floats 2342)
        lpr = 16;
        rep = 1;
    }
    // K of 17..32, rows of 32 and more that are neither split nor paired: 16 lanes of one
    // dword, two loads per lane (4 items per wavefront instead of 8): 9-19 % faster than
    // 8 lanes x dwordx4 on the community and clique inputs of the validation sets; rows
    // of 20-27 and road-like inputs keep the 16-byte shape.
    if (!p.S && !wide_scatter && !pair_long && d_hat >= 32.0 && K > 16 && K <= 32) {
        lpr = 16;
        vec = 1;
        rep = 2;
    }
    p.lanes_per_row = lpr;
    p.vec = vec;
    p.rep = rep;
    // Shape to launch in its place (see resolve_launch).  All figures: uniform columns, 12 to 136
    // per row, R-MAT scale 20, a shuffled community graph.
    int wide = 0, wide_rep = 1;
    bool pair = false, beyond = false;
    const bool dword = wide_scatter || (lpr == 16 && vec == 1 && rep == 2 && K <= 32);
    if (K > 64 && K % 32 != 0 && (p.S || scattered || K % 4 != 0)) {
        // one tile for the whole row instead of slices of 64: 1.06-1.36x (0.96x on rows of 96, K = 300)
        wide_shape(K, 64, &wide, &wide_rep);
    } else if (K > 32 && K <= 64 && K % 32 != 0 && !p.S && !banded && scattered && d_hat >= 8.0 && b_bytes > 24.0 * 1048576.0) {
        // half a wavefront per scattered row: 0-6 % where B is gathered from the memory side, 20-30 %
        // slower where L2 holds it (uniform columns, 9 to 200 per row; on a par at 20-25 MB)
        wide = 32;
    } else if (K % 4 != 0 && K > 16 && !dword) {
        // 16 lanes of two floats for K up to 32 unless rows are short: 8 % on clique inputs
        pair = K <= 32 && !p.S && d_hat >= 8.0;
        wide_shape(K, lpr_cap, &wide, &wide_rep);
        if (pair) wide = 16;
    } else if (quads) {
        wide = 16;
    } else if (narrow && p.S && K % 4 == 0) {
        // Items of 8 lanes of a dword are for up to 8 columns: others as 4 lanes of 16 bytes (R-MAT 2^20, a handle for K = 8: K = 16 337 us
        // and 238, K = 64 1423 and 960, K = 256 6153 and 3834).
        wide = 4;
        beyond = true;
    } else if (wide_scatter && !banded && d_hat < 32.0 && b_bytes <= 16.0 * 1048576.0) {
        // and a dword a lane of rows in L2 for up to 32 (20,000 rows of 22, a handle for K = 24: K = 192 29.0 us and 27.1, K = 256
        // 36.3 and 33.4)
        wide = K % 4 == 0 ? 8 : 16;
        pair = K % 4 != 0;
        beyond = true;
    }
    // Rows that are not split for K = 64 and more: few columns of them are best left to the library (150,000 rows of 60, a handle
    // for K = 64: K = 4, 8, 16 and 24 146, 144, 170 and 187 us in its shape, 91, 91, 99 and 168 when its rows were split, 50, 60,
    // 77 and 127 in auto shapes).
    // So are those of rows of 8 to 40 whose shape only stands in (20,000 rows of 22, a handle for K = 128, K = 16 11.0 us in halves of
    // two floats, 7.6 in 16 lanes of 16 bytes, 6.6 in auto shapes).
    const bool auto_narrow = quads || (long_uniform && K >= 64 && !p.S && p.V == 1);
    if (auto_narrow) p.flags |= kAutoNarrow | stands_for(lpr, vec, rep);
    if (wide) {
        int code = 1;
        while (4 << code >> 1 < wide) ++code;
        p.flags |= code << kWideShift | (pair ? kWidePair : 0) | (wide_rep == 2 ? kWideTwice : 0) | (beyond ? kWideBeyond : 0) | stands_for(lpr, vec, rep);
    }
    // Workgroup size: four wavefronts, two for short rows and for paired long rows (eight
    // were 4-7 % slower than four on every unsplit input of the later validation sets).
    p.waves_per_wg = p.S ? 4 : (d_hat >= 16.0 && !pair_long ? 4 : 2);
    p.items_per_group = 1;
    p.col_window = 0;
    // (Also where long rows are neither split nor paired but in one band: for its sums.)
    if ((banded || (pairs && !pair_long) || (long_uniform && K >= 64)) && p.V == 1 && !p.S) p.flags |= PCSR_FLAG_COLUMN_BANDS;
    // Column-window blocking: rows that gather from a neighbourhood of their own index (most
    // nonzeros within 512 columns of the diagonal) and are long enough that every staged row
    // of B is used dozens of times.  A 500-node community graph of degree 48 runs 1.1x
    // (K = 64) to 1.4x (K = 512) faster from LDS than from L2; cliques of 25 or blocks of 50
    // nodes do not repay the staging.  The build drops the window again if the blocks it
    // finds are poor.
    if (windowed) {
        p.V = 1;
        p.col_window = 512;
        p.flags |= PCSR_FLAG_WINDOW_IF_USEFUL;
        p.lanes_per_row = 16; // 64-column slices of the window (136 KiB of LDS)
        p.rep = 1;
        p.waves_per_wg = 16;
    }
    *out = p;
    return PCSR_OK;
}

int32_t pcsr_mac_job_gap(int32_t dim, int32_t F, int32_t omega)
{
    if (dim <= 0 || F <= 0 || omega <= 0) return -1;
    const int64_t span = (int64_t)F * omega;
    const int64_t tn = dim < span ? dim : span;
    const int64_t tr = dim % span;
    return tr == 0 ? 0 : (int32_t)(tn - tr);
}

const char *pcsr_strerror(int code)
{
    switch (code) {
    case PCSR_OK: return "ok";
    case PCSR_E_INVALID_ARG: return "invalid argument";
    case PCSR_E_BAD_CSR: return "malformed CSR (rowptr not monotone, column out of range, unsorted or duplicate columns)";
    case PCSR_E_UNSUPPORTED: return "unsupported parameter value";
    case PCSR_E_TOO_LARGE: return "size does not fit 32-bit indexing, or the fixed workspace";
    case PCSR_E_OOM: return "out of memory";
    case PCSR_E_HIP: return "HIP runtime error";
    }
    return "unknown error";
}

int pcsr_last_hip_error(void) { return g_last_hip; }

} // extern "C"
