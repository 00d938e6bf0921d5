// PCSR generation on the GPU (internal to the library).
#pragma once
#include <cstdint>

#include "pcsr_kernels.h"
#include "pcsr_pool.h"

namespace pcsr {

// Device arrays produced by build_device; ownership passes to the caller (pool_free).
struct DeviceBuild {
    int32_t *rowptr = nullptr; // M+1
    int32_t *colidx = nullptr; // nnz_v
    float *val = nullptr;      // nnz_v * V
    int32_t *trow = nullptr;   // M (S only)
    int32_t *split = nullptr;  // panels with more than one item (S only), ascending, n_split entries
    int32_t *item_slot = nullptr;   // per item (S only): workspace slot, -1 for a sole item
    int32_t *split_slot = nullptr;  // first workspace slot of each of them, n_split + 1 entries
    int32_t *long_list = nullptr;   // positions in split of the panels with more than kLongPanelSlots items
    int32_t *sched = nullptr;       // column-ordered schedule, 4 int32 per launch position (or null)
    int64_t P = 0, M = 0, nnz_v = 0, n_split = 0, n_split_items = 0, n_long = 0, max_item_len = 0;
    int32_t S = 0, SG = 0;
    bool vals_due = false;  // val is still to be filled, once `late` is there
    int32_t *bands = nullptr; // band_ends of the rows (or null), kColumnBands - 1 of them one after the other
    bool clustered = false; // the schedule runs the rows community by community
    bool dropped = false;   // something that the product can do without did not fit in memory
    struct {                // the arrays of a product with windows of communities (blocks 0: none)
        int32_t *rowptr = nullptr, *colidx = nullptr, *rows = nullptr, *ptr = nullptr, *hi = nullptr;
        float *val = nullptr;
        int64_t blocks = 0;
    } win;
    int32_t xcd_bounds[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
};

// late: the copy that fills d_vals, if it is still under way (null: it is not).  With V = 1 nothing but val needs the
// values: the call then leaves that to the caller (vals_due); else it waits.
// d_rowptr / d_colidx / d_vals are device pointers.  Returns PCSR_OK or a PCSR_E_* code;
// on PCSR_E_HIP *hip_err holds the hipError_t.  Synchronous.
// known: what the check counts, of arrays that have been checked (null: they are checked if `validate`, and counted).
// clusters: where the rows turn out to form communities, S = 1 with items of kClusterItem and the schedule by community;
// windows: and, where they fit in LDS, out->win beside it.
// bands: S = 0 and V = 1, where it stays so: out->bands, if there is memory for it.
constexpr int kColumnBands = 12;
constexpr int32_t kClusterItem = 1024;
struct RowStats {
    int64_t longest, nonempty;
};
int build_device(int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t *d_rowptr,
                 const int32_t *d_colidx, const float *d_vals, int32_t V, int32_t S, int32_t SG,
                 int32_t omega, bool validate, bool column_order, bool clusters, bool windows, bool bands, const RowStats *known, Late *late,
                 DeviceBuild *out, int *hip_err);

// Whether rows share more columns than chance has them: enqueues the count of a sample on the null stream (d_out: two
// sums, zeros on entry), and what the sums say.  The arrays need not have been checked.
hipError_t cluster_probe(int64_t n, int64_t nnz, const int32_t *d_rowptr, const int32_t *d_colidx, unsigned long long *d_out);
bool cluster_probe_says(const unsigned long long found[2], int64_t n);
// A label in [0, n) for every row of a checked square CSR, rows of a community having the same one; null where too few do for
// an order by label to pay.  Ownership passes to the caller.  The same labels on every run.  *mean_size: of the label that
// a row has.  Synchronous.
int cluster_rows(int64_t n, const int32_t *d_rowptr, const int32_t *d_colidx, int32_t **labels, double *mean_size, int *hip_err);
// Keys of cluster_key_bits(n) bits by which items sort into the order of their rows' labels (enqueued on the null stream).
int cluster_key_bits(int64_t n);
hipError_t cluster_keys(int64_t n, const int32_t *d_labels, int64_t n_items, const int32_t *d_items, const int32_t *d_rows,
                        uint32_t *d_key);

// out->win of a square CSR whose rows have these labels: rows sorted by label, cut into blocks of communities, each row's
// vectors partitioned.  Nothing where too few vectors lie inside the blocks.  Synchronous.
int cluster_windows(int64_t n, int64_t nnz, const int32_t *d_rowptr, const int32_t *d_colidx, const float *d_vals,
                    const int32_t *d_labels, DeviceBuild *out, int *hip_err);

// Enqueues: `words` words from device memory to pinned host memory, then seq to *flag there.
hipError_t deliver(void *to, const void *from, int words, unsigned *flag, unsigned seq, hipStream_t stream);

// The check build_device makes, alone: PCSR_OK or PCSR_E_BAD_CSR (or HIP, OOM).  Synchronous.
int validate_device(int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t *d_rowptr, const int32_t *d_colidx,
                    int *hip_err);

// Table 3 features (order as in pcsr.h) from CSR arrays in device memory.  The CSR is
// assumed valid (pcsr_build validates).  Synchronous.
int features_device(int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t *d_rowptr,
                    const int32_t *d_colidx, int32_t omega, double *out, int *hip_err);

// Window blocks of S = 0 arrays in device memory, the same ones choose_windows picks.
// UNSUPPORTED where a stretch of items has more vectors than a workgroup can sort (the caller
// then takes the host builder).  Ownership of the arrays passes to the caller.  Synchronous.
struct DeviceWindows {
    int32_t *ptr = nullptr, *start = nullptr, *lo = nullptr, *hi = nullptr;
    int64_t blocks = 0, hits = 0;
};
int windows_device(int64_t M, int64_t n_cols, int32_t win, const int32_t *d_rowptr, const int32_t *d_colidx,
                   DeviceWindows *out, int *hip_err);

// CSR of the transpose from CSR arrays in device memory, as pcsr_transpose_csr gives it; the
// outputs (n_cols + 1, nnz, nnz) are allocated here, ownership passes to the caller.  Synchronous.
// d_vals null (only where transpose_in_two_passes says so): *t_vals gets the bits of the place that each value has in the
// array to come, and turned_values puts the values there, in the same place.
hipError_t turned_values(int64_t nnz, const float *d_vals, float *t_vals); // enqueued on setup_stream()
int transpose_device(int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t *d_rowptr, const int32_t *d_colidx,
                     const float *d_vals, int32_t **t_rowptr, int32_t **t_colidx, float **t_vals, int *hip_err);

} // namespace pcsr
