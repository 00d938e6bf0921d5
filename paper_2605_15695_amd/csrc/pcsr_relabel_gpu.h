// GPU side of the relabelling pre-step and the transpose (internal to the library).  Results are
// those of the host code in pcsr_reorder.cpp, bit for bit.
#pragma once
#include <cstdint>

namespace pcsr {

// Whether a GPU is there and `nnz` is enough for it to be the faster side.
bool relabel_on_gpu(int64_t nnz);

// Returned where the host code has to decide: arrays it would treat in a way of its own (row
// pointer not monotone, columns out of range or repeated), or the GPU cannot (memory).
constexpr int kUseHost = 1;

// pcsr_reorder / pcsr_permute_csr on host arrays.  PCSR_OK or kUseHost; outputs are only
// written with PCSR_OK.
int reorder_gpu(int64_t n, const int32_t *rowptr, const int32_t *colidx, int32_t max_rounds, int32_t *perm,
                int64_t *n_clusters);
int permute_gpu(int64_t n, const int32_t *rowptr, const int32_t *colidx, const float *vals, const int32_t *perm,
                int32_t *out_rowptr, int32_t *out_colidx, float *out_vals);
int transpose_gpu(int64_t n_rows, int64_t n_cols, const int32_t *rowptr, const int32_t *colidx, const float *vals,
                  int32_t *out_rowptr, int32_t *out_colidx, float *out_vals);
int degree_order_gpu(int64_t n, const int32_t *rowptr, const int32_t *colidx, int32_t *perm);

// transpose_device for matrices that it takes (bits of a column, of a row, enough nonzeros): outputs in device memory.
bool transpose_in_two_passes(int64_t n_rows, int64_t n_cols, int64_t nnz);
int transpose_two_passes(int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t *d_rowptr, const int32_t *d_colidx,
                         const float *d_vals, int32_t *t_rowptr, int32_t *t_colidx, float *t_vals, int *hip_err);

} // namespace pcsr
