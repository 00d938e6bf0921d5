// Dense side of a GNN layer (internal to the package: gnn.py calls these through ctypes).
// The layers around an SpMM are tall and narrow - n rows of tens of features against a weight
// matrix of a few kilobytes - so every product is bound by reading and writing the n-row
// arrays, and what belongs to one of them (bias, ReLU, its backward mask, column sums) is done
// in the same pass.  All fp32, products on the fp32 matrix instructions.
#pragma once
#include <cstdint>

#include "../../include/pcsr.h"

// widest side of a weight matrix the kernels take
#define PCSR_GNN_MAX_WIDTH 128

extern "C" {

// What the SpMM's write-back does to each element before it is stored:
//   v = acc + bias[k] + (1 + *self_eps) * self[row][k];  relu: v = max(v, 0);
//   mask: v = 0 where mask[row][k] <= 0.     Any pointer may be null.
typedef struct {
    const float *bias;     // K
    const float *self;     // n_rows x K
    const float *self_eps; // one fp32 in device memory (null: 0)
    const float *mask;     // n_rows x K
    int32_t relu;
    int32_t reserved;
} pcsr_epilogue_t;

// pcsr_spmm with an epilogue.  UNSUPPORTED with PCSR_FLAG_ATOMIC_SPLIT on a handle that has
// split panels (its partial sums meet in C).
int pcsr_spmm_epilogue(pcsr_handle_t h, const float *B, float *C, int32_t K, const pcsr_epilogue_t *epi,
                       void *stream);

// Both directions of a matrix, set up in device memory from one upload (or from arrays there
// already: PCSR_FLAG_DEVICE_CSR in p->flags): the CSR is checked, each direction gets the
// parameters pcsr_select picks for width K with the launch shape left on auto, or the caller's
// (reserved[0] = 0), and is built.  out[0]: A, out[1]: its transpose (with_transpose, else null).
// p may be null.  Errors as pcsr_build.
enum { PCSR_OPERATOR_SELECT = 1 }; // in p->reserved[0]: p only carries flags
int pcsr_operator_build(int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t *rowptr, const int32_t *colidx,
                        const float *vals, const pcsr_params_t *p, int32_t K, int32_t with_transpose,
                        pcsr_handle_t out[2]);

// Floats of workspace a call below needs for weights of b x a.
int64_t pcsr_gnn_workspace_floats(int32_t a, int32_t b);

// Y[n x b] = X[n x a] * op(W) with W[b x a] (op: transpose) or, w_transposed = 1, W[a x b];
// then v += bias; relu; dot_out += sum(v * dot_aux); mask as above; colsum_out = column sums of Y.
// Y may be null (only dot_out wanted).  Widths up to PCSR_GNN_MAX_WIDTH.
int pcsr_gnn_linear(int64_t n, int32_t a, int32_t b, const float *X, const float *W, int32_t w_transposed,
                    const float *bias, int32_t relu, const float *mask, const float *dot_aux, float *Y,
                    float *colsum_out, float *dot_out, float *ws, void *stream);

// The two layers of a GIN layer in one pass: Z[n x m] = relu(X[n x a] W1^T + b1), Y[n x m] =
// Z W2^T + b2, ReLU if asked.  UNSUPPORTED unless both widths are 16, 32, 48 or 64 and the arrays
// 16-byte aligned; the calls above do the same then.
int pcsr_gnn_mlp(int64_t n, int32_t a, int32_t m, const float *X, const float *W1, const float *b1, const float *W2,
                 const float *b2, int32_t relu, float *Z, float *Y, void *stream);

// Its backward from G = dL/dY: dW2 = G^T Z, db2, G1 = (G W2) where Z > 0, dW1 = G1^T A, db1, dA =
// G1 W1 (may be null), dot = sum(dA * H) (may be null).  Same widths.
int pcsr_gnn_mlp_backward(int64_t n, int32_t a, int32_t m, const float *G, const float *Z, const float *A,
                          const float *H, const float *W1, const float *W2, float *dA, float *dW1, float *db1,
                          float *dW2, float *db2, float *dot, float *ws, void *stream);

// Backward of Y = X W^T, W[b x a], from G = dL/dY: dW = G^T X, dX = G W (where X > 0 if masked; may be
// null), db and colsum = column sums of G and of dX (may be null).  Same widths.
int pcsr_gnn_linear_backward(int64_t n, int32_t a, int32_t b, const float *G, const float *X, const float *W,
                             int32_t masked, float *dX, float *dW, float *db, float *colsum, float *ws,
                             void *stream);

// dW[b x a] = G^T X, db[b] = column sums of G (db may be null) for G[n x b], X[n x a].
int pcsr_gnn_wgrad(int64_t n, int32_t a, int32_t b, const float *G, const float *X, float *dW, float *db,
                   float *ws, void *stream);

// out[b] = column sums of G[n x b].
int pcsr_gnn_colsum(int64_t n, int32_t b, const float *G, float *out, float *ws, void *stream);
}
