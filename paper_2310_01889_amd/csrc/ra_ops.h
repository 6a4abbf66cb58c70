// Internal host-side building blocks shared by the C-ABI translation units.
#pragma once

#include <hip/hip_runtime.h>

#include "ra_gemm.h"

namespace ra {

// Validation of a row-blocked product [T, d_in] x [d_in, d_out]; sets the error text.
int check_gemm_dims(int T, int d_in, int d_out, int block);
// One GEMM launch (timed when kernel timing is enabled); RA_OK or an ra_status.
int gemm(const GemmArgs& g, bool ta, bool tb, int epi, hipStream_t st);

// A product C [M, N] = A B (K deep) with the leading dimensions of its operands.
GemmArgs gemm_args(const void* A, long long lda, const void* B, long long ldb, void* C, long long ldc, int M, int N,
                   int K);

// Row-wise products of bf16 operands (x [T, din], dy and y [T, dout], w [din, dout]).  They have
// no intermediate, so all row blocks go in one launch:
//   proj:  y (bf16) = x w (+ residual)       dgrad: dx (bf16) = dy w^T
//   wgrad: dw (f32, overwritten) = x^T dy, the sums of blocks of `block` rows added up (n of
//          them with one x: n <= 3)
int proj(const void* x, const void* w, const void* residual, void* y, int T, int din, int dout, hipStream_t st);
int proj3(const void* x, const void* const* w, void* const* y, int T, int din, int dout, hipStream_t st);
int dgrad(const void* dy, const void* w, void* dx, int T, int din, int dout, hipStream_t st);
int wgrad(const void* x, const void* const* dy, float* const* dw, int n, int T, int din, int dout, int block,
          hipStream_t st);
// The input gradient of n (2 or 3) products of one input, the sum of dy[i] w[i]^T: bf16 with a
// residual added before the one rounding (dx), one launch that sums all pairs in its
// accumulators, or float32 (dx32), a launch a pair: a chain of sums is then no longer than a
// pair's (float32 tiles that hold two sets of sums would cost more than reading dx32 again).
int dgrad_pairs(const void* const* dy, const void* const* w, int n, float* dx32, const void* residual, void* dx, int T,
                int din, int dout, hipStream_t st);

// Workspace of a feed-forward network of d_model x d_ff: row_bytes of intermediates per row plus
// fixed bytes.  The rows are worked on in groups of whole blocks.  256 tiles of 256 x 256 fill the
// chip, so a group is the rows that give the narrower product kFillRounds times as many (4096
// wide: 8192 rows, the intermediates of a backward at d_ff = 4 d_model then 1 GiB), but no more
// than kGroupBytes hold; one block where that is more, or where memory is short.  Forward +
// backward in groups of one round, two, four, ms: 8192 x 4096 x 16384 7.35, 7.08, 7.07; 16384 x
// 2048 x 5120 2.86, 2.65, 2.65; LLaMA step of 16384 x 4096 x 11008 70.1, 68.6, 68.8.
// *rows: rows of a group (the last one may have fewer).
constexpr int kFillRounds = 2;
constexpr size_t kGroupBytes = (size_t)5 << 28;
struct CallResources;
int alloc_row_groups(CallResources& R, int T, int d_model, int d_ff, int block, size_t row_bytes, size_t fixed,
                     int* rows);

// Blockwise FFN forward: y = act(x W1 + b1) W2 + b2 (+ residual); arguments validated.
int ffn_forward(const void* x, const void* w1, const void* b1, const void* w2, const void* b2, const void* residual,
                void* y, int T, int d_model, int d_ff, int block, int act, hipStream_t stream);
// Blockwise FFN backward; dx = dy_ffn (+ dx_residual).  Weight gradients overwritten.
int ffn_backward(const void* x, const void* w1, const void* b1, const void* w2, const void* dy, const void* dx_residual,
                 void* dx, float* dw1, float* db1, float* dw2, float* db2, int T, int d_model, int d_ff, int block,
                 int act, hipStream_t stream);

}  // namespace ra
