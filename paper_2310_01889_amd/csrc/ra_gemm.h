// Interface of the bf16 GEMM kernel family and the column-sum reduction.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

namespace ra {

enum GemmEpilogue {
  EPI_BF16 = 0,           // C = acc (+ bias[n]) (+ residual[m][n]), stored bf16
  EPI_ACT_BF16 = 1,       // C = act(acc + bias[n]) (+ residual), stored bf16
  EPI_ACT_STORE_H = 2,    // aux_f32 = acc + bias (pre-activation, float32); C = act(aux_f32), bf16
  EPI_ACT_GRAD_BF16 = 3,  // C = acc * act'(aux_f32[m][n]), stored bf16
  EPI_F32 = 4,            // C = acc (or C += acc if accumulate), float32
  EPI_GLU_BF16 = 5,       // with u = A B[0], w = A B[1]: C = silu(u) * w, bf16; aux_f32 = u, aux2_f32 = w unless null
  EPI_GLU_GRAD = 6,       // with u = aux_f32, w = aux2_f32: C = acc * w * silu'(u), C2 = acc * silu(u) (bf16)
  EPI_F32_SEGMENTS = 7    // EPI_F32 with kseg < K (launch_gemm's choice)
};

struct GemmArgs {
  // nb products C[z] = A[z] B[z] of one shape in one launch, or (ns > 1) one product
  // C[0] = sum over s < ns of A[s] B[s]
  const void* A[3];       // bf16, [M][lda] (or [K][lda] when transposed)
  const void* B[3];       // bf16, [K][ldb] (or [N][ldb] when transposed)
  void* C[3];             // bf16 or float32 [M][ldc]
  const void* bias;       // bf16 [N] or null
  const void* residual;   // bf16 [M][ldc] or null
  float* aux_f32;         // float32 [M][ldc]: pre-activation (written or read)
  float* aux2_f32;        // float32 [M][ldc]: second gate input of the GLU epilogues
  void* C2;               // bf16 [M][ldc]: second output of EPI_GLU_GRAD
  long long lda, ldb, ldc;
  int M, N, K, act, accumulate;
  int nb = 1, ns = 1;
  int kseg = 0;           // EPI_F32: terms of K summed by themselves (0: all); not with ns > 1
};

// ta: A stored as [K][M]; tb: B stored as [N][K].  M, N, K and kseg must be multiples of 256,
// K one of kseg.
hipError_t launch_gemm(const GemmArgs& g, bool ta, bool tb, int epi, hipStream_t st);

// out[n] (+)= sum_m x[m][n] for bf16 x [M][N]; part: colsum_workspace_floats(N) floats.
hipError_t launch_colsum_bf16(const void* x, float* part, float* out, int M, int N, int accumulate,
                              hipStream_t st);
size_t colsum_workspace_floats(int N);

}  // namespace ra
