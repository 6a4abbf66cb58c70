// C ABI of the blockwise feed-forward network and the per-block projections.
//
// The feed-forward network of Section 2 is applied to `block` rows at a time
// (Blockwise Parallel Transformers, Section 2; the feed-forward step of Algorithm 1),
// so the [rows, d_ff] intermediate exists for a bounded number of blocks only.  Every product
// runs in the bf16 matrix-core GEMM; bias, activation, residual and activation-derivative are
// fused into its epilogue.  The backward pass recomputes each group's pre-activation
// (gradient checkpointing) and accumulates weight gradients in float32.
#include <algorithm>

#include "ra_gemm.h"
#include "ra_ops.h"
#include "ra_runtime.h"
#include "ringattn.h"

namespace ra {

int check_gemm_dims(int T, int d_in, int d_out, int block) {
  if (!(T > 0 && d_in > 0 && d_out > 0 && block > 0))
    return set_err(RA_EINVAL, "sizes must be positive (T=%d d_in=%d d_out=%d block=%d)", T, d_in, d_out, block);
  if (T % block) return set_err(RA_EUNSUPPORTED, "T=%d is not a multiple of block=%d", T, block);
  if (block % 256 || d_in % 256 || d_out % 256)
    return set_err(RA_EUNSUPPORTED, "block=%d, d_in=%d and d_out=%d must be multiples of 256", block, d_in, d_out);
  if ((long long)T * d_in >= (1ll << 31) || (long long)T * d_out >= (1ll << 31) ||
      (long long)block * d_in >= (1ll << 31) || (long long)d_in * d_out >= (1ll << 31))
    return set_err(RA_EUNSUPPORTED, "tensor sizes exceed 2^31-1 elements");
  return RA_OK;
}

int gemm(const GemmArgs& g, bool ta, bool tb, int epi, hipStream_t st) {
  RA_HIP(timed_launch(RA_KERNEL_GEMM, st, [&] { return launch_gemm(g, ta, tb, epi, st); }));
  return RA_OK;
}

GemmArgs gemm_args(const void* A, long long lda, const void* B, long long ldb, void* C, long long ldc, int M, int N,
                   int K) {
  GemmArgs g{};
  g.A[0] = A;
  g.B[0] = B;
  g.C[0] = C;
  g.lda = lda;
  g.ldb = ldb;
  g.ldc = ldc;
  g.M = M;
  g.N = N;
  g.K = K;
  return g;
}

int proj(const void* x, const void* w, const void* residual, void* y, int T, int din, int dout, hipStream_t st) {
  GemmArgs g = gemm_args(x, din, w, dout, y, dout, T, dout, din);
  g.residual = residual;
  return gemm(g, false, false, EPI_BF16, st);
}

int proj3(const void* x, const void* const* w, void* const* y, int T, int din, int dout, hipStream_t st) {
  GemmArgs g = gemm_args(x, din, w[0], dout, y[0], dout, T, dout, din);
  g.nb = 3;
  for (int i = 0; i < 3; ++i) {
    g.A[i] = x;
    g.B[i] = w[i];
    g.C[i] = y[i];
  }
  return gemm(g, false, false, EPI_BF16, st);
}

int dgrad(const void* dy, const void* w, void* dx, int T, int din, int dout, hipStream_t st) {
  return gemm(gemm_args(dy, dout, w, dout, dx, din, T, din, dout), false, true, EPI_BF16, st);
}

int wgrad(const void* x, const void* const* dy, float* const* dw, int n, int T, int din, int dout, int block,
          hipStream_t st) {
  GemmArgs g = gemm_args(x, din, dy[0], dout, dw[0], dout, din, dout, T);
  g.nb = n;
  g.kseg = block;
  for (int i = 0; i < n; ++i) {
    g.A[i] = x;
    g.B[i] = dy[i];
    g.C[i] = dw[i];
  }
  return gemm(g, true, false, EPI_F32, st);
}

int dgrad_pairs(const void* const* dy, const void* const* w, int n, float* dx32, const void* residual, void* dx, int T,
                int din, int dout, hipStream_t st) {
  GemmArgs g = gemm_args(dy[0], dout, w[0], dout, dx32 ? (void*)dx32 : dx, din, T, din, dout);
  if (!dx32) {
    g.ns = n;
    for (int i = 0; i < n; ++i) {
      g.A[i] = dy[i];
      g.B[i] = w[i];
    }
    g.residual = residual;
    return gemm(g, false, true, EPI_BF16, st);
  }
  for (int i = 0; i < n; ++i) {
    g.A[0] = dy[i];
    g.B[0] = w[i];
    g.accumulate = i > 0;
    if (int rc = gemm(g, false, true, EPI_F32, st)) return rc;
  }
  return RA_OK;
}

int alloc_row_groups(CallResources& R, int T, int d_model, int d_ff, int block, size_t row_bytes, size_t fixed,
                     int* rows) {
  const int blocks = T / block;
  const long long fill = (long long)kFillRounds * 256 * 256 * 256 / std::min(d_model, d_ff);
  const long long fit = (long long)(kGroupBytes / ((size_t)block * row_bytes));
  int per = (int)std::max(1ll, std::min({(fill + block - 1) / block, fit, (long long)blocks}));
  const int groups = (blocks + per - 1) / per;
  per = (blocks + groups - 1) / groups;  // groups of equal size
  int rc = R.alloc((size_t)per * block * row_bytes + fixed);
  if (rc == RA_ENOMEM && per > 1) {
    (void)hipGetLastError();
    g_err.clear();
    per = 1;
    rc = R.alloc((size_t)block * row_bytes + fixed);
  }
  *rows = per * block;
  return rc;
}

int ffn_forward(const void* x, const void* w1, const void* b1, const void* w2, const void* b2, const void* residual,
                void* y, int T, int d_model, int d_ff, int block, int act, hipStream_t stream) {
  CallResources R(stream);
  int rows, rc;
  if ((rc = alloc_row_groups(R, T, d_model, d_ff, block, (size_t)d_ff * 2, 0, &rows))) return rc;
  void* a = R.ws;  // activation of one group of blocks, bf16 [rows, d_ff]
  for (int r0 = 0; r0 < T; r0 += rows) {
    const int m = T - r0 < rows ? T - r0 : rows;
    const size_t off = (size_t)r0 * d_model * 2;
    GemmArgs up = gemm_args((const char*)x + off, d_model, w1, d_ff, a, d_ff, m, d_ff, d_model);
    up.bias = b1;
    up.act = act;
    if ((rc = gemm(up, false, false, EPI_ACT_BF16, stream))) return rc;
    GemmArgs dn = gemm_args(a, d_ff, w2, d_model, (char*)y + off, d_model, m, d_model, d_ff);
    dn.bias = b2;
    dn.residual = residual ? (const char*)residual + off : nullptr;
    if ((rc = gemm(dn, false, false, EPI_BF16, stream))) return rc;
  }
  return RA_OK;
}

int ffn_backward(const void* x, const void* w1, const void* b1, const void* w2, const void* dy, const void* dx_residual,
                 void* dx, float* dw1, float* db1, float* dw2, float* db2, int T, int d_model, int d_ff, int block,
                 int act, hipStream_t stream) {
  const size_t part = colsum_workspace_floats(d_ff > d_model ? d_ff : d_model);
  CallResources R(stream);
  int rows, rc;
  if ((rc = alloc_row_groups(R, T, d_model, d_ff, block, (size_t)d_ff * 8, part * 4, &rows))) return rc;
  const size_t nb = (size_t)rows * d_ff;
  float* h = (float*)R.ws;                       // pre-activation, float32 [rows, d_ff]
  void* a = (char*)R.ws + nb * 4;                // activation, bf16
  void* dh = (char*)R.ws + nb * 6;               // gradient of the pre-activation, bf16
  float* parts = (float*)((char*)R.ws + nb * 8);  // column-sum partials
  for (int r0 = 0; r0 < T; r0 += rows) {
    const int m = T - r0 < rows ? T - r0 : rows;
    const size_t off = (size_t)r0 * d_model * 2;
    const char* xb = (const char*)x + off;
    const char* dyb = (const char*)dy + off;
    // recompute H = x W1 + b1 and A = act(H)
    GemmArgs up = gemm_args(xb, d_model, w1, d_ff, a, d_ff, m, d_ff, d_model);
    up.bias = b1;
    up.aux_f32 = h;
    up.act = act;
    if ((rc = gemm(up, false, false, EPI_ACT_STORE_H, stream))) return rc;
    // dH = (dy W2^T) * act'(H)
    GemmArgs gA = gemm_args(dyb, d_model, w2, d_model, dh, d_ff, m, d_ff, d_model);
    gA.aux_f32 = h;
    gA.act = act;
    if ((rc = gemm(gA, false, true, EPI_ACT_GRAD_BF16, stream))) return rc;
    // dW2 (+)= A^T dy
    GemmArgs gw2 = gemm_args(a, d_ff, dyb, d_model, dw2, d_model, d_ff, d_model, m);
    gw2.accumulate = r0 > 0;
    gw2.kseg = block;
    if ((rc = gemm(gw2, true, false, EPI_F32, stream))) return rc;
    if (db2) RA_HIP(launch_colsum_bf16(dyb, parts, db2, m, d_model, r0 > 0, stream));
    // dW1 (+)= x^T dH
    GemmArgs gw1 = gemm_args(xb, d_model, dh, d_ff, dw1, d_ff, d_model, d_ff, m);
    gw1.accumulate = r0 > 0;
    gw1.kseg = block;
    if ((rc = gemm(gw1, true, false, EPI_F32, stream))) return rc;
    if (db1) RA_HIP(launch_colsum_bf16(dh, parts, db1, m, d_ff, r0 > 0, stream));
    // dx = dH W1^T
    GemmArgs gx = gemm_args(dh, d_ff, w1, d_ff, (char*)dx + off, d_model, m, d_model, d_ff);
    gx.residual = dx_residual ? (const char*)dx_residual + off : nullptr;
    if ((rc = gemm(gx, false, true, EPI_BF16, stream))) return rc;
  }
  return RA_OK;
}

}  // namespace ra

using namespace ra;

extern "C" {

int blockwise_ffn(const void* x, const void* w1, const void* b1, const void* w2, const void* b2, void* y, int T,
                  int d_model, int d_ff, int block, int act, hipStream_t stream) {
  g_err.clear();
  if (!x || !w1 || !w2 || !y) return set_err(RA_EINVAL, "null pointer argument");
  if (int e = check_aligned({x, w1, b1, w2, b2, y})) return e;
  if (act < 0 || act > 2) return set_err(RA_EINVAL, "act=%d is not an ra_act value", act);
  int rc = check_gemm_dims(T, d_model, d_ff, block);
  if (rc) return rc;
  return ffn_forward(x, w1, b1, w2, b2, nullptr, y, T, d_model, d_ff, block, act, stream);
}

int blockwise_ffn_bwd(const void* x, const void* w1, const void* b1, const void* w2, const void* dy, void* dx,
                      float* dw1, float* db1, float* dw2, float* db2, int T, int d_model, int d_ff, int block,
                      int act, hipStream_t stream) {
  g_err.clear();
  if (!x || !w1 || !w2 || !dy || !dx || !dw1 || !dw2) return set_err(RA_EINVAL, "null pointer argument");
  if (int e = check_aligned({x, w1, b1, w2, dy, dx, dw1, db1, dw2, db2})) return e;
  if (act < 0 || act > 2) return set_err(RA_EINVAL, "act=%d is not an ra_act value", act);
  int rc = check_gemm_dims(T, d_model, d_ff, block);
  if (rc) return rc;
  return ffn_backward(x, w1, b1, w2, dy, nullptr, dx, dw1, db1, dw2, db2, T, d_model, d_ff, block, act, stream);
}

int blockwise_linear(const void* x, const void* w, const void* residual, void* y, int T, int d_in, int d_out,
                     int block, hipStream_t stream) {
  g_err.clear();
  if (!x || !w || !y) return set_err(RA_EINVAL, "null pointer argument");
  if (int e = check_aligned({x, w, residual, y})) return e;
  int rc = check_gemm_dims(T, d_in, d_out, block);
  if (rc) return rc;
  return proj(x, w, residual, y, T, d_in, d_out, stream);
}

int blockwise_linear_bwd(const void* x, const void* w, const void* dy, void* dx, float* dw, int T, int d_in,
                         int d_out, int block, hipStream_t stream) {
  g_err.clear();
  if (!x || !w || !dy || !dw) return set_err(RA_EINVAL, "null pointer argument");
  if (int e = check_aligned({x, w, dy, dx, dw})) return e;
  int rc = check_gemm_dims(T, d_in, d_out, block);
  if (rc) return rc;
  if (dx && (rc = dgrad(dy, w, dx, T, d_in, d_out, stream))) return rc;
  return wgrad(x, &dy, &dw, 1, T, d_in, d_out, block, stream);
}

}  // extern "C"
