// bf16 matrix-core GEMM for gfx950 with fused epilogues, and the column-sum reduction.
//
// C[M][N] = sum_k A[m][k] B[k][n] with A stored row-major [M][K] (TA = 0) or as its
// transpose [K][M] (TA = 1), B stored row-major [K][N] (TB = 0) or as [N][K] (TB = 1).
// Workgroup tile 256 x 256, 8 waves (two per SIMD) each owning a 128 x 64 sub-tile (8
// accumulators of 32 x 32): while one wave waits for operands or the barrier, the other
// keeps the matrix core busy.  K advances 32 at a time through a ring of five LDS stages
// (all 160 KB of the CU's LDS) filled by direct-to-LDS buffer loads four steps ahead of
// their use.  Products with too few such tiles for the chip's 256 CUs take 128 x 128 tiles,
// 4 waves of 64 x 64, two workgroups a CU (see tile_size); weight gradients of several row blocks
// these or 256 x 128 (see small_sums).  Tiles are kept in their
// memory layout, unpadded, with 16-byte chunks XOR-swizzled per row so that both the row
// reads and the transpose reads (an operand whose registers must run along its contiguous
// dimension) are free of bank conflicts.  Each wave computes C^T = B^T A^T so that a lane
// owns one row m of C and four consecutive columns n per register group: epilogues then
// read bias / residual / pre-activation and write C with vector accesses.
//
// One launch covers up to three products of one shape (the query, key and value projections
// of a layer) or one product whose reduction runs over up to three operand pairs (the sum of
// their input gradients, which so stays in the accumulators).
#include "ra_common.h"
#include "ra_dma.h"
#include "ra_gemm.h"
#include "ringattn.h"

namespace ra {
namespace {

constexpr int kTK = 32;
constexpr int kNS = 5;  // ring stages

// Tile layouts in LDS (no padding; chunk = 16 bytes = 8 elements):
//   row tile   [T][32] (T rows or columns of C; A with TA = 0, B with TB = 1): 64-byte rows of 4 chunks, logical
//              chunk c of row r stored at c ^ ((r >> 2) & 3);
//   k-major    [32][T] (A with TA = 1, B with TB = 0): rows of T / 8 chunks,
//              logical chunk c of row r stored at c ^ (4 (r & 3)).
// A one-wave direct-to-LDS load fills 1 KB: 16 rows of a row tile, or 512 / T rows of a k-major
// tile, lane i landing at byte 16 i; the swizzle is applied to the global address.
__device__ __forceinline__ int swz_row(int r) { return (r >> 2) & 3; }
__device__ __forceinline__ int swz_kmaj(int r) { return 4 * (r & 3); }

// sigmoid(u); silu(u) = u sigmoid(u) has derivative sigmoid(u) (1 + u (1 - sigmoid(u)))
// (SwiGLU gate)
__device__ __forceinline__ float sigmoid_f(float u) { return __builtin_amdgcn_rcpf(1.f + __expf(-u)); }

// Exact GeLU h Phi(h) and Phi(h), phi(h) (standard normal CDF and density) from the erfc
// approximation of Abramowitz and Stegun, formula 7.1.26: with a = |h| / sqrt(2),
//   0.5 erfc(a) = Phi(-|h|) ~ t (b1 + t (b2 + t (b3 + t (b4 + t b5)))) exp(-a^2),
//   t = 1 / (1 + p a), p = 0.3275911, b_i half the published a_i
// (absolute error below 1.5e-7 in erf).  The lower tail is formed directly, without the
// cancellation of 1 + erf for negative h; one reciprocal and one exponential, a third of
// the instructions of a library erf in the epilogue.
__device__ __forceinline__ float gauss_lower(float h, float& e) {  // Phi(-|h|); e = exp(-h^2 / 2)
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f * 0.7071067811865476f, fabsf(h), 1.f));
  e = fast_exp2(h * (h * (-0.5f * kLog2e)));
  const float poly =
      t * fmaf(t, fmaf(t, fmaf(t, fmaf(t, 0.5307027145f, -0.7265760135f), 0.7107068705f), -0.142248368f), 0.127414796f);
  return poly * e;
}
__device__ __forceinline__ float gelu_erf(float h) {
  float e;
  const float hl = h * gauss_lower(h, e);
  return h >= 0.f ? h - hl : hl;
}
__device__ __forceinline__ float gauss_cdf(float h, float& pdf) {
  float e;
  const float lower = gauss_lower(h, e);
  pdf = 0.3989422804014327f * e;
  return h >= 0.f ? 1.f - lower : lower;
}

template <int ACT>
__device__ __forceinline__ float act_apply(float h) {
  constexpr int act = ACT;
  if (act == 1) return fmaxf(h, 0.f);
  if (act == 2) {  // 0.5 (1 + tanh(u)) = sigmoid(2 u)
    const float u = 0.7978845608028654f * (h + 0.044715f * h * h * h);
    return h * sigmoid_f(2.f * u);
  }
  return gelu_erf(h);
}


template <int ACT>
__device__ __forceinline__ float act_grad(float h) {
  constexpr int act = ACT;
  if (act == 1) return h > 0.f ? 1.f : 0.f;
  if (act == 2) {  // with s = sigmoid(2 u): 0.5 (1 + tanh u) = s, 0.5 (1 - tanh^2 u) = 2 s (1 - s)
    const float u = 0.7978845608028654f * (h + 0.044715f * h * h * h);
    const float sg = sigmoid_f(2.f * u);
    const float du = 0.7978845608028654f * (1.f + 3.f * 0.044715f * h * h);
    return sg + 2.f * h * sg * (1.f - sg) * du;
  }
  float pdf;
  const float cdf = gauss_cdf(h, pdf);
  return cdf + h * pdf;
}


// ACT: the activation of the ACT epilogues (an ra_act value, fixed at compile time so
// that each kernel holds the code of one activation only).
// EPI_GLU_BF16 (256 x 256, TB = 0) forms two products over the same A at once: the B tile is 128
// columns of B[0] beside the same 128 columns of B[1], two k-major [32][128] tiles, so that the
// epilogue finds u = A B[0] and w = A B[1] of an element in one row of the transposed tile.
// EPI_F32_SEGMENTS (SUMS, TN = 128) sums K in segments of g.kseg, each by itself, and adds up
// the segments' sums in a second set of accumulators: the error of one chain of sums grows with
// its length (x^T dy of 16384 rows, relative: 8.2e-7 in one chain, 2.8e-7 in segments of 2048).
// A wave's 64 x 64 leaves the registers for it; the 128 x 64 of a 256 x 256 tile do not, and a
// running total in C, read and written from behind the L2 at each segment, took longer (dW of
// 4096 x 16384 over 8192 rows in segments of 1024: 1368 us, 1033 so, 838 in one chain; 2048 x 5120
// over 16384 in 256: 1036, 411, 302).
template <int TM, int TN, bool TA, bool TB, int EPI, int ACT>
__global__ __launch_bounds__(TM == 256 ? 512 : 256, TM == 256 ? 1 : 2) void gemm_kernel(const GemmArgs g) {
  constexpr bool DUAL = EPI == EPI_GLU_BF16, SUMS = EPI == EPI_F32_SEGMENTS;
  static_assert(!DUAL || (TM == 256 && TN == 256 && !TB), "two-product tiles are 256 x (128 + 128), k-major");
  static_assert((TM == TN && !SUMS) || (TM >= TN && TN == 128 && SUMS), "256 x 256, 128 x 128 or (float32) 256 x 128");
  constexpr int NWAVE = TM == 256 ? 8 : 4;
  constexpr int WN = TN / 64, WM = NWAVE / WN; // waves across N and M
  constexpr int NI = 2;                        // 32-column groups of a wave (64 columns)
  constexpr int MI = TM / WM / 32;             // 32-row groups of a wave
  constexpr int TNC = DUAL ? TN / 2 : TN;      // columns of C per workgroup
  constexpr int BW = DUAL ? TN / 2 : TN;       // columns of a k-major B tile
  constexpr int kTileA = TM * kTK * 2, kTileB = TN * kTK * 2;  // bytes of the operand tiles
  constexpr int LA = kTileA / 1024 / NWAVE, LB = kTileB / 1024 / NWAVE;  // 1 KB loads per wave
  constexpr int LPS = LA + LB;                 // loads per step per wave
  // one LDS object per stage (A tile, then B tile), so that reads of one stage are known not
  // to alias the direct-to-LDS loads in flight into the others
  __shared__ __attribute__((aligned(1024))) char sS0[kTileA + kTileB];
  __shared__ __attribute__((aligned(1024))) char sS1[kTileA + kTileB];
  __shared__ __attribute__((aligned(1024))) char sS2[kTileA + kTileB];
  __shared__ __attribute__((aligned(1024))) char sS3[kTileA + kTileB];
  __shared__ __attribute__((aligned(1024))) char sS4[kTileA + kTileB];
  auto stage = [&](auto Sc) __attribute__((always_inline)) -> char* {
    constexpr int S = decltype(Sc)::value % kNS;
    if constexpr (S == 0) return sS0; else if constexpr (S == 1) return sS1; else if constexpr (S == 2) return sS2;
    else if constexpr (S == 3) return sS3; else return sS4;
  };

  // tile order: XCD-contiguous ranges over the products of the launch, then groups of 8
  // tile-rows sweeping across N
  const int tiles_m = g.M / TM, tiles_n = g.N / TNC;
  const int total = tiles_m * tiles_n;
  const int Lz = xcd_swizzle(blockIdx.x, total * g.nb);
  const int z = Lz / total, L = Lz - z * total;
  const int GM = 2048 / TM;
  const int group = L / (GM * tiles_n);
  const int first_m = group * GM;
  const int gsize = min(GM, tiles_m - first_m);
  const int tm = first_m + (L % (GM * tiles_n)) % gsize;
  const int tn = (L % (GM * tiles_n)) / gsize;
  const int m0 = tm * TM, n0 = tn * TNC;

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
  const int wm = wave / WN, wn = wave % WN;  // TM / WM rows x 64 columns per wave
  void* const Cz = g.C[z];
  const int nk1 = g.K / kTK, nk = nk1 * g.ns;  // steps of one operand pair, of all

  f32x16 acc[NI][MI];  // [n tile][m tile] of C^T
#pragma unroll
  for (int a = 0; a < NI; ++a)
#pragma unroll
    for (int b = 0; b < MI; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;
  // the sum of the segments so far, from C's own values where they are added to
  f32x16 tot[SUMS ? NI : 1][SUMS ? MI : 1];
  if constexpr (SUMS) {
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) {
        tot[ni][mi] = f32x16{};
        if (g.accumulate) {
          const float* c = (const float*)Cz + (long long)(m0 + wm * (TM / WM) + 32 * mi + l32) * g.ldc + n0 + 64 * wn +
                           32 * ni + 4 * hi;
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            const f32x4 t = *(const f32x4*)(c + 8 * q4);
#pragma unroll
            for (int e = 0; e < 4; ++e) tot[ni][mi][4 * q4 + e] = t[e];
          }
        }
      }
  }

  // ---- direct-to-LDS loads: per-lane byte offsets from the tile origin (fixed), and
  // the tile origin, which moves by kTK along K (scalar) ------------------------------
  // load j of this wave's L of a tile fills LDS bytes [blk * 1024, +1024) of it, blk = wave * L + j
  // (two-product B tiles: blk = j * 8 + wave, so that load j is of B[j])
  auto lane_off = [&](bool kmajor, int width, long long ld, int blk) __attribute__((always_inline)) -> int {
    if (!kmajor) {  // 16 rows x 4 chunks
      const int r = blk * 16 + (lane >> 2), pc = lane & 3;
      return (int)(2 * (r * ld + 8 * (pc ^ swz_row(r))));
    }
    const int cpr = width / 8;
    const int r = blk * (64 / cpr) + lane / cpr, pc = lane % cpr;
    return (int)(2 * (r * ld + 8 * (pc ^ swz_kmaj(r))));
  };
  int aoff[LA], boff[LB];
#pragma unroll
  for (int j = 0; j < LA; ++j) aoff[j] = lane_off(TA, TM, g.lda, wave * LA + j);
#pragma unroll
  for (int j = 0; j < LB; ++j) boff[j] = lane_off(!TB, BW, g.ldb, DUAL ? wave : wave * LB + j);
  // extent of a tile's reads (bytes from its origin), for the buffer descriptors
  const int a_ext = (int)(2 * (TA ? (long long)(kTK - 1) * g.lda + TM : (long long)(TM - 1) * g.lda + kTK));
  const int b_ext = (int)(2 * (TB ? (long long)(TN - 1) * g.ldb + kTK : (long long)(kTK - 1) * g.ldb + BW));
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const bf16* const A0 = (const bf16*)g.A[z];
  const bf16* const B0 = (const bf16*)g.B[z];
  auto load_stage = [&](int kt, auto Sc) __attribute__((always_inline)) {
    const bf16 *A = A0, *B = B0;
    int k0 = kt * kTK;
    if (g.ns > 1 && kt >= nk1) {  // the second or third operand pair
      const int sgm = kt >= 2 * nk1 ? 2 : 1;
      A = (const bf16*)g.A[sgm];
      B = (const bf16*)g.B[sgm];
      k0 -= sgm * g.K;
    }
    const bf16* at = TA ? A + (long long)k0 * g.lda + m0 : A + (long long)m0 * g.lda + k0;
    const long long boffs = TB ? (long long)n0 * g.ldb + k0 : (long long)k0 * g.ldb + n0;
    const __amdgpu_buffer_rsrc_t ra_ = make_rsrc(at, a_ext), rb_ = make_rsrc(B + boffs, b_ext);
    const unsigned st = lds_addr(stage(Sc));
    const unsigned sa = st + wave_u * LA * 1024, sb = st + kTileA + (DUAL ? wave_u : wave_u * LB) * 1024;
    if constexpr (DUAL) {
      const __amdgpu_buffer_rsrc_t rb2 = make_rsrc((const bf16*)g.B[1] + boffs, b_ext);
      dma_lds16(ra_, sa, aoff[0]);
      dma_lds16(rb_, sb, boff[0]);
      dma_lds16(ra_, sa + 1024, aoff[1]);
      dma_lds16(rb2, sb + kTileB / 2, boff[1]);
    } else {
#pragma unroll
      for (int j = 0; j < LA; ++j) {
        dma_lds16(ra_, sa + j * 1024, aoff[j]);  // tile loads the loop waits for itself
        if (j < LB) dma_lds16(rb_, sb + j * 1024, boff[j]);
      }
    }
  };

  // ---- LDS read offsets (bytes within an operand tile) --------------------------------
  // row-tile operand: rows base + l32 (base a multiple of 32), logical chunk 2 kk + hi
  int roff[2];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) roff[kk] = l32 * 64 + 16 * ((2 * kk + hi) ^ swz_row(l32));
  // k-major operand by transpose reads: rows 16 kk + 8 hi + li / 4 (and + 4), columns
  // base + 32 t + 16 (gq & 1) + 4 (li & 3) for t < MI (A: base TM / WM wm) or t < NI (B: base 64 wn)
  const int gq = lane >> 4, li = lane & 15;
  const int trow = 8 * hi + (li >> 2);
  auto tr_off = [&](int width, int col) __attribute__((always_inline)) -> int {
    return trow * width * 2 + 16 * ((col >> 3) ^ swz_kmaj(trow)) + 2 * (col & 7);
  };
  int toff[MI], tboff[NI];
#pragma unroll
  for (int t = 0; t < MI; ++t) toff[t] = tr_off(TM, wm * (TM / WM) + 32 * t + 16 * (gq & 1) + 4 * (li & 3));
#pragma unroll
  for (int t = 0; t < NI; ++t) {
    const int col = 64 * wn + 32 * t + 16 * (gq & 1) + 4 * (li & 3);
    tboff[t] = DUAL ? (wn >> 1) * (kTileB / 2) + tr_off(BW, col & (BW - 1)) : tr_off(BW, col);
  }
  // operand fetch for k-slice kk of a stage: A operand rows m (bop: B^T rows n)
  auto fetch = [&](const char* st, int kk, bf16x8* aop, bf16x8* bop) __attribute__((always_inline)) {
    const char* as = st;
    const char* bs = st + kTileA;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      if (!TA) {
        aop[i] = *(const bf16x8*)(as + (wm * (TM / WM) + 32 * i) * 64 + roff[kk]);
      } else {
        const char* p = as + kk * 16 * TM * 2 + toff[i];
        const bf16x4 lo = lds_read_tr16((const bf16*)p), up = lds_read_tr16((const bf16*)(p + 4 * TM * 2));
        aop[i] = bf16x8{lo[0], lo[1], lo[2], lo[3], up[0], up[1], up[2], up[3]};
      }
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      if (TB) {
        bop[i] = *(const bf16x8*)(bs + (wn * 64 + 32 * i) * 64 + roff[kk]);
      } else {
        const char* p = bs + kk * 16 * BW * 2 + tboff[i];
        const bf16x4 lo = lds_read_tr16((const bf16*)p), up = lds_read_tr16((const bf16*)(p + 4 * BW * 2));
        bop[i] = bf16x8{lo[0], lo[1], lo[2], lo[3], up[0], up[1], up[2], up[3]};
      }
    }
  };
  auto mfmas = [&](const bf16x8* aop, const bf16x8* bop) __attribute__((always_inline)) {
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) acc[ni][mi] = mfma32(bop[ni], aop[mi], acc[ni][mi]);
  };

  // ---- main loop ----------------------------------------------------------------------
  // Step kt (stage kt % kNS): issue the loads of step kt + kNS - 1 into the stage step kt-1 used;
  // slice 0's products while slice 1's operands are read; then wait for step kt+1's loads
  // (those of later steps may stay in flight -- loads complete in issue order), the
  // barrier (every read of this stage has been issued by now), and step kt+1's slice-0
  // reads, covered by slice 1's products.
  bf16x8 a0[MI], b0[NI], a1[MI], b1[NI];
  static_for<0, kNS - 1>([&](auto Sc) __attribute__((always_inline)) { load_stage(decltype(Sc)::value, Sc); });
  // stage 0 has landed (the others may stay in flight: K is at least 8 steps)
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kNS - 2) * LPS) : "memory");
  lds_barrier();
  fetch(sS0, 0, a0, b0);
  const int seg = g.kseg / kTK;  // SUMS: steps of a segment
  int seg_end = seg;
  auto step = [&](auto Sc, int kt) __attribute__((always_inline)) {
    constexpr int S = decltype(Sc)::value;
    if (kt + kNS - 1 < nk) load_stage(kt + kNS - 1, std::integral_constant<int, (S + kNS - 1) % kNS>{});
    fetch(stage(Sc), 1, a1, b1);
    mfmas(a0, b0);
    // step kt+1 must have landed: at most the loads of steps kt+2 .. kt + kNS - 1 outstanding
    if (kt + 4 < nk)
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * LPS) : "memory");
    else if (kt + 3 < nk)
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * LPS) : "memory");
    else if (kt + 2 < nk)
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LPS) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
    if (kt + 1 < nk) fetch(stage(std::integral_constant<int, S + 1>{}), 0, a0, b0);
    mfmas(a1, b1);
    if constexpr (SUMS) {
      if (__builtin_expect(kt + 1 == seg_end, 0)) {
        seg_end += seg;
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
          for (int mi = 0; mi < MI; ++mi) {
            tot[ni][mi] += acc[ni][mi];
            acc[ni][mi] = f32x16{};
          }
      }
    }
  };
  int kt = 0;
  for (; kt + kNS - 1 < nk; kt += kNS)
    static_for<0, kNS>([&](auto Sc) __attribute__((always_inline)) { step(Sc, kt + decltype(Sc)::value); });
  static_for<0, kNS - 1>([&](auto Sc) __attribute__((always_inline)) {
    if (kt < nk) step(Sc, kt++);
  });
  const f32x16(&res)[NI][MI] = [&]() -> const f32x16(&)[NI][MI] {
    if constexpr (SUMS) return tot; else return acc;
  }();

  // ---- epilogue --------------------------------------------------------------------
  // The float32 accumulators pass through LDS (the stage buffers are free now) in passes of
  // 128 rows, 32 rows per stage buffer (rows of TN floats; 16-byte chunk c of row r stored at
  // c ^ (r & 15), so both the writes -- 32 rows at one column -- and the row reads are free of
  // bank conflicts): the waves owning those rows write them, then every wave takes a share of
  // each buffer's rows and a lane handles 4 consecutive columns, so bias, residual,
  // pre-activation and output accesses are contiguous along rows.
  // What an epilogue reads of a row (residual, pre-activation, C itself) is loaded a chunk of
  // rows ahead, the first chunk before the accumulators go through LDS: one row at a time,
  // each paid a memory round trip (8192 x 16384 x 4096 with the activation gradient: 1285 us
  // instead of the plain product's 890).
  struct Pre { f32x4 x, y; bf16x4 r; };
  constexpr bool READS1 = EPI == EPI_ACT_GRAD_BF16 || EPI == EPI_GLU_GRAD, READS2 = EPI == EPI_GLU_GRAD;
  constexpr bool RES = EPI == EPI_BF16 || EPI == EPI_ACT_BF16 || EPI == EPI_ACT_STORE_H;
  auto prefetch = [&](int m, int n) __attribute__((always_inline)) -> Pre {
    Pre q;
    const long long off = (long long)m * g.ldc + n;
    if constexpr (READS1) q.x = *(const f32x4*)(g.aux_f32 + off);
    if constexpr (READS2) q.y = *(const f32x4*)(g.aux2_f32 + off);
    if constexpr (EPI == EPI_F32) {
      if (g.accumulate) q.x = *(const f32x4*)((const float*)Cz + off);
    }
    if constexpr (RES) {
      if (g.residual) q.r = *(const bf16x4*)((const bf16*)g.residual + off);
    }
    return q;
  };
  auto epi4 = [&](int m, int n, float* v, const float* v2, const Pre& q) __attribute__((always_inline)) {
    const long long off = (long long)m * g.ldc + n;
    if (RES) {
      if (g.bias) {
        const bf16x4 bb = *(const bf16x4*)((const bf16*)g.bias + n);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] += (float)bb[e];
      }
      if (EPI == EPI_ACT_STORE_H) *(f32x4*)(g.aux_f32 + off) = f32x4{v[0], v[1], v[2], v[3]};
      if (EPI != EPI_BF16) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = act_apply<ACT>(v[e]);
      }
      if (g.residual) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] += (float)q.r[e];
      }
      *(u32x2*)((bf16*)Cz + off) = u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
    } else if (EPI == EPI_ACT_GRAD_BF16) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] *= act_grad<ACT>(q.x[e]);
      *(u32x2*)((bf16*)Cz + off) = u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
    } else if (EPI == EPI_GLU_BF16) {
      if (g.aux_f32) *(f32x4*)(g.aux_f32 + off) = f32x4{v[0], v[1], v[2], v[3]};
      if (g.aux2_f32) *(f32x4*)(g.aux2_f32 + off) = f32x4{v2[0], v2[1], v2[2], v2[3]};
      float o[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = v2[e] * (v[e] * sigmoid_f(v[e]));
      *(u32x2*)((bf16*)Cz + off) = u32x2{pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3])};
    } else if (EPI == EPI_GLU_GRAD) {
      const f32x4 u = q.x, w = q.y;
      float du[4], dw[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float sg = sigmoid_f(u[e]);
        du[e] = v[e] * w[e] * sg * (1.f + u[e] * (1.f - sg));
        dw[e] = v[e] * u[e] * sg;
      }
      *(u32x2*)((bf16*)Cz + off) = u32x2{pack_bf16x2(du[0], du[1]), pack_bf16x2(du[2], du[3])};
      *(u32x2*)((bf16*)g.C2 + off) = u32x2{pack_bf16x2(dw[0], dw[1]), pack_bf16x2(dw[2], dw[3])};
    } else {  // EPI_F32: overwrite, or add into C
      f32x4* cp = (f32x4*)((float*)Cz + off);
      if (EPI == EPI_F32 && g.accumulate)
        *cp = f32x4{q.x[0] + v[0], q.x[1] + v[1], q.x[2] + v[2], q.x[3] + v[3]};
      else
        *cp = f32x4{v[0], v[1], v[2], v[3]};
    }
  };
  constexpr int ROWB = TN * 4;               // bytes of a row in LDS
  constexpr int LPR = TNC / 4;               // lanes per row
  constexpr int RPI = 64 / LPR;              // rows a wave handles at once
  constexpr int RPWV = 32 / NWAVE;           // rows of a buffer per wave
  constexpr int PASSES = TM / 128;
  constexpr int NR = RPWV / RPI;             // row groups of a buffer per wave
  constexpr int CH = RES || DUAL ? 8 : 4;    // row groups of a prefetched chunk (8 float4 rows spill)
  constexpr int NCH = 4 * NR / CH;           // chunks of a pass
  const int cl = lane % LPR;                 // this lane's 4 columns
#pragma unroll
  for (int pass = 0; pass < PASSES; ++pass) {
    // row group i of the pass: local row lr of buffer i / NR
    auto row_of = [&](int i) __attribute__((always_inline)) { return RPWV * wave + (i % NR) * RPI + lane / LPR; };
    Pre pre[2][CH];
    auto fetch_chunk = [&](auto Cc) __attribute__((always_inline)) {
      constexpr int C = decltype(Cc)::value;
#pragma unroll
      for (int k = 0; k < CH; ++k) {
        const int i = C * CH + k;
        pre[C & 1][k] = prefetch(m0 + 128 * pass + 32 * (i / NR) + row_of(i), n0 + 4 * cl);
      }
    };
    fetch_chunk(std::integral_constant<int, 0>{});
    // the rows of wave row wmp: m groups wmp * MI + mi of the tile, buffer (that) % 4
    static_for<0, WM>([&](auto Wp) __attribute__((always_inline)) {
      constexpr int wmp = decltype(Wp)::value;
      if (wm == wmp && wmp * MI / 4 == pass) {
        // lane: row l32 of the buffer, columns 64 wn + 32 ni + 8 q4 + 4 hi .. +3
        static_for<0, MI>([&](auto Mi) __attribute__((always_inline)) {
          constexpr int mi = decltype(Mi)::value;
          char* sb = stage(std::integral_constant<int, (wmp * MI + mi) % 4>{}) + l32 * ROWB;
#pragma unroll
          for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
              const int c = 16 * wn + 8 * ni + 2 * q4 + hi;
              *(f32x4*)(sb + 16 * (c ^ (l32 & 15))) =
                  f32x4{res[ni][mi][4 * q4], res[ni][mi][4 * q4 + 1], res[ni][mi][4 * q4 + 2], res[ni][mi][4 * q4 + 3]};
            }
        });
      }
    });
    lds_barrier();
    static_for<0, NCH>([&](auto Cc) __attribute__((always_inline)) {
      constexpr int C = decltype(Cc)::value;
      if constexpr (C + 1 < NCH) fetch_chunk(std::integral_constant<int, C + 1>{});
      static_for<0, CH>([&](auto Kc) __attribute__((always_inline)) {
        constexpr int k = decltype(Kc)::value, i = C * CH + k;
        const char* sb = stage(std::integral_constant<int, i / NR>{});
        const int lr = row_of(i);
        const f32x4 t = *(const f32x4*)(sb + lr * ROWB + 16 * (cl ^ (lr & 15)));
        float v[4] = {t[0], t[1], t[2], t[3]}, v2[4] = {};
        if constexpr (DUAL) {
          const f32x4 t2 = *(const f32x4*)(sb + lr * ROWB + 16 * ((cl + LPR) ^ (lr & 15)));
#pragma unroll
          for (int e = 0; e < 4; ++e) v2[e] = t2[e];
        }
        epi4(m0 + 128 * pass + 32 * (i / NR) + lr, n0 + 4 * cl, v, v2, pre[C & 1][k]);
      });
    });
    if (pass + 1 < PASSES) lds_barrier();
  }
}

// Column sums of a bf16 [M, N] matrix (N a multiple of 8), deterministic two-pass reduction:
// pass 1 writes partial sums of row slabs, a thread taking 8 columns (16-byte loads) of every
// fourth row of its slab, in turn into four sums; pass 2 adds the slabs, in eight sums, into out
// (+= or =).  HBM-bound.  Short chains of sums keep the error near one rounding (16384 rows of
// N(0, 1), relative: 5.5e-8, in one chain a thread 1.1e-7).
constexpr int kCS = 64;  // row slabs
__global__ __launch_bounds__(256) void colsum_partial_kernel(const bf16* x, float* part, int M, int N) {
  __shared__ float red[4][64][9];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = (blockIdx.x * 64 + lane) * 8;
  const int slab = blockIdx.y;
  const int rows = (M + kCS - 1) / kCS;
  const int r0 = slab * rows, r1 = min(M, r0 + rows);
  float s[4][8] = {};
  if (n < N)
    for (int r = r0 + wave; r < r1; r += 16) {
      bf16x8 v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j)  // past the slab: its last row, not added
        v[j] = *(const bf16x8*)(x + (long long)min(r + 4 * j, r1 - 1) * N + n);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (j == 0 || r + 4 * j < r1) {
#pragma unroll
          for (int e = 0; e < 8; ++e) s[j][e] += (float)v[j][e];
        }
    }
#pragma unroll
  for (int e = 0; e < 8; ++e) red[wave][lane][e] = (s[0][e] + s[1][e]) + (s[2][e] + s[3][e]);
  __syncthreads();
  for (int i = threadIdx.x; i < 512; i += 256) {
    const int l = i >> 3, e = i & 7, c = blockIdx.x * 512 + i;
    if (c < N) part[(long long)slab * N + c] = (red[0][l][e] + red[1][l][e]) + (red[2][l][e] + red[3][l][e]);
  }
}
__global__ __launch_bounds__(256) void colsum_final_kernel(const float* part, float* out, int N, int accumulate) {
  const int n = blockIdx.x * 256 + threadIdx.x;
  if (n >= N) return;
  float p[8] = {};
  float v[kCS];
#pragma unroll
  for (int sl = 0; sl < kCS; ++sl) v[sl] = part[(long long)sl * N + n];
  __builtin_amdgcn_sched_barrier(0);  // all loads in flight at once: few waves, one memory latency
#pragma unroll
  for (int sl = 0; sl < kCS; ++sl) p[sl % 8] += v[sl];
  const float s = ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
  out[n] = accumulate ? out[n] + s : s;
}

// 256 x 256 tiles, or 128 x 128 where they finish sooner.  A round of the chip is 256 big
// tiles, one a CU, or 512 small ones, two a CU, which hold half the work and run at 1 / kSmall
// of the big tiles' rate (8192 x 4096 x 4096: 219 us in big tiles, 288 in small ones).  Big
// tiles against small ones where the rule turns, us: 2048 x 4096 x 4096 (128 big tiles) 83, 72;
// 4096^3 (256) 113, 145; 5120 x 1280 x 4864 (380) 74.4, 76.2; 2048 x 1024 x 1024 (32) 25.7, 13.6;
// 2048 x 4096 x 1024 (32, deep) 76, 37.
constexpr double kSmall = 1.35;
int tile_size(const GemmArgs& g) {
  const long long big = (long long)(g.M / 256) * (g.N / 256) * g.nb;
  const long long r256 = (big + 255) / 256, r128 = (4 * big + 511) / 512;
  return 0.5 * kSmall * (double)r128 < (double)r256 ? 128 : 256;
}
// Float32 sums of several segments: 256 x 128 tiles, one workgroup a CU, or 128 x 128, up to two.
// At 8192 rows a round of the chip is 112 us in the former, in the latter 62 us for each tile of
// a CU and 14 more for one that is alone at the end: ahead for an odd count of them, up to five.
// 256 x 128 against 128 x 128 tiles, us: 2048^2 (128 of the former) 101, 81; 3072 x 2048 (192) 115,
// 125; 4096 x 3072 (384) 216, 198; 4096 x 3584 (448) 227, 244; 4352 x 4096 (544) 332, 305; 4096 x
// 6400 (800) 445, 458.
bool small_sums(const GemmArgs& g) {
  const long long per_cu = ((long long)(g.M / 128) * (g.N / 128) * g.nb + 255) / 256;
  return per_cu % 2 == 1 && per_cu <= 5;
}

template <int TM, int TN, bool TA, bool TB, int EPI, int ACT>
void launch_tile(const GemmArgs& g, hipStream_t st) {
  const int cols = EPI == EPI_GLU_BF16 ? TN / 2 : TN;
  hipLaunchKernelGGL((gemm_kernel<TM, TN, TA, TB, EPI, ACT>), dim3((unsigned)((g.M / TM) * (g.N / cols) * g.nb)),
                     dim3(TM == 256 ? 512 : 256), 0, st, g);
}

template <bool TA, bool TB, int EPI, int ACT>
hipError_t launch_t(const GemmArgs& g, hipStream_t st) {
  if constexpr (EPI == EPI_GLU_BF16) {
    launch_tile<256, 256, TA, TB, EPI, ACT>(g, st);
  } else if constexpr (EPI == EPI_F32_SEGMENTS) {
    if (small_sums(g))
      launch_tile<128, 128, TA, TB, EPI, ACT>(g, st);
    else
      launch_tile<256, 128, TA, TB, EPI, ACT>(g, st);
  } else {
    if (tile_size(g) == 128)
      launch_tile<128, 128, TA, TB, EPI, ACT>(g, st);
    else
      launch_tile<256, 256, TA, TB, EPI, ACT>(g, st);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm(const GemmArgs& g, bool ta, bool tb, int epi, hipStream_t st) {
  if (g.M % 256 || g.N % 256 || g.K % 256 || g.K <= 0 || g.nb < 1 || g.nb > 3 || g.ns < 1 || g.ns > 3 || (g.nb > 1 && g.ns > 1))
    return hipErrorInvalidValue;
  if (epi == EPI_GLU_BF16 && (g.nb > 1 || g.ns > 1)) return hipErrorInvalidValue;
  if (g.kseg < 0 || g.kseg % 256 || (g.kseg && (g.ns > 1 || g.K % g.kseg))) return hipErrorInvalidValue;
  if (epi == EPI_F32 && g.kseg && g.kseg < g.K) epi = EPI_F32_SEGMENTS;
#define RA_GEMM_CASE(TA_, TB_, E_) \
  if (ta == TA_ && tb == TB_ && epi == E_) return launch_t<TA_, TB_, E_, 0>(g, st);
#define RA_GEMM_CASE_ACT(TA_, TB_, E_)                                                 \
  if (ta == TA_ && tb == TB_ && epi == E_) {                                           \
    if (g.act == RA_ACT_RELU) return launch_t<TA_, TB_, E_, RA_ACT_RELU>(g, st);       \
    if (g.act == RA_ACT_GELU_TANH) return launch_t<TA_, TB_, E_, RA_ACT_GELU_TANH>(g, st); \
    return launch_t<TA_, TB_, E_, RA_ACT_GELU_ERF>(g, st);                             \
  }
  RA_GEMM_CASE(false, false, EPI_BF16)
  RA_GEMM_CASE_ACT(false, false, EPI_ACT_BF16)
  RA_GEMM_CASE_ACT(false, false, EPI_ACT_STORE_H)
  RA_GEMM_CASE(false, true, EPI_BF16)
  RA_GEMM_CASE_ACT(false, true, EPI_ACT_GRAD_BF16)
  RA_GEMM_CASE(true, false, EPI_F32)
  RA_GEMM_CASE(false, true, EPI_F32)
  RA_GEMM_CASE(true, false, EPI_F32_SEGMENTS)
  RA_GEMM_CASE(false, false, EPI_GLU_BF16)
  RA_GEMM_CASE(false, true, EPI_GLU_GRAD)
#undef RA_GEMM_CASE
#undef RA_GEMM_CASE_ACT
  return hipErrorInvalidValue;
}

hipError_t launch_colsum_bf16(const void* x, float* part, float* out, int M, int N, int accumulate,
                              hipStream_t st) {
  hipLaunchKernelGGL(colsum_partial_kernel, dim3((N + 511) / 512, kCS), dim3(256), 0, st, (const bf16*)x, part, M,
                     N);
  hipLaunchKernelGGL(colsum_final_kernel, dim3((N + 255) / 256), dim3(256), 0, st, part, out, N, accumulate);
  return hipGetLastError();
}

size_t colsum_workspace_floats(int N) { return (size_t)kCS * N; }

}  // namespace ra
