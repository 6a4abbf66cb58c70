// Ring-attention backward step kernels for gfx950.
//
// The backward pass of the paper's Appendix A keeps dq on the host and lets dk, dv
// travel with their key/value block; each step adds one block's contribution.  With
// the saved log-sum-exp of each query row, the normalised probabilities are recomputed
// (gradient checkpointing: nothing of size [queries, keys] is stored) and
//     P = exp(s - lse),  dV += P^T dO,  dP = dO V^T,  dS = P * (dP - Delta),
//     dQ += dS K / sqrt(D),  dK += dS^T Q / sqrt(D),   Delta_r = sum_d dO_rd O_rd.
// Two kernels: one owning key tiles (dK, dV in registers, looping over the query tiles that
// see them) and one owning query tiles (dQ in registers, looping over key tiles).  Both write
// their tile once, so no atomics are needed.
//
// In bf16 each covers the whole ring in one launch, or one ring step of the listed hosts.
// Over the whole ring the gradients stay in registers; a launch per step read and wrote them
// in float32 at every step (3.7 GB at 16384 tokens x 16 heads, all workgroups of a step at
// once, a quarter of a dV/dK wave's life) and had a grid tail each.  Backward of 16384 x 16,
// 8 hosts: 4190 us in 16 launches, 3220 in two; 4 x 2048 x 12 heads of 64, 4 hosts: 405, 215;
// 2 x 3001 x 8, 8 hosts (ragged): 457 without the staging copies, 165.
#include <type_traits>

#include "ra_common.h"
#include "ra_dma.h"
#include "ra_kernels.h"

namespace ra {
namespace {


// -------------------------------------------------------------------------------------
// Delta_r = sum_d dO_rd * O_rd  (float32 [B, H, S]).  A workgroup takes a tile of kPreR
// consecutive query rows x kPreH consecutive heads of one batch: TPR threads per (row,
// head) read that row of o and dO, heads fastest (so a row's kPreH heads are one contiguous
// run of memory); the sums pass through LDS, and the results (and lse) are then written
// (read) head by head as runs of kPreR consecutive floats.
// The bf16 step kernels take -Delta and -lse sqrt(D) (their accumulators start there:
// the score accumulators hold q.k, in units of the unscaled products).
// -------------------------------------------------------------------------------------
constexpr int kPreR = 16, kPreH = 8, kPreTile = kPreR * kPreH;

__device__ __forceinline__ void pre_tile(int S, int H, int& b, int& r0, int& h0) {
  const int nht = (H + kPreH - 1) / kPreH, nrt = (S + kPreR - 1) / kPreR;
  const int t = blockIdx.x;
  h0 = (t % nht) * kPreH;
  r0 = ((t / nht) % nrt) * kPreR;
  b = t / (nht * nrt);
}

template <int D>
__global__ __launch_bounds__(256) void bwd_pre_bf16_kernel(const bf16* o, const bf16* dO, const float* lse,
                                                           float* ndelta, float* nlse_s, int B, int S, int H) {
  constexpr int TPR = D / 8;      // threads per (row, head)
  constexpr int RPP = 256 / TPR;  // (row, head) pairs per pass
  constexpr int NP = kPreTile / RPP;
  __shared__ float sums[kPreTile];
  int b, r0, h0;
  pre_tile(S, H, b, r0, h0);
  const int c = (threadIdx.x % TPR) * 8;
  float s[NP];
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    const int q = k * RPP + threadIdx.x / TPR, r = r0 + q / kPreH, h = h0 + q % kPreH;
    s[k] = 0.f;
    if (r < S && h < H) {
      const long long row = ((long long)b * S + r) * H + h;
      const bf16x8 a = *(const bf16x8*)(o + row * D + c);
      const bf16x8 g = *(const bf16x8*)(dO + row * D + c);
#pragma unroll
      for (int e = 0; e < 8; ++e) s[k] = fmaf((float)a[e], (float)g[e], s[k]);
    }
  }
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    for (int off = TPR / 2; off > 0; off >>= 1) s[k] += __shfl_xor(s[k], off, 64);
    if (threadIdx.x % TPR == 0) sums[k * RPP + threadIdx.x / TPR] = s[k];
  }
  __syncthreads();
  if (threadIdx.x < kPreTile) {
    const int r = r0 + threadIdx.x % kPreR, h = h0 + threadIdx.x / kPreR;
    if (r < S && h < H) {
      const long long idx = ((long long)b * H + h) * S + r;
      ndelta[idx] = -sums[(threadIdx.x % kPreR) * kPreH + threadIdx.x / kPreR];
      nlse_s[idx] = -lse[idx] * sqrtf((float)D);  // lse / scale: units of q.k
    }
  }
}

template <int D>
__global__ __launch_bounds__(256) void bwd_pre_f32_kernel(const float* o, const float* dO, float* delta,
                                                          int B, int S, int H) {
  constexpr int TPR = D / 4;
  constexpr int RPP = 256 / TPR;
  constexpr int NP = kPreTile / RPP;
  __shared__ float sums[kPreTile];
  int b, r0, h0;
  pre_tile(S, H, b, r0, h0);
  const int c = (threadIdx.x % TPR) * 4;
  float s[NP];
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    const int q = k * RPP + threadIdx.x / TPR, r = r0 + q / kPreH, h = h0 + q % kPreH;
    s[k] = 0.f;
    if (r < S && h < H) {
      const long long row = ((long long)b * S + r) * H + h;
      const f32x4 a = *(const f32x4*)(o + row * D + c);
      const f32x4 g = *(const f32x4*)(dO + row * D + c);
#pragma unroll
      for (int e = 0; e < 4; ++e) s[k] = fmaf(a[e], g[e], s[k]);
    }
  }
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    for (int off = TPR / 2; off > 0; off >>= 1) s[k] += __shfl_xor(s[k], off, 64);
    if (threadIdx.x % TPR == 0) sums[k * RPP + threadIdx.x / TPR] = s[k];
  }
  __syncthreads();
  if (threadIdx.x < kPreTile) {
    const int r = r0 + threadIdx.x % kPreR, h = h0 + threadIdx.x / kPreR;
    if (r < S && h < H) delta[((long long)b * H + h) * S + r] = sums[(threadIdx.x % kPreR) * kPreH + threadIdx.x / kPreR];
  }
}

// Accumulators of a workgroup's dK (DK) or dV (lanes over keys, accumulated transposed:
// register 4 gg + e of product tile dt holds d = 32 dt + 8 gg + 4 hi + e).
// dkdv_start: their values before the first tile -- zero, or what the block's earlier ring
// steps accumulated.  dkdv_finish: the whole ring done, dK and dV go out in bf16 (dK carries
// the 1/sqrt(D)); steps to come, the accumulators are saved as they are, so that a call cut
// into steps adds up in the order of a call made of one launch; one host's share: its
// contribution is added to the float32 gradient that travels with the block.
template <int NDT, bool DK, class P>
__device__ __forceinline__ void dkdv_start(const P& p, int slot, int b, int h, int key_in_blk, int hi,
                                           f32x16 (&acc)[NDT]) {
  constexpr int D = 32 * NDT;
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[dt][i] = 0.f;
  if constexpr (std::is_same_v<P, BwdStep>) {
    if (!p.whole || (p.dkv_flags[slot] & kFirst)) return;
    const long long row = min(p.dkv_row0[slot] + key_in_blk, p.Skv - 1);
    const float* g32 = (DK ? p.dk : p.dv) + (long long)b * p.dkv_bstride + row * (p.H * D) + h * D;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int gg = 0; gg < 4; ++gg) {
        const f32x4 c4 = *(const f32x4*)(g32 + 32 * dt + 8 * gg + 4 * hi);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[dt][4 * gg + e] = c4[e];
      }
  }
}

template <int NDT, bool DK, class P>
__device__ __forceinline__ void dkdv_finish(const P& p, int slot, int b, int h, int key_in_blk, int hi,
                                            f32x16 (&acc)[NDT]) {
  constexpr int D = 32 * NDT;
  constexpr bool STEP = std::is_same_v<P, BwdStep>;
  const int rs = p.H * D;
  const float sc = DK ? p.scale : 1.f;
  bool out16 = true;
  long long grow;
  bf16* o16;
  if constexpr (STEP) {
    const int row = p.dkv_row0[slot] + key_in_blk;
    if (row >= p.Skv) return;
    grow = (long long)b * p.dkv_bstride + (long long)row * rs + h * D;
    out16 = p.whole && (p.dkv_flags[slot] & kLast);
    o16 = (bf16*)(DK ? p.dk_out : p.dv_out);
  } else {
    if (key_in_blk >= p.S) return;
    grow = (long long)b * p.bstride + (long long)key_in_blk * rs + h * D;
    o16 = (bf16*)(DK ? p.dk : p.dv);
  }
  if (out16) {
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int gg = 0; gg < 4; ++gg) {
        const f32x16& a = acc[dt];
        *(u32x2*)(o16 + grow + 32 * dt + 8 * gg + 4 * hi) =
            u32x2{pack_bf16x2(a[4 * gg] * sc, a[4 * gg + 1] * sc), pack_bf16x2(a[4 * gg + 2] * sc, a[4 * gg + 3] * sc)};
      }
  } else if constexpr (STEP) {
    float* g32 = (DK ? p.dk : p.dv) + grow;
    if (!p.whole) {  // every carried value loaded before the first store
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int gg = 0; gg < 4; ++gg) {
          const f32x4 c4 = *(const f32x4*)(g32 + 32 * dt + 8 * gg + 4 * hi);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[dt][4 * gg + e] = DK ? c4[e] + acc[dt][4 * gg + e] * sc : c4[e] + acc[dt][4 * gg + e];
        }
    }
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int gg = 0; gg < 4; ++gg) {
        const f32x16& a = acc[dt];
        *(f32x4*)(g32 + 32 * dt + 8 * gg + 4 * hi) = f32x4{a[4 * gg], a[4 * gg + 1], a[4 * gg + 2], a[4 * gg + 3]};
      }
  }
}

// What a dK/dV workgroup works on: 128 keys and the 32-query tiles that see them, in ring
// order.  One ring step: the tiles of the host that holds the block (rows q_row0 of q space).
// The whole ring: the hosts that fold block j do so in the order j, j + 1, ... (mod N), so
// their queries are simply the rows from block j on (causal: to the end; else around the
// ring, back to row wrap).
struct KeyTile {
  int slot, bh;
  int key0;            // first key (row of k / v, from the block's base)
  int kpos0;           // its global position
  int kv_rows;         // rows of k / v that exist
  int q_row0, q_pos0;  // q-space row and position of query tile 0
  int q_rows;          // rows of q space that exist
  int qt0, qt_free, n; // first tile, first one without mask (relative to tile 0), tiles visited
  int wrap;            // tile index at which the walk continues at row 0 of q space
  long long q_bs, kv_bs;
  const bf16 *k, *v;
};

template <int D, class P>
__device__ __forceinline__ bool key_tile(const P& p, KeyTile& t) {
  constexpr int kKB = 128, kQB = 32;
  if constexpr (std::is_same_v<P, BwdRing>) {
    const int n_kt = (p.S + kKB - 1) / kKB;
    int tile;
    if (!ring_item(blockIdx.x, p.B * p.H, n_kt, (long long)p.S * (D * 4), t.bh, tile)) return false;
    const int kt = n_kt - 1 - tile;  // under the causal mask the first keys have the most queries
    const int n_q = (p.S + kQB - 1) / kQB;
    t.slot = 0;
    t.key0 = t.kpos0 = kt * kKB;
    t.kv_rows = t.q_rows = p.S;
    t.q_row0 = t.q_pos0 = 0;
    t.q_bs = t.kv_bs = p.bstride;
    t.wrap = n_q;
    if (p.causal) {
      t.qt0 = t.key0 / kQB;
      t.qt_free = t.qt0 + kKB / kQB;
      t.n = n_q - t.qt0;
    } else {
      t.qt0 = t.key0 / p.c * (p.c / kQB);
      t.qt_free = t.qt0;
      t.n = n_q;
    }
    t.k = (const bf16*)p.k;
    t.v = (const bf16*)p.v;
  } else {
    const int n_kt = p.c / kKB, BH = p.B * p.H;
    const int id = xcd_swizzle(blockIdx.x, p.n_slots * BH * n_kt);
    const int grp = id / n_kt, kt = id % n_kt;
    t.slot = grp / BH;
    t.bh = grp % BH;
    const StepHost& hs = p.host[t.slot];
    t.key0 = kt * kKB;
    t.kpos0 = hs.k_pos0 + t.key0;
    t.kv_rows = hs.kv_rows;
    t.q_row0 = hs.q_row0;
    t.q_pos0 = hs.q_pos0;
    t.q_rows = p.Sq;
    t.q_bs = p.q_bstride;
    t.kv_bs = hs.kv_bstride;
    const int n_q = (min(p.c, p.Sq - hs.q_row0) + kQB - 1) / kQB;  // <= 0: the host has no rows
    t.wrap = 0x7fffffff;
    t.qt0 = t.qt_free = 0;
    if (p.causal) {
      const int rel = t.kpos0 - hs.q_pos0;
      t.qt0 = rel <= 0 ? 0 : max(0, min(n_q, rel / kQB));
      t.qt_free = max(t.qt0, rel + kKB <= 0 ? 0 : (rel + kKB - 1 + kQB - 1) / kQB);
    }
    t.n = max(0, n_q - t.qt0);
    t.k = (const bf16*)hs.k;
    t.v = (const bf16*)hs.v;
  }
  return t.key0 < t.kv_rows;
}

// =====================================================================================
// bf16 dK/dV kernel (D = 64; D = 128 runs the split kernel below, whose waves hold the
// same products): 4 waves x 32 keys = 128 keys per workgroup; loops over 32-query tiles
// of the host's block.  Per wave, lanes run over the wave's keys:
//   S' = Q K^T - lse sqrt(D)   [query x key] (A = Q rows from LDS with row bits 2 and 3
//        swapped, B = K of the wave's keys in registers, as stored: the products are
//        exact in float32; the accumulator starts at -lse sqrt(D) of its query)
//   P  = exp2(S' log2e / sqrt(D))  (the scale in float32)       (masked -> 0)
//   dP = dO V^T - Delta   (A = dO rows, B = V in registers; starts at -Delta)
//   dS = P * dP
//   dV^T += dO^T P        (A = dO^T by LDS transpose read, B = P)
//   dK^T += Q^T dS        (A = Q^T by LDS transpose read, B = dS)
// Q and dO tiles (XOR-swizzled rows) and the tile's -lse sqrt(D) and -Delta are filled by
// direct-to-LDS buffer loads into a ring of three buffers (25.5 KB for D = 64, so every
// LDS address fits the reads' immediate offsets).  The loop is software pipelined: while
// tile t's P and dS are formed on the vector ALUs and its dV, dK products run, the S' and
// dP products of tile t+1 are issued and tile t+2 streams in.
// Two workgroups a CU (204 registers): with one wave a SIMD the matrix core idled during its
// vector work and LDS waits.  Backward with one, two waves a SIMD, us: 16384 x 16 heads, causal
// 2254, 1871; 4 x 2048 x 12, bidirectional 238, 204; 1024 x 8 53, 52.
// =====================================================================================
constexpr int kKB = 128, kQB = 32, kBT = 256;

template <int D, class P>
__global__ __launch_bounds__(kBT, 2) void bwd_dkdv_bf16_kernel(const P p) {
  constexpr int NKK = D / 16, NDT = D / 32, CPR = D / 8;
  constexpr int ROWS_PER_LOAD = 64 / CPR, LOADS = kQB / 4 / ROWS_PER_LOAD;
  static_assert(LOADS >= 1, "each wave fills at least one 1 KB row group");
  // one LDS object per buffer, so that reads of one are known not to alias the
  // direct-to-LDS loads in flight into another (else the compiler waits for them)
  __shared__ __attribute__((aligned(1024))) bf16 sQ0[kQB * D];
  __shared__ __attribute__((aligned(1024))) bf16 sQ1[kQB * D];
  __shared__ __attribute__((aligned(1024))) bf16 sQ2[kQB * D];
  __shared__ __attribute__((aligned(1024))) bf16 sO0[kQB * D];  // dO tiles
  __shared__ __attribute__((aligned(1024))) bf16 sO1[kQB * D];
  __shared__ __attribute__((aligned(1024))) bf16 sO2[kQB * D];
  // -lse sqrt(D) and -Delta: 64 floats each, as a one-wave 4-byte load writes 256 bytes
  // (lanes past the tile read zero)
  __shared__ __attribute__((aligned(256))) float sL0[64];  // -lse sqrt(D)
  __shared__ __attribute__((aligned(256))) float sL1[64];
  __shared__ __attribute__((aligned(256))) float sL2[64];
  __shared__ __attribute__((aligned(256))) float sD0[64];  // -Delta
  __shared__ __attribute__((aligned(256))) float sD1[64];
  __shared__ __attribute__((aligned(256))) float sD2[64];
  auto pick = [](auto Bc, auto* a, auto* b, auto* c) __attribute__((always_inline)) {
    constexpr int B = decltype(Bc)::value % 3;
    if constexpr (B == 0) return a; else if constexpr (B == 1) return b; else return c;
  };

  KeyTile kt;
  if (!key_tile<D>(p, kt)) return;
  const int b = kt.bh / p.H, h = kt.bh % p.H;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);  // uniform: LDS destinations in scalar registers
  const int rs = p.H * D;
  const float sl2 = p.scale * kLog2e;

  const int key_in_blk = kt.key0 + wave * 32 + l32;  // this lane's key (B-operand column)
  const int kpos = kt.kpos0 + wave * 32 + l32;
  bf16x8 kreg[NKK], vreg[NKK];
  {
    const long long off = (long long)b * kt.kv_bs + (long long)min(key_in_blk, kt.kv_rows - 1) * rs + h * D;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      kreg[kk] = *(const bf16x8*)(kt.k + off + 16 * kk + 8 * hi);
      vreg[kk] = *(const bf16x8*)(kt.v + off + 16 * kk + 8 * hi);
    }
  }
  f32x16 dkacc[NDT], dvacc[NDT];
  dkdv_start<NDT, true>(p, kt.slot, b, h, key_in_blk, hi, dkacc);
  dkdv_start<NDT, false>(p, kt.slot, b, h, key_in_blk, hi, dvacc);

  const bf16* qbase = (const bf16*)p.q + (long long)b * kt.q_bs + h * D;
  const bf16* obase = (const bf16*)p.dO + (long long)b * kt.q_bs + h * D;
  const long long lrow0 = (long long)kt.bh * kt.q_rows;
  constexpr int RPW = kQB / 4;  // tile rows each wave fills
  int goff[LOADS];
#pragma unroll
  for (int j = 0; j < LOADS; ++j) {
    const int r = wave * RPW + j * ROWS_PER_LOAD + lane / CPR;
    goff[j] = 2 * (r * rs + 8 * ((lane % CPR) ^ swz<D>(r)));
  }
  auto load_tile = [&](int i, auto Bc) __attribute__((always_inline)) {
    const int row = kt.q_row0 + (kt.qt0 + i - (kt.qt0 + i >= kt.wrap ? kt.wrap : 0)) * kQB;
    const int rows = min(kQB, kt.q_rows - row);
    const long long t0 = (long long)row * rs;
#pragma unroll
    for (int j = 0; j < LOADS; ++j) {
      buffer_load_lds16(qbase + t0, rows * rs * 2, pick(Bc, sQ0, sQ1, sQ2) + (wave_u * RPW + j * ROWS_PER_LOAD) * D,
                        goff[j]);
      buffer_load_lds16(obase + t0, rows * rs * 2, pick(Bc, sO0, sO1, sO2) + (wave_u * RPW + j * ROWS_PER_LOAD) * D,
                        goff[j]);
    }
    if (wave_u == 0) buffer_load_lds4(p.lse + lrow0 + row, rows * 4, pick(Bc, sL0, sL1, sL2), 4 * lane);
    if (wave_u == 1) buffer_load_lds4(p.delta + lrow0 + row, rows * 4, pick(Bc, sD0, sD1, sD2), 4 * lane);
  };
  const int qrow = swap_bits23(l32);
  int roff[NKK];
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) roff[kk] = qrow * D + 8 * ((2 * kk + hi) ^ swz<D>(qrow));
  const int g16 = lane >> 4, li = lane & 15;
  int toff[2][NDT];
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) {
      const int row = 8 * hi + 4 * r + (li >> 2);
      const int d = 32 * dt + 16 * (g16 & 1) + 4 * (li & 3);
      toff[r][dt] = row * D + 8 * ((d >> 3) ^ swz<D>(row)) + (d & 7);
    }

  // accumulator starts of S' (-lse sqrt(D)) and dP (-Delta), stored negated by the
  // preprocess kernel, of a tile: register 8 g + e of a lane holds query 16 g + 8 hi + e
  auto inits = [&](auto Bc, f32x16& si, f32x16& di) __attribute__((always_inline)) {
    const float* sl = pick(Bc, sL0, sL1, sL2);
    const float* sd = pick(Bc, sD0, sD1, sD2);
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const int q0 = 16 * g + 8 * hi;
      const f32x4 la = *(const f32x4*)&sl[q0], lb = *(const f32x4*)&sl[q0 + 4];
      const f32x4 da = *(const f32x4*)&sd[q0], db = *(const f32x4*)&sd[q0 + 4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        si[8 * g + e] = la[e];
        si[8 * g + 4 + e] = lb[e];
        di[8 * g + e] = da[e];
        di[8 * g + 4 + e] = db[e];
      }
    }
  };
  // P and dS (bf16 pairs) of group g (16 queries) of a tile, pair u of the group's 4
  auto unit = [&](auto Mc, const f32x16& sc, const f32x16& dpc, int qpos0, int g, int u, uint32_t& w1,
                  uint32_t& w2) __attribute__((always_inline)) {
    constexpr bool MASK = decltype(Mc)::value;
    float pv[2], dsv[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int r = 8 * g + 2 * u + e;
      float pr = fast_exp2(sc[r] * sl2);
      if (MASK && kpos > qpos0 + 16 * g + 8 * hi + 2 * u + e) pr = 0.f;
      pv[e] = pr;
      dsv[e] = pr * dpc[r];
    }
    w1 = pack_bf16x2(pv[0], pv[1]);
    w2 = pack_bf16x2(dsv[0], dsv[1]);
  };

  // One tile t (buffer Bc): loads of tile t+2 (buffer Bc+2), the S'/dP products of tile t+1
  // (buffer Bc+1; Nc: it exists) and, for tile t, P and dS in two groups of 16 queries, each
  // followed by its dV and dK products; then the wait for tile t+2 and the barrier that frees
  // buffer Bc.
  auto tile = [&](auto Bc, auto Mc, auto Nc, int i, f32x16& s_cur, f32x16& dp_cur) __attribute__((always_inline)) {
    constexpr int B = decltype(Bc)::value;
    constexpr bool NX = decltype(Nc)::value;
    using Bn = std::integral_constant<int, (B + 1) % 3>;
    using Bl = std::integral_constant<int, (B + 2) % 3>;
    if (i + 2 < kt.n) load_tile(i + 2, Bl{});
    const bf16* qn = pick(Bn{}, sQ0, sQ1, sQ2);  // next tile: row reads
    const bf16* on = pick(Bn{}, sO0, sO1, sO2);
    const bf16* qc = pick(Bc, sQ0, sQ1, sQ2);    // this tile: transpose reads
    const bf16* oc = pick(Bc, sO0, sO1, sO2);
    const int qpos0 = kt.q_pos0 + (kt.qt0 + i) * kQB;
    f32x16 s_nx, dp_nx;
    if constexpr (NX) inits(Bn{}, s_nx, dp_nx);
    if constexpr (NX) {
#pragma unroll
      for (int kk = 0; kk < NKK; ++kk) {
        s_nx = mfma32(*(const bf16x8*)(qn + roff[kk]), kreg[kk], s_nx);
        dp_nx = mfma32(*(const bf16x8*)(on + roff[kk]), vreg[kk], dp_nx);
      }
    }
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      uint32_t wp[4], ws[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) unit(Mc, s_cur, dp_cur, qpos0, g, u, wp[u], ws[u]);
      const bf16x8 pbg = __builtin_bit_cast(bf16x8, u32x4{wp[0], wp[1], wp[2], wp[3]});
      const bf16x8 dsg = __builtin_bit_cast(bf16x8, u32x4{ws[0], ws[1], ws[2], ws[3]});
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) {
        const bf16x4 olo = lds_read_tr16(oc + 16 * g * D + toff[0][dt]);
        const bf16x4 oup = lds_read_tr16(oc + 16 * g * D + toff[1][dt]);
        dvacc[dt] = mfma32(bf16x8{olo[0], olo[1], olo[2], olo[3], oup[0], oup[1], oup[2], oup[3]}, pbg, dvacc[dt]);
        const bf16x4 qlo = lds_read_tr16(qc + 16 * g * D + toff[0][dt]);
        const bf16x4 qup = lds_read_tr16(qc + 16 * g * D + toff[1][dt]);
        dkacc[dt] = mfma32(bf16x8{qlo[0], qlo[1], qlo[2], qlo[3], qup[0], qup[1], qup[2], qup[3]}, dsg, dkacc[dt]);
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // tile t+2 landed
    __syncthreads();                                   // and buffer Bc is free again
    if constexpr (NX) {
      s_cur = s_nx;
      dp_cur = dp_nx;
    }
  };

  if (kt.n > 0) {
    load_tile(0, std::integral_constant<int, 0>{});
    if (kt.n > 1) load_tile(1, std::integral_constant<int, 1>{});
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    f32x16 s_cur, dp_cur;  // S' and dP of the tile being processed
    inits(std::integral_constant<int, 0>{}, s_cur, dp_cur);
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      s_cur = mfma32(*(const bf16x8*)(sQ0 + roff[kk]), kreg[kk], s_cur);
      dp_cur = mfma32(*(const bf16x8*)(sO0 + roff[kk]), vreg[kk], dp_cur);
    }
    // buffer of tile i is i % 3, known at compile time in a loop unrolled by 3; tiles [a, e)
    // all have a successor
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    auto run = [&](auto Mc, int a, int e) __attribute__((always_inline)) {
      int it = a;
      if (it < e && it % 3 == 1) tile(I1{}, Mc, std::true_type{}, it++, s_cur, dp_cur);
      if (it < e && it % 3 == 2) tile(I2{}, Mc, std::true_type{}, it++, s_cur, dp_cur);
      for (; it + 2 < e; it += 3) {
        tile(I0{}, Mc, std::true_type{}, it, s_cur, dp_cur);
        tile(I1{}, Mc, std::true_type{}, it + 1, s_cur, dp_cur);
        tile(I2{}, Mc, std::true_type{}, it + 2, s_cur, dp_cur);
      }
      if (it < e) tile(I0{}, Mc, std::true_type{}, it++, s_cur, dp_cur);
      if (it < e) tile(I1{}, Mc, std::true_type{}, it++, s_cur, dp_cur);
    };
    const int il = kt.n - 1;
    const int split = max(0, min(kt.qt_free - kt.qt0, il));  // masked tiles first
    run(std::true_type{}, 0, split);
    run(std::false_type{}, split, il);
    // last tile: no successor
    const int ph = il % 3;
    auto last = [&](auto Mc) __attribute__((always_inline)) {
      if (ph == 0) tile(I0{}, Mc, std::false_type{}, il, s_cur, dp_cur);
      else if (ph == 1) tile(I1{}, Mc, std::false_type{}, il, s_cur, dp_cur);
      else tile(I2{}, Mc, std::false_type{}, il, s_cur, dp_cur);
    };
    if (kt.qt0 + il < kt.qt_free) last(std::true_type{}); else last(std::false_type{});
  }

  dkdv_finish<NDT, true>(p, kt.slot, b, h, key_in_blk, hi, dkacc);
  dkdv_finish<NDT, false>(p, kt.slot, b, h, key_in_blk, hi, dvacc);
}

// =====================================================================================
// bf16 dK/dV kernel for D = 128 with the work of each 32-key column split over three
// waves: 12 waves and 128 keys per workgroup, three waves on every SIMD.
//   row wave (w < 4, column w): holds K and V of keys 32 w .. 32 w + 31 in registers and,
//     per 32-query tile, runs the products contracted over D and the vector work
//       S' = Q K^T - lse sqrt(D),  dP = dO V^T - Delta,
//       P = exp2(S' log2e / sqrt(D)) (masked -> 0),  dS = P * dP,
//     and stores P and dS, packed to bf16 in the lane order of a B operand, to LDS;
//   dV wave (w = 4 + column), one tile later:  dV^T += dO^T P;
//   dK wave (w = 8 + column), one tile later:  dK^T += Q^T dS
//     (A operands by LDS transpose reads; each of the two holds 64 accumulator registers).
// At 162 registers a wave, three waves share each SIMD: the row wave is mostly vector
// work, the other two only matrix products and LDS reads, so each covers the others'
// waits for LDS and for the barrier (with one wave per SIMD, as in the kernel above, those
// waits leave the matrix core idle).  The operands and their order of accumulation are
// those of the one-wave kernel, so the results are the same bit for bit.
// Q and dO tiles (XOR-swizzled rows) with the tile's -lse sqrt(D) and -Delta stream by
// direct-to-LDS loads (waves 0-7, 4 rows each) into a ring of four buffers: in the region
// of tile t the row waves read tile t+1, the dV and dK waves tile t-1, and tile t+2 streams
// in.  The packed P and dS pass through two exchange buffers; one barrier per tile.
// =====================================================================================
constexpr int kPT = 768;

template <class P>
__global__ __launch_bounds__(kPT) void bwd_dkdv_split_kernel(const P p) {
  constexpr int D = 128, NKK = D / 16, NDT = D / 32, CPR = D / 8, ROWS_PER_LOAD = 64 / CPR;
  static_assert(kQB == 8 * ROWS_PER_LOAD, "waves 0-7 fill 4 rows of a tile each");
  // Q tiles 0-3, then dO tiles 0-3, in one LDS object, so that every read of a ring buffer
  // is one lane offset plus an immediate; filled by direct-to-LDS loads the compiler does
  // not track (the region's explicit vmcnt wait and barrier order them)
  __shared__ __attribute__((aligned(1024))) bf16 sQO[8 * kQB * D];
  // -lse sqrt(D) of tiles 0-3, then -Delta: 64 floats each, as a one-wave 4-byte load
  // writes 256 bytes (lanes past the tile read zero)
  __shared__ __attribute__((aligned(1024))) float sLD[8 * 64];
  // packed P and dS of a tile: [column][P of queries 0-15, 16-31, dS of 0-15, 16-31][lane]
  __shared__ __attribute__((aligned(1024))) u32x4 sX0[4 * 4 * 64];
  __shared__ __attribute__((aligned(1024))) u32x4 sX1[4 * 4 * 64];
  auto qt_lds = [&](auto Bc) __attribute__((always_inline)) { return sQO + (decltype(Bc)::value % 4) * kQB * D; };
  auto ot_lds = [&](auto Bc) __attribute__((always_inline)) { return sQO + (4 + decltype(Bc)::value % 4) * kQB * D; };
  auto l_lds = [&](auto Bc) __attribute__((always_inline)) { return sLD + (decltype(Bc)::value % 4) * 64; };
  auto d_lds = [&](auto Bc) __attribute__((always_inline)) { return sLD + (4 + decltype(Bc)::value % 4) * 64; };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;

  KeyTile kt;
  if (!key_tile<D>(p, kt)) return;
  const int b = kt.bh / p.H, h = kt.bh % p.H;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
  const int wave_u = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: LDS destinations in scalar registers
  const int col = wave_u & 3;                                   // the wave's 32-key column
  const int rs = p.H * D;
  const int key_in_blk = kt.key0 + col * 32 + l32;  // this lane's key (B-operand column)
  const int n = kt.n;  // tiles visited

  const bf16* qbase = (const bf16*)p.q + (long long)b * kt.q_bs + h * D;
  const bf16* obase = (const bf16*)p.dO + (long long)b * kt.q_bs + h * D;
  const long long lrow0 = (long long)kt.bh * kt.q_rows;
  const int lrow = (wave_u & 7) * ROWS_PER_LOAD + lane / CPR;  // the tile row this lane fills (waves 0-7)
  const int goff = 2 * (lrow * rs + 8 * ((lane % CPR) ^ swz<D>(lrow)));
  // tile i into ring buffer buf: the Q and dO rows by waves 0-7, -lse sqrt(D) by wave 0,
  // -Delta by wave 1
  auto load_tile = [&](int i, int buf) __attribute__((always_inline)) {
    const int row = kt.q_row0 + (kt.qt0 + i - (kt.qt0 + i >= kt.wrap ? kt.wrap : 0)) * kQB;
    const int rows = min(kQB, kt.q_rows - row);  // rows past the end read as zero
    const long long t0 = (long long)row * rs;
    if (wave_u < 8) {
      dma_lds16(make_rsrc(qbase + t0, rows * rs * 2), lds_addr(sQO + (buf * kQB + wave_u * ROWS_PER_LOAD) * D), goff);
      dma_lds16(make_rsrc(obase + t0, rows * rs * 2), lds_addr(sQO + ((4 + buf) * kQB + wave_u * ROWS_PER_LOAD) * D),
                goff);
    }
    if (wave_u == 0) dma_lds4(make_rsrc(p.lse + lrow0 + row, rows * 4), lds_addr(sLD + buf * 64), 4 * lane);
    if (wave_u == 1) dma_lds4(make_rsrc(p.delta + lrow0 + row, rows * 4), lds_addr(sLD + (4 + buf) * 64), 4 * lane);
  };
  // regions [a, e) with the buffer of region i (i % 4) known at compile time
  auto run4 = [&](int a, int e, auto&& f) __attribute__((always_inline)) {
    int i = a;
    if (i < e && (i & 3) == 1) f(I1{}, i++);
    if (i < e && (i & 3) == 2) f(I2{}, i++);
    if (i < e && (i & 3) == 3) f(I3{}, i++);
    for (; i + 3 < e; i += 4) {
      f(I0{}, i);
      f(I1{}, i + 1);
      f(I2{}, i + 2);
      f(I3{}, i + 3);
    }
    if (i < e) f(I0{}, i++);
    if (i < e) f(I1{}, i++);
    if (i < e) f(I2{}, i++);
  };
  auto at = [&](int i, auto&& f) __attribute__((always_inline)) {  // one region, buffer i % 4
    switch (i & 3) {
      case 0: f(I0{}, i); break;
      case 1: f(I1{}, i); break;
      case 2: f(I2{}, i); break;
      default: f(I3{}, i); break;
    }
  };
  auto sync = [&]() __attribute__((always_inline)) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's loads of tile i+2 landed
    __syncthreads();                                   // every wave's; the exchange written
  };

  if (n > 0) {
    load_tile(0, 0);
    if (n > 1) load_tile(1, 1);
  }

  if (wave_u < 4) {
    // ---------------------------------------------------------------- row wave
    const int kpos = kt.kpos0 + col * 32 + l32;
    const float sl2 = p.scale * kLog2e;
    bf16x8 kreg[NKK], vreg[NKK];
    {
      const long long off = (long long)b * kt.kv_bs + (long long)min(key_in_blk, kt.kv_rows - 1) * rs + h * D;
#pragma unroll
      for (int kk = 0; kk < NKK; ++kk) {
        kreg[kk] = *(const bf16x8*)(kt.k + off + 16 * kk + 8 * hi);
        vreg[kk] = *(const bf16x8*)(kt.v + off + 16 * kk + 8 * hi);
      }
    }
    if (n == 0) return;
    const int qrow = swap_bits23(l32);
    int roff[NKK];
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) roff[kk] = qrow * D + 8 * ((2 * kk + hi) ^ swz<D>(qrow));
    // accumulator starts of S' (-lse sqrt(D)) and dP (-Delta) of a tile: register 8 g + e
    // of a lane holds query 16 g + 8 hi + e
    auto inits = [&](auto Bc, f32x16& si, f32x16& di) __attribute__((always_inline)) {
      const float* sl = l_lds(Bc);
      const float* sd = d_lds(Bc);
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const int q0 = 16 * g + 8 * hi;
        const f32x4 la = *(const f32x4*)&sl[q0], lb = *(const f32x4*)&sl[q0 + 4];
        const f32x4 da = *(const f32x4*)&sd[q0], db = *(const f32x4*)&sd[q0 + 4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          si[8 * g + e] = la[e];
          si[8 * g + 4 + e] = lb[e];
          di[8 * g + e] = da[e];
          di[8 * g + 4 + e] = db[e];
        }
      }
    };
    // P and dS (bf16 pairs) of group g (16 queries) of a tile, pair u of the group's 4
    auto unit = [&](auto Mc, const f32x16& sc, const f32x16& dpc, int qpos0, int g, int u, uint32_t& w1,
                    uint32_t& w2) __attribute__((always_inline)) {
      constexpr bool MASK = decltype(Mc)::value;
      float pv[2], dsv[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int r = 8 * g + 2 * u + e;
        float pr = fast_exp2(sc[r] * sl2);
        if (MASK && kpos > qpos0 + 16 * g + 8 * hi + 2 * u + e) pr = 0.f;
        pv[e] = pr;
        dsv[e] = pr * dpc[r];
      }
      w1 = pack_bf16x2(pv[0], pv[1]);
      w2 = pack_bf16x2(dsv[0], dsv[1]);
    };
    sync();
    f32x16 s_cur, dp_cur;  // S' and dP of the tile whose P and dS are formed next
    inits(I0{}, s_cur, dp_cur);
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      s_cur = mfma32(*(const bf16x8*)(qt_lds(I0{}) + roff[kk]), kreg[kk], s_cur);
      dp_cur = mfma32(*(const bf16x8*)(ot_lds(I0{}) + roff[kk]), vreg[kk], dp_cur);
    }
    // Region of tile i (buffer Bc; Nc: tile i+1 exists): loads of tile i+2, the S'/dP
    // products of tile i+1 in 16 fenced steps (S' and dP alternate; operand reads two
    // steps ahead), and P, dS of tile i, one pair unit at every even step; each group's
    // packed P and dS go to the exchange buffer of tile i once formed.
    auto region = [&](auto Bc, auto Mc, auto Nc, int i) __attribute__((always_inline)) {
      constexpr int B = decltype(Bc)::value;
      constexpr bool NX = decltype(Nc)::value;
      using Bn = std::integral_constant<int, (B + 1) % 4>;
      using Bl = std::integral_constant<int, (B + 2) % 4>;
      if (i + 2 < n) load_tile(i + 2, Bl::value);
      const bf16* qn = qt_lds(Bn{});
      const bf16* on = ot_lds(Bn{});
      u32x4* xw = ((B & 1) ? sX1 : sX0) + col * 4 * 64 + lane;
      const int qpos0 = kt.q_pos0 + (kt.qt0 + i) * kQB;
      f32x16 s_nx, dp_nx;
      if constexpr (NX) inits(Bn{}, s_nx, dp_nx);
      bf16x8 aop[16];
      uint32_t wp[2][4], ws[2][4];
      constexpr int kPF = 2;
      auto read_a = [&](auto Sc) __attribute__((always_inline)) {  // product s: kk = s / 2, dP if odd
        constexpr int S = decltype(Sc)::value;
        aop[S] = *(const bf16x8*)(((S & 1) ? on : qn) + roff[S / 2]);
      };
      if constexpr (NX) static_for<0, kPF>([&](auto Sc) __attribute__((always_inline)) { read_a(Sc); });
      static_for<0, 16>([&](auto Sc) __attribute__((always_inline)) {
        constexpr int S = decltype(Sc)::value;
        if constexpr (NX && S + kPF < 16) read_a(std::integral_constant<int, S + kPF>{});
        if constexpr (NX) {
          if constexpr (S & 1)
            dp_nx = mfma32(aop[S], vreg[S / 2], dp_nx);
          else
            s_nx = mfma32(aop[S], kreg[S / 2], s_nx);
        }
        if constexpr (S % 2 == 0) {
          constexpr int g = S / 8, u = (S % 8) / 2;
          unit(Mc, s_cur, dp_cur, qpos0, g, u, wp[g][u], ws[g][u]);
        }
        if constexpr (S % 8 == 7) {
          constexpr int g = S / 8;
          xw[g * 64] = u32x4{wp[g][0], wp[g][1], wp[g][2], wp[g][3]};
          xw[(2 + g) * 64] = u32x4{ws[g][0], ws[g][1], ws[g][2], ws[g][3]};
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      sync();
      if constexpr (NX) {
        s_cur = s_nx;
        dp_cur = dp_nx;
      }
    };
    // masked tiles first; every tile but the last has a successor
    const int ms = max(0, min(kt.qt_free - kt.qt0, n - 1));
    run4(0, ms, [&](auto Bc, int i) __attribute__((always_inline)) {
      region(Bc, std::true_type{}, std::true_type{}, i);
    });
    run4(ms, n - 1, [&](auto Bc, int i) __attribute__((always_inline)) {
      region(Bc, std::false_type{}, std::true_type{}, i);
    });
    if (kt.qt0 + n - 1 < kt.qt_free)
      at(n - 1, [&](auto Bc, int i) __attribute__((always_inline)) { region(Bc, std::true_type{}, std::false_type{}, i); });
    else
      at(n - 1, [&](auto Bc, int i) __attribute__((always_inline)) { region(Bc, std::false_type{}, std::false_type{}, i); });
    return;
  }

  // ------------------------------------------------------------------ column waves
  // waves 4-7 accumulate dV, waves 8-11 dK, of the column
  auto column = [&](auto Kc) __attribute__((always_inline)) {
    constexpr bool DK = decltype(Kc)::value;
    f32x16 acc[NDT];
    dkdv_start<NDT, DK>(p, kt.slot, b, h, key_in_blk, hi, acc);
    if (n > 0) {
      const int g16 = lane >> 4, li = lane & 15;
      int toff[2][NDT];
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) {
          const int row = 8 * hi + 4 * r + (li >> 2);
          const int d = 32 * dt + 16 * (g16 & 1) + 4 * (li & 3);
          toff[r][dt] = row * D + 8 * ((d >> 3) ^ swz<D>(row)) + (d & 7);
        }
      sync();
      for (int i = 0; i <= n; ++i) {
        if (i + 2 < n) load_tile(i + 2, (i + 2) & 3);
        if (i >= 1) {
          const u32x4* xr = (((i - 1) & 1) ? sX1 : sX0) + col * 4 * 64 + lane + (DK ? 128 : 0);
          const bf16x8 bop[2] = {__builtin_bit_cast(bf16x8, xr[0]), __builtin_bit_cast(bf16x8, xr[64])};
          const bf16* src = sQO + ((DK ? 0 : 4) + ((i - 1) & 3)) * kQB * D;
          bf16x8 top[8];
          constexpr int kPF = 2;
          auto read_t = [&](auto Qc) __attribute__((always_inline)) {  // product q: group q / 4, dt q % 4
            constexpr int Q = decltype(Qc)::value, g = Q / 4, dt = Q % 4;
            const bf16x4 lo = lds_read_tr16(src + 16 * g * D + toff[0][dt]);
            const bf16x4 up = lds_read_tr16(src + 16 * g * D + toff[1][dt]);
            top[Q] = bf16x8{lo[0], lo[1], lo[2], lo[3], up[0], up[1], up[2], up[3]};
          };
          static_for<0, kPF>([&](auto Qc) __attribute__((always_inline)) { read_t(Qc); });
          static_for<0, 8>([&](auto Qc) __attribute__((always_inline)) {
            constexpr int Q = decltype(Qc)::value, g = Q / 4, dt = Q % 4;
            if constexpr (Q + kPF < 8) read_t(std::integral_constant<int, Q + kPF>{});
            acc[dt] = mfma32(top[Q], bop[g], acc[dt]);
            __builtin_amdgcn_sched_barrier(0);
          });
        }
        if (i < n) sync();
      }
    }
    dkdv_finish<NDT, DK>(p, kt.slot, b, h, key_in_blk, hi, acc);
  };
  if (wave_u >= 8) column(std::true_type{});
  else column(std::false_type{});
}

// bf16 dQ kernel: 4 waves x 32 queries = 128 queries per workgroup; loops over 64-key
// tiles of the block.  Per wave, lanes run over queries:
//   S^T  = K Q^T            (A = K rows from LDS, B = Q in registers)
//   dP^T = V dO^T - Delta   (A = V rows, B = dO in registers; the accumulator starts at
//                            -Delta of the lane's query, so the subtraction is free)
//   P^T  = exp2(S^T log2e/sqrt(D) - lse log2e),  dS^T = P^T * dP^T   (masked -> 0), the
//          scale applied in float32
//   dQ^T += K^T dS^T        (A = K^T by LDS transpose read, B = dS^T)
// K and V tiles are filled by direct-to-LDS buffer loads into XOR-swizzled unpadded rows
// (see swz), double buffered: tile it+1 streams in while tile it is processed.
// =====================================================================================
constexpr int kQQ = 128, kKK = 64;

template <int D, class P>
__global__ __launch_bounds__(kBT, 2) void bwd_dq_bf16_kernel(const P p) {
  constexpr bool RING = std::is_same_v<P, BwdRing>;
  constexpr int NKK = D / 16, NDT = D / 32, CPR = D / 8;
  constexpr int ROWS_PER_LOAD = 64 / CPR, LOADS = kKK / 4 / ROWS_PER_LOAD;
  // one LDS array (K0, K1, V0, V1 tiles), filled by direct-to-LDS loads the compiler does
  // not track (each tile's loads are waited for before the barrier that ends the tile), so
  // that every read address is one register plus an immediate offset
  __shared__ __attribute__((aligned(1024))) bf16 lds[4 * kKK * D];
  bf16* const sK0 = lds;
  bf16* const sK1 = lds + kKK * D;
  bf16* const sV0 = lds + 2 * kKK * D;
  bf16* const sV1 = lds + 3 * kKK * D;
  auto pick = [](auto Bc, auto* a, auto* b) __attribute__((always_inline)) {
    if constexpr (decltype(Bc)::value == 0) return a; else return b;
  };

  // the workgroup's query rows and the blocks it folds (as in the forward kernel)
  int bh, q_tile_row, tile_first_q, k_pos0, kv_rows, q_rows, host = 0, flags = kFirst | kLast;
  long long q_bs;
  const bf16 *kbase, *vbase;
  const int blk_tiles = p.c / kKK;
  if constexpr (RING) {
    const int n_qt = (p.S + kQQ - 1) / kQQ;
    int qt;
    if (!ring_item(blockIdx.x, p.B * p.H, n_qt, (long long)p.S * (D * 4), bh, qt)) return;
    q_tile_row = tile_first_q = qt * kQQ;
    host = q_tile_row / p.c;
    k_pos0 = host * p.c;
    kv_rows = q_rows = p.S;
    q_bs = p.bstride;
    const long long off = (long long)(bh / p.H) * p.bstride + (bh % p.H) * D;
    kbase = (const bf16*)p.k + off;
    vbase = (const bf16*)p.v + off;
  } else {
    const int n_qt = p.c / kQQ;
    const int BH = p.B * p.H;
    const int L = xcd_swizzle(blockIdx.x, p.n_slots * BH * n_qt);
    const int grp = L / n_qt, qt = n_qt - 1 - (L % n_qt);
    const StepHost& hs = p.host[grp / BH];
    bh = grp % BH;
    q_tile_row = hs.q_row0 + qt * kQQ;
    tile_first_q = hs.q_pos0 + qt * kQQ;
    k_pos0 = hs.k_pos0;
    kv_rows = hs.kv_rows;
    q_rows = p.Sq;
    q_bs = p.q_bstride;
    flags = hs.flags;
    const long long off = (long long)(bh / p.H) * hs.kv_bstride + (bh % p.H) * D;
    kbase = (const bf16*)hs.k + off;
    vbase = (const bf16*)hs.v + off;
    if (q_tile_row >= p.Sq) return;
  }
  const int b = bh / p.H, h = bh % p.H;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);  // uniform: LDS destinations in scalar registers
  const int rs = p.H * D;

  const int qr = q_tile_row + wave * 32 + l32;
  const int qpos = tile_first_q + wave * 32 + l32;
  const int qr_ld = min(qr, q_rows - 1);  // rows past the end: any row (nothing of them is stored)
  const long long lrow = (long long)bh * q_rows + qr_ld;
  const long long qoff = (long long)b * q_bs + (long long)qr_ld * rs + h * D;
  const float nlse_s = p.lse[lrow];  // -lse sqrt(D) (written by the preprocess kernel)
  const float ndlt = p.delta[lrow];  // -Delta

  bf16x8 qreg[NKK], oreg[NKK];
  {
    const long long off = qoff + 8 * hi;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      qreg[kk] = *(const bf16x8*)((const bf16*)p.q + off + 16 * kk);
      oreg[kk] = *(const bf16x8*)((const bf16*)p.dO + off + 16 * kk);
    }
    // consume the loads here: otherwise the compiler, unsure whether they are still in
    // flight, waits on the load counter inside the loop, where it also counts the
    // prefetch of the next tile
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) asm volatile("" ::"v"(qreg[kk]), "v"(oreg[kk]));
  }
  // dQ^T: zero, or what the host's earlier ring steps accumulated
  f32x16 dqacc[NDT];
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) dqacc[dt][i] = 0.f;
  if constexpr (!RING) {
    if (!(flags & kFirst)) {
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int gg = 0; gg < 4; ++gg) {
          const f32x4 c4 = *(const f32x4*)(p.dq + qoff + 32 * dt + 8 * gg + 4 * hi);
#pragma unroll
          for (int e = 0; e < 4; ++e) dqacc[dt][4 * gg + e] = c4[e];
        }
    }
  }

  // tiles of the first block (the last ones under the mask), then the other blocks in ring
  // order: the walk of the forward kernel
  int n_own = blk_tiles, n_full = blk_tiles;
  if (p.causal) {
    n_own = min(n_own, max(0, (tile_first_q + kQQ - k_pos0 + kKK - 1) / kKK));
    n_own = min(n_own, (max(0, RING ? kv_rows - k_pos0 : kv_rows) + kKK - 1) / kKK);
    n_full = min(n_own, max(0, (tile_first_q - k_pos0 + 1) / kKK));
  }
  int nt = n_own;
  if constexpr (RING) nt += (p.causal ? host : p.N - 1) * blk_tiles;
  int w_row = RING ? k_pos0 : 0, w_left = n_own, w_blk = host;  // next tile to load

  // direct-to-LDS staging: load j of wave w fills rows j * 4 ROWS_PER_LOAD + w ROWS_PER_LOAD +
  // lane / CPR.  The swizzle of those rows does not depend on j, so all loads of a lane read
  // at one byte offset goff plus a wave-uniform j * 8 ROWS_PER_LOAD * rs bytes.
  static_assert(16 == LOADS * ROWS_PER_LOAD, "each wave fills LOADS row groups");
  const int goff = 2 * ((wave * ROWS_PER_LOAD + lane / CPR) * rs +
                        8 * ((lane % CPR) ^ swz<D>(wave * ROWS_PER_LOAD + lane / CPR)));
  auto load_tile = [&](auto Bc) __attribute__((always_inline)) {  // the next tile of the walk
    const long long t0 = (long long)w_row * rs;
    const int bytes = min(kKK, kv_rows - w_row) * rs * 2;  // rows past the end read as zero
    w_row += kKK;
    if constexpr (RING) {
      if (--w_left == 0) {
        w_blk = w_blk == 0 ? p.N - 1 : w_blk - 1;
        w_row = w_blk * p.c;
        w_left = blk_tiles;
      }
    }
    const __amdgpu_buffer_rsrc_t rk = make_rsrc(kbase + t0, bytes), rv = make_rsrc(vbase + t0, bytes);
#pragma unroll
    for (int j = 0; j < LOADS; ++j) {
      const int row = (j * 4 + wave_u) * ROWS_PER_LOAD, so = j * 8 * ROWS_PER_LOAD * rs;
      dma_lds16_so(rk, lds_addr(pick(Bc, sK0, sK1) + row * D), goff, so);
      dma_lds16_so(rv, lds_addr(pick(Bc, sV0, sV1) + row * D), goff, so);
    }
  };
  // row reads (A operand, rows 32 mt + swap_bits23(l32)) and transpose reads of the tiles
  const int krow = swap_bits23(l32);
  int roff[NKK];
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) roff[kk] = krow * D + 8 * ((2 * kk + hi) ^ swz<D>(krow));
  const int g16 = lane >> 4, li = lane & 15;
  int toff[2][NDT];
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) {
      const int row = 8 * hi + 4 * r + (li >> 2);
      const int d = 32 * dt + 16 * (g16 & 1) + 4 * (li & 3);
      toff[r][dt] = row * D + 8 * ((d >> 3) ^ swz<D>(row)) + (d & 7);
    }
  const float sl2 = p.scale * kLog2e;
  const float nl2 = nlse_s * sl2;  // -lse log2(e): the exponent is q.k sl2 + nl2 in float32

  // One 64-key tile, laid out by hand in fenced steps: the S^T and dP^T products of the
  // first 32 keys (the two chains alternating), then those of the last 32 keys while the
  // first 32 keys' probabilities and dS are formed, then the 16 dQ^T products while the
  // last 32 keys' dS are formed; operand reads PF steps ahead.
  auto body_sched = [&](auto Bc, auto Mc, int it) __attribute__((always_inline)) {
    constexpr int B = decltype(Bc)::value;
    constexpr bool MASK = decltype(Mc)::value;
    if (it + 1 < nt) load_tile(std::integral_constant<int, B ^ 1>{});
    const bf16* kt = pick(Bc, sK0, sK1);
    const bf16* vt = pick(Bc, sV0, sV1);
    constexpr int NA = 2 * NKK;       // S^T and dP^T products of one 32-key half
    constexpr int NQ = 4 * NDT;       // dQ^T products of the tile
    constexpr int NST = 2 * NA + NQ;  // steps
    constexpr int PF = 2;
    f32x16 sacc[2], dpacc[2];
    bf16x8 aop[2 * NA], top[NQ];
    u32x4 w[4];  // dS^T of the four 16-key groups, packed bf16: the B operands as they are
    const int kpos0 = k_pos0 + it * kKK;
    // step S < 2 NA: half h = S / NA, product j = S % NA of it (S^T if j even, dP^T if odd,
    // reduction slice kk = j / 2); step S >= 2 NA: dQ^T product q = S - 2 NA (keys of group
    // kb = q / NDT, dims 32 (q % NDT)..)
    auto fetch = [&](auto Sc) __attribute__((always_inline)) {
      constexpr int S = decltype(Sc)::value;
      if constexpr (S < 2 * NA) {
        constexpr int h = S / NA, j = S % NA, kk = j / 2;
        aop[S] = *(const bf16x8*)(((j & 1) ? vt : kt) + 32 * h * D + roff[kk]);
      } else {
        constexpr int q = S - 2 * NA, kb = q / NDT, dt = q % NDT;
        const bf16x4 lo = lds_read_tr16(kt + 16 * kb * D + toff[0][dt]);
        const bf16x4 up = lds_read_tr16(kt + 16 * kb * D + toff[1][dt]);
        top[q] = bf16x8{lo[0], lo[1], lo[2], lo[3], up[0], up[1], up[2], up[3]};
      }
    };
    // pair jj of the 4 of key group kb: probabilities and dS, packed bf16
    auto unit = [&](int kb, int jj) __attribute__((always_inline)) {
      float ds2[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int i = 8 * (kb & 1) + 2 * jj + e;
        const int mt = kb >> 1;
        float pv = fast_exp2(fmaf(sacc[mt][i], sl2, nl2));
        if (MASK) {
          const int kpos = kpos0 + 32 * mt + 16 * (i >> 3) + 8 * hi + (i & 7);
          if (kpos > qpos) pv = 0.f;
        }
        ds2[e] = pv * dpacc[mt][i];
      }
      w[kb][jj] = pack_bf16x2(ds2[0], ds2[1]);
    };
    // vector work: group kb's four pairs at steps VSTEP(kb) .. + 3 (groups 0, 1 once the
    // first half's chains are complete, groups 2, 3 once the second half's are)
    static_assert(NKK == 8 && NDT == 4, "hand schedule written for D = 128");
    constexpr int V0 = NA + 2, V2 = 2 * NA;
    static_for<0, PF>([&](auto Sc) __attribute__((always_inline)) { fetch(Sc); });
    static_for<0, NST>([&](auto Sc) __attribute__((always_inline)) {
      constexpr int S = decltype(Sc)::value;
      if constexpr (S + PF < NST) fetch(std::integral_constant<int, S + PF>{});
      if constexpr (S < 2 * NA) {
        constexpr int h = S / NA, j = S % NA, kk = j / 2;
        if constexpr (j == 1) {  // dP^T of half h starts at -Delta (set here: shorter live range)
#pragma unroll
          for (int i = 0; i < 16; ++i) dpacc[h][i] = ndlt;
        }
        if constexpr (j & 1)
          dpacc[h] = mfma32(aop[S], oreg[kk], dpacc[h]);
        else
          sacc[h] = mfma32(aop[S], qreg[kk], kk == 0 ? f32x16{} : sacc[h]);
      } else {
        constexpr int q = S - 2 * NA, kb = q / NDT, dt = q % NDT;
        dqacc[dt] = mfma32(top[q], __builtin_bit_cast(bf16x8, w[kb]), dqacc[dt]);
      }
      if constexpr (S >= V0 && S < V0 + 8) unit((S - V0) / 4, (S - V0) % 4);
      if constexpr (S >= V2 && S < V2 + 8) unit(2 + (S - V2) / 4, (S - V2) % 4);
      __builtin_amdgcn_sched_barrier(0);
    });
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };
  // other head dims: the same work, ordered by the compiler
  auto body_plain = [&](auto Bc, auto Mc, int it) __attribute__((always_inline)) {
    constexpr int B = decltype(Bc)::value;
    constexpr bool MASK = decltype(Mc)::value;
    if (it + 1 < nt) load_tile(std::integral_constant<int, B ^ 1>{});
    const bf16* kt = pick(Bc, sK0, sK1);
    const bf16* vt = pick(Bc, sV0, sV1);
    f32x16 sacc[2], dpacc[2];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        sacc[mt][i] = 0.f;
        dpacc[mt][i] = ndlt;
      }
#pragma unroll
      for (int kk = 0; kk < NKK; ++kk) {
        sacc[mt] = mfma32(*(const bf16x8*)(kt + 32 * mt * D + roff[kk]), qreg[kk], sacc[mt]);
        dpacc[mt] = mfma32(*(const bf16x8*)(vt + 32 * mt * D + roff[kk]), oreg[kk], dpacc[mt]);
      }
    }
    const int kpos0 = k_pos0 + it * kKK;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      u32x4 w;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float ds2[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int i = 8 * (kb & 1) + 2 * j + e;
          const int mt = kb >> 1;
          float pv = fast_exp2(fmaf(sacc[mt][i], sl2, nl2));
          if (MASK) {
            const int kpos = kpos0 + 32 * mt + 16 * (i >> 3) + 8 * hi + (i & 7);
            if (kpos > qpos) pv = 0.f;
          }
          ds2[e] = pv * dpacc[mt][i];
        }
        w[j] = pack_bf16x2(ds2[0], ds2[1]);
      }
      const bf16x8 dsb = __builtin_bit_cast(bf16x8, w);
      // dQ^T += K^T dS^T for these 16 keys
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) {
        const bf16x4 lo = lds_read_tr16(kt + 16 * kb * D + toff[0][dt]);
        const bf16x4 up = lds_read_tr16(kt + 16 * kb * D + toff[1][dt]);
        const bf16x8 a = {lo[0], lo[1], lo[2], lo[3], up[0], up[1], up[2], up[3]};
        dqacc[dt] = mfma32(a, dsb, dqacc[dt]);
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };
  auto body = [&](auto Bc, auto Mc, int it) __attribute__((always_inline)) {
    if constexpr (D == 128)
      body_sched(Bc, Mc, it);
    else
      body_plain(Bc, Mc, it);
  };
  auto run = [&](auto Mc, int a, int e) __attribute__((always_inline)) {
    int it = a;
    if ((it & 1) && it < e) body(std::integral_constant<int, 1>{}, Mc, it++);
    for (; it + 1 < e; it += 2) {
      body(std::integral_constant<int, 0>{}, Mc, it);
      body(std::integral_constant<int, 1>{}, Mc, it + 1);
    }
    if (it < e) body(std::integral_constant<int, 0>{}, Mc, it);
  };
  if (nt > 0) load_tile(std::integral_constant<int, 0>{});
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  run(std::false_type{}, 0, n_full);
  run(std::true_type{}, n_full, n_own);
  if constexpr (RING) run(std::false_type{}, n_own, nt);

  // the host's last step writes dq = scale * dQ in bf16; earlier ones save the accumulators
  if (qr >= q_rows) return;
  if (flags & kLast) {
    bf16* out = [&] { if constexpr (RING) return (bf16*)p.dq; else return (bf16*)p.dq_out; }() + qoff;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int gg = 0; gg < 4; ++gg) {
        const f32x16& a = dqacc[dt];
        *(u32x2*)(out + 32 * dt + 8 * gg + 4 * hi) =
            u32x2{pack_bf16x2(a[4 * gg] * p.scale, a[4 * gg + 1] * p.scale),
                  pack_bf16x2(a[4 * gg + 2] * p.scale, a[4 * gg + 3] * p.scale)};
      }
  } else if constexpr (!RING) {
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int gg = 0; gg < 4; ++gg) {
        const f32x16& a = dqacc[dt];
        *(f32x4*)(p.dq + qoff + 32 * dt + 8 * gg + 4 * hi) = f32x4{a[4 * gg], a[4 * gg + 1], a[4 * gg + 2], a[4 * gg + 3]};
      }
  }
}

}  // namespace

hipError_t launch_bwd_pre_bf16(const void* o, const void* dO, const float* lse, float* delta, float* nlse_s, int B,
                               int S, int H, int D, hipStream_t st) {
  const long long blocks = (long long)B * ((S + kPreR - 1) / kPreR) * ((H + kPreH - 1) / kPreH);
  if (D == 128)
    hipLaunchKernelGGL(bwd_pre_bf16_kernel<128>, dim3(blocks), dim3(256), 0, st, (const bf16*)o, (const bf16*)dO, lse, delta, nlse_s, B, S, H);
  else
    hipLaunchKernelGGL(bwd_pre_bf16_kernel<64>, dim3(blocks), dim3(256), 0, st, (const bf16*)o, (const bf16*)dO, lse, delta, nlse_s, B, S, H);
  return hipGetLastError();
}

hipError_t launch_bwd_pre_f32(const float* o, const float* dO, float* delta, int B, int S, int H, int D,
                              hipStream_t st) {
  const long long blocks = (long long)B * ((S + kPreR - 1) / kPreR) * ((H + kPreH - 1) / kPreH);
  if (D == 128)
    hipLaunchKernelGGL(bwd_pre_f32_kernel<128>, dim3(blocks), dim3(256), 0, st, o, dO, delta, B, S, H);
  else
    hipLaunchKernelGGL(bwd_pre_f32_kernel<64>, dim3(blocks), dim3(256), 0, st, o, dO, delta, B, S, H);
  return hipGetLastError();
}

hipError_t launch_bwd_bf16(const BwdStep& s, int D, hipStream_t st) {
  if (s.n_slots == 0) return hipSuccess;
  // a last touch needs the bf16 outputs
  if (s.whole && (s.dk_out == nullptr || s.dv_out == nullptr)) return hipErrorInvalidValue;
  const int g1 = s.n_slots * s.B * s.H * (s.c / kKB);
  const int g2 = s.n_slots * s.B * s.H * (s.c / kQQ);
  if (D == 128) {
    hipLaunchKernelGGL(bwd_dkdv_split_kernel<BwdStep>, dim3(g1), dim3(kPT), 0, st, s);
    hipLaunchKernelGGL((bwd_dq_bf16_kernel<128, BwdStep>), dim3(g2), dim3(kBT), 0, st, s);
  } else {
    hipLaunchKernelGGL((bwd_dkdv_bf16_kernel<64, BwdStep>), dim3(g1), dim3(kBT), 0, st, s);
    hipLaunchKernelGGL((bwd_dq_bf16_kernel<64, BwdStep>), dim3(g2), dim3(kBT), 0, st, s);
  }
  return hipGetLastError();
}

hipError_t launch_bwd_ring_bf16(const BwdRing& s, int D, hipStream_t st) {
  const int g1 = ring_grid(s.B * s.H, (s.S + kKB - 1) / kKB);
  const int g2 = ring_grid(s.B * s.H, (s.S + kQQ - 1) / kQQ);
  if (D == 128) {
    hipLaunchKernelGGL(bwd_dkdv_split_kernel<BwdRing>, dim3(g1), dim3(kPT), 0, st, s);
    hipLaunchKernelGGL((bwd_dq_bf16_kernel<128, BwdRing>), dim3(g2), dim3(kBT), 0, st, s);
  } else {
    hipLaunchKernelGGL((bwd_dkdv_bf16_kernel<64, BwdRing>), dim3(g1), dim3(kBT), 0, st, s);
    hipLaunchKernelGGL((bwd_dq_bf16_kernel<64, BwdRing>), dim3(g2), dim3(kBT), 0, st, s);
  }
  return hipGetLastError();
}

}  // namespace ra
