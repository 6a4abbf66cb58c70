// float32 ring attention for gfx950 on the float32 matrix cores: every product and sum is
// float32 (v_mfma_f32_32x32x2_f32, one fused multiply-add per term), nothing is rounded to
// bf16.  The whole ring runs in one launch (backward: one after the Delta pass); every
// workgroup walks the blocks it meets in ring order, where they lie.
//
// A workgroup owns 32 G rows (queries, or keys for dK/dV) in its 4 waves; R = 4 / G waves
// share 32 rows and take every R-th 32-row tile of the other operand, their partial results
// being combined through LDS at the end: a tile of 64 rows by 32 takes its wave thousands of
// cycles (64 a product), so short sequences need the split to fill the chip and a causal
// launch needs short workgroups to balance, while the matrix cores leave the L2 idle enough
// (about 8 bytes a cycle and CU) that sharing a tile between fewer rows costs nothing.
// D = 128: G = 2, R = 2; D = 64: G = 1, R = 4 (130 and 132 KB of LDS, double buffered).
//
// Lane layouts: S^T = K Q^T takes A = K rows from LDS (16-byte chunks, lane half h holding dims
// 8 u + 4 h + e) and B = Q in registers in the same order; register i of the result holds key
// 8 (i / 4) + 4 h + i % 4 of the lane's query, which is just the B operand of the next
// product over keys, O^T += V^T P^T, whose A operand is read from V's rows, D / 32 dims a lane.
//
// Bound by the float32 matrix cores (157 TFLOP/s), with one wave a SIMD the exponentials and
// rescaling on top; short sequences by the chain of tiles of one wave.  Forward + backward
// against one thread per row on the vector units (a launch a ring step, blocks copied), us:
// 4096 tokens x 8 heads of 128, 8 hosts 50500 -> 1595 (executed: 18 D flop a pair, 97 TFLOP/s);
// 1024 x 1 of 64, 4 hosts 3476 -> 89.  Errors against float64 are below that kernel's (o 3.5e-7,
// it 6.1e-7; dV 4.7e-7, 7.1e-7 at 4096 x 8).
#include "ra_common.h"
#include "ra_dma.h"
#include "ra_kernels.h"

namespace ra {
namespace {

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

constexpr int kFT = 32;  // rows of a tile

template <int D>
struct F32Tile {
  static constexpr int G = D / 64, R = 4 / G;     // row groups of a workgroup, waves per group
  static constexpr int ROWS = kFT * G;            // rows a workgroup owns
  static constexpr int NU = D / 8, NDT = D / 32;  // 16-byte chunk pairs of a row; dims per lane and output row
  static constexpr int CPR = D / 4, RB = D * 4;   // chunks, bytes of a row
  static constexpr int TILE = kFT * RB;           // bytes of one operand tile
  static constexpr int RPL = 64 / CPR;            // rows of a 1 KB load
  static constexpr int LOADS = kFT / G / RPL;     // loads per wave and operand tile
  static constexpr int BUF = 2 * TILE + 512;      // both operands and two 64-float row vectors
};

// Chunk c of row r lies at c ^ (r & 15): 16 consecutive rows read at one chunk, and one row
// read across its chunks, both touch 16 distinct chunk positions.
template <int D>
struct F32Wave {
  using T = F32Tile<D>;
  int lane, l32, hi, g, r;  // lane; wave's row group and its share of the tiles
  int goff[T::LOADS];       // byte offsets of this lane's loads from a tile's first row
  int rs;                   // row stride (elements)

  __device__ __forceinline__ F32Wave(int row_stride) : rs(row_stride) {
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    lane = tid & 63;
    l32 = lane & 31;
    hi = lane >> 5;
    g = wave % T::G;
    r = wave / T::G;
#pragma unroll
    for (int j = 0; j < T::LOADS; ++j) {
      const int row = g * (kFT / T::G) + j * T::RPL + lane / T::CPR;
      goff[j] = 4 * row * rs + 16 * ((lane % T::CPR) ^ (row & 15));
    }
  }
  // this wave's rows of both operand tiles (rows [row, row + 32) of a and b) into buf
  __device__ __forceinline__ void load(const float* a, const float* b, int row, unsigned buf) const {
    const __amdgpu_buffer_rsrc_t ra_ = make_rsrc(a + (long long)row * rs, kFT * rs * 4);
    const __amdgpu_buffer_rsrc_t rb_ = make_rsrc(b + (long long)row * rs, kFT * rs * 4);
#pragma unroll
    for (int j = 0; j < T::LOADS; ++j) {
      const unsigned at = buf + (g * (kFT / T::G) + j * T::RPL) * T::RB;
      dma_lds16(ra_, at, goff[j]);
      dma_lds16(rb_, at + T::TILE, goff[j]);
    }
  }
  // operand registers of row `row` (B operand, contracted over dims)
  __device__ __forceinline__ void row_regs(const float* base, int row, float (&x)[D / 2]) const {
    const float* p = base + (long long)row * rs + 4 * hi;
#pragma unroll
    for (int u = 0; u < T::NU; ++u) {
      const f32x4 t = *(const f32x4*)(p + 8 * u);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[4 * u + e] = t[e];
    }
  }
  // tile rows (A) times x (B), contracted over dims: lane's row of x against 32 tile rows
  __device__ __forceinline__ f32x16 dots(const char* tile, const float (&x)[D / 2]) const {
    f32x16 s = {};
    const char* p = tile + l32 * T::RB;
#pragma unroll
    for (int u = 0; u < T::NU; ++u) {
      const f32x4 a = *(const f32x4*)(p + 16 * ((2 * u + hi) ^ (l32 & 15)));
#pragma unroll
      for (int e = 0; e < 4; ++e) s = mfma_f32(a[e], x[4 * u + e], s);
    }
    return s;
  }
  // acc[dt] += tile^T w, contracted over the tile's 32 rows: register i of acc[dt] is dim
  // NDT (8 (i / 4) + 4 hi + i % 4) + dt of the lane's row.  The tile's sum is formed by itself
  // and then added: chained into acc term by term, a sum over thousands of rows rounds once a
  // row at the size of the whole (4096 tokens: dV 1.2e-6 off float64 instead of 4.7e-7,
  // for 5 % of the time).
  __device__ __forceinline__ void accum(const char* tile, const f32x16& w, f32x16 (&sum)[T::NDT]) const {
    f32x16 acc[T::NDT];
#pragma unroll
    for (int dt = 0; dt < T::NDT; ++dt) acc[dt] = f32x16{};
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int row0 = 8 * (i / 4) + i % 4, row = row0 + 4 * hi;
      if constexpr (D == 128) {
        const f32x4 a = *(const f32x4*)(tile + row * T::RB + 16 * (l32 ^ (row & 15)));
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) acc[dt] = mfma_f32(a[dt], w[i], acc[dt]);
      } else {
        const f32x2 a = *(const f32x2*)(tile + row * T::RB + 16 * ((l32 >> 1) ^ (row & 15)) + 8 * (l32 & 1));
#pragma unroll
        for (int dt = 0; dt < 2; ++dt) acc[dt] = mfma_f32(a[dt], w[i], acc[dt]);
      }
    }
#pragma unroll
    for (int dt = 0; dt < T::NDT; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) sum[dt][i] += acc[dt][i];
  }
  // dims of accumulator register group i: offset of the lane's NDT consecutive dims
  __device__ __forceinline__ int dim_of(int i) const { return T::NDT * (8 * (i / 4) + 4 * hi + i % 4); }
  __device__ __forceinline__ void store(float* out, const f32x16 (&acc)[T::NDT], float sc) const {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if constexpr (D == 128)
        *(f32x4*)(out + dim_of(i)) = f32x4{acc[0][i] * sc, acc[1][i] * sc, acc[2][i] * sc, acc[3][i] * sc};
      else
        *(f32x2*)(out + dim_of(i)) = f32x2{acc[0][i] * sc, acc[1][i] * sc};
    }
  }
  // partial accumulators through LDS, one slot a wave: [dt][i][lane]
  __device__ __forceinline__ void put(float* slot, const f32x16 (&acc)[T::NDT]) const {
#pragma unroll
    for (int dt = 0; dt < T::NDT; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) slot[(dt * 16 + i) * 64 + lane] = acc[dt][i];
  }
  __device__ __forceinline__ void add(const float* slot, f32x16 (&acc)[T::NDT], float w) const {
#pragma unroll
    for (int dt = 0; dt < T::NDT; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[dt][i] = fmaf(slot[(dt * 16 + i) * 64 + lane], w, acc[dt][i]);
  }
};

__device__ __forceinline__ void tiles_landed() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  lds_barrier();
}

// Walk over the key tiles of a query tile: n_own tiles of its host's block, then the other
// blocks in ring order, host - 1, host - 2, ... (mod N).
struct KeyWalk {
  int host, k_pos0, n_own, n, blk_tiles, c, N;
  __device__ __forceinline__ KeyWalk(int q0, int rows, int c_, int N_, int causal) : c(c_), N(N_) {
    host = q0 / c;
    k_pos0 = host * c;
    blk_tiles = c / kFT;
    n_own = causal ? (q0 + rows - k_pos0) / kFT : blk_tiles;
    n = n_own + (causal ? host : N - 1) * blk_tiles;
  }
  __device__ __forceinline__ int row(int p) const {
    if (p < n_own) return k_pos0 + p * kFT;
    const int b = (p - n_own) / blk_tiles;
    int j = host - 1 - b;
    if (j < 0) j += N;
    return j * c + (p - n_own - b * blk_tiles) * kFT;
  }
};

template <int D>
__global__ __launch_bounds__(256) void fwd_f32_kernel(const FwdRing p) {
  using T = F32Tile<D>;
  __shared__ __attribute__((aligned(1024))) char lds[2 * T::R * T::BUF];
  int bh, qt;
  if (!ring_item(blockIdx.x, p.B * p.H, p.S / T::ROWS, (long long)p.S * (D * 8), bh, qt)) return;
  const int b = bh / p.H, h = bh % p.H, q0 = qt * T::ROWS;
  const F32Wave<D> w(p.H * D);
  const long long off = (long long)b * p.bstride + h * D;
  const float *kb = (const float*)p.k + off, *vb = (const float*)p.v + off;
  const KeyWalk walk(q0, T::ROWS, p.c, p.N, p.causal);
  const int qw0 = q0 + kFT * w.g, qr = qw0 + w.l32;  // the wave's first query, the lane's
  auto buf = [&](int it) __attribute__((always_inline)) { return lds + ((it & 1) * T::R + w.r) * T::BUF; };
  const int iters = (walk.n + T::R - 1) / T::R;
  if (w.r < walk.n) w.load(kb, vb, walk.row(w.r), lds_addr(buf(0)));

  float q[D / 2];
  w.row_regs((const float*)p.q + off, qr, q);
  f32x16 acc[T::NDT];
#pragma unroll
  for (int dt = 0; dt < T::NDT; ++dt) acc[dt] = f32x16{};
  float m = -INFINITY, l = 0.f;
  tiles_landed();
  for (int it = 0; it < iters; ++it) {
    const int t = it * T::R + w.r;
    if (t + T::R < walk.n) w.load(kb, vb, walk.row(t + T::R), lds_addr(buf(it + 1)));
    const int k0 = t < walk.n ? walk.row(t) : 0;
    // rows of a wave and tiles are aligned to 32: a tile is seen whole, on its diagonal, or not
    if (t < walk.n && !(p.causal && k0 > qw0)) {
      const char* kt = buf(it);
      f32x16 s = w.dots(kt, q);
      float mx = -INFINITY;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        s[i] *= p.scale;
        if (p.causal && k0 == qw0 && 8 * (i / 4) + 4 * w.hi + i % 4 > w.l32) s[i] = -INFINITY;
        mx = fmaxf(mx, s[i]);
      }
      // a maximum of -inf (so far only scores of -inf, which weigh 0) would make inf - inf of them
      const float m_new = fmaxf(m, pair_max(mx)), m_use = m_new == -INFINITY ? 0.f : m_new;
      const float alpha = expf(m - m_use);
      m = m_new;
      l *= alpha;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        s[i] = expf(s[i] - m_use);
        l += s[i];
      }
#pragma unroll
      for (int dt = 0; dt < T::NDT; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[dt][i] *= alpha;
      w.accum(kt + T::TILE, s, acc);
    }
    tiles_landed();
  }
  // combine the R waves of a row group (the tile buffers are free): the first takes the others'
  l = pair_sum(l);
  float* slots = (float*)lds;
  constexpr int SLOT = D * 32 + 64;
  if (w.r > 0) {
    float* s = slots + ((w.r - 1) * T::G + w.g) * (SLOT + 64);
    w.put(s, acc);
    s[D * 32 + w.lane] = m;
    s[D * 32 + 64 + w.lane] = l;
  }
  __syncthreads();
  if (w.r > 0) return;
  float mt = m;
#pragma unroll
  for (int j = 0; j < T::R - 1; ++j) mt = fmaxf(mt, slots[(j * T::G + w.g) * (SLOT + 64) + D * 32 + w.lane]);
  const float mt_use = mt == -INFINITY ? 0.f : mt;
  const float a0 = expf(m - mt_use);
  l *= a0;
#pragma unroll
  for (int dt = 0; dt < T::NDT; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[dt][i] *= a0;
#pragma unroll
  for (int j = 0; j < T::R - 1; ++j) {
    const float* s = slots + (j * T::G + w.g) * (SLOT + 64);
    const float aj = expf(s[D * 32 + w.lane] - mt_use);
    l = fmaf(s[D * 32 + 64 + w.lane], aj, l);
    w.add(s, acc, aj);
  }
  w.store((float*)p.o + off + (long long)qr * w.rs, acc, 1.f / l);
  if (!w.hi) p.lse[(long long)bh * p.S + qr] = mt + logf(l);
}

// dK and dV of the workgroup's keys: lanes over keys, tiles of 32 queries in ring order (rows
// from the keys' own block on; non-causal around the ring).
template <int D>
__device__ __forceinline__ void bwd_f32_dkdv(const BwdRing& p, int id, char* lds) {
  using T = F32Tile<D>;
  const int n_kt = p.S / T::ROWS;
  int bh, tile;
  if (!ring_item(id, p.B * p.H, n_kt, (long long)p.S * (D * 8), bh, tile)) return;
  const int b = bh / p.H, h = bh % p.H, key0 = (n_kt - 1 - tile) * T::ROWS;  // first keys have most queries
  const F32Wave<D> w(p.H * D);
  const long long off = (long long)b * p.bstride + h * D;
  const float *qb = (const float*)p.q + off, *ob = (const float*)p.dO + off;
  const int start = p.causal ? key0 : key0 / p.c * p.c;
  const int n = (p.causal ? p.S - key0 : p.S) / kFT;
  auto row = [&](int t) __attribute__((always_inline)) {
    const int x = start + t * kFT;
    return x >= p.S ? x - p.S : x;
  };
  auto buf = [&](int it) __attribute__((always_inline)) { return lds + ((it & 1) * T::R + w.r) * T::BUF; };
  const float* lse = p.lse + (long long)bh * p.S;
  const float* delta = p.delta + (long long)bh * p.S;
  auto load = [&](int t, int it) __attribute__((always_inline)) {
    const unsigned at = lds_addr(buf(it));
    const int q0 = row(t);
    w.load(qb, ob, q0, at);
    if (w.g == 0) {  // lse and Delta of the tile's queries (lanes past them write zeros)
      dma_lds4(make_rsrc(lse + q0, kFT * 4), at + 2 * T::TILE, 4 * w.lane);
      dma_lds4(make_rsrc(delta + q0, kFT * 4), at + 2 * T::TILE + 256, 4 * w.lane);
    }
  };
  const int iters = (n + T::R - 1) / T::R;
  if (w.r < n) load(w.r, 0);
  const int kw0 = key0 + kFT * w.g, key = kw0 + w.l32;
  float k[D / 2], v[D / 2];
  w.row_regs((const float*)p.k + off, key, k);
  w.row_regs((const float*)p.v + off, key, v);
  f32x16 dk[T::NDT], dv[T::NDT];
#pragma unroll
  for (int dt = 0; dt < T::NDT; ++dt) dk[dt] = dv[dt] = f32x16{};
  tiles_landed();
  for (int it = 0; it < iters; ++it) {
    const int t = it * T::R + w.r;
    if (t + T::R < n) load(t + T::R, it + 1);
    const int q0 = t < n ? row(t) : 0;
    if (t < n && !(p.causal && q0 < kw0)) {
      const char* bt = buf(it);
      const f32x16 s = w.dots(bt, k);
      const f32x16 dp = w.dots(bt + T::TILE, v);
      const float* sl = (const float*)(bt + 2 * T::TILE);
      f32x16 pr, ds;
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const f32x4 ls = *(const f32x4*)(sl + 8 * i4 + 4 * w.hi), dl = *(const f32x4*)(sl + 64 + 8 * i4 + 4 * w.hi);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int i = 4 * i4 + e;
          float x = expf(s[i] * p.scale - ls[e]);
          if (p.causal && q0 == kw0 && 8 * i4 + 4 * w.hi + e < w.l32) x = 0.f;
          pr[i] = x;
          ds[i] = x * (dp[i] - dl[e]);
        }
      }
      w.accum(bt + T::TILE, pr, dv);
      w.accum(bt, ds, dk);
    }
    tiles_landed();
  }
  float* slots = (float*)lds;
  constexpr int SLOT = 2 * D * 32;
  if (w.r > 0) {
    float* s = slots + ((w.r - 1) * T::G + w.g) * SLOT;
    w.put(s, dk);
    w.put(s + D * 32, dv);
  }
  __syncthreads();
  if (w.r > 0) return;
#pragma unroll
  for (int j = 0; j < T::R - 1; ++j) {
    const float* s = slots + (j * T::G + w.g) * SLOT;
    w.add(s, dk, 1.f);
    w.add(s + D * 32, dv, 1.f);
  }
  w.store((float*)p.dk + off + (long long)key * w.rs, dk, p.scale);
  w.store((float*)p.dv + off + (long long)key * w.rs, dv, 1.f);
}

// dQ of the workgroup's queries: lanes over queries, key tiles in ring order.
template <int D>
__device__ __forceinline__ void bwd_f32_dq(const BwdRing& p, int id, char* lds) {
  using T = F32Tile<D>;
  int bh, qt;
  if (!ring_item(id, p.B * p.H, p.S / T::ROWS, (long long)p.S * (D * 8), bh, qt)) return;
  const int b = bh / p.H, h = bh % p.H, q0 = qt * T::ROWS;
  const F32Wave<D> w(p.H * D);
  const long long off = (long long)b * p.bstride + h * D;
  const float *kb = (const float*)p.k + off, *vb = (const float*)p.v + off;
  const KeyWalk walk(q0, T::ROWS, p.c, p.N, p.causal);
  const int qw0 = q0 + kFT * w.g, qr = qw0 + w.l32;
  auto buf = [&](int it) __attribute__((always_inline)) { return lds + ((it & 1) * T::R + w.r) * T::BUF; };
  const int iters = (walk.n + T::R - 1) / T::R;
  if (w.r < walk.n) w.load(kb, vb, walk.row(w.r), lds_addr(buf(0)));
  float q[D / 2], o[D / 2];
  w.row_regs((const float*)p.q + off, qr, q);
  w.row_regs((const float*)p.dO + off, qr, o);
  const float lse = p.lse[(long long)bh * p.S + qr], delta = p.delta[(long long)bh * p.S + qr];
  f32x16 dq[T::NDT];
#pragma unroll
  for (int dt = 0; dt < T::NDT; ++dt) dq[dt] = f32x16{};
  tiles_landed();
  for (int it = 0; it < iters; ++it) {
    const int t = it * T::R + w.r;
    if (t + T::R < walk.n) w.load(kb, vb, walk.row(t + T::R), lds_addr(buf(it + 1)));
    const int k0 = t < walk.n ? walk.row(t) : 0;
    if (t < walk.n && !(p.causal && k0 > qw0)) {
      const char* kt = buf(it);
      const f32x16 s = w.dots(kt, q);
      const f32x16 dp = w.dots(kt + T::TILE, o);
      f32x16 ds;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        float x = expf(s[i] * p.scale - lse);
        if (p.causal && k0 == qw0 && 8 * (i / 4) + 4 * w.hi + i % 4 > w.l32) x = 0.f;
        ds[i] = x * (dp[i] - delta);
      }
      w.accum(kt, ds, dq);
    }
    tiles_landed();
  }
  float* slots = (float*)lds;
  if (w.r > 0) w.put(slots + ((w.r - 1) * T::G + w.g) * (D * 32), dq);
  __syncthreads();
  if (w.r > 0) return;
#pragma unroll
  for (int j = 0; j < T::R - 1; ++j) w.add(slots + (j * T::G + w.g) * (D * 32), dq, 1.f);
  w.store((float*)p.dq + off + (long long)qr * w.rs, dq, p.scale);
}

// One launch: workgroups [0, n_dkdv) take key tiles, the rest query tiles.  The two halves are
// independent; together they fill the chip on short sequences and share one tail.
template <int D>
__global__ __launch_bounds__(256) void bwd_f32_kernel(const BwdRing p, int n_dkdv) {
  using T = F32Tile<D>;
  __shared__ __attribute__((aligned(1024))) char lds[2 * T::R * T::BUF];
  if ((int)blockIdx.x < n_dkdv)
    bwd_f32_dkdv<D>(p, blockIdx.x, lds);
  else
    bwd_f32_dq<D>(p, blockIdx.x - n_dkdv, lds);
}

}  // namespace

hipError_t launch_fwd_ring_f32(const FwdRing& s, int D, hipStream_t st) {
  const int G = s.B * s.H;
  if (D == 128)
    hipLaunchKernelGGL(fwd_f32_kernel<128>, dim3(ring_grid(G, s.S / F32Tile<128>::ROWS)), dim3(256), 0, st, s);
  else
    hipLaunchKernelGGL(fwd_f32_kernel<64>, dim3(ring_grid(G, s.S / F32Tile<64>::ROWS)), dim3(256), 0, st, s);
  return hipGetLastError();
}

hipError_t launch_bwd_ring_f32(const BwdRing& s, int D, hipStream_t st) {
  const int n = ring_grid(s.B * s.H, s.S / (D == 128 ? F32Tile<128>::ROWS : F32Tile<64>::ROWS));
  if (D == 128)
    hipLaunchKernelGGL(bwd_f32_kernel<128>, dim3(2 * n), dim3(256), 0, st, s, n);
  else
    hipLaunchKernelGGL(bwd_f32_kernel<64>, dim3(2 * n), dim3(256), 0, st, s, n);
  return hipGetLastError();
}

}  // namespace ra
