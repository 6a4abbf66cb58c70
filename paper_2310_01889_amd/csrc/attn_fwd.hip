// Ring-attention forward kernels for gfx950.
//
// One launch folds either every block of the ring, or, for every host listed in one ring
// step, the key/value block that host holds, into the hosts' running state -- running row maximum m, running denominator l and
// unnormalised output (numerator) acc -- as the online-softmax recurrence of the
// paper's blockwise attention (Section 2 "Blockwise Parallel Transformers"; Section 3;
// the carry of the Appendix A forward scan):
//     m' = max(m, rowmax(s)),  p = exp(s - m'),
//     l' = l * exp(m - m') + rowsum(p),  acc' = acc * exp(m - m') + p v
// with s = q k^T / sqrt(D), masked (causal, by global position) keys giving p = 0.
// On a host's first active step the state starts from (m=-inf, l=0, acc=0) in
// registers; on its last it is finalised into o = acc / l and lse = m + ln l.
//
// The bf16 whole-ring launch is bound by the matrix cores at the board's power limit and the
// key/value tile loads.  Against one launch a step (state saved and loaded in float32, blocks
// copied from host to host, a grid tail each step) it takes, in us: 32768 tokens x 32 heads,
// 8 hosts 7490 (steps 7919; 1.18 PFLOP/s); 16384 x 16, 8 hosts 955 (1120); 4 x 2048 x 12 heads
// of 64, bidirectional, 4 hosts 63 (110); 2048 x 8, 4 hosts 35 (71).
#include <type_traits>

#include "ra_common.h"
#include "ra_kernels.h"

namespace ra {

// ===================================================================================
// bf16 kernel: NW = 4 or 8 waves, 32 queries per wave (128 or 256 per workgroup), 64-key
// tiles.
//
// Per wave, scores are formed transposed, S^T = K Q^T (32x32x16 MFMA, A = K rows from
// LDS, B = Q held in registers), so that each lane owns one query: its row max and
// row sum are in-lane reductions plus one exchange with lane l^32.  K rows are loaded
// with bits 2 and 3 of the row index swapped, which makes each lane half hold 8
// consecutive keys per 16-key group; the probabilities P^T then serve directly as the
// B operand of O^T += V^T P^T, whose A operand is read from the row-major V tile with
// the LDS transpose read.  O^T (128 dims x 32 queries per wave) stays in registers.
// ===================================================================================
namespace {

constexpr int kBM = 128, kBN = 64, kThreads = 256;
constexpr float kSumMax = 65536.f;  // overflow test: a lane's row sum over a tile below this


// LDS tiles are unpadded [64 rows][D] with the 16-byte chunks of each row permuted by
// an XOR swizzle, so that every read pattern below is free of bank conflicts:
//   * row reads (A operand of S^T): 16 lanes read 16 consecutive rows at one chunk;
//   * transpose reads (V^T): 16 lanes read 4 consecutive rows x 32 contiguous bytes.
// For D = 128 (16 chunks per row): chunk c of row r lives at c ^ (4 (r & 3) + ((r >> 2) & 3));
// for D = 64 (8 chunks, two rows per 256-byte bank sweep) at c ^ s, s = (r >> 1) & 7 with
// bit 2 flipped on odd s.  Tiles are filled with direct-to-LDS loads (no registers):
// lane i of a 1 KB load lands at byte 16 i of its destination, so each lane fetches the
// logical chunk that the swizzle puts there.
// RING: the whole ring in one launch.  A workgroup walks the tiles of every block its host
// folds, in ring order -- its own block first, then its predecessors' -- reading them where
// they lie, so the state never leaves the registers.  Otherwise one ring step: the tiles of
// the one block the slot names.
template <int D, int NW, bool RING>
__global__ __launch_bounds__(64 * NW, NW == 4 ? 2 : 1) void fwd_bf16_kernel(
    const typename std::conditional<RING, FwdRing, FwdStep>::type p) {
  constexpr int BM = 32 * NW;  // queries per workgroup (32 per wave)
  constexpr int NKK = D / 16;  // 16-wide reduction steps of q.k
  constexpr int NDT = D / 32;  // 32-row output tiles of O^T
  constexpr int CPR = D / 8;   // 16-byte chunks per row
  constexpr int ROWS_PER_LOAD = 64 / CPR;               // rows filled by one 1 KB wave load
  constexpr int RPW = kBN / NW;                          // tile rows each wave fills
  constexpr int LOADS = RPW / ROWS_PER_LOAD;             // 1 KB loads per wave per tile
  constexpr int TILE = kBN * D;                          // elements per tile
  // Four separate LDS objects (not one [2][TILE] array per operand): the compiler then
  // knows that reads of one buffer do not alias direct-to-LDS loads in flight into the
  // other, and does not wait for those loads before every read.
  __shared__ __attribute__((aligned(1024))) bf16 sK0[TILE];
  __shared__ __attribute__((aligned(1024))) bf16 sK1[TILE];
  __shared__ __attribute__((aligned(1024))) bf16 sV0[TILE];
  __shared__ __attribute__((aligned(1024))) bf16 sV1[TILE];
  auto kbuf = [&](auto Bc) __attribute__((always_inline)) -> bf16* {
    if constexpr (decltype(Bc)::value == 0) return sK0; else return sK1;
  };
  auto vbuf = [&](auto Bc) __attribute__((always_inline)) -> bf16* {
    if constexpr (decltype(Bc)::value == 0) return sV0; else return sV1;
  };

  // ---- the workgroup's query rows and the blocks it folds ----------------------------
  int bh, q_tile_row;     // (batch, head); first q-space row of the workgroup
  int tile_first_q;       // its global position
  int k_pos0;             // global position of the first block's first key
  int host = 0;           // RING: the host that owns the rows
  int flags = kFirst | kLast;
  int kv_rows;            // key rows that exist, from kbase (reads past them give zero)
  int nt, n_full;         // key tiles visited; tiles [n_full, n_own) need the causal mask
  int n_own;              // tiles of the first block
  const int blk_tiles = p.c / kBN;
  const bf16 *kbase, *vbase;
  if constexpr (RING) {
    const int n_qt = (p.S + BM - 1) / BM;
    int qt;
    if (!ring_item(blockIdx.x, p.B * p.H, n_qt, (long long)p.S * (D * 4), bh, qt)) return;
    q_tile_row = tile_first_q = qt * BM;
    host = q_tile_row / p.c;
    k_pos0 = host * p.c;
    kv_rows = p.S;
    const long long off = (long long)(bh / p.H) * p.bstride + (bh % p.H) * D;
    kbase = (const bf16*)p.k + off;
    vbase = (const bf16*)p.v + off;
  } else {
    const int n_qt = p.c / BM;
    const int BH = p.B * p.H;
    const int L = xcd_swizzle(blockIdx.x, p.n_slots * BH * n_qt);
    const int grp = L / n_qt;
    const int qt = n_qt - 1 - (L % n_qt);  // longest causal rows first
    const StepHost& hs = p.host[grp / BH];
    bh = grp % BH;
    q_tile_row = hs.q_row0 + qt * BM;
    tile_first_q = hs.q_pos0 + qt * BM;
    k_pos0 = hs.k_pos0;
    kv_rows = hs.kv_rows;
    flags = hs.flags;
    const long long off = (long long)(bh / p.H) * hs.kv_bstride + (bh % p.H) * D;
    kbase = (const bf16*)hs.k + off;
    vbase = (const bf16*)hs.v + off;
    if (q_tile_row >= p.Sq) return;
  }
  const int b = bh / p.H, h = bh % p.H;

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);  // uniform: LDS destinations in scalar registers
  const int l32 = lane & 31, hi = lane >> 5;
  const int rs = p.H * D;  // row stride of q / k / v / o (elements)
  const int q_rows = [&] { if constexpr (RING) return p.S; else return p.Sq; }();  // query rows that exist
  const long long q_bs = [&] { if constexpr (RING) return p.bstride; else return p.q_bstride; }();

  const int qr = q_tile_row + wave * 32 + l32;       // this lane's query row
  const int qpos = tile_first_q + wave * 32 + l32;
  const bf16* qbase = (const bf16*)p.q + (long long)b * q_bs + h * D;

  // key tiles of the first block with at least one visible key; the first n_full need no mask
  n_own = n_full = blk_tiles;
  if (p.causal) {
    const int vis = tile_first_q + BM - k_pos0;  // keys visible to the last row
    n_own = min(n_own, max(0, (vis + kBN - 1) / kBN));
    n_own = min(n_own, (max(0, RING ? kv_rows - k_pos0 : kv_rows) + kBN - 1) / kBN);
    n_full = min(n_own, max(0, (tile_first_q - k_pos0 + 1) / kBN));
  }
  nt = n_own;
  if constexpr (RING) nt += (p.causal ? host : p.N - 1) * blk_tiles;
  // Walk over the key tiles: row of the next tile (from kbase) and the tiles left in its
  // block.  The blocks follow one another in ring order, host, host - 1, ... (mod N).
  struct Walk { int row, left, blk; };
  auto next_row = [&](Walk& w) __attribute__((always_inline)) -> int {
    const int r = w.row;
    w.row += kBN;
    if constexpr (RING) {
      if (--w.left == 0) {
        w.blk = w.blk == 0 ? p.N - 1 : w.blk - 1;
        w.row = w.blk * p.c;
        w.left = blk_tiles;
      }
    }
    return r;
  };
  Walk wk{RING ? k_pos0 : 0, n_own, host}, wv = wk;

  // ---- running state -------------------------------------------------------------
  f32x16 oacc[NDT];
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[dt][i] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  if constexpr (!RING) {
    if (!(flags & kFirst)) {
      const f32x4* acc_tile = (const f32x4*)(p.acc + ((long long)bh * (p.Sp / BM) + q_tile_row / BM) * (BM * D));
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 t = acc_tile[((wave * NDT + dt) * 4 + g) * 64 + lane];
#pragma unroll
          for (int e = 0; e < 4; ++e) oacc[dt][4 * g + e] = t[e];
        }
      const long long st_row = (long long)bh * p.Sp + qr;
      m_run = p.m[st_row];
      l_run = p.l[2 * st_row + hi];
    }
  }

  // ---- Q in registers: B operand of S^T = K Q^T (n = query, k = dim) ---------------
  // Q as stored (bf16): the products q.k are exact in the float32 accumulators, and the
  // scale log2(e)/sqrt(D) is applied in float32 (the paper's float32 logits), once per
  // score, fused with the subtraction of the running maximum: x = fma(q.k, sl2, -m_eff).
  const float sl2 = p.scale * kLog2e;
  bf16x8 qreg[NKK];
  {
    const bf16* qrow = qbase + (long long)min(qr, q_rows - 1) * rs;  // rows past the end: any row
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) qreg[kk] = *(const bf16x8*)(qrow + 16 * kk + 8 * hi);
  }
  // Running maximum without a per-tile maximum.  m_eff = the running maximum in log2 units
  // (0 while it is still -inf); the probabilities of a tile are formed against it, and the
  // tile's exact maximum is taken -- m raised, O^T and l rescaled, the probabilities formed
  // again -- only when a lane's row sum over the tile is not below kSumMax (or not finite),
  // or while m is still -inf (thrs = -1).  Every probability that reaches the products is
  // thus at most kSumMax, which bf16 and float32 hold exactly in range; the offset cancels
  // in o and is carried in lse.
  float m_eff = (m_run == -INFINITY) ? 0.f : m_run;
  float thrs = (m_run == -INFINITY) ? -1.f : kSumMax;
  const f32x16 zero16 = {};

  // ---- direct-to-LDS staging: each wave fills RPW rows of a tile ---------------------
  // load j of wave w covers rows j * NW ROWS_PER_LOAD + w ROWS_PER_LOAD + lane / CPR; the
  // lane's physical chunk is lane % CPR, its logical (global) chunk that ^ swz(row).  With
  // rows interleaved over the waves this way, swz(row) is the same for all loads of a lane
  // (the row bits it reads do not depend on j), so every load of the lane reads at one
  // byte offset goff plus a wave-uniform j * 2 NW ROWS_PER_LOAD * rs bytes.
  static_assert(RPW == LOADS * ROWS_PER_LOAD, "each wave fills LOADS row groups");
  const int goff = 2 * ((wave * ROWS_PER_LOAD + lane / CPR) * rs +
                        8 * ((lane % CPR) ^ swz<D>(wave * ROWS_PER_LOAD + lane / CPR)));
  // buffer loads with the LDS flag: the tile base is a wave-uniform descriptor, so the
  // per-tile address update is scalar work; reads past the tile return zero
  auto dload = [&](const bf16* src, int row, bf16* dst_tile) __attribute__((always_inline)) {
    const bf16* src_tile = src + (long long)row * rs;
    const int bytes = min(kBN, kv_rows - row) * rs * 2;
#pragma unroll
    for (int j = 0; j < LOADS; ++j)
      buffer_load_lds16_so(src_tile, bytes, dst_tile + (j * NW + wave_u) * ROWS_PER_LOAD * D, goff,
                           j * 2 * NW * ROWS_PER_LOAD * rs);
  };
  // the next tile of the walk (called once per tile, in order)
  auto load_k = [&](auto Bc) __attribute__((always_inline)) { dload(kbase, next_row(wk), kbuf(Bc)); };
  auto load_v = [&](auto Bc) __attribute__((always_inline)) { dload(vbase, next_row(wv), vbuf(Bc)); };

  // ---- per-lane LDS read offsets (elements), fixed across tiles ----------------------
  // row reads of K: row 32 mt + swap_bits23(l32), logical chunk 2 kk + hi
  const int krow = swap_bits23(l32);
  int koff[NKK];
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) koff[kk] = krow * D + 8 * ((2 * kk + hi) ^ swz<D>(krow));
  // transpose reads of V: rows 16 kb + 8 hi + 4 r + li / 4, dims 32 dt + 16 (g & 1) + 4 (li & 3)
  const int g16 = lane >> 4, li = lane & 15;
  int voff[2][NDT];
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) {
      const int row = 8 * hi + 4 * r + (li >> 2);
      const int d = 32 * dt + 16 * (g16 & 1) + 4 * (li & 3);
      voff[r][dt] = row * D + 8 * ((d >> 3) ^ swz<D>(row)) + (d & 7);
    }

  // ---- three-stage tile pipeline -----------------------------------------------------
  // Region t (one straight-line stretch of code per tile): the score products of tile t+1
  // (into s_nx), the exponentials of tile t (from s_cur, into the packed probabilities w)
  // and O^T += V^T P^T of tile t-1 (from pprev), interleaved step by step; the overflow
  // test of tile t closes the region, so that the only branch (the rare exact path) sits
  // between regions and tile t's probabilities are known good before tile t+1's region
  // multiplies them into O^T.  K runs one tile ahead of the scores, V one tile behind.
  // Region t reads K(t+1) and V(t-1) from buffer (t+1) % 2 and loads K(t+2), V(t) into
  // buffer t % 2.
  constexpr int NS = 2 * NKK;    // score products per tile (two 32-key halves)
  constexpr int NP = 4 * NDT;    // PV products per tile (four 16-key groups)
  constexpr int NSTEP = NS + NP;
  constexpr int PF = 2;          // operand reads issued this many steps ahead
  static_assert(NS == NP, "as many score as PV products per tile");
  f32x16 s_cur[2], s_nx[2];      // raw q.k of tiles t and t+1 (masked keys -inf)
  bf16x8 pprev[4];               // P^T of tile t-1, four 16-key groups
  float l_tile = 0.f;            // this lane's row sum of tile t's probabilities

  auto mask_tile = [&](f32x16* sc, int it) __attribute__((always_inline)) {
    const int kpos0 = k_pos0 + it * kBN;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int kpos = kpos0 + 32 * mt + 16 * (i >> 3) + 8 * hi + (i & 7);
        if (kpos > qpos) sc[mt][i] = -INFINITY;
      }
  };
  // probabilities of pair u (keys 2u, 2u+1 of this lane's 32) of a tile, packed bf16
  auto expo_pair = [&](const f32x16* sc, int u) __attribute__((always_inline)) -> uint32_t {
    const int kb = u / 4, jj = u % 4, i0 = 8 * (kb & 1) + 2 * jj;
    return pack_bf16x2(fast_exp2(fmaf(sc[kb >> 1][i0], sl2, -m_eff)), fast_exp2(fmaf(sc[kb >> 1][i0 + 1], sl2, -m_eff)));
  };
  // exact path of a tile whose probabilities failed the test: its maximum, the rescale of
  // the state, the probabilities again (w, l_tile)
  auto exact = [&](const f32x16* sc, uint32_t* w) __attribute__((always_inline)) {
    float mx = -INFINITY;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int i = 0; i < 16; ++i) mx = fmaxf(mx, sc[mt][i]);
    const float mx2 = pair_max(mx) * sl2;  // masked keys -inf; every scale positive
    const float m_new = fmaxf(m_run, mx2);
    const float alpha = (m_run == -INFINITY) ? 0.f : fast_exp2(m_run - m_new);
    l_run *= alpha;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) oacc[dt][i] *= alpha;
    m_run = m_new;
    m_eff = (m_new == -INFINITY) ? 0.f : m_new;
    thrs = (m_new == -INFINITY) ? -1.f : kSumMax;
    float r0 = 0.f, r1 = 0.f;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      w[u] = expo_pair(sc, u);
      if (u & 1) r1 = dot2_bf16_ones(w[u], r1); else r0 = dot2_bf16_ones(w[u], r0);
    }
    l_tile = r0 + r1;
  };
  // end of region: the test, then the tile's probabilities become pprev
  auto close_tile = [&](const f32x16* sc, uint32_t* w) __attribute__((always_inline)) {
    if (__builtin_amdgcn_ballot_w64(!(l_tile < thrs))) exact(sc, w);
    l_run += l_tile;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) pprev[kb] = __builtin_bit_cast(bf16x8, u32x4{w[4 * kb], w[4 * kb + 1], w[4 * kb + 2], w[4 * kb + 3]});
  };

  // Region t.  Bc = t % 2 (buffer loaded), NX: tile t+1 exists, PV: tile t-1 exists, MC:
  // tile t needs the causal mask.  Step s issues MFMA s -- the PV products of tile t-1 in
  // the first half of the region, the score products of tile t+1 in the second, so that
  // the probabilities of tile t-1 and the scores of tile t+1 are never live together --,
  // operand reads PF steps ahead, and the vector work of pair u = s * 16 / NSTEP of tile t:
  // its exponentials at that step, its packing one step later, its row-sum term two steps
  // later.
  auto region = [&](auto Bc, auto NXc, auto PVc, auto MCc, int it) __attribute__((always_inline)) {
    constexpr int B = decltype(Bc)::value;
    constexpr bool NX = decltype(NXc)::value, PV = decltype(PVc)::value, MC = decltype(MCc)::value;
    if (NX && it + 2 < nt) load_k(Bc);
    load_v(Bc);  // read by region t+1 or, after the last region, by the final products
    const bf16* kt = kbuf(std::integral_constant<int, B ^ 1>{});
    const bf16* vt = vbuf(std::integral_constant<int, B ^ 1>{});
    if constexpr (MC) mask_tile(s_cur, it);
    if constexpr (!PV) {
      if (it >= n_full && it < n_own) mask_tile(s_cur, it);
    }
    bf16x8 kop[NS], vop[NP];
    uint32_t w[16];
    float pe[16][2];
    float rs2[4] = {0.f, 0.f, 0.f, 0.f};
    auto fetch = [&](auto Sc) __attribute__((always_inline)) {
      constexpr int S = decltype(Sc)::value;
      if constexpr (S >= NP) {
        constexpr int I = S - NP;  // score product I: key half I % 2, dims 16 (I / 2)..
        if constexpr (NX) kop[I] = *(const bf16x8*)(kt + 32 * (I % 2) * D + koff[I / 2]);
      } else {
        constexpr int Q = S;  // PV product Q: keys 16 (Q / NDT).., dims 32 (Q % NDT)..
        if constexpr (PV) {
          const bf16x4 lo = lds_read_tr16(vt + 16 * (Q / NDT) * D + voff[0][Q % NDT]);
          const bf16x4 up = lds_read_tr16(vt + 16 * (Q / NDT) * D + voff[1][Q % NDT]);
          vop[Q] = bf16x8{lo[0], lo[1], lo[2], lo[3], up[0], up[1], up[2], up[3]};
        }
      }
    };
    constexpr int UPS = NSTEP / 16;  // steps per probability pair
    static_for<0, PF>([&](auto Sc) __attribute__((always_inline)) { fetch(Sc); });
    static_for<0, NSTEP + 2 * UPS>([&](auto Sc) __attribute__((always_inline)) {
      constexpr int S = decltype(Sc)::value;
      if constexpr (S + PF < NSTEP) fetch(std::integral_constant<int, S + PF>{});
      if constexpr (S < NSTEP && S >= NP) {
        constexpr int I = S - NP, mt = I % 2, kk = I / 2;
        if constexpr (NX) s_nx[mt] = mfma32(kop[I], qreg[kk], kk == 0 ? zero16 : s_nx[mt]);
      } else if constexpr (S < NP) {
        constexpr int Q = S;
        if constexpr (PV) oacc[Q % NDT] = mfma32(vop[Q], pprev[Q / NDT], oacc[Q % NDT]);
      }
      if constexpr (S % UPS == 0 && S / UPS < 16) {
        constexpr int u = S / UPS, kb = u / 4, jj = u % 4, i0 = 8 * (kb & 1) + 2 * jj;
        pe[u][0] = fast_exp2(fmaf(s_cur[kb >> 1][i0], sl2, -m_eff));
        pe[u][1] = fast_exp2(fmaf(s_cur[kb >> 1][i0 + 1], sl2, -m_eff));
      }
      if constexpr (S % UPS == 0 && S / UPS >= 1 && S / UPS <= 16) {
        constexpr int u = S / UPS - 1;
        w[u] = pack_bf16x2(pe[u][0], pe[u][1]);
      }
      if constexpr (S % UPS == 0 && S / UPS >= 2 && S / UPS <= 17) {
        constexpr int u = S / UPS - 2;
        rs2[u % 4] = dot2_bf16_ones(w[u], rs2[u % 4]);  // row sum of the bf16 probabilities used
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    l_tile = (rs2[0] + rs2[1]) + (rs2[2] + rs2[3]);
    close_tile(s_cur, w);
    if constexpr (NX) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // K(t+2) and V(t) landed
      __syncthreads();
      s_cur[0] = s_nx[0];
      s_cur[1] = s_nx[1];
    }
  };

  // regions [a, e) that have a successor and a predecessor, two at a time so that the
  // buffer parity is a constant; MC: their tiles need the mask (a branch inside a region
  // copies the scores' registers on every tile: 1 % at 4096 tokens and up)
  auto run = [&](auto MCc, int a, int e) __attribute__((always_inline)) {
    int it = a;
    if ((it & 1) && it < e) region(std::integral_constant<int, 1>{}, std::true_type{}, std::true_type{}, MCc, it++);
    for (; it + 1 < e; it += 2) {
      region(std::integral_constant<int, 0>{}, std::true_type{}, std::true_type{}, MCc, it);
      region(std::integral_constant<int, 1>{}, std::true_type{}, std::true_type{}, MCc, it + 1);
    }
    if (it < e) region(std::integral_constant<int, 0>{}, std::true_type{}, std::true_type{}, MCc, it);
  };
  // the last region (no successor): one instance for any parity, mask and predecessor,
  // its two buffers chosen at run time (the compiler then waits for the in-flight load of
  // V(t) before reading V(t-1) from the other buffer: once per workgroup)
  auto last = [&](int it) __attribute__((always_inline)) {
    if (it >= n_full && it < n_own) mask_tile(s_cur, it);
    bf16* vld = (it & 1) ? sV1 : sV0;
    const bf16* vt = (it & 1) ? sV0 : sV1;
    dload(vbase, next_row(wv), vld);  // V(t) for the final products
    uint32_t w[16];
    float rs2[4] = {0.f, 0.f, 0.f, 0.f};  // row sums in the order of the other regions
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      w[u] = expo_pair(s_cur, u);
      rs2[u % 4] = dot2_bf16_ones(w[u], rs2[u % 4]);
    }
    if (it > 0) {
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        const bf16x4 lo = lds_read_tr16(vt + 16 * (q / NDT) * D + voff[0][q % NDT]);
        const bf16x4 up = lds_read_tr16(vt + 16 * (q / NDT) * D + voff[1][q % NDT]);
        oacc[q % NDT] = mfma32(bf16x8{lo[0], lo[1], lo[2], lo[3], up[0], up[1], up[2], up[3]}, pprev[q / NDT], oacc[q % NDT]);
      }
    }
    l_tile = (rs2[0] + rs2[1]) + (rs2[2] + rs2[3]);
    close_tile(s_cur, w);
  };

  if (nt > 0) {
    // K(0) and K(1); the scores of tile 0
    load_k(std::integral_constant<int, 0>{});
    if (nt > 1) load_k(std::integral_constant<int, 1>{});
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      s_cur[mt] = mfma32(*(const bf16x8*)(sK0 + 32 * mt * D + koff[0]), qreg[0], zero16);
#pragma unroll
      for (int kk = 1; kk < NKK; ++kk) s_cur[mt] = mfma32(*(const bf16x8*)(sK0 + 32 * mt * D + koff[kk]), qreg[kk], s_cur[mt]);
    }
    // region 0 loads K(2) into the buffer of K(0): every wave must have read it
    if (nt > 2) __syncthreads();
    if (nt > 1) {
      // region 0: no predecessor
      region(std::integral_constant<int, 0>{}, std::true_type{}, std::false_type{}, std::false_type{}, 0);
      const int m0 = max(1, min(nt - 1, n_full)), m1 = max(m0, min(nt - 1, n_own));  // masked: [m0, m1)
      run(std::false_type{}, 1, m0);
      run(std::true_type{}, m0, m1);
      if constexpr (RING) run(std::false_type{}, m1, nt - 1);
    }
    last(nt - 1);
    // O^T += V^T P^T of the last tile, from V(nt-1) in buffer (nt-1) % 2
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const bf16* vt = ((nt - 1) & 1) ? sV1 : sV0;
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const bf16x4 lo = lds_read_tr16(vt + 16 * (q / NDT) * D + voff[0][q % NDT]);
      const bf16x4 up = lds_read_tr16(vt + 16 * (q / NDT) * D + voff[1][q % NDT]);
      oacc[q % NDT] = mfma32(bf16x8{lo[0], lo[1], lo[2], lo[3], up[0], up[1], up[2], up[3]}, pprev[q / NDT], oacc[q % NDT]);
    }
  }

  // ---- end of step: finalise or save the running state -------------------------------
  // The per-lane indices are recomputed here from an opaque copy of the thread index, so
  // that none of them is kept live (or spilled) across the tile loop.
  int tid_e = threadIdx.x;
  asm volatile("" : "+v"(tid_e));
  const int lane_e = tid_e & 63, wave_e = tid_e >> 6, hi_e = lane_e >> 5;
  const int qr_e = q_tile_row + wave_e * 32 + (lane_e & 31);
  if (flags & kLast) {
    const float l_tot = pair_sum(l_run);
    const float inv = 1.f / l_tot;
    if (qr_e < q_rows) {
      bf16* orow = (bf16*)p.o + (long long)b * q_bs + (long long)qr_e * rs + h * D;
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int d = 32 * dt + 8 * g + 4 * hi_e;
          u32x2 w = {pack_bf16x2(oacc[dt][4 * g] * inv, oacc[dt][4 * g + 1] * inv),
                     pack_bf16x2(oacc[dt][4 * g + 2] * inv, oacc[dt][4 * g + 3] * inv)};
          *(u32x2*)(orow + d) = w;
        }
      if (!hi_e) {
        float ln_l = logf(l_tot);
        asm volatile("" : "+v"(ln_l));  // no contraction into the logarithm: the same bits in every instance
        p.lse[(long long)bh * q_rows + qr_e] = fmaf(m_run, kLn2, ln_l);
      }
    }
  } else if constexpr (!RING) {
    // the two half sums of a row's denominator go out as they are, so that a call made of
    // several launches adds them up in the order of a call made of one
    f32x4* acc_tile = (f32x4*)(p.acc + ((long long)bh * (p.Sp / BM) + q_tile_row / BM) * (BM * D));
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 t = {oacc[dt][4 * g], oacc[dt][4 * g + 1], oacc[dt][4 * g + 2], oacc[dt][4 * g + 3]};
        acc_tile[((wave_e * NDT + dt) * 4 + g) * 64 + lane_e] = t;
      }
    const long long st_row = (long long)bh * p.Sp + qr_e;
    if (!hi_e) p.m[st_row] = m_run;
    p.l[2 * st_row + hi_e] = l_run;
  }
}

}  // namespace

// Long blocks (D = 128, at least 16384 keys, a multiple of 256) run the eight-wave kernel:
// 256 queries per workgroup, so each key/value tile is loaded once for twice the queries
// (one workgroup per CU instead of two).  One ring step at a time its longer start and end
// outweigh the saved loads at 4096-8192 keys; over the whole ring in one launch the two are
// within 2 % of each other at 16384 tokens x 16 heads (4 waves 955 us, 8 waves 943) and 65536
// x 8 (7288, 7244), the four-wave kernel ahead at 32768 x 32 (7490, 7860) and wherever the
// workgroups are few (2048 x 8: 35.5, 52.7; 16384 x 12: 776, 840).  The choice depends only on
// (D, c), so a call cut into steps uses one kernel and the float32 state keeps one layout.
static bool fwd_bf16_wide(int D, int c) { return D == 128 && c % 256 == 0 && c >= 16384; }

hipError_t launch_fwd_bf16(const FwdStep& s, int D, hipStream_t st) {
  const int total = s.n_slots * s.B * s.H * (s.c / kBM);
  if (total == 0) return hipSuccess;
  if (fwd_bf16_wide(D, s.c))
    hipLaunchKernelGGL((fwd_bf16_kernel<128, 8, false>), dim3(total / 2), dim3(512), 0, st, s);
  else if (D == 128)
    hipLaunchKernelGGL((fwd_bf16_kernel<128, 4, false>), dim3(total), dim3(kThreads), 0, st, s);
  else
    hipLaunchKernelGGL((fwd_bf16_kernel<64, 4, false>), dim3(total), dim3(kThreads), 0, st, s);
  return hipGetLastError();
}

hipError_t launch_fwd_ring_bf16(const FwdRing& s, int D, hipStream_t st) {
  const int G = s.B * s.H;
  if (fwd_bf16_wide(D, s.c))
    hipLaunchKernelGGL((fwd_bf16_kernel<128, 8, true>), dim3(ring_grid(G, (s.S + 255) / 256)), dim3(512), 0, st, s);
  else if (D == 128)
    hipLaunchKernelGGL((fwd_bf16_kernel<128, 4, true>), dim3(ring_grid(G, (s.S + kBM - 1) / kBM)), dim3(kThreads), 0, st, s);
  else
    hipLaunchKernelGGL((fwd_bf16_kernel<64, 4, true>), dim3(ring_grid(G, (s.S + kBM - 1) / kBM)), dim3(kThreads), 0, st, s);
  return hipGetLastError();
}

}  // namespace ra
