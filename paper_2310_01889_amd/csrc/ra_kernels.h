// Step descriptors passed by value to the kernels, and the launchers the ring
// scheduler calls.  One kernel launch covers every virtual host that has work in one
// ring step; each host contributes one "slot".
#pragma once

#include <hip/hip_runtime.h>

namespace ra {

constexpr int kMaxSlots = 64;        // hosts per launch (= maximum ring size)
constexpr int kFirst = 1;            // host's first active step: start from m=-inf, l=0, acc=0
constexpr int kLast = 2;             // host's last active step: finalize o = acc / l, lse

// One host's work in one ring step.
struct StepHost {
  const void* k;          // key block, row 0 (batch 0, head 0)
  const void* v;          // value block, row 0
  long long kv_bstride;   // elements between consecutive batches of k / v
  int q_row0;             // first row of the host's queries in q / o / lse / state rows
  int q_pos0;             // global position of that row (causal mask)
  int k_pos0;             // global position of the key block's first row
  int kv_rows;            // rows of the block that exist (the rest read as zero)
  int flags;              // kFirst | kLast
};

// Forward step, bf16: fold one key/value block into every listed host's running state.
struct FwdStep {
  StepHost host[kMaxSlots];
  const void* q;          // [B, Sq, H, D]
  void* o;                // [B, Sq, H, D]
  float* lse;             // [B, H, Sq]
  float* acc;             // running numerator, float32, B*H*Sp*D
  float* m;               // running max (log2 units of the scaled scores), [B, H, Sp]
  float* l;               // running denominator in two halves, [B, H, Sp, 2]
  long long q_bstride;    // Sq * H * D
  int n_slots, B, H, Sq, c, causal;
  int Sp;                 // rows of the state: the hosts' blocks in full (Sq, rounded up to blocks)
  float scale;            // 1 / sqrt(D)
};

// Forward over the whole ring in one launch, bf16 or float32 tensors: every host's queries
// against every block, read where the blocks lie (rows [j c, (j + 1) c) of k and v).
struct FwdRing {
  const void *q, *k, *v;  // [B, S, H, D]
  void* o;                // [B, S, H, D]
  float* lse;             // [B, H, S]
  long long bstride;      // S * H * D
  int B, H, S, c, N, causal;  // bf16, causal: S need not fill the N blocks of c rows
  float scale;            // 1 / sqrt(D)
};

// Backward step, bf16: one key/value block per host; dq accumulates per host, dk/dv per block.
struct BwdStep {
  StepHost host[kMaxSlots];
  const void* q;          // [B, Sq, H, D]
  const void* dO;         // [B, Sq, H, D]
  const float* lse;       // [B, H, Sq]  -lse sqrt(D)
  const float* delta;     // [B, H, Sq]  -rowsum(dO * o)
  float* dq;              // float32 [B, Sq, H, D]: accumulators between the host's steps
  float* dk;              // float32 [B, Skv, H, D]: gradient of the block each host holds
  float* dv;              //   (home position of that block: see dkv_row0)
  int dkv_row0[kMaxSlots];// first row of the host's current block in dk / dv
  long long q_bstride;    // Sq * H * D
  long long dkv_bstride;  // elements between consecutive batches of dk / dv
  int n_slots, B, H, Sq, c, causal;
  int Skv;                // rows of dk / dv that exist
  float scale;
  // whole: the call holds every contribution to dk / dv, so these hold the
  // accumulators between steps; the block a slot holds is touched for the first (kFirst: start
  // from zero) or the last time (kLast: the sum goes out, rounded, to dk_out / dv_out).
  // Otherwise contributions are added into dk / dv.
  int whole;
  unsigned char dkv_flags[kMaxSlots];
  void* dk_out;           // bf16 [B, Skv, H, D] results (rows at the block's home position)
  void* dv_out;
  void* dq_out;           // bf16 [B, Sq, H, D], written on a host's kLast step
};

// Backward over the whole ring: bf16, one launch for dK and dV, one for dQ; float32, one for
// all three.
struct BwdRing {
  const void *q, *k, *v, *dO;  // [B, S, H, D]
  const float *lse, *delta;    // [B, H, S]: -lse sqrt(D) and -Delta (bf16), lse and Delta (float32)
  void *dq, *dk, *dv;          // [B, S, H, D]
  long long bstride;           // S * H * D
  int B, H, S, c, N, causal;   // bf16, causal: S need not fill the N blocks of c rows
  float scale;
};

hipError_t launch_fwd_bf16(const FwdStep& s, int D, hipStream_t st);
hipError_t launch_fwd_ring_bf16(const FwdRing& s, int D, hipStream_t st);
hipError_t launch_fwd_ring_f32(const FwdRing& s, int D, hipStream_t st);
// -Delta = -rowsum(dO * o) and -lse * sqrt(D), both [B, H, S] (for the bf16 step kernels)
hipError_t launch_bwd_pre_bf16(const void* o, const void* dO, const float* lse, float* ndelta, float* nlse_s,
                               int B, int S, int H, int D, hipStream_t st);
hipError_t launch_bwd_pre_f32(const float* o, const float* dO, float* delta, int B, int S, int H,
                              int D, hipStream_t st);
hipError_t launch_bwd_bf16(const BwdStep& s, int D, hipStream_t st);
hipError_t launch_bwd_ring_bf16(const BwdRing& s, int D, hipStream_t st);
hipError_t launch_bwd_ring_f32(const BwdRing& s, int D, hipStream_t st);

}  // namespace ra
