// Host-side runtime helpers shared by the C-ABI translation units: thread-local error
// text, HIP error mapping, stream-ordered per-call workspace, optional kernel timing.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <initializer_list>
#include <string>
#include <vector>

#include "ringattn.h"

namespace ra {

extern thread_local std::string g_err;
int set_err(int code, const char* fmt, ...);

#define RA_HIP(expr)                                                                   \
  do {                                                                                 \
    hipError_t e_ = (expr);                                                            \
    if (e_ != hipSuccess)                                                              \
      return set_err(e_ == hipErrorOutOfMemory ? RA_ENOMEM : RA_EHIP, "%s failed: %s", \
                     #expr, hipGetErrorString(e_));                                    \
  } while (0)

// Tensors made of rows of elements are read and written with 16-byte vector accesses from
// their start, so they must begin on a 16-byte boundary (rows16); float32 per-row vectors
// such as lse on a 4-byte one (vec4).  A null pointer (an absent optional argument) passes.
inline int check_aligned(std::initializer_list<const void*> rows16, std::initializer_list<const void*> vec4 = {}) {
  for (const void* p : rows16)
    if (reinterpret_cast<uintptr_t>(p) & 15u) return set_err(RA_EINVAL, "tensor pointer %p is not 16-byte aligned", p);
  for (const void* p : vec4)
    if (reinterpret_cast<uintptr_t>(p) & 3u) return set_err(RA_EINVAL, "pointer %p is not 4-byte aligned", p);
  return RA_OK;
}

// The current device's workspace pool: a stream-ordered memory pool owned by the library
// (created on first use, release threshold unlimited, so workspace freed at the end of a
// call is reused by the next call instead of being unmapped and mapped again).  The
// device's default pool is left as it is.
int workspace_pool(hipMemPool_t* out);

// Small workspaces of the default (null) stream are kept between calls: allocating from the
// pool and freeing cost the host 12 us a call, as much as a short call's kernels.  A block given
// back after a call goes to the next one: stream order keeps the two apart, and the null
// stream of a device is never destroyed (another stream's handle can come back as a new
// stream's, which need not be ordered after the old one's work, so other streams' workspaces
// go to the pool and back, as does what a capture allocates, the null stream taking part in
// none).  At most kWsKeepCount blocks a device of at most kWsKeepBlock bytes, kWsKeepTotal in
// all, are kept; ring_attn_release_workspace() returns them.
constexpr size_t kWsKeepBlock = (size_t)64 << 20, kWsKeepTotal = (size_t)256 << 20;
constexpr int kWsKeepCount = 32;
// A kept block of the device of at least `bytes` (its size in *got), or null.
void* workspace_take(int dev, size_t bytes, size_t* got);
// Offers a block whose last use is enqueued on the device's null stream; false: free it.
bool workspace_give(int dev, void* p, size_t bytes);
// Gives the current device's kept blocks, and what else the pool has free, back to the driver;
// true if there were any.  Waits for the null stream if so.
bool workspace_drop_kept();

// Stream-ordered workspace and events owned by one call; released on every exit path.
// side: the library's side stream when the call enqueued work on it.  Before the workspace
// goes back the caller stream waits for everything enqueued on the side stream
// so far -- also on an error return in the middle of a call, where the call's own final
// join was never enqueued -- so that no copy still queued there can write into memory a
// later call has been given.
struct CallResources {
  hipStream_t stream;
  hipStream_t side = nullptr;
  void* ws = nullptr;
  size_t ws_bytes = 0;
  int keep_dev = -1;  // the device that may keep ws, or -1
  std::vector<hipEvent_t> events;
  explicit CallResources(hipStream_t s) : stream(s) {}
  ~CallResources() {
    if (ws && side && side != stream) {
      hipEvent_t e;
      if (hipEventCreateWithFlags(&e, hipEventDisableTiming) == hipSuccess) {
        (void)hipEventRecord(e, side);
        (void)hipStreamWaitEvent(stream, e, 0);
        (void)hipEventDestroy(e);
      } else {
        (void)hipStreamSynchronize(side);
      }
    }
    if (ws && !(keep_dev >= 0 && workspace_give(keep_dev, ws, ws_bytes))) (void)hipFreeAsync(ws, stream);
    for (hipEvent_t e : events) (void)hipEventDestroy(e);
  }
  int alloc(size_t bytes) {
    if (bytes == 0) return RA_OK;
    if (stream == nullptr && bytes <= kWsKeepBlock) {
      RA_HIP(hipGetDevice(&keep_dev));
      if ((ws = workspace_take(keep_dev, bytes, &ws_bytes))) return RA_OK;
      // sizes in steps of an eighth of their power of two, so that near sizes share a block
      size_t step = (size_t)64 << 10;
      while (step * 16 < bytes) step *= 2;
      bytes = (bytes + step - 1) / step * step;
    }
    hipMemPool_t pool;
    int rc = workspace_pool(&pool);
    if (rc) return rc;
    hipError_t e = hipMallocFromPoolAsync(&ws, bytes, pool, stream);
    if (e == hipErrorOutOfMemory && workspace_drop_kept()) {  // whichever stream asks
      (void)hipGetLastError();
      e = hipMallocFromPoolAsync(&ws, bytes, pool, stream);
    }
    RA_HIP(e);
    ws_bytes = bytes;
    return RA_OK;
  }
  int event(hipEvent_t* e) {
    RA_HIP(hipEventCreateWithFlags(e, hipEventDisableTiming));
    events.push_back(*e);
    return RA_OK;
  }
};

// Kernel timing (ring_attn_timing_enable): true when launches are to be bracketed.
bool timing_on();
void timing_push(int kind, hipEvent_t a, hipEvent_t b);

// Runs f() (which enqueues kernels on st) between two timing events when timing is on.
template <class F>
hipError_t timed_launch(int kind, hipStream_t st, F&& f) {
  if (!timing_on()) return f();
  // no system-scope fences: the events only carry timestamps, and the fences of a default
  // event widen the gap between consecutive launches by about 3 us per event
  hipEvent_t a, b;
  hipError_t e = hipEventCreateWithFlags(&a, hipEventDisableSystemFence);
  if (e != hipSuccess) return e;
  if ((e = hipEventCreateWithFlags(&b, hipEventDisableSystemFence)) != hipSuccess) {
    (void)hipEventDestroy(a);
    return e;
  }
  (void)hipEventRecord(a, st);
  e = f();
  (void)hipEventRecord(b, st);
  timing_push(kind, a, b);
  return e;
}

}  // namespace ra
