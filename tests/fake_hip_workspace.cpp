// The library's workspace code against a model of the HIP runtime, on the host.
//
// The model: a driver with kDriver bytes; a stream-ordered pool whose blocks count against them
// from their allocation until a trim after the stream that freed them has been waited for.  A
// block that two calls hold at once, or that is freed twice, is an error.
#include <stdio.h>
#include <stdlib.h>

#include <map>
#include <memory>
#include <mutex>
#include <thread>
#include <vector>

#include "ra_runtime.h"

namespace {
constexpr size_t kMiB = (size_t)1 << 20, kDriver = 1024 * kMiB;
std::mutex mu;
struct Block {
  size_t bytes;
  bool freed, waited;  // by its owner; and the stream it was freed on waited for
  hipStream_t on;
};
std::map<void*, Block> blocks;
size_t used = 0;
int waits = 0;
uintptr_t next_ptr = 0x100000;

void check(bool ok, const char* what) {
  if (ok) return;
  printf("FAILED: %s\n", what);
  fflush(stdout);
  abort();
}
size_t live() {  // blocks not freed
  std::lock_guard<std::mutex> lk(mu);
  size_t n = 0;
  for (auto& b : blocks) n += !b.second.freed;
  return n;
}
}  // namespace

extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "model"; }
hipError_t hipMemPoolCreate(hipMemPool_t* p, const hipMemPoolProps*) { *p = (hipMemPool_t)0x10; return hipSuccess; }
hipError_t hipMemPoolSetAttribute(hipMemPool_t, hipMemPoolAttr, void*) { return hipSuccess; }
hipError_t hipMemPoolDestroy(hipMemPool_t) { return hipSuccess; }
hipError_t hipMallocFromPoolAsync(void** p, size_t bytes, hipMemPool_t, hipStream_t) {
  std::lock_guard<std::mutex> lk(mu);
  if (used + bytes > kDriver) return hipErrorOutOfMemory;
  *p = (void*)next_ptr;
  next_ptr += bytes + 256;
  blocks[*p] = {bytes, false, false, nullptr};
  used += bytes;
  return hipSuccess;
}
hipError_t hipFreeAsync(void* p, hipStream_t s) {
  std::lock_guard<std::mutex> lk(mu);
  auto it = blocks.find(p);
  check(it != blocks.end() && !it->second.freed, "block freed once");
  it->second.freed = true;
  it->second.on = s;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  std::lock_guard<std::mutex> lk(mu);
  ++waits;
  for (auto& b : blocks)
    if (b.second.freed && b.second.on == s) b.second.waited = true;
  return hipSuccess;
}
hipError_t hipMemPoolTrimTo(hipMemPool_t, size_t) {
  std::lock_guard<std::mutex> lk(mu);
  for (auto it = blocks.begin(); it != blocks.end();)
    if (it->second.freed && it->second.waited) {
      used -= it->second.bytes;
      it = blocks.erase(it);
    } else {
      ++it;
    }
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)0x20; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
}

namespace ra {
thread_local std::string g_err;
int set_err(int code, const char*, ...) { return code; }
}  // namespace ra
using namespace ra;

static void* call(size_t bytes, hipStream_t s) {
  CallResources R(s);
  check(R.alloc(bytes) == RA_OK, "allocation");
  return R.ws;
}

// Kept blocks are reused, bounded, and returned by a release in one go.
static void release() {
  void* a = call(8 * kMiB, nullptr);
  check(call(8 * kMiB, nullptr) == a, "a kept block is used again");
  check(call(7 * kMiB, nullptr) == a, "for a near size too");
  for (int i = 0; i < 200; ++i) {
    CallResources R[3] = {CallResources(nullptr), CallResources(nullptr), CallResources(nullptr)};
    for (auto& r : R) check(r.alloc((size_t)(1 + (i * 37) % 64) * kMiB) == RA_OK, "allocation");
    check(R[0].ws != R[1].ws && R[1].ws != R[2].ws && R[0].ws != R[2].ws, "calls in flight share no block");
    if (i % 20 == 0) {  // blocks given up for others are free by now
      hipStreamSynchronize(nullptr);
      hipMemPoolTrimTo(nullptr, 0);
    }
  }
  check(live() <= (size_t)kWsKeepCount, "bounded count");
  hipStreamSynchronize(nullptr);
  hipMemPoolTrimTo(nullptr, 0);
  check(used > 0 && used <= kWsKeepTotal, "bounded bytes");
  const int before = waits;
  check(workspace_drop_kept() && used == 0, "a release returns every kept block to the driver");
  check(waits == before + 1, "it waits for the null stream");
  check(!workspace_drop_kept() && waits == before + 1, "and for nothing when nothing is kept");
}

// Kept blocks make room for a workspace of any stream.
static void short_of_memory() {
  hipStream_t other = (hipStream_t)0x30;
  for (hipStream_t s : {(hipStream_t) nullptr, other}) {
    {
      CallResources A(nullptr), B(nullptr), C(nullptr);
      for (auto* r : {&A, &B, &C}) check(r->alloc(60 * kMiB) == RA_OK, "allocation");
    }
    check(live() == 3, "three blocks kept");
    auto R = std::make_unique<CallResources>(s);
    check(R->alloc(kDriver - 100 * kMiB) == RA_OK, "kept blocks make room");
    {
      CallResources Q(s);
      check(Q.alloc(200 * kMiB) == RA_ENOMEM && Q.ws == nullptr, "no room: an error");
    }
    R.reset();
    hipStreamSynchronize(s);
    hipMemPoolTrimTo(nullptr, 0);
    check(used == 0, "all returned");
  }
}

// Host threads on the null stream: a block belongs to one call at a time.
static void threads() {
  std::mutex own_mu;
  std::map<void*, int> owner;
  std::vector<std::thread> ts;
  for (int t = 0; t < 6; ++t)
    ts.emplace_back([&, t] {
      unsigned x = 12345u + t;
      for (int i = 0; i < 4000; ++i) {
        x = x * 1664525u + 1013904223u;
        CallResources R(nullptr);
        check(R.alloc(((size_t)(x >> 8) % (4 * kMiB)) + 1) == RA_OK, "allocation");
        {
          std::lock_guard<std::mutex> lk(own_mu);
          check(owner.emplace(R.ws, t).second, "a block belongs to one call");
        }
        if (x % 7 == 0) std::this_thread::yield();
        {
          std::lock_guard<std::mutex> lk(own_mu);
          owner.erase(R.ws);
        }
        if (t == 0 && i % 500 == 0) workspace_drop_kept();
      }
    });
  for (auto& t : ts) t.join();
  workspace_drop_kept();
  check(used == 0, "all returned");
}

int main() {
  release();
  short_of_memory();
  threads();
  printf("ok\n");
  return 0;
}
