// The workspace pool of each device and the blocks of it kept for the null streams.
#include <mutex>
#include <new>
#include <vector>

#include "ra_runtime.h"

namespace ra {

namespace {
std::mutex g_pool_mu;
hipMemPool_t g_pool[64];
}  // namespace

int workspace_pool(hipMemPool_t* out) {
  int dev = 0;
  RA_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) return set_err(RA_EHIP, "device index %d out of range", dev);
  std::lock_guard<std::mutex> lk(g_pool_mu);
  if (!g_pool[dev]) {
    hipMemPoolProps props{};
    props.allocType = hipMemAllocationTypePinned;
    props.handleTypes = hipMemHandleTypeNone;
    props.location.type = hipMemLocationTypeDevice;
    props.location.id = dev;
    hipMemPool_t pool;
    RA_HIP(hipMemPoolCreate(&pool, &props));
    uint64_t thr = ~0ull;
    hipError_t e = hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &thr);
    if (e != hipSuccess) {
      (void)hipMemPoolDestroy(pool);
      return set_err(RA_EHIP, "hipMemPoolSetAttribute failed: %s", hipGetErrorString(e));
    }
    g_pool[dev] = pool;
  }
  *out = g_pool[dev];
  return RA_OK;
}

// Kept workspaces of the null streams (see ra_runtime.h).
namespace {
struct KeptBlock {
  void* p;
  size_t bytes;
  int dev;
};
std::mutex g_kept_mu;
std::vector<KeptBlock> g_kept;
}  // namespace

void* workspace_take(int dev, size_t bytes, size_t* got) {
  std::lock_guard<std::mutex> lk(g_kept_mu);
  int best = -1;
  for (int i = 0; i < (int)g_kept.size(); ++i) {
    const KeptBlock& b = g_kept[i];
    if (b.dev == dev && b.bytes >= bytes && b.bytes <= 2 * bytes + ((size_t)1 << 20) &&
        (best < 0 || b.bytes < g_kept[best].bytes))
      best = i;
  }
  if (best < 0) return nullptr;
  void* p = g_kept[best].p;
  *got = g_kept[best].bytes;
  g_kept.erase(g_kept.begin() + best);
  return p;
}

bool workspace_give(int dev, void* p, size_t bytes) {
  std::lock_guard<std::mutex> lk(g_kept_mu);
  int count = 0, first = -1;
  size_t total = 0;
  for (int i = 0; i < (int)g_kept.size(); ++i)
    if (g_kept[i].dev == dev) {
      if (first < 0) first = i;
      ++count;
      total += g_kept[i].bytes;
    }
  // full: the block kept longest makes room (the freed memory stays in the pool)
  if (first >= 0 && (count >= kWsKeepCount || total + bytes > kWsKeepTotal)) {
    (void)hipFreeAsync(g_kept[first].p, nullptr);
    total -= g_kept[first].bytes;
    --count;
    g_kept.erase(g_kept.begin() + first);
  }
  if (count >= kWsKeepCount || total + bytes > kWsKeepTotal) return false;
  try {
    g_kept.push_back({p, bytes, dev});
  } catch (const std::bad_alloc&) {  // called from a destructor: nothing may escape
    return false;
  }
  return true;
}

bool workspace_drop_kept() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return false;
  bool any = false;
  {
    std::lock_guard<std::mutex> lk(g_kept_mu);
    for (int i = (int)g_kept.size() - 1; i >= 0; --i)
      if (g_kept[i].dev == dev) {
        (void)hipFreeAsync(g_kept[i].p, nullptr);
        g_kept.erase(g_kept.begin() + i);
        any = true;
      }
  }
  hipMemPool_t pool;
  if (!any || workspace_pool(&pool)) return any;
  // until the null stream has passed the frees a trim finds nothing to return
  (void)hipStreamSynchronize(nullptr);
  (void)hipMemPoolTrimTo(pool, 0);
  return true;
}

}  // namespace ra
