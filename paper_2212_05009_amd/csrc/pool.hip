// Device memory kept between calls.
//
// hipMalloc / hipFree cost tens of microseconds each, hipFree waits for the device, and large blocks are mapped anew:
// building the 11.8 M entry graph of R-MAT 2^18 spent 6 of 8.5 ms in them, and up to 80 ms when builds follow each
// other directly.  Handle arrays, workspaces and the temporaries of build / induced / partition calls therefore come
// from a pool of freed blocks.
//
//  * A block enters the pool only when no enqueued work can touch it: the temporaries of a call after the call has
//    waited for its stream, a handle's arrays after gcn_csr_free has waited for the handle's device.  Any thread and any
//    stream may therefore take it at once.  Where the wait fails (another thread captures a graph), it is not kept.
//  * A block serves requests of at least 3/4 of its size, so what is held and not used stays small.
//  * Bounded: at most 1/64 of the device's memory is kept (4.5 of 288 GB), least recently freed blocks go first; a block
//    that lies unused over 256 later returns goes back to the runtime; a failed hipMalloc empties the pool and retries;
//    gcn_release_memory empties it on demand.
//  * The lock covers the lists only.  hipFree, which waits for the device, runs outside it: a thread that gives blocks back
//    holds up no other thread's calls, on this GPU or another.
#include <condition_variable>
#include <list>
#include <map>
#include <mutex>
#include <new>
#include <unordered_map>
#include <vector>

#include "common.h"

namespace gcn {
namespace {

constexpr int kPoolDevices = 64;
constexpr uint64_t kIdleReturns = 256;

struct Block { void* p; size_t bytes; uint64_t freed_at; };
typedef std::list<Block> BlockList;

struct DevicePool {
  BlockList by_age;                                       // oldest first
  std::multimap<size_t, BlockList::iterator> by_size;
  size_t held = 0, limit = 0;
  uint64_t returns = 0;
  int leaving = 0;                                        // threads with blocks taken off the lists but not yet freed
};

struct Pool {
  std::mutex mu;
  std::condition_variable left;                             // some DevicePool::leaving has fallen
  std::unordered_map<void*, std::pair<int, size_t>> live;   // block -> device, size
  DevicePool dev[kPoolDevices];
  std::vector<void*> pinned;                                // idle pinned host pages
};

// In memory of its own: the first use allocates nothing, so it cannot throw, and it is never destroyed (at process end the
// runtime takes the device memory back).
Pool& pool() {
  alignas(Pool) static unsigned char place[sizeof(Pool)];
  static Pool* p = new (place) Pool();
  return *p;
}

// moves the oldest block from the lists to `gone` (under the lock; no allocation)
void drop_oldest(DevicePool& d, BlockList& gone) {
  BlockList::iterator b = d.by_age.begin();
  auto r = d.by_size.equal_range(b->bytes);
  for (auto i = r.first; i != r.second; ++i)
    if (i->second == b) { d.by_size.erase(i); break; }
  d.held -= b->bytes;
  gone.splice(gone.end(), d.by_age, b);
}

// frees what has been taken off the lists of d; called with the lock held, which is open while hipFree runs
void free_gone(Pool& P, DevicePool& d, BlockList& gone, std::unique_lock<std::mutex>& lock) {
  if (gone.empty()) return;
  ++d.leaving;
  lock.unlock();
  for (const Block& b : gone) (void)hipFree(b.p);
  lock.lock();
  --d.leaving;
  P.left.notify_all();
}

// sizes in steps of 1/8 of a power of two, so that requests of similar size share blocks
size_t pool_size(size_t bytes) {
  if (bytes < 4096) return 4096;
  size_t step = 512;
  while (step * 16 <= bytes) step <<= 1;
  return (bytes + step - 1) / step * step;
}

}  // namespace

int pool_alloc(void** out, size_t bytes) {
  *out = nullptr;
  int device = 0;
  GCN_HIP(hipGetDevice(&device));
  const size_t want = pool_size(bytes);
  try {
    Pool& P = pool();
    const bool pooled = device >= 0 && device < kPoolDevices;
    if (pooled) {
      std::lock_guard<std::mutex> lock(P.mu);
      DevicePool& d = P.dev[device];
      auto i = d.by_size.lower_bound(want);
      if (i != d.by_size.end() && i->first - i->first / 4 <= want) {
        BlockList::iterator b = i->second;
        P.live.emplace(b->p, std::make_pair(device, b->bytes));
        *out = b->p;
        d.held -= b->bytes;
        d.by_size.erase(i);
        d.by_age.erase(b);
        return GCN_OK;
      }
    }
    void* p = nullptr;
    hipError_t e = hipMalloc(&p, want);
    if (e == hipErrorOutOfMemory && pooled) {
      (void)hipGetLastError();
      {
        std::unique_lock<std::mutex> lock(P.mu);
        DevicePool& d = P.dev[device];
        BlockList gone;
        while (!d.by_age.empty()) drop_oldest(d, gone);
        free_gone(P, d, gone, lock);
        P.left.wait(lock, [&] { return d.leaving == 0; });      // what other threads are giving back counts too
      }
      e = hipMalloc(&p, want);
    }
    if (e != hipSuccess) return fail(e == hipErrorOutOfMemory ? GCN_ENOMEM : GCN_EHIP, "hipMalloc(%zu bytes): %s", want, hipGetErrorString(e));
    *out = p;
    if (pooled) {
      try {
        std::lock_guard<std::mutex> lock(P.mu);
        P.live.emplace(p, std::make_pair(device, want));
      } catch (const std::bad_alloc&) {        // not on the list: pool_free returns it to the runtime
      }
    }
    return GCN_OK;
  } catch (const std::bad_alloc&) {
    return fail(GCN_ENOMEM, "host allocation failed");
  }
}

void pool_free(void* p, bool idle) {
  if (!p) return;
  Pool& P = pool();
  std::unique_lock<std::mutex> lock(P.mu);
  auto i = P.live.find(p);
  if (i == P.live.end()) {
    lock.unlock();
    (void)hipFree(p);
    return;
  }
  const int device = i->second.first;
  const size_t bytes = i->second.second;
  P.live.erase(i);
  DevicePool& d = P.dev[device];
  if (!d.limit) {
    hipDeviceProp_t prop;
    d.limit = hipGetDeviceProperties(&prop, device) == hipSuccess ? prop.totalGlobalMem / 64 : (size_t)1 << 30;
  }
  ++d.returns;
  BlockList gone;
  bool kept = false;
  if (idle && bytes <= d.limit) {
    const size_t listed = d.by_age.size();
    try {
      d.by_age.push_back(Block{p, bytes, d.returns});
      d.by_size.emplace(bytes, std::prev(d.by_age.end()));
      d.held += bytes;
      kept = true;
    } catch (const std::bad_alloc&) {
      if (d.by_age.size() > listed) d.by_age.pop_back();
    }
  }
  if (kept) {
    while (d.held > d.limit || d.by_age.front().freed_at + kIdleReturns < d.returns) drop_oldest(d, gone);
    free_gone(P, d, gone, lock);
    return;
  }
  ++d.leaving;
  lock.unlock();
  (void)hipFree(p);
  lock.lock();
  --d.leaving;
  P.left.notify_all();
}

// Pinned host pages: at most kMaxPinned are kept.
constexpr size_t kMaxPinned = 16;

int pinned_take(void** out) {
  *out = nullptr;
  {
    Pool& P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    if (!P.pinned.empty()) { *out = P.pinned.back(); P.pinned.pop_back(); return GCN_OK; }
  }
  GCN_HIP(hipHostMalloc(out, kPinnedBytes, hipHostMallocPortable));
  return GCN_OK;
}

void pinned_give(void* p) {
  if (!p) return;
  try {
    Pool& P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    if (P.pinned.size() < kMaxPinned) { P.pinned.push_back(p); return; }
  } catch (const std::bad_alloc&) {
  }
  (void)hipHostFree(p);
}

}  // namespace gcn

extern "C" int gcn_release_memory(void) {
  using namespace gcn;
  clear_error();
  Pool& P = pool();
  std::unique_lock<std::mutex> lock(P.mu);
  for (DevicePool& d : P.dev) {
    BlockList gone;
    while (!d.by_age.empty()) drop_oldest(d, gone);
    free_gone(P, d, gone, lock);
  }
  std::vector<void*> pages;
  pages.swap(P.pinned);
  lock.unlock();
  for (void* p : pages) (void)hipHostFree(p);
  return GCN_OK;
}
