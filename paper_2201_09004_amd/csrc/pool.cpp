// Working memory of the calls: device blocks of vectors and reduction buffers,
// and the small pinned host blocks of the solver states, kept for reuse.
//
// Every call takes its vectors here and gives them back when it ends.  The
// runtime's stream-ordered pool served them before; on a 2 GB block its free
// alone took 1 ms, and a call whose blocks it did not find again went to the
// driver every time (71.8 ms for a 3.3 ms Schur application at 24^3x64).
//
// A block that is given back waits in the list of its thread and stream and is
// handed out again to that thread on that stream only, so the stream's own
// order keeps its two users apart.  When a call of the library has waited for
// its stream, the blocks of its list move to one that serves every stream, so
// that a caller's streams may come and go (with a list kept per stream, twenty
// Schur applications at 24^3x64 on streams of their own held 27 GiB; on one, 1.4
// GiB).  So do the blocks of a stream that the library destroys.
// hipStreamPerThread names another stream on every thread, as the lists do.
//
// What waits is bounded by a quarter of the device's memory: beyond that blocks
// go back to the device (hipFree, which waits for the device's work), as all of
// them do when an allocation fails and when the last context of the device is
// finalized; the pinned blocks go with the last context of all.  HISQ with 12
// columns and 8 masses at 32^3x96, all sites, which reaches the bound in every
// call: 3.94 s, with three quarters as the bound 3.91 s.
#include <map>
#include <mutex>
#include <thread>
#include <unordered_map>
#include <vector>

#include "pool.h"

namespace lq {
namespace {

constexpr int kMaxDevices = 64;
using Sized = std::multimap<size_t, void*>;

// 4 KiB steps up to 1 MiB, 2 MiB steps above: widths that differ little share blocks
size_t block_size(size_t n) {
  const size_t step = n <= ((size_t)1 << 20) ? 4096 : (size_t)2 << 20;
  return (n + step - 1) / step * step;
}

// the smallest block that holds n and wastes at most a quarter
void* take(Sized& l, size_t n, size_t* got) {
  auto it = l.lower_bound(n);
  if (it == l.end() || it->first > n + n / 4) return nullptr;
  void* p = it->second;
  *got = it->first;
  l.erase(it);
  return p;
}

using Owner = std::pair<hipStream_t, std::thread::id>;
Owner me(hipStream_t s) { return {s, std::this_thread::get_id()}; }

struct DevicePool {
  std::map<Owner, Sized> by_owner;
  Sized idle;  // blocks without pending work
  size_t waiting = 0, limit = 0;
  int contexts = 0;

  // removes blocks from the lists until at most `keep` bytes wait: idle ones
  // first, then the largest (the caller frees them, outside the lock)
  std::vector<void*> shrink(size_t keep) {
    std::vector<void*> out;
    while (waiting > keep) {
      Sized* from = idle.empty() ? nullptr : &idle;
      if (!from)
        for (auto& kv : by_owner)
          if (!kv.second.empty() && (!from || kv.second.rbegin()->first > from->rbegin()->first)) from = &kv.second;
      if (!from) break;
      auto it = std::prev(from->end());
      waiting -= it->first;
      out.push_back(it->second);
      from->erase(it);
    }
    return out;
  }
};

struct Handed {  // a block in use
  size_t bytes;
  int device;
};

struct Pools {
  std::mutex m;
  int contexts = 0;  // of all devices
  DevicePool dev[kMaxDevices];
  std::unordered_map<void*, Handed> used;
};
Pools& pools() {
  static Pools* p = new Pools;  // never destroyed: what is left at process exit is the driver's to free
  return *p;
}
int current_device() {
  int d = 0;
  (void)hipGetDevice(&d);
  return d < 0 || d >= kMaxDevices ? 0 : d;
}
void give_back(const std::vector<void*>& v) {
  for (void* p : v) (void)hipFree(p);
}

// pinned host blocks by size, at most kPinnedKept of them
constexpr size_t kPinnedKept = 64;
struct PinnedPool {
  std::mutex m;
  Sized blocks;
};
PinnedPool& pinned() {
  static PinnedPool* p = new PinnedPool;
  return *p;
}

}  // namespace

void* work_alloc(size_t bytes, hipStream_t s) {
  Pools& P = pools();
  const int dev = current_device();
  const size_t n = block_size(bytes);
  {
    std::lock_guard<std::mutex> lk(P.m);
    DevicePool& d = P.dev[dev];
    size_t got = 0;
    void* p = nullptr;
    auto it = d.by_owner.find(me(s));
    if (it != d.by_owner.end()) p = take(it->second, n, &got);
    if (!p) p = take(d.idle, n, &got);
    if (p) {
      d.waiting -= got;
      P.used[p] = {got, dev};
      return p;
    }
  }
  void* p = device_malloc(n);
  if (!p) return nullptr;
  std::lock_guard<std::mutex> lk(P.m);
  P.used[p] = {n, dev};
  return p;
}

void work_free(void* p, hipStream_t s) {
  if (!p) return;
  Pools& P = pools();
  std::vector<void*> out;
  {
    std::lock_guard<std::mutex> lk(P.m);
    auto it = P.used.find(p);
    if (it == P.used.end()) return;
    const Handed h = it->second;
    P.used.erase(it);
    DevicePool& d = P.dev[h.device];
    d.by_owner[me(s)].emplace(h.bytes, p);
    d.waiting += h.bytes;
    if (!d.limit) {
      size_t total = 0;
      (void)hipDeviceTotalMem(&total, h.device);
      d.limit = total / 4 + 1;
    }
    if (d.waiting > d.limit) out = d.shrink(d.limit);
  }
  give_back(out);
}

void work_stream_gone(int device, hipStream_t s) {
  Pools& P = pools();
  std::lock_guard<std::mutex> lk(P.m);
  DevicePool& d = P.dev[device];
  for (auto it = d.by_owner.begin(); it != d.by_owner.end();) {
    if (it->first.first != s) {
      ++it;
      continue;
    }
    d.idle.insert(it->second.begin(), it->second.end());
    it = d.by_owner.erase(it);
  }
}

WorkCall::~WorkCall() {
  Pools& P = pools();
  DevicePool& d = P.dev[device];
  {
    std::lock_guard<std::mutex> lk(P.m);
    auto it = d.by_owner.find(me(s));
    if (it == d.by_owner.end()) return;
  }
  if (!idle && hipStreamSynchronize(s) != hipSuccess) {
    (void)hipGetLastError();
    return;
  }
  std::lock_guard<std::mutex> lk(P.m);
  auto it = d.by_owner.find(me(s));
  if (it == d.by_owner.end()) return;
  d.idle.insert(it->second.begin(), it->second.end());
  d.by_owner.erase(it);
}

static void release_all(int device) {
  Pools& P = pools();
  std::vector<void*> out;
  {
    std::lock_guard<std::mutex> lk(P.m);
    out = P.dev[device].shrink(0);
  }
  give_back(out);
}

void* device_malloc(size_t bytes) {
  void* p = nullptr;
  if (hipMalloc(&p, bytes) == hipSuccess) return p;
  (void)hipGetLastError();
  release_all(current_device());
  if (hipMalloc(&p, bytes) == hipSuccess) return p;
  (void)hipGetLastError();
  return nullptr;
}

void work_context(int device, int change) {
  Pools& P = pools();
  bool last = false, last_of_all = false;
  {
    std::lock_guard<std::mutex> lk(P.m);
    P.dev[device].contexts += change;
    P.contexts += change;
    last = P.dev[device].contexts <= 0;
    last_of_all = P.contexts <= 0;
  }
  if (last) release_all(device);
  if (!last_of_all) return;
  Sized blocks;
  {
    std::lock_guard<std::mutex> lk(pinned().m);
    blocks.swap(pinned().blocks);
  }
  for (auto& kv : blocks) (void)hipHostFree(kv.second);
}

double* pinned_alloc(size_t bytes, size_t* got) {
  const size_t n = (bytes + 4095) / 4096 * 4096;
  PinnedPool& h = pinned();
  {
    std::lock_guard<std::mutex> lk(h.m);
    if (void* p = take(h.blocks, n, got)) return (double*)p;
  }
  void* p = nullptr;
  if (hipHostMalloc(&p, n, hipHostMallocPortable) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  *got = n;
  return (double*)p;
}

void pinned_free(double* p, size_t n) {
  if (!p) return;
  PinnedPool& h = pinned();
  {
    std::lock_guard<std::mutex> lk(h.m);
    if (n <= ((size_t)1 << 20) && h.blocks.size() < kPinnedKept) {
      h.blocks.emplace(n, p);
      return;
    }
  }
  (void)hipHostFree(p);
}

}  // namespace lq
