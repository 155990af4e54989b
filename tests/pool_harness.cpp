// The working memory of the library over a stand-in for the runtime that
// counts: run by test_pool.py on the CPU.  Exits 0, or prints the check that
// does not hold.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <set>
#include <thread>

#include "../paper_2201_09004_amd/csrc/pool.h"

namespace {
std::map<void*, size_t> dev_blocks, host_blocks;
size_t dev_used = 0, dev_total = (size_t)1 << 30;
int syncs = 0;
bool sync_ok = true;
char* next_addr = (char*)0x100000;
}  // namespace

extern "C" {
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceTotalMem(size_t* n, hipDevice_t) { return *n = dev_total, hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return ++syncs, sync_ok ? hipSuccess : hipErrorStreamCaptureUnsupported; }
hipError_t hipMalloc(void** p, size_t n) {
  if (dev_used + n > dev_total) return hipErrorOutOfMemory;
  *p = next_addr;
  next_addr += n + 4096;
  dev_blocks[*p] = n;
  dev_used += n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (!dev_blocks.count(p)) std::abort();
  dev_used -= dev_blocks[p];
  dev_blocks.erase(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = std::malloc(n);
  host_blocks[*p] = n;
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  if (!host_blocks.erase(p)) std::abort();
  std::free(p);
  return hipSuccess;
}
}

#define CHECK(x)                                      \
  do {                                                \
    if (!(x)) {                                       \
      std::printf("line %d: %s\n", __LINE__, #x);     \
      std::exit(1);                                   \
    }                                                 \
  } while (0)

int main() {
  using namespace lq;
  const hipStream_t a = (hipStream_t)0x10, b = (hipStream_t)0x20;
  const size_t MB = (size_t)1 << 20;
  work_context(0, 1);
  void* p;
  {  // inside a call a block stays with its thread and stream
    WorkCall call(0, a);
    p = work_alloc(MB, a);
    work_free(p, a);
    void* q = work_alloc(MB, b);
    CHECK(q != p);
    void* o = nullptr;
    std::thread([&] {
      o = work_alloc(MB, a);
      work_free(o, a);
    }).join();
    CHECK(o != p);
    CHECK(work_alloc(MB, a) == p);
    work_free(p, a);
    work_free(q, b);
    sync_ok = false;  // a stream that cannot be waited for keeps its blocks
  }
  CHECK(syncs == 1);
  CHECK(work_alloc(MB, a) == p);
  work_free(p, a);
  sync_ok = true;
  { WorkCall call(0, a); }
  CHECK(syncs == 2);
  {
    WorkCall call(0, b);
    call.idle = true;  // b's block, and with it the call's own two
    void *x = work_alloc(MB, b), *y = work_alloc(MB, b);
    CHECK(x == p || y == p);
    CHECK(dev_blocks.size() == 3);
    work_free(x, b);
    work_free(y, b);
  }
  { WorkCall call(0, (hipStream_t)0x30); }  // nothing left behind: nothing waited for
  CHECK(syncs == 2);
  work_stream_gone(0, a);  // the other thread's block on a
  {
    std::set<void*> s;
    for (int k = 0; k < 3; ++k) s.insert(work_alloc(MB, (hipStream_t)0x40));
    CHECK(s.size() == 3 && dev_blocks.size() == 3);
    for (void* v : s) work_free(v, (hipStream_t)0x40);
  }
  // what waits is at most a quarter of the device
  {
    void* big[6];
    for (auto& v : big) v = work_alloc(100 * MB, a);
    for (auto& v : big) work_free(v, a);
    CHECK(dev_used <= dev_total / 4 + 1);
  }
  // waiting blocks make room
  {
    void* v = work_alloc(dev_total - 2 * MB, b);
    CHECK(v && dev_blocks.size() == 1);
    CHECK(!work_alloc(4 * MB, b));
    work_free(v, b);
  }
  // pinned blocks are kept and, like the device's, given back with the last context
  size_t n1 = 0, n2 = 0;
  double* h = pinned_alloc(100, &n1);
  pinned_free(h, n1);
  CHECK(pinned_alloc(200, &n2) == h && n1 == n2);
  pinned_free(h, n2);
  p = work_alloc(MB, a);
  work_free(p, a);
  work_context(0, 1);
  work_context(0, -1);
  CHECK(host_blocks.size() == 1 && dev_used > 0);
  work_context(1, 1);
  work_context(0, -1);
  CHECK(host_blocks.size() == 1 && dev_used == 0);
  work_context(1, -1);
  CHECK(host_blocks.empty());
  return 0;
}
