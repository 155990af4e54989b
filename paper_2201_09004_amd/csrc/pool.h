// Working memory of the calls (pool.cpp).
#pragma once

#include <hip/hip_runtime.h>

namespace lq {

// Device blocks in the order of stream s: given back, a block serves later
// requests of the thread on s.  nullptr when the device has no room.
void* work_alloc(size_t bytes, hipStream_t s);
void work_free(void* p, hipStream_t s);
// a library stream is gone, its work done: its blocks may serve any stream
void work_stream_gone(int device, hipStream_t s);
// One call of the library on stream s, made before the call's first block: at
// its end the stream is idle (waited for, unless the call says that it did), and
// the blocks that the calling thread gave back on it may serve any stream.
struct WorkCall {
  int device;
  hipStream_t s;
  bool idle = false;
  WorkCall(int dev, hipStream_t st) : device(dev), s(st) {}
  WorkCall(const WorkCall&) = delete;
  WorkCall& operator=(const WorkCall&) = delete;
  ~WorkCall();
};
// contexts of a device (+1, -1): the last one gives every waiting block back
void work_context(int device, int change);
// hipMalloc for what lives with a field; waiting blocks make room when it fails
void* device_malloc(size_t bytes);
// pinned host blocks; *got is the size to give back
double* pinned_alloc(size_t bytes, size_t* got);
void pinned_free(double* p, size_t got);

}  // namespace lq
