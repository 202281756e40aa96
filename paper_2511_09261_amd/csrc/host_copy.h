// Copies between the caller's (pageable) host memory and the device through a ring of pinned memory that a context
// owns.  Nothing here is part of the public ABI (see include/gco.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

namespace gco {

// Not for use by two threads at a time (as a context is not).  Every copy is enqueued on the stream given to it, which
// has to be the same for all copies of an object.
class HostCopies {
 public:
  ~HostCopies() { release(); }
  // Allocates the ring if there is none yet.  false: there is no pinned memory to be had; copy without.
  bool allocate();
  void release();
  // Device to host; returns when dst is filled (the stream has then run everything before the copy).
  hipError_t out(void* dst, const void* dev, size_t bytes, hipStream_t st);
  // Host to device; src is the caller's again on return, the device side follows in stream order.
  hipError_t in(void* dev, const void* src, size_t bytes, hipStream_t st);

 private:
  static constexpr int kSlots = 4;
  static constexpr size_t kSlot = size_t{2} << 20;
  hipError_t wait(int slot);           // until the copies that last used the slot are done
  hipError_t leave(hipStream_t st);    // on to the next slot
  char* base_ = nullptr;
  hipEvent_t done_[kSlots] = {};
  bool busy_[kSlots] = {};             // the event is recorded and not waited for
  int slot_ = 0;                       // in use, up to used_ bytes
  size_t used_ = 0;
};

}  // namespace gco
