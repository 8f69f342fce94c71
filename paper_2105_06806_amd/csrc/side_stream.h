#pragma once
#include <hip/hip_runtime.h>

#include "slot_pool.h"

namespace edx {

// A second stream for a call, with an event to order it behind the caller's;
// the destructor waits for what is still running on it and gives it back.
class SideStream {
 public:
  SideStream() = default;
  SideStream(const SideStream&) = delete;
  SideStream& operator=(const SideStream&) = delete;
  ~SideStream() {
    if (!slot_) return;
    (void)hipStreamSynchronize(slot_->st);
    SlotPool<Slot>::give(slot_);
  }
  // its work starts after what is on `st` now; false: no stream to be had, or
  // `st` is being captured (the stream would become part of the graph)
  bool fork(hipStream_t st) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cs) != hipSuccess) return failed();
    if (cs != hipStreamCaptureStatusNone) return false;
    slot_ = SlotPool<Slot>::take();
    if (!slot_) return false;
    if (hipEventRecord(slot_->ev, st) == hipSuccess &&
        hipStreamWaitEvent(slot_->st, slot_->ev, 0) == hipSuccess)
      return true;
    return failed();
  }
  hipStream_t stream() const { return slot_->st; }

 private:
  struct Slot {
    static constexpr int kKeep = 16;
    hipStream_t st = nullptr;
    hipEvent_t ev = nullptr;
    int device = 0;
    int64_t serial = 0;
    Slot* next = nullptr;
    bool make() {
      return hipStreamCreateWithFlags(&st, hipStreamNonBlocking) == hipSuccess &&
             hipEventCreateWithFlags(&ev, hipEventDisableTiming) == hipSuccess;
    }
    void drop() {
      if (ev) (void)hipEventDestroy(ev);
      if (st) (void)hipStreamDestroy(st);
    }
  };
  static bool failed() {
    (void)hipGetLastError();   // the call goes on without the stream
    return false;
  }
  Slot* slot_ = nullptr;
};

}  // namespace edx
