#pragma once
#include <hip/hip_runtime.h>

#include <mutex>
#include <vector>

namespace edx {

// A second stream for a call, with an event to order it behind the caller's:
// kept for the life of the process (at most kMax of them), held by one call at
// a time; the destructor waits for what is still running on it.
class SideStream {
 public:
  SideStream() = default;
  SideStream(const SideStream&) = delete;
  SideStream& operator=(const SideStream&) = delete;
  ~SideStream() {
    if (!slot_) return;
    (void)hipStreamSynchronize(slot_->st);
    std::lock_guard<std::mutex> lk(mutex());
    slot_->used = false;
  }
  // its work starts after what is on `st` now; false: no stream to be had
  bool fork(hipStream_t st) {
    slot_ = acquire();
    return slot_ && hipEventRecord(slot_->ev, st) == hipSuccess &&
           hipStreamWaitEvent(slot_->st, slot_->ev, 0) == hipSuccess;
  }
  hipStream_t stream() const { return slot_->st; }

 private:
  struct Slot {
    hipStream_t st = nullptr;
    hipEvent_t ev = nullptr;
    int device = 0;
    bool used = false;
  };
  static constexpr int kMax = 16;
  static std::mutex& mutex() {
    static std::mutex* m = new std::mutex;   // never destroyed: calls may outlive statics
    return *m;
  }
  static Slot* acquire() {
    static std::vector<Slot*>* all = new std::vector<Slot*>;
    int device = -1;
    if (hipGetDevice(&device) != hipSuccess) return nullptr;
    std::lock_guard<std::mutex> lk(mutex());
    for (Slot* q : *all)
      if (!q->used && q->device == device) {
        q->used = true;
        return q;
      }
    if ((int)all->size() >= kMax) return nullptr;
    Slot q;
    q.device = device;
    q.used = true;
    if (hipStreamCreateWithFlags(&q.st, hipStreamNonBlocking) != hipSuccess) return nullptr;
    if (hipEventCreateWithFlags(&q.ev, hipEventDisableTiming) != hipSuccess) {
      (void)hipStreamDestroy(q.st);
      return nullptr;
    }
    all->push_back(new Slot(q));
    return all->back();
  }
  Slot* slot_ = nullptr;
};

}  // namespace edx
