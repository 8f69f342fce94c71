#pragma once
#include <hip/hip_runtime.h>

#include <mutex>
#include <new>

namespace edx {

// Runtime objects (streams, events, pinned memory) that a call uses by itself
// and that take too long to make for each call.  S has make() and drop(), a
// device and a next link, and kKeep.  A call always gets one, made if none is
// free; given back, up to kKeep of them a device are kept for the next calls
// and the others dropped.  nullptr: the runtime has none to give, which is not
// an error of the call that can do without (its trace in the runtime's last
// error is cleared).
template <typename S>
class SlotPool {
 public:
  static S* take() {
    int device = -1;
    if (hipGetDevice(&device) != hipSuccess) return none();
    {
      std::lock_guard<std::mutex> lk(mutex());
      for (S** p = &free_list(); *p; p = &(*p)->next)
        if ((*p)->device == device) {
          S* s = *p;
          *p = s->next;
          return s;
        }
    }
    S* s = new (std::nothrow) S;
    if (!s) return nullptr;
    s->device = device;
    if (s->make()) return s;
    s->drop();
    delete s;
    return none();
  }
  static void give(S* s) {
    {
      std::lock_guard<std::mutex> lk(mutex());
      int kept = 0;
      for (S* q = free_list(); q; q = q->next) kept += q->device == s->device ? 1 : 0;
      if (kept < S::kKeep) {
        s->next = free_list();
        free_list() = s;
        return;
      }
    }
    s->drop();
    delete s;
  }

 private:
  static S* none() {
    (void)hipGetLastError();
    return nullptr;
  }
  static std::mutex& mutex() {
    static std::mutex* m = new std::mutex;   // never destroyed: calls may outlive statics
    return *m;
  }
  static S*& free_list() {
    static S* head = nullptr;
    return head;
  }
};

}  // namespace edx
