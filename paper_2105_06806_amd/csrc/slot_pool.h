#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>
#include <new>

namespace edx {

// Runtime objects (streams, events, pinned memory) that a call uses by itself
// and that take too long to make for each call.  S has make() and drop(), a
// device, a serial number and a next link, and kKeep.  A call always gets one,
// made if none is free; given back, up to kKeep of them a device are kept for the
// next calls and the others dropped.  The one made first goes out first: the
// runtime spreads streams over a few hardware queues in the order in which they
// are made, and later ones share the queue of the caller's stream (Green's
// function with its branches at once, Ns=12 FP64: 4.1-4.6 ms on the stream made
// first, 6.1 ms on the eighth).
// nullptr: the runtime has none to give, which is not an error of the call that
// can do without (its trace in the runtime's last error is cleared).
template <typename S>
class SlotPool {
 public:
  static S* take() {
    int device = -1;
    if (hipGetDevice(&device) != hipSuccess) return none();
    int64_t serial = 0;
    {
      std::lock_guard<std::mutex> lk(mutex());
      for (S** p = &free_list(); *p; p = &(*p)->next)
        if ((*p)->device == device) {
          S* s = *p;
          *p = s->next;
          return s;
        }
      static int64_t made = 0;
      serial = made++;
    }
    S* s = new (std::nothrow) S;
    if (!s) return nullptr;
    s->device = device;
    s->serial = serial;
    if (s->make()) return s;
    s->drop();
    delete s;
    return none();
  }
  static void give(S* s) {
    S* extra = nullptr;
    {
      std::lock_guard<std::mutex> lk(mutex());
      S** at = &free_list();   // the list runs by serial number
      while (*at && (*at)->serial < s->serial) at = &(*at)->next;
      s->next = *at;
      *at = s;
      int kept = 0;
      for (S** p = &free_list(); *p; p = &(*p)->next)
        if ((*p)->device == s->device && ++kept > S::kKeep) {
          extra = *p;
          *p = extra->next;
          break;
        }
    }
    if (!extra) return;
    extra->drop();
    delete extra;
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
