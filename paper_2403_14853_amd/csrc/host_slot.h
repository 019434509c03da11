// A little pinned host memory: values that the device writes for the host to read after a synchronisation.
#pragma once
#include <atomic>
#include "isp_internal.h"

// Counters that the device writes for the host to read after a synchronisation: one page, allocated at first use and
// kept until the process ends, handed out in slots.  Any number of threads; with every slot taken (or no page) the
// caller copies instead.
class host_slot {
 public:
  static constexpr int SIZE = 128, COUNT = 32;
  ~host_slot() {
    if (index_ >= 0) busy().fetch_and(~(1u << index_));
  }
  void* get() {
    static char* const page = [] {
      void* p = nullptr;
      if (hipHostMalloc(&p, SIZE * COUNT, hipHostMallocPortable) != hipSuccess) {
        (void)hipGetLastError();
        p = nullptr;
      }
      return static_cast<char*>(p);
    }();
    if (!page) return nullptr;
    uint32_t b = busy().load();
    while (~b != 0) {
      const int k = __builtin_ctz(~b);
      if (busy().compare_exchange_weak(b, b | (1u << k))) {
        index_ = k;
        return page + k * SIZE;
      }
    }
    return nullptr;
  }

 private:
  static std::atomic<uint32_t>& busy() {
    static std::atomic<uint32_t> b{0};
    return b;
  }
  int index_ = -1;
};
