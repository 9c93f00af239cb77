// Device memory of the library's allocations: large blocks stay with it between
// their uses.
#pragma once
#include <stddef.h>

#include <chrono>
#include <mutex>

namespace gt {

// Large device blocks between their uses.  Freeing gigabytes and allocating
// them again makes the driver clear them, 28 ms per GB once its cleared pages
// have run out (measured: 80 ms of the 83 ms of a repeated 200,000 x 1000
// build; up to seconds in single calls), so freed blocks of kPoolMin bytes or
// more are kept for the next allocation of their size.  At most kPoolMax bytes
// per device stay here, the oldest leave first, blocks idle for kPoolIdle
// leave with the next allocation or free of any size, and everything leaves
// when one fails.  A block is only kept once the device has finished all work
// (what hipFree waits for too), so it carries no stream.  Nothing here throws:
// the pool's entries are an array.
template <class Dev>
class BlockPool {
 public:
  static constexpr size_t kPoolMin = size_t(32) << 20;
  static constexpr size_t kPoolMax = size_t(4) << 30;
  static constexpr std::chrono::seconds kPoolIdle{2};

  typename Dev::Error alloc(void** p, size_t bytes) {
    std::lock_guard<std::mutex> lock(mu_);
    drop_idle();
    const int dev = Dev::current();
    for (int k = 0; k < count_; ++k)
      if (idle_[k].dev == dev && idle_[k].bytes == bytes) {
        *p = idle_[k].p;
        erase(k);
        return Dev::kOk;
      }
    typename Dev::Error e = Dev::alloc(p, bytes);
    if (e == Dev::kNoMemory && count_ > 0) {
      while (count_ > 0) drop(0);
      e = Dev::alloc(p, bytes);
    }
    return e;
  }

  // bytes: as it was allocated with
  void free(void* p, size_t bytes) {
    std::lock_guard<std::mutex> lock(mu_);
    drop_idle();
    const int dev = Dev::current();
    if (bytes < kPoolMin || bytes > kPoolMax || dev < 0 || !Dev::is_block(p, bytes, dev) ||
        !Dev::synchronize()) {
      Dev::free(p);
      return;
    }
    size_t held = bytes;
    for (int k = 0; k < count_; ++k) held += idle_[k].dev == dev ? idle_[k].bytes : 0;
    for (int k = 0; k < count_ && held > kPoolMax;) {  // oldest first
      if (idle_[k].dev == dev) {
        held -= idle_[k].bytes;
        drop(k);
      } else {
        ++k;
      }
    }
    if (count_ == kEntries) drop(0);
    idle_[count_++] = {p, dev, bytes, Dev::now()};
  }

 private:
  static constexpr int kEntries = 2 * (int)(kPoolMax / kPoolMin);  // (of all devices)
  struct Idle {
    void* p;
    int dev;
    size_t bytes;
    typename Dev::Time since;
  };
  void erase(int k) {
    for (--count_; k < count_; ++k) idle_[k] = idle_[k + 1];
  }
  void drop(int k) {
    void* p = idle_[k].p;
    erase(k);
    Dev::free(p);
  }
  void drop_idle() {
    const auto now = Dev::now();
    while (count_ > 0 && now - idle_[0].since > kPoolIdle) drop(0);
  }
  std::mutex mu_;
  Idle idle_[kEntries];  // in the order of their freeing
  int count_ = 0;
};

}  // namespace gt
