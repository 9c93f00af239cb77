// Device memory of the library's allocations: large blocks stay with it between
// their uses.
#pragma once
#include <stddef.h>

#include <chrono>
#include <list>
#include <mutex>
#include <unordered_map>

namespace gt {

// Large device blocks between their uses.  Freeing gigabytes and allocating
// them again makes the driver clear them, 28 ms per GB once its cleared pages
// have run out (measured: 80 ms of the 83 ms of a repeated 200,000 x 1000
// build; up to seconds in single calls), so freed blocks of kPoolMin bytes or
// more are kept for the next allocation that fits them closely.  At most
// kPoolMax bytes per device stay here, the oldest leave first, blocks idle for
// kPoolIdle leave with the next allocation or free of any size, and everything
// leaves when one fails.  A block is only kept once the device has finished
// all work (what hipFree waits for too), so it carries no stream.
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
    if (bytes < kPoolMin || dev < 0) return take(p, bytes);
    auto best = idle_.end();
    for (auto it = idle_.begin(); it != idle_.end(); ++it)
      if (it->dev == dev && it->bytes >= bytes && it->bytes <= bytes + bytes / 8 &&
          (best == idle_.end() || it->bytes < best->bytes))
        best = it;
    if (best != idle_.end()) {
      *p = best->p;
      live_[best->p] = {dev, best->bytes};
      idle_.erase(best);
      return Dev::kOk;
    }
    const typename Dev::Error e = take(p, bytes);
    if (e == Dev::kOk) live_[*p] = {dev, bytes};
    return e;
  }

  void free(void* p) {
    std::lock_guard<std::mutex> lock(mu_);
    drop_idle();
    const int dev = Dev::current();
    const auto it = live_.find(p);
    if (it == live_.end()) {
      Dev::free(p);
      return;
    }
    const Live b = it->second;
    live_.erase(it);
    if (b.bytes > kPoolMax || dev != b.dev || !Dev::synchronize()) {
      Dev::free(p);
      return;
    }
    size_t held = b.bytes;
    for (const Idle& x : idle_) held += x.dev == dev ? x.bytes : 0;
    for (auto x = idle_.begin(); x != idle_.end() && held > kPoolMax;) {  // oldest first
      if (x->dev == dev) {
        held -= x->bytes;
        x = drop(x);
      } else {
        ++x;
      }
    }
    idle_.push_back({p, dev, b.bytes, Dev::now()});
  }

 private:
  struct Live {
    int dev;
    size_t bytes;
  };
  struct Idle {
    void* p;
    int dev;
    size_t bytes;
    typename Dev::Time since;
  };
  // A device allocation; without memory for it, again after everything left.
  typename Dev::Error take(void** p, size_t bytes) {
    typename Dev::Error e = Dev::alloc(p, bytes);
    if (e == Dev::kNoMemory && !idle_.empty()) {
      while (!idle_.empty()) drop(idle_.begin());
      e = Dev::alloc(p, bytes);
    }
    return e;
  }
  typename std::list<Idle>::iterator drop(typename std::list<Idle>::iterator it) {
    Dev::free(it->p);
    return idle_.erase(it);
  }
  void drop_idle() {
    const auto now = Dev::now();
    while (!idle_.empty() && now - idle_.front().since > kPoolIdle) drop(idle_.begin());
  }
  std::mutex mu_;
  std::unordered_map<void*, Live> live_;
  std::list<Idle> idle_;  // in the order of their freeing
};

}  // namespace gt
