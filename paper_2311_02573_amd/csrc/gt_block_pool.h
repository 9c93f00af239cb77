// Device memory of the library's allocations: large blocks stay with it between
// their uses.
#pragma once
#include <stddef.h>
#include <unistd.h>

#include <chrono>
#include <condition_variable>
#include <mutex>
#include <thread>

namespace gt {

// Large device blocks between their uses.  Freeing gigabytes and allocating
// them again makes the driver clear them, 28 ms per GB once its cleared pages
// have run out (measured: 80 ms of the 83 ms of a repeated 200,000 x 1000
// build; up to seconds in single calls), so freed blocks of kPoolMin bytes or
// more are kept for the next allocation of their size.  At most kPoolMax bytes
// per device stay here, the oldest leave first, blocks idle for kPoolIdle
// leave by themselves (a thread that lives while blocks are idle frees them:
// a program that has closed its indexes makes no call that could), and
// everything leaves when an allocation fails.  A block is only kept once the
// device has finished all work (what hipFree waits for too), so it carries no
// stream.  Nothing here throws: the pool's entries are an array, and without a
// thread nothing is kept.
template <class Dev>
class BlockPool {
 public:
  static constexpr size_t kPoolMin = size_t(32) << 20;
  static constexpr size_t kPoolMax = size_t(4) << 30;
  static constexpr std::chrono::seconds kPoolIdle{2};

  ~BlockPool() {
    stop();
    give_back([](const Idle&) { return true; });
  }

  typename Dev::Error alloc(void** p, size_t bytes) {
    give_expired();
    const int dev = Dev::current();
    {
      std::lock_guard<std::mutex> lock(mu_);
      for (int k = 0; k < count_; ++k)
        if (idle_[k].dev == dev && idle_[k].bytes == bytes) {
          *p = idle_[k].p;
          erase(k);
          return Dev::kOk;
        }
    }
    typename Dev::Error e = Dev::alloc(p, bytes);
    if (e == Dev::kNoMemory) {
      // again after every idle block, and those that other threads are giving
      // back, have left; until then none is kept
      change_short(1);
      give_back([](const Idle&) { return true; });
      e = Dev::alloc(p, bytes);
      change_short(-1);
    }
    return e;
  }

  // bytes: as it was allocated with
  void free(void* p, size_t bytes) {
    give_expired();
    const int dev = Dev::current();
    if (bytes < kPoolMin || bytes > kPoolMax || dev < 0 || !Dev::is_block(p, bytes, dev) ||
        getpid() != pid_ || !Dev::synchronize()) {
      Dev::free(p);
      return;
    }
    const Idle x = {p, dev, bytes, Dev::now()};
    {
      std::lock_guard<std::mutex> lock(mu_);
      if (fits(x) && start()) {
        idle_[count_++] = x;
        return;
      }
    }
    give_back([&](const Idle& o) {  // the oldest
      return short_ == 0 && ((o.dev == dev && held(dev) + bytes > kPoolMax) || count_ == kEntries);
    }, &x);
  }

  // Ends the thread; nothing is kept from then on.  For the process's exit (a
  // forked child has no such thread to end).
  void stop() {
    if (getpid() != pid_) return;
    std::thread t;
    {
      std::lock_guard<std::mutex> lock(mu_);
      stopped_ = true;
      t.swap(thread_);
    }
    wake_.notify_all();
    if (t.joinable()) t.join();
  }

 private:
  static constexpr int kEntries = 2 * (int)(kPoolMax / kPoolMin);  // (of all devices)
  struct Idle {
    void* p;
    int dev;
    size_t bytes;
    typename Dev::Time since;
  };
  // (mu_ is held)
  size_t held(int dev) const {
    size_t n = 0;
    for (int k = 0; k < count_; ++k) n += idle_[k].dev == dev ? idle_[k].bytes : 0;
    return n;
  }
  bool fits(const Idle& x) const {
    return !stopped_ && short_ == 0 && count_ < kEntries && held(x.dev) + x.bytes <= kPoolMax;
  }
  void change_short(int by) {
    std::lock_guard<std::mutex> lock(mu_);
    short_ += by;
  }
  void erase(int k) {
    for (--count_; k < count_; ++k) idle_[k] = idle_[k + 1];
  }
  // Frees the blocks of which `leaves` is true, then keeps `add`.  The entries
  // are locked while the blocks are picked, not while the device frees them;
  // giving back is one thread's at a time, so that who waits for its turn finds
  // the memory of the others' blocks.
  template <class F>
  void give_back(F leaves, const Idle* add = nullptr) {
    std::lock_guard<std::mutex> turn(turn_);
    void* out[kEntries];
    int n = 0;
    {
      std::lock_guard<std::mutex> lock(mu_);
      for (int k = 0; k < count_;) {
        if (leaves(idle_[k])) {
          out[n++] = idle_[k].p;
          erase(k);
        } else {
          ++k;
        }
      }
      if (add && fits(*add) && start())
        idle_[count_++] = *add;
      else if (add)
        out[n++] = add->p;
    }
    for (int k = 0; k < n; ++k) Dev::free(out[k]);
  }
  void give_expired() {
    const auto now = Dev::now();
    auto expired = [&](const Idle& x) { return now - x.since > kPoolIdle; };
    {
      std::lock_guard<std::mutex> lock(mu_);
      if (count_ == 0 || !expired(idle_[0])) return;
    }
    give_back(expired);
  }
  // Starts the thread that frees expired blocks, where none runs (it ends when it
  // finds no block idle); the caller holds mu_ until it has added one.
  bool start() {
    if (running_) return true;
    try {
      if (thread_.joinable()) thread_.join();  // (it has ended: it let go of mu_ with running_ cleared)
      thread_ = std::thread([this] { expire(); });
    } catch (...) {
      return false;
    }
    return running_ = true;
  }
  void expire() {
    Dev::thread_starts();
    for (;;) {
      {
        std::unique_lock<std::mutex> lock(mu_);
        if (stopped_ || count_ == 0) {
          running_ = false;
          return;
        }
        const auto until = idle_[0].since + kPoolIdle;
        if (Dev::now() <= until) Dev::wait(wake_, lock, until);
      }
      give_expired();
    }
  }
  std::mutex turn_;  // taken before mu_
  std::mutex mu_;    // of the entries; no device call is made under it
  Idle idle_[kEntries];  // in the order of their freeing
  int count_ = 0;
  int short_ = 0;        // threads that found no memory
  std::condition_variable wake_;
  std::thread thread_;
  bool running_ = false, stopped_ = false;
  const pid_t pid_ = getpid();
};

}  // namespace gt
