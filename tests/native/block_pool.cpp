// The pool of freed device blocks over a made-up device of a few GiB, with a
// clock of its own.  Prints the name of each check that held.
#include "gt_block_pool.h"

#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <atomic>
#include <future>
#include <map>
#include <thread>

namespace {

constexpr size_t MB = size_t(1) << 20;

struct FakeMemory {
  using Error = int;
  using Time = std::chrono::steady_clock::time_point;
  static constexpr Error kOk = 0, kNoMemory = 2;
  static std::map<char*, size_t> blocks;
  static std::map<char*, int> home;
  static size_t limit, used;
  static int dev;
  static std::atomic<int> syncs;
  static std::atomic<double> clock;  // seconds
  static char* next;

  static std::mutex mu;
  static std::atomic<bool> busy, waiting;  // the device has work: synchronize() waits

  static Error alloc(void** p, size_t bytes) {
    std::lock_guard<std::mutex> lock(mu);
    if (used + bytes > limit) return kNoMemory;
    blocks[next] = bytes;
    home[next] = dev;
    used += bytes;
    *p = next;
    next += bytes;
    return kOk;
  }
  static void free(void* p) {
    std::lock_guard<std::mutex> lock(mu);
    const auto it = blocks.find(static_cast<char*>(p));
    if (it == blocks.end()) abort();  // freed twice, or never allocated
    used -= it->second;
    blocks.erase(it);
  }
  static int current() { return dev; }
  static bool is_block(void* p, size_t bytes, int d) {
    std::lock_guard<std::mutex> lock(mu);
    char* c = static_cast<char*>(p);
    return home.at(c) == d && blocks.at(c) >= bytes;
  }
  static bool synchronize() {
    ++syncs;
    while (busy) {
      waiting = true;
      std::this_thread::yield();
    }
    return true;
  }
  static Time now() {
    return Time(std::chrono::duration_cast<Time::duration>(std::chrono::duration<double>(clock.load())));
  }
  static void thread_starts() { ++threads; }
  static void wait(std::condition_variable& wake, std::unique_lock<std::mutex>& lock, Time) {
    wake.wait_for(lock, std::chrono::milliseconds(1));
  }
  static std::atomic<int> threads;
};
std::map<char*, size_t> FakeMemory::blocks;
std::map<char*, int> FakeMemory::home;
size_t FakeMemory::limit = 0, FakeMemory::used = 0;
int FakeMemory::dev = 0;
std::atomic<int> FakeMemory::syncs{0}, FakeMemory::threads{0};
std::mutex FakeMemory::mu;
std::atomic<bool> FakeMemory::busy{false}, FakeMemory::waiting{false};
std::atomic<double> FakeMemory::clock{0.0};
char* FakeMemory::next = reinterpret_cast<char*>(uintptr_t(1) << 40);

using Mem = FakeMemory;
using Pool = gt::BlockPool<Mem>;

void reset(size_t limit) {
  if (Mem::used != 0) abort();
  Mem::limit = limit;
  Mem::dev = 0;
  Mem::syncs = 0;
}
void* take(Pool& p, size_t bytes) {
  void* q = nullptr;
  if (p.alloc(&q, bytes) != Mem::kOk) return nullptr;
  return q;
}
void check(bool ok, const char* what) {
  if (!ok) {
    printf("FAILED %s\n", what);
    exit(1);
  }
  printf("%s\n", what);
  fflush(stdout);
}
// Waits until nothing is allocated, with no further call of the pool.
bool gone() {
  for (int k = 0; k < 20000; ++k) {
    {
      std::lock_guard<std::mutex> lock(Mem::mu);
      if (Mem::used == 0) return true;
    }
    std::this_thread::sleep_for(std::chrono::milliseconds(1));
  }
  return false;
}
void pass(double s) {
  Mem::clock = Mem::clock + s;
}

}  // namespace

int main() {
  {
    reset(1000 * MB);
    Pool p;
    void* a = take(p, 400 * MB);
    p.free(a, 400 * MB);
    check(Mem::used == 400 * MB && take(p, 400 * MB) == a, "a freed block serves the next allocation");
    p.free(a, 400 * MB);
    a = take(p, 390 * MB);
    check(Mem::used == 790 * MB, "a block serves its own size only: what is counted is what is held");
    Mem::free(a);
    void* b = take(p, 700 * MB);
    check(b && Mem::used == 700 * MB, "a large allocation without memory has the idle blocks back");
    p.free(b, 700 * MB);
    void* c = take(p, 290 * MB);
    void* d = take(p, 20 * MB);
    check(d && Mem::used == 310 * MB, "so has a small one");
    p.free(c, 290 * MB);
    p.free(d, 20 * MB);
    check(Mem::used == 290 * MB, "small blocks are freed");
    pass(3.0);
    d = take(p, MB);
    check(Mem::used == MB, "idle blocks leave with a small allocation");
    c = take(p, 100 * MB);
    p.free(c, 100 * MB);
    pass(3.0);
    p.free(d, MB);
    check(Mem::used == 0, "and with a small free");
  }
  {
    reset(20000 * MB);
    Pool p;
    void* b[6];
    for (auto& x : b) x = take(p, 1000 * MB);
    for (auto& x : b) p.free(x, 1000 * MB);
    check(Mem::used == 4000 * MB, "at most 4 GiB stay");
    void* r = take(p, 1000 * MB);
    check(r >= b[2], "the oldest left");
    Mem::dev = 1;
    void* o = take(p, 1000 * MB);
    check(Mem::used == 5000 * MB, "another device has blocks of its own");
    Mem::dev = 0;
    p.free(o, 1000 * MB);
    check(Mem::used == 4000 * MB, "a block freed with another device current is not kept");
    p.free(r, 1000 * MB);
  }
  {
    reset(2000 * MB);
    Pool p;
    void* a = take(p, 400 * MB);
    void* b = take(p, 100 * MB);
    p.free(b, 100 * MB);
    Mem::busy = true;  // one thread's free waits for the device
    std::thread t([&] { p.free(a, 400 * MB); });
    while (!Mem::waiting) std::this_thread::yield();
    auto other = std::async(std::launch::async, [&] {
      void* c = take(p, 100 * MB);
      void* d = take(p, 50 * MB);
      Mem::free(c);
      Mem::free(d);
      return c == b && d;
    });
    const bool ended = other.wait_for(std::chrono::seconds(20)) == std::future_status::ready;
    Mem::busy = false;
    t.join();
    check(ended && other.get(), "another thread allocates while one waits for the device");
    check(Mem::used == 400 * MB && take(p, 400 * MB) == a, "whose block is kept when it is done");
    Mem::free(a);
  }
  {
    // four threads on blocks of three sizes, memory for less than they keep
    reset(1200 * MB);
    Pool p;
    std::atomic<int> failed{0};
    std::thread t[4];
    for (int k = 0; k < 4; ++k)
      t[k] = std::thread([&, k] {
        for (int i = 0; i < 3000; ++i) {
          const size_t n = (60 + 70 * ((k + i) % 3)) * MB;
          void* x = take(p, n);
          if (!x) ++failed;
          if (x) p.free(x, n);
        }
      });
    for (auto& x : t) x.join();
    check(failed == 0, "no allocation fails for memory that others are giving back");
    pass(3.0);
    p.free(take(p, MB), MB);
    check(Mem::used == 0, "and all of it comes back");
  }
  {
    reset(2000 * MB);
    Pool p;
    for (int round = 0; round < 3; ++round) {
      void* a = take(p, 300 * MB);
      void* b = take(p, 100 * MB);
      p.free(a, 300 * MB);
      pass(1.0);
      p.free(b, 100 * MB);
      pass(1.5);
      pass(1.0);
      check(gone(), "idle blocks leave by themselves");
    }
    void* a = take(p, 300 * MB);
    p.free(a, 300 * MB);
    p.stop();
    pass(3.0);
    a = take(p, 300 * MB);
    p.free(a, 300 * MB);
    check(Mem::used == 0, "after the end nothing is kept");
  }
  for (int k = 0; k < 200; ++k) {
    // a thread that ends as the next block comes
    static Pool p;
    void* a = take(p, 300 * MB);
    p.free(a, 300 * MB);
    pass(2.5);
    if (k % 3) std::this_thread::sleep_for(std::chrono::microseconds(300 * (k % 7)));
    if (k == 199) {
      check(gone(), "the last block leaves too");
      p.stop();
    }
  }
  printf("done\n");
  return 0;
}
