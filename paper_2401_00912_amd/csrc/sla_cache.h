// A host-side table of per-kernel, per-device launch figures, filled on first use.  No
// HIP header is needed, so that it can be compiled and checked on the host.
#pragma once
#include <atomic>
#include <mutex>

namespace sla {

// value(key, dev), computed on first use.  Host threads may look up concurrently: an
// entry is written whole before the count that publishes it, and never changes after.
template <int N>
class LaunchTable {
 public:
  template <class F>
  int get(const void* key, int dev, F compute) {
    const int known = find(count_.load(std::memory_order_acquire), key, dev);
    if (known >= 0) return entries_[known].value;
    const int value = compute();
    std::lock_guard<std::mutex> lock(mu_);
    const int n = count_.load(std::memory_order_relaxed);
    if (n < N && find(n, key, dev) < 0) {   // a full table computes again
      entries_[n] = Entry{key, dev, value};
      count_.store(n + 1, std::memory_order_release);
    }
    return value;
  }

 private:
  struct Entry {
    const void* key;
    int dev, value;
  };
  int find(int n, const void* key, int dev) const {
    for (int i = 0; i < n; ++i)
      if (entries_[i].key == key && entries_[i].dev == dev) return i;
    return -1;
  }
  Entry entries_[N] = {};
  std::atomic<int> count_{0};
  std::mutex mu_;
};

}  // namespace sla
