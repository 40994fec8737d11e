// Host-side order between threads that call the library.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <atomic>
#include <mutex>

namespace saap {

// Held by every entry point while it enqueues: the launches of one call follow each other on their stream.  Threads that
// share a stream may share a workspace; between the launches of a call nothing else may use it.  One lock for several
// streams (a stream's address chooses it), recursive since some calls are made of others.
class InOrder {
 public:
  explicit InOrder(const void* stream) : lock_(lock_of(stream)) {}

 private:
  static std::recursive_mutex& lock_of(const void* stream) {
    constexpr size_t kLocks = 16;
    static std::recursive_mutex locks[kLocks];
    const uint64_t mixed = (uint64_t)(uintptr_t)stream * 0x9E3779B97F4A7C15ull;
    return locks[mixed >> 60];
  }
  std::lock_guard<std::recursive_mutex> lock_;
};

// Raises a limit to `need` by set(need) and remembers it: one thread at a time, so that what is remembered is what was set
// last, and never down, since another thread may be about to launch with the larger one.
template <typename Set>
bool raise_limit(std::atomic<int>& limit, int need, Set set) {
  if (limit.load(std::memory_order_acquire) >= need) return true;
  static std::mutex one;
  const std::lock_guard<std::mutex> lock(one);
  if (limit.load(std::memory_order_relaxed) >= need) return true;
  if (!set(need)) return false;
  limit.store(need, std::memory_order_release);
  return true;
}

}  // namespace saap
