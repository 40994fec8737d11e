// Host-side order between threads that call the library.
#pragma once

#include <stddef.h>
#include <stdint.h>

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

}  // namespace saap
