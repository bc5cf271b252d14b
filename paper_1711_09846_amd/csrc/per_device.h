// What has to happen once on every GPU of the process.
#pragma once
#include <atomic>
#include <cstdint>

namespace pbt {

// set() unless it has succeeded on `device` before; zero is success.  Several threads may come at once (set() may then run more than once, which a function
// attribute allows), a failure is reported to its caller and tried again by the next, and devices past the 64th always call.
template <class Set>
auto once_per_device(std::atomic<uint64_t>& done, int device, Set set) -> decltype(set()) {
  const uint64_t bit = device >= 0 && device < 64 ? (uint64_t)1 << device : 0;
  if (done.load(std::memory_order_acquire) & bit) return decltype(set())();
  const auto result = set();
  if (result == decltype(set())()) done.fetch_or(bit, std::memory_order_release);
  return result;
}

}  // namespace pbt
