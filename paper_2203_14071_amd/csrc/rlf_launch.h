// Launch sizes.
#pragma once

#include <hip/hip_runtime.h>

#include <map>
#include <mutex>
#include <utility>

namespace rlf {

// Resident blocks of a kernel on the current device (kept per kernel and
// device; the value is a property of both, and found once).
template <class K>
int64_t resident_blocks(K kernel, int threads) {
  static std::mutex mu;
  static std::map<std::pair<const void *, int>, int64_t> cache;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  std::lock_guard<std::mutex> lock(mu);
  int64_t &n = cache[{reinterpret_cast<const void *>(kernel), dev}];
  if (!n) {
    int per_cu = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
      (void)hipGetLastError();
      return 0;
    }
    n = (int64_t)per_cu * cus;
  }
  return n;
}

}  // namespace rlf
