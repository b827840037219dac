#include "lds_grant.h"

#include <map>
#include <mutex>
#include <utility>

namespace erem {

hipError_t lds_grant(const void* kernel, int bytes) {
  static std::mutex mu;  // contexts may be created and run on several threads
  static std::map<std::pair<int, const void*>, int> granted;
  int device = 0;
  hipError_t e = hipGetDevice(&device);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lock(mu);
  int& have = granted[{device, kernel}];
  if (bytes <= have) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) have = bytes;
  return e;
}

}  // namespace erem
