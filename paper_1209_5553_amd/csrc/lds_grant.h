// Dynamic LDS past 64 KB: the attribute a kernel needs before its launch.
#pragma once

#include <hip/hip_runtime_api.h>

namespace erem {

// Lets `kernel` be launched with up to `bytes` of dynamic LDS on the current
// device.  The attribute belongs to a kernel on a device: the largest size granted
// so far is kept for each pair, behind a lock, so a second context on the device
// costs a look-up and a first one on another device sets it there.
hipError_t lds_grant(const void* kernel, int bytes);

}  // namespace erem
