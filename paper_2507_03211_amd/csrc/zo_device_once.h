// What has to be done once on every device before a kernel's first launch there (dynamic LDS beyond the default limit).
#pragma once
#include <hip/hip_runtime_api.h>
#include <atomic>
#include <stdint.h>

namespace zo {

// `done`: one bit per device, set after f() has succeeded on it.  Threads that meet here first may each call f().  Devices
// past the 64th call it every time.
template <class F> hipError_t once_per_device(std::atomic<uint64_t> &done, F &&f)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev < 64 ? 1ull << dev : 0;
    if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
    e = f();
    if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
    return e;
}

}  // namespace zo
