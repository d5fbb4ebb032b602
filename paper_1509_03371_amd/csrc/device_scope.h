#pragma once
// The current device of a stretch of host code (internal to the host code).
#include <hip/hip_runtime.h>

namespace sk {

// a device as the calling thread's current one, for as long as this lives
struct DeviceScope {
    int old = 0;
    bool moved = false;
    hipError_t status;
    explicit DeviceScope(int device) : status(hipGetDevice(&old))
    {
        if (status != hipSuccess || old == device) return;
        status = hipSetDevice(device);
        moved = status == hipSuccess;
    }
    ~DeviceScope()
    {
        if (moved) (void)hipSetDevice(old);
    }
    DeviceScope(const DeviceScope &) = delete;
    DeviceScope &operator=(const DeviceScope &) = delete;
};

}  // namespace sk
