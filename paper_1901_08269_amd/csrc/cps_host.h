// cps_host.h -- host helpers shared by the C entry points.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace cps {

// Whether kernels on device dev may work on a caller's array where it lies: all of its bytes are in
// one allocation of that device.  Every other array (host memory, another device's, one that runs
// past its allocation) goes through a copy, which the runtime checks and which can fail, where a
// kernel would fault.
inline bool device_array(const void *p, size_t bytes, int dev)
{
    hipPointerAttribute_t a{};
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    if (hipPointerGetAttributes(&a, p) != hipSuccess ||
        (a.type == hipMemoryTypeDevice && a.device == dev &&
         hipMemGetAddressRange(&base, &size, const_cast<void *>(p)) != hipSuccess)) {
        (void)hipGetLastError();              // an answer, not the program's error
        return false;
    }
    const size_t off = (size_t)((uintptr_t)p - (uintptr_t)base);
    return base && (uintptr_t)p >= (uintptr_t)base && off <= size && bytes <= size - off;
}

}  // namespace cps
