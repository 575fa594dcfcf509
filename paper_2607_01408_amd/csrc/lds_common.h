// LDS helpers shared by the kernels: the order of a wave's exchanges between its lanes, and
// the limit of dynamic LDS.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>

namespace spingtp {
namespace {

// Orders a wave's LDS accesses across its lanes: LDS executes a wave's instructions in
// order, and the fence keeps the compiler from moving one lane's reads over another lane's
// writes (the barrier alone orders no memory).
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Raises a kernel's dynamic LDS limit to the 160 KB of a CU, once per device.
template <auto KERNEL>
hipError_t raise_lds_limit() {
    constexpr int kMaxDevices = 64;
    static std::atomic<bool> raised[kMaxDevices];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    if (!raised[dev].load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(KERNEL),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        raised[dev].store(true, std::memory_order_release);
    }
    return hipSuccess;
}

}  // namespace
}  // namespace spingtp
