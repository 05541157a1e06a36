// The LDS limit of a kernel that asks for more than the 64 KiB of dynamic LDS a launch gets by default.  The limit belongs to the
// kernel on one GPU, so it is raised once per GPU that the kernel is launched on; an attempt that failed is made again.
#pragma once
#include <hip/hip_runtime_api.h>
#include <stdint.h>
#include <atomic>

namespace specv {

class LdsLimit {                              // one per kernel, with static storage
    std::atomic<uint64_t> raised_{0};         // bit i: raised on GPU i (beyond 63 it is set at every launch)

public:
    // on the calling thread's current GPU
    hipError_t raise(const void* kernel, int bytes)
    {
        int gpu = 0;
        hipError_t e = hipGetDevice(&gpu);
        if (e != hipSuccess) return e;
        const uint64_t bit = gpu < 64 ? 1ull << gpu : 0;
        if (raised_.load(std::memory_order_acquire) & bit) return hipSuccess;
        e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e == hipSuccess) raised_.fetch_or(bit, std::memory_order_release);
        return e;
    }
};

}  // namespace specv
