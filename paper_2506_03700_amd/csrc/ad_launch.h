// Launches of the library's kernels.  Not installed.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>

namespace ad {

// Launches Kernel with the arguments as its parameters; returns a hipError_t.  The kernel's handle on each device is
// looked up once and kept: <<< >>> finds it by the host function's address at every launch, 0.25 us of 2.5, which is what the parameters
// of the projections cost beyond one block of arguments (20 launches of a tiny model's layers take the host 56 us with both and with neither).
template <class T>
struct Param { using type = T; };
template <auto Kernel, class... Params>
int launch_as_is(void (*)(Params...), dim3 grid, dim3 block, size_t lds, hipStream_t s, typename Param<Params>::type... params) {
    constexpr int kMaxDevices = 64;
    static std::atomic<hipFunction_t> handle[kMaxDevices];
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return (int)e;
    if (dev < 0 || dev >= kMaxDevices) return (int)hipErrorInvalidDevice;
    hipFunction_t f = handle[dev].load(std::memory_order_acquire);
    if (!f) {
        e = hipGetFuncBySymbol(&f, (const void *)Kernel);
        if (e != hipSuccess) return (int)e;
        handle[dev].store(f, std::memory_order_release);
    }
    void *p[] = {&params...};
    e = hipModuleLaunchKernel(f, grid.x, grid.y, grid.z, block.x, block.y, block.z, (unsigned)lds, s, p, nullptr);
    if (e != hipSuccess) (void)hipGetLastError();               // (reported here, and not by the next call that asks)
    return (int)e;
}
template <auto Kernel, class... Args>
int launch(dim3 grid, dim3 block, size_t lds, hipStream_t s, const Args &...args) {
    return launch_as_is<Kernel>(Kernel, grid, block, lds, s, args...);
}

}  // namespace ad
