// Launches of the library's kernels.  Not installed.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>

#include "ad_internal.h"

namespace ad {

// Launches Kernel with the arguments as its parameters; returns a hipError_t.  The kernel's handle on each device is looked up once and
// kept: <<< >>> finds it by the host function's address at every launch, 0.25 us of some 3, which is what the parameters of the
// projections cost beyond one block of arguments.  The handle is that of the stream's device (c.device), whatever device the calling
// thread has current; that costs a question to the runtime, which is asked once per entry of the library and not per launch (a tiny model's
// token, 22 launches: the host takes 71.3 us with one block of arguments and <<< >>>, 70.3 with the parameters and a question per
// launch, 69.1 now).  hipGetFuncBySymbol answers for the current device: while that is another one, and for streams that have no answer, <<< >>>.
template <class T>
struct Param { using type = T; };
template <auto Kernel, class... Params>
int launch_as_is(void (*)(Params...), const LaunchCtx &c, dim3 grid, dim3 block, size_t lds, typename Param<Params>::type... params) {
    constexpr int kMaxDevices = 64;
    static std::atomic<hipFunction_t> handle[kMaxDevices];
    const hipStream_t s = (hipStream_t)c.stream;
    hipFunction_t f = nullptr;
    if (c.device >= 0 && c.device < kMaxDevices) {
        f = handle[c.device].load(std::memory_order_acquire);
        int current = -1;
        if (!f && hipGetDevice(&current) == hipSuccess && current == c.device) {
            if (hipGetFuncBySymbol(&f, (const void *)Kernel) == hipSuccess) {
                handle[c.device].store(f, std::memory_order_release);
            } else {
                f = nullptr;
                (void)hipGetLastError();
            }
        }
    }
    if (!f) {
        hipLaunchKernelGGL(Kernel, grid, block, lds, s, params...);
        return (int)hipGetLastError();
    }
    void *p[] = {&params...};
    const hipError_t e = hipModuleLaunchKernel(f, grid.x, grid.y, grid.z, block.x, block.y, block.z, (unsigned)lds, s, p, nullptr);
    if (e != hipSuccess) (void)hipGetLastError();               // (reported here, and not by the next call that asks)
    return (int)e;
}
template <auto Kernel, class... Args>
int launch(const LaunchCtx &c, dim3 grid, dim3 block, size_t lds, const Args &...args) {
    return launch_as_is<Kernel>(Kernel, c, grid, block, lds, args...);
}

}  // namespace ad
