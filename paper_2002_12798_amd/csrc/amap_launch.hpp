// One kernel launch, and the LDS it may ask for.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <initializer_list>
#include <tuple>
#include <type_traits>

namespace amap_detail {

// The launch's own status, taken from the call: an error that an earlier, unrelated HIP call left on this thread is neither read
// as this launch's nor cleared.  (Asked for with hipGetLastError before and after, with the whole 4 KB argument block copied
// twice more on the way, a call from C was issued in 4.5 us against 4.2.)  Blocks of 1.5 KB where a launch has few pieces: level.
template <class... P, class... A>
inline hipError_t launch_kernel(void (*kernel)(P...), dim3 grid, dim3 block, uint32_t lds, hipStream_t stream, const A &...args) {
    static_assert(std::is_same<std::tuple<P...>, std::tuple<A...>>::value, "the kernel's own argument types");
    void *at[] = {const_cast<void *>(static_cast<const void *>(&args))...};
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(kernel), grid, block, at, lds, stream);
    if (e != hipSuccess) (void)hipGetLastError();   // reported here, not to the next caller who asks
    return e;
}

// Dynamic LDS beyond 64 KB is an attribute of a kernel on one device: asked for once per device, whichever thread comes first.
// (Two threads may both ask; devices from the 65th on are asked for at every launch.)
class LdsReservation {
  public:
    hipError_t on_current_device(std::initializer_list<const void *> kernels, int bytes) {
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        const uint64_t bit = dev >= 0 && dev < 64 ? 1ull << dev : 0;
        if (e == hipSuccess && (devices_.load(std::memory_order_acquire) & bit)) return hipSuccess;
        for (const void *kernel : kernels)
            if (e == hipSuccess) e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e == hipSuccess)
            devices_.fetch_or(bit, std::memory_order_release);
        else
            (void)hipGetLastError();
        return e;
    }

  private:
    std::atomic<uint64_t> devices_{0};
};

}  // namespace amap_detail
