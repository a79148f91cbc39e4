// One kernel launch.
#pragma once

#include <hip/hip_runtime.h>

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

}  // namespace amap_detail
