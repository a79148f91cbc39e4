// One kernel launch, and the LDS it may ask for.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <initializer_list>
#include <tuple>
#include <type_traits>

namespace amap_detail {

// A call runs on its stream's device: that one is current while this object lives, the caller's again afterwards.  Kernel handles and
// reserved LDS belong to a device, and are asked for on the current one.  (The null stream is the current device's.  A stream that the
// runtime cannot tell of is left to the launch.)
class StreamDevice {
  public:
    explicit StreamDevice(hipStream_t stream) {
        int here = 0;
        hipDevice_t there = 0;
        if (!stream) return;
        if (hipGetDevice(&here) != hipSuccess || hipStreamGetDevice(stream, &there) != hipSuccess) {
            (void)hipGetLastError();
            return;
        }
        if ((int)there == here) return;
        status_ = hipSetDevice((int)there);
        if (status_ == hipSuccess)
            back_to_ = here;
        else
            (void)hipGetLastError();
    }
    ~StreamDevice() {
        if (back_to_ >= 0 && hipSetDevice(back_to_) != hipSuccess) (void)hipGetLastError();
    }
    StreamDevice(const StreamDevice &) = delete;
    StreamDevice &operator=(const StreamDevice &) = delete;
    hipError_t status() const { return status_; }

  private:
    hipError_t status_ = hipSuccess;
    int back_to_ = -1;
};

// A kernel's handle on each device, asked for at its first launch there; null where there is none, and no error of the asking is left.
class KernelHandle {
  public:
    hipFunction_t on_current_device(const void *kernel) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) return none();
        if (dev < 0 || dev >= kDevices) return nullptr;
        hipFunction_t f = at_[dev].load(std::memory_order_acquire);
        if (!f) {   // (two threads may both ask, and are told the same)
            if (hipGetFuncBySymbol(&f, kernel) != hipSuccess) return none();
            at_[dev].store(f, std::memory_order_release);
        }
        return f;
    }

  private:
    static hipFunction_t none() {
        (void)hipGetLastError();
        return nullptr;
    }
    static constexpr int kDevices = 64;
    std::atomic<hipFunction_t> at_[kDevices] = {};
};

// The launch's own status, taken from the call: an error that an earlier, unrelated HIP call left on this thread is neither read
// as this launch's nor cleared.  (Asked for with hipGetLastError before and after, with the whole 4 KB argument block copied
// twice more on the way, a call from C was issued in 4.5 us against 4.2.)  Blocks of 1.5 KB where a launch has few pieces: level.
// Launched by the kernel's handle: by its address the runtime looks it up and copies the arguments once more, a stream of launches with
// 1.2 to 3.8 KB of them 4.24 us each against 3.85 (352 bytes 3.51 and 3.57).  Without a handle the address has to do.
template <auto KERNEL>
inline hipError_t launch_kernel_of(dim3 grid, dim3 block, uint32_t lds, hipStream_t stream, void **at) {
    static KernelHandle handle;
    const void *const address = reinterpret_cast<const void *>(KERNEL);
    const hipFunction_t f = handle.on_current_device(address);
    const hipError_t e = f ? hipModuleLaunchKernel(f, grid.x, grid.y, grid.z, block.x, block.y, block.z, lds, stream, at, nullptr)
                           : hipLaunchKernel(address, grid, block, at, lds, stream);
    if (e != hipSuccess) (void)hipGetLastError();   // reported here, not to the next caller who asks
    return e;
}
template <auto KERNEL, class... P, class... A>
inline hipError_t launch_kernel_as(void (*)(P...), dim3 grid, dim3 block, uint32_t lds, hipStream_t stream, const A &...args) {
    static_assert(std::is_same<std::tuple<P...>, std::tuple<A...>>::value, "the kernel's own argument types");
    void *at[] = {const_cast<void *>(static_cast<const void *>(&args))...};
    return launch_kernel_of<KERNEL>(grid, block, lds, stream, at);
}
template <auto KERNEL, class... A>
inline hipError_t launch_kernel(dim3 grid, dim3 block, uint32_t lds, hipStream_t stream, const A &...args) {
    return launch_kernel_as<KERNEL>(KERNEL, grid, block, lds, stream, args...);
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
