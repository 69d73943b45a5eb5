// What a launch needs to find out or set once per device (a kernel's LDS
// attribute, how many workgroups are resident), for any number of host threads.
#pragma once

#include <hip/hip_runtime.h>

#include <mutex>

namespace pfk {

template <typename T>
class PerDevice {
    static constexpr int kDevices = 64;  // of those kept; for others `fill` runs every time
    std::mutex lock;
    bool ready[kDevices] = {};
    T value[kDevices] = {};

public:
    // The current device's value; fill(device, value) -> hipError_t makes it, and
    // again at the next call if it fails.
    template <typename Fill>
    hipError_t get(T &out, Fill fill) {
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        if (dev < 0 || dev >= kDevices) return fill(dev, out);
        std::lock_guard<std::mutex> guard(lock);
        if (!ready[dev]) {
            T v{};
            e = fill(dev, v);
            if (e != hipSuccess) return e;
            value[dev] = v;
            ready[dev] = true;
        }
        out = value[dev];
        return hipSuccess;
    }
};

// Dynamic LDS above 64 KB needs an attribute of the kernel on each device.
class LargeLds {
    PerDevice<bool> set;

public:
    template <typename... Kernels>
    hipError_t allow(size_t bytes, Kernels... kernels) {
        bool done;
        return set.get(done, [&](int, bool &) {
            hipError_t e = hipSuccess;
            for (const void *k : {reinterpret_cast<const void *>(kernels)...})
                if (e == hipSuccess) e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
            return e;
        });
    }
};

}  // namespace pfk
