// A setting that HIP keeps per device (a kernel's limit of dynamic LDS), made once on each device that the
// process runs on.  Host code without HIP calls of its own.
#pragma once
#include <atomic>
#include <cstdint>

namespace itq3s {

class DeviceOnce {
    std::atomic<uint64_t> done_{0};  // bit d: made on device d

public:
    // Calls set() unless it has succeeded on this device before; devices beyond the 64 remembered set it on
    // every call.  Two threads may both call it (the setting is the same).  False if set() failed.
    template <typename Set>
    bool operator()(int device, Set set) {
        const uint64_t bit = device >= 0 && device < 64 ? 1ull << device : 0;
        if ((done_.load(std::memory_order_acquire) & bit) != 0) return true;
        if (!set()) return false;
        done_.fetch_or(bit, std::memory_order_release);
        return true;
    }
};

}  // namespace itq3s
