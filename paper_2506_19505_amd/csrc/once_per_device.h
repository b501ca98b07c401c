// Set-up that has to be made once on every device of the process.
#pragma once

#include <atomic>
#include <stdint.h>

namespace antkv {

// A kernel's attributes (the dynamic LDS it may ask for) belong to the device that is current while they are set: a second device
// needs them too.  A set-up that failed is tried again by the next call.  Two threads may both make it, which does no harm.
class OncePerDevice {
public:
    // set() returns a status whose zero value means success
    template <typename Set>
    auto operator()(int device, Set&& set) -> decltype(set())
    {
        const uint64_t bit = device >= 0 && device < 64 ? 1ull << device : 0ull;      // (other devices: on every call)
        if (done_.load(std::memory_order_acquire) & bit) return decltype(set()){};
        const auto status = set();
        if (status == decltype(set()){}) done_.fetch_or(bit, std::memory_order_release);
        return status;
    }

private:
    std::atomic<uint64_t> done_{0};
};

}  // namespace antkv
