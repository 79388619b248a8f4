// What each device needs once, before a kernel's first launch there.
#pragma once
#include <atomic>
#include <cstdint>

namespace lrd {

// Remembers on which devices (of the first 64; on others it is done each time) something has been done, for any thread.  Two
// threads that come first together both do it: for things that are harmless twice.
class OncePerDevice {
    std::atomic<uint64_t> done_{0};

public:
    // what() if it has not succeeded on `device` yet; its zero means success
    template <class What>
    auto operator()(int device, What what) -> decltype(what())
    {
        const uint64_t bit = device >= 0 && device < 64 ? uint64_t(1) << device : 0;
        if (done_.load(std::memory_order_acquire) & bit) return {};
        const auto failed = what();
        if (failed == decltype(what()){}) done_.fetch_or(bit, std::memory_order_release);
        return failed;
    }
};

}  // namespace lrd
