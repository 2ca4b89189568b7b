// Host settings that hold for one device only (a kernel's LDS limit), made once on each.
#pragma once

#include <atomic>
#include <cstdint>

namespace moe {

// run(device, f) calls f the first time it sees `device`.  Threads that meet there may each call it (f is idempotent), and
// none returns before f has been done on its device; devices past the 64th set it every time.
class OncePerDevice {
    std::atomic<uint64_t> done_{0};

public:
    template <typename F>
    void run(int device, F&& f) {
        const uint64_t bit = device >= 0 && device < 64 ? 1ull << device : 0;
        if (done_.load(std::memory_order_acquire) & bit) return;
        f();
        done_.fetch_or(bit, std::memory_order_release);
    }
};

}  // namespace moe
