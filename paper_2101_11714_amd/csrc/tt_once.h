// Something done once per device of the process, from any thread: `done(dev, f)` calls f unless it has returned 0 for that
// device before, and passes its result on.  (Two threads may both be first; f has to bear that.)  A kernel's attributes
// belong to a device, so one flag for all of them would leave every device but the first without.
#pragma once

#include <atomic>
#include <stdint.h>

namespace tt {

class OncePerDevice {
    std::atomic<uint64_t> devices_{0};

public:
    template <typename F>
    int operator()(int dev, F f)
    {
        const uint64_t bit = dev >= 0 && dev < 64 ? 1ull << dev : 0ull;         // (others: every time)
        if (devices_.load(std::memory_order_acquire) & bit) return 0;
        const int e = f();
        if (e == 0) devices_.fetch_or(bit, std::memory_order_release);
        return e;
    }
};

}  // namespace tt
