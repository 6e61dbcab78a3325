// Which devices a per-device setting of the process (a kernel's LDS limit) has been made on.  Plain C++.
#pragma once

#include <atomic>

namespace rs {

class DeviceOnce {
public:
    bool done(int device) const { return device >= 0 && device < 64 && (made_.load(std::memory_order_acquire) >> device & 1); }
    // (ordinals past 63 are never remembered: their setting is made again, which is harmless)
    void mark(int device) { if (device >= 0 && device < 64) made_.fetch_or(1ull << device, std::memory_order_release); }

private:
    std::atomic<unsigned long long> made_{0};
};

}  // namespace rs
