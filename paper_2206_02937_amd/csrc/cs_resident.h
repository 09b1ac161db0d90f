// cs_resident.h -- numbers that depend on the device a launch goes to (how
// many workgroups of a kernel fit it at once), looked up once per device.
// Host code, without HIP.
#pragma once

#include <atomic>
#include <cstdint>

namespace cs {

// Two counts, both positive; {0, 0}: not known.
struct Resident {
    int64_t per_cu, cus;
};

// Contexts of several devices and threads share one of these per kernel: an
// entry per device, written whole (threads that look a device up at the same
// time find and store the same counts).
class ResidentCache {
   public:
    // The counts of device `dev`, from look_up() unless they are known; what
    // look_up does not find is not kept.
    template <typename F>
    Resident get(int dev, const F& look_up) {
        const bool kept = dev >= 0 && dev < kDevices;
        if (kept) {
            const uint64_t w = known_[dev].load(std::memory_order_relaxed);
            if (w) return {(int64_t)(w >> 32), (int64_t)(w & 0xFFFFFFFFu)};
        }
        const Resident r = look_up();
        if (r.per_cu <= 0 || r.cus <= 0) return {0, 0};
        if (kept) known_[dev].store((uint64_t)r.per_cu << 32 | (uint64_t)r.cus, std::memory_order_relaxed);
        return r;
    }

   private:
    static constexpr int kDevices = 64;
    std::atomic<uint64_t> known_[kDevices] = {};
};

}  // namespace cs
