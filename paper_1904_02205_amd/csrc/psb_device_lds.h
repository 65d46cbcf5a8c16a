// More than 64 KB of dynamic LDS for a kernel: asked for once per kernel and device.
//
// The attribute belongs to the kernel as loaded on one device, so a process that uses a second GPU has to ask there as well.  A refusal
// sends the call to another kernel; the runtime's last error is cleared then, or that kernel's launch would be reported as failed.
// Host code only (no HIP types), so that it can be tested with a runtime that refuses and counts.
#pragma once
#include <stddef.h>

#include <atomic>

namespace psb {

// One per kernel, with static lifetime.  Threads may ask at the same time: the answer is the same.
class LdsGrant {
    static constexpr int kDevices = 64;        // beyond: asked for on every call
    enum : signed char { unknown = 0, granted = 1, refused = 2 };
    std::atomic<signed char> state_[kDevices] = {};

public:
    // Runtime: bool device(int*), bool request(bytes), void clear_error()
    template <class Runtime>
    bool operator()(size_t bytes, Runtime&& runtime)
    {
        if (bytes <= 65536) return true;
        int device = 0;
        if (!runtime.device(&device)) {
            runtime.clear_error();
            return false;
        }
        const bool kept = device >= 0 && device < kDevices;
        if (kept) {
            const signed char s = state_[device].load(std::memory_order_relaxed);
            if (s != unknown) return s == granted;
        }
        const bool ok = runtime.request(bytes);
        if (!ok) runtime.clear_error();
        if (kept) state_[device].store(ok ? granted : refused, std::memory_order_relaxed);
        return ok;
    }
};

}  // namespace psb
