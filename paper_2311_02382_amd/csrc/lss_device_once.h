// Something that has to be done once for every GPU of the process, such as raising a kernel's limit of dynamic LDS, which
// HIP keeps per GPU.  No HIP header: a host program can drive it.
#pragma once
#include <atomic>
#include <stdint.h>

namespace lss {

// Runs `f` (0 = done) for GPU `dev` until it has succeeded there.  Concurrent first calls may each run it: it must be idempotent.
// GPUs whose ids do not fit the mask run it every time.
class DeviceOnce {
    std::atomic<uint64_t> done{0};

public:
    template <typename F>
    auto run(int dev, F &&f) -> decltype(f())
    {
        const uint64_t bit = dev >= 0 && dev < 64 ? (uint64_t)1 << dev : 0;
        if (done.load(std::memory_order_acquire) & bit) return {};
        const auto e = f();
        if (e == decltype(e){}) done.fetch_or(bit, std::memory_order_release);
        return e;
    }
};

} // namespace lss
