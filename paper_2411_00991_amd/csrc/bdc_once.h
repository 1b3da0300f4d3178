// bdc_once.h -- work done once per device.
#pragma once

#include <stdint.h>

#include <atomic>

namespace bdc {

// A kernel's attributes belong to its device, so that a process with several has to set
// them on each.  Threads that come together may each do the work; a failure is reported
// to its caller and not kept.
class OncePerDevice {
public:
    template <class E, class F>
    E run(int device, E ok, F&& work) {
        const uint64_t bit = device >= 0 && device < 64 ? (uint64_t)1 << device : 0;
        if (done.load(std::memory_order_acquire) & bit) return ok;
        const E e = work();
        if (e == ok) done.fetch_or(bit, std::memory_order_release);
        return e;
    }

private:
    std::atomic<uint64_t> done{0};
};

}  // namespace bdc
