// What is asked of the runtime once per GPU and kernel, from any thread (host code without HIP).
#pragma once

#include <atomic>
#include <stdint.h>

namespace hgf {

// Asks with `ask()` unless it has succeeded (returned 0) for this device before; its answer else.  Two threads may
// both ask.  Devices from 64 on are asked every time.
class OncePerDevice {
public:
    template <class F>
    int operator()(int device, F ask)
    {
        const uint64_t bit = device >= 0 && device < 64 ? uint64_t(1) << device : 0;
        if (done.load(std::memory_order_acquire) & bit) return 0;
        const int answer = ask();
        if (answer == 0) done.fetch_or(bit, std::memory_order_release);
        return answer;
    }

private:
    std::atomic<uint64_t> done{0};
};

}  // namespace hgf
