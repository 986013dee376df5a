// When to try again what failed for want of memory: a failed allocation costs
// the library's cached blocks, so it is not tried at every step.
#pragma once

#include <cstdint>

namespace pm {

struct Backoff {
    static constexpr uint32_t kMost = 64;
    // Is this one to be left out?  After the n-th failure in a row
    // min(2^(n - 1), kMost) are.
    bool skip()
    {
        if (left == 0) return false;
        --left;
        return true;
    }
    void failed()
    {
        left = next;
        next = next < kMost ? 2 * next : kMost;
    }
    void succeeded() { next = 1; }

private:
    uint32_t left = 0, next = 1;
};

}  // namespace pm
