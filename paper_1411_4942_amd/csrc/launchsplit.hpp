// How many samples one launch may take: every wave counts its samples' classes
// in 32 bits, so it must sample fewer than 2^32.
#pragma once

#include <algorithm>
#include <cstdint>

namespace pm {

constexpr unsigned kBlockWaves = 4;  // waves of a block of the sampling kernels

// 2^31 a wave: whole waves step through the ids, 64 (or a few times 64) a
// round, so a wave's share is over an equal split by less than a round.
constexpr uint64_t max_launch_samples(unsigned blocks) { return (uint64_t)blocks * kBlockWaves << 31; }

// f(first sample, samples) for the launches of `blocks` blocks that k samples take.
template <typename F>
inline void for_launches(uint64_t k, unsigned blocks, F f)
{
    const uint64_t most = max_launch_samples(blocks);
    for (uint64_t at = 0; at < k;) {
        const uint64_t kc = std::min(k - at, most);
        f(at, kc);
        at += kc;
    }
}

}  // namespace pm
