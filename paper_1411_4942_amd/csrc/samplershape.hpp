// The sampling kernels' launch shape, process-wide (pm_set_sampler_shape).
#pragma once

#include <atomic>

namespace pm {

class SamplerShape {
public:
    // Blocks per compute unit of a draw-ordered launch while no shape is set:
    // its blocks sweep one window of the graph together, so more of them hide
    // more latency without holding more of the graph.  1e7 + 1e7 samples took
    // 1.33, 1.21, 1.16 and 1.33 ms at 4, 5, 6 and 7 blocks on 1e6 edges, 1.66,
    // 1.60, 1.57 and 1.87 on 1e7, 2.56, 2.50, 2.51 and 3.01 on 1.2e8.  In id
    // order 4 stay best (2e6 + 2e6 on 1e7 edges: 0.65 ms at 4, 0.69 at 6, 0.75
    // at 7).  A shape that is set is taken as given for both.
    static constexpr int kBlocks = 4, kOrderBlocks = 6;

    void set(int samples_per_lane, int blocks_per_cu)
    {
        per_lane_.store(samples_per_lane);
        blocks_.store(blocks_per_cu);
        order_blocks_.store(blocks_per_cu);
    }
    int per_lane() const { return per_lane_.load(); }
    int blocks() const { return blocks_.load(); }
    int order_blocks() const { return order_blocks_.load(); }

private:
    std::atomic<int> per_lane_{1}, blocks_{kBlocks}, order_blocks_{kOrderBlocks};
};

}  // namespace pm
