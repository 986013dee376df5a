// Host check of the launch shape (paper_1411_4942_amd/csrc/samplershape.hpp):
// the draw-ordered launches have a default of their own, and a shape that is
// set holds for both orders, also the values of the default.
#include <cstdio>
#include <initializer_list>

#include "../paper_1411_4942_amd/csrc/samplershape.hpp"

int main()
{
    pm::SamplerShape s;
    if (s.per_lane() != 1 || s.blocks() != 4 || s.order_blocks() != 6) return puts("defaults"), 1;
    for (int lanes : {1, 2, 4})
        for (int blocks : {4, 1, 6, 64}) {
            s.set(lanes, blocks);
            if (s.per_lane() != lanes || s.blocks() != blocks || s.order_blocks() != blocks)
                return printf("(%d, %d) is not taken as given\n", lanes, blocks), 1;
        }
    puts("ok");
    return 0;
}
