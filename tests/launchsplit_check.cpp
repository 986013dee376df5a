// Host check of the split of large sample budgets into launches
// (paper_1411_4942_amd/csrc/launchsplit.hpp): the launches take every sample
// once, in order, and in none of them does a wave count 2^32 samples.  The
// first wave of a launch of `blocks` blocks takes the ids [base + q T, + 64)
// for q < U, base = 0, T U, 2 T U, ... below the launch's samples, T the
// launch's threads.
#include <cstdio>

#include "../paper_1411_4942_amd/csrc/launchsplit.hpp"

int main()
{
    const uint64_t ks[] = {1,           64, (1ull << 40) - 1, 1ull << 40, (1ull << 41) + 77, (1ull << 44) + 1,
                           (1ull << 50) + 12345};
    for (unsigned blocks : {1u, 32u, 128u, 256u, 1024u, 16384u})
        for (uint64_t k : ks)
            for (uint64_t U : {1u, 2u, 4u}) {
                uint64_t next = 0, launches = 0;
                bool ok = true;
                pm::for_launches(k, blocks, [&](uint64_t at, uint64_t kc) {
                    const uint64_t T = (uint64_t)blocks * pm::kBlockWaves * 64;
                    const uint64_t rounds = (kc + T * U - 1) / (T * U);
                    ok = ok && at == next && kc > 0 && rounds * U * 64 < 1ull << 32;
                    next = at + kc;
                    ++launches;
                });
                if (!ok || next != k) {
                    printf("blocks %u k %llu U %llu: %llu launches to %llu\n", blocks, (unsigned long long)k,
                           (unsigned long long)U, (unsigned long long)launches, (unsigned long long)next);
                    return 1;
                }
            }
    puts("ok");
    return 0;
}
