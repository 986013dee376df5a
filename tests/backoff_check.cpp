// Host check of Backoff (paper_1411_4942_amd/csrc/backoff.hpp): without memory
// the tries come 1, 2, 4, ..., 64, 64, ... steps apart; with memory again the
// next try succeeds and every step after it tries.
#include <cstdio>

#include "../paper_1411_4942_amd/csrc/backoff.hpp"

int main()
{
    pm::Backoff b;
    for (int round = 0; round < 2; ++round) {
        unsigned want = 1;
        if (b.skip()) return puts("the first step is left out"), 1;
        b.failed();
        for (int tries = 0; tries < 20; ++tries) {
            unsigned out = 0;
            while (out <= 64 && b.skip()) ++out;
            if (out != want) return printf("%u steps left out, not %u\n", out, want), 1;
            want = want < 64 ? 2 * want : 64;
            if (tries < 19)
                b.failed();
            else
                b.succeeded();  // memory again, within 64 steps
        }
        for (int i = 0; i < 100; ++i)
            if (b.skip()) return puts("a step after a success is left out"), 1;
    }
    puts("ok");
    return 0;
}
