// Host check of the ingest's row starts (paper_1411_4942_amd/csrc/
// rowstarts.hpp): the spans of the entries 0 .. K set every row's start once
// and to the number of keys below it, and (built with AddressSanitizer) no word
// outside the max(K, 1) given is read, also for the entries after K (the rest
// of the last block).
// Usage: rowstarts_check <K> <n> <seed>
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "../paper_1411_4942_amd/csrc/rowstarts.hpp"

int main(int, char **argv)
{
    const int64_t K = strtoll(argv[1], nullptr, 10), n = strtoll(argv[2], nullptr, 10);
    std::mt19937_64 rng(strtoull(argv[3], nullptr, 10));
    std::vector<uint32_t> key((size_t)std::max<int64_t>(K, 1));
    for (auto &k : key) k = (uint32_t)(rng() % (uint64_t)n);
    std::sort(key.begin(), key.end());
    key.shrink_to_fit();
    std::vector<int64_t> start((size_t)n + 1, -1);
    const int64_t launched = (K / 1024 + 1) * 1024;  // whole blocks of 256 threads, 4 entries each
    for (int64_t i = 0; i < launched; ++i) {
        const pm::RowSpan r = pm::row_span(key.data(), K, n, i);
        if (i > K) continue;  // read like the others, but of no entry
        for (int64_t v = r.first; v <= (int64_t)r.last; ++v) {
            if (start[(size_t)v] != -1) return printf("row %lld set twice\n", (long long)v), 1;
            start[(size_t)v] = i;
        }
    }
    for (int64_t v = 0; v <= n; ++v) {
        const int64_t below = std::lower_bound(key.begin(), key.begin() + K, (uint32_t)v) - key.begin();
        if (start[(size_t)v] != below) return printf("start[%lld] = %lld, not %lld\n", (long long)v,
                                                     (long long)start[(size_t)v], (long long)below), 1;
    }
    puts("ok");
    return 0;
}
