// Row starts of K ascending keys: start[v] = entries with a key below v, for
// the rows v in [0, n].
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace pm {

// Rows [first, last]; none when first > last.
struct RowSpan {
    uint32_t first, last;
};

// The rows whose start is i: those after entry i - 1's key up to entry i's, a
// virtual entry K ending at row n; none for i > K.  Only keys [0, K) are read
// (none when there are none).
__host__ __device__ __forceinline__ RowSpan row_span(const uint32_t *__restrict__ key, int64_t K, int64_t n,
                                                     int64_t i)
{
    RowSpan r{1u, 0u};
    if (i > K) return r;
    r.first = i > 0 ? key[i - 1] + 1 : 0u;
    r.last = i < K ? key[i] : (uint32_t)n;
    return r;
}

}  // namespace pm
