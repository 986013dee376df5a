// Stable LSD radix sort of (uint32 key, uint32 value) elements, digits of up
// to 11 bits.
//
// What bounds a pass is memory traffic and, nearly as much, the instructions
// that rank an element among equal digits, so the passes are as few as
// 2048-way digits allow (two for keys of 12 to 22 bits) and an element's rank
// costs four vector instructions per digit bit.  One pass:
//   1. histogram: a block counts the digits of a chunk of up to kRadixChunk
//      tiles (8192 elements each), storing before each tile what it counted so
//      far (16 bits suffice) and at the end the chunk's counts;
//   2. column scan: each digit's chunk counts scanned over the chunks, in
//      place, and the digit's total;
//   3. scatter, a tile per block: the elements are ranked per wave in input
//      order with ballots and 16-bit per-wave digit counters, the counters
//      become positions, and the tile leaves through one LDS buffer grouped by
//      digit, first the keys, then the values (4 bytes per element at a time:
//      72 KiB in all, so two blocks of eight waves share a CU).
// Neighbouring tiles run at the same time on one XCD, so that the 16-byte
// runs they write side by side meet in its L2 (1.13 times the bytes reach
// memory; a block that went through four tiles in turn wrote 1.95 times).
// Against three passes of 8-bit digits ranked with seven instructions a bit:
// pm_count_motifs 1003 -> 676 us at 2e6 slots, where launches count (three per
// pass instead of five), and 12.50 -> 11.62 ms at 2.4e8 slots; a pass over
// 1.3e8 pairs takes 0.17 + 0.02 + 0.5..0.7 ms, of which 0.28 are the ranking's
// instructions and 0.4 its 2.1 GB at the copy rate.
// Elements come from a Src functor and leave through a Dst functor, so a sort
// can read its first pass from, and write its last pass to, whatever layout
// its neighbours use:
//   Src: uint32_t key(int64_t i); void load(int64_t i, uint32_t &k, uint32_t &v);
//        void check(const uint32_t (&k)[kRadixItems]): the scatter's keys of one
//        lane once loaded (0 past the end)
//   Dst: static constexpr bool kKeys (are keys written?); void key(uint32_t
//        dst, uint32_t k); void val(uint32_t dst, uint32_t v)
#pragma once

#include <algorithm>
#include <string>

#include "profile.hpp"
#include "scan.hpp"

namespace pm {

// The kernels have internal linkage: each translation unit that sorts keeps
// its own copy.

constexpr int kRadixBits = 11;      // widest digit
constexpr int kRadixThreads = 512;  // threads per histogram / scatter block
constexpr int kRadixWaves = kRadixThreads / kWave;
constexpr int kRadixItems = 16;
constexpr int kRadixTile = kRadixThreads * kRadixItems;  // 8192 elements
constexpr int kRadixWaveSpan = kWave * kRadixItems;      // a wave's contiguous share of a tile
// tiles per histogram block: more than one only when there are blocks enough
// to fill the chip (1024 are resident)
constexpr int kRadixChunk = 8;
constexpr int64_t kRadixFill = 1024;
static_assert((kRadixChunk - 1) * kRadixTile <= 65535, "counts before a chunk's last tile fit 16 bits");

inline int64_t radix_tiles(int64_t N) { return std::max<int64_t>(1, (N + kRadixTile - 1) / kRadixTile); }
inline int radix_chunk(int64_t tiles)
{
    return (int)std::max<int64_t>(1, std::min<int64_t>(kRadixChunk, tiles / kRadixFill));
}

// A read of data that the pass reads once: past the caches, which the runs
// being written need.
template <typename T>
__device__ __forceinline__ T read_once(const T *p)
{
    return __builtin_nontemporal_load(p);
}

// Workgroups are dealt round-robin to the 8 XCDs, each with its own L2.  Give
// every XCD a contiguous run of blocks so that the digit runs that
// neighbouring blocks write next to each other meet in the same L2 and leave
// it as whole lines.
constexpr int kXcds = 8;

__device__ __forceinline__ int64_t xcd_tile(int64_t b, int64_t nb)
{
    const int64_t x = b % kXcds, i = b / kXcds;
    const int64_t per = nb / kXcds, extra = nb % kXcds;
    return x * per + (x < extra ? x : extra) + i;
}

// Digit counts of one chunk: before[tile][d] = elements with digit d in the
// chunk's earlier tiles, counts[chunk][d] = in the chunk.  kHistCopies LDS
// histograms (lane & 3 picks one) cut the atomic conflicts of skewed digits.
constexpr int kHistCopies = 4;

template <int BITS, typename Src>
static __global__ __launch_bounds__(kRadixThreads) void radix_histogram(Src src, int64_t N, int64_t tiles, int chunk,
                                                                        int shift, uint32_t mask,
                                                                        uint16_t *__restrict__ before,
                                                                        uint32_t *__restrict__ counts)
{
    constexpr int BINS = 1 << BITS;
    __shared__ uint32_t hist[kHistCopies][BINS];
    const int t = threadIdx.x;
    for (int j = t; j < kHistCopies * BINS; j += kRadixThreads) (&hist[0][0])[j] = 0;
    uint32_t *const mine = hist[lane_id() & (kHistCopies - 1)];
    const auto sum_of = [&](int d) {
        uint32_t c = 0;
#pragma unroll
        for (int i = 0; i < kHistCopies; ++i) c += hist[i][d];
        return c;
    };
    const int64_t first = (int64_t)blockIdx.x * chunk;
    const int64_t end = first + chunk < tiles ? first + chunk : tiles;
    __syncthreads();
    for (int64_t tile = first; tile < end; ++tile) {  // block-uniform
        const int64_t tile0 = tile * kRadixTile;
        const bool full = tile0 + kRadixTile <= N;
        uint32_t k[kRadixItems];
        if (full) {
#pragma unroll
            for (int i = 0; i < kRadixItems; ++i) k[i] = src.key(tile0 + i * kRadixThreads + t);
        }
        for (int d = t; d < BINS; d += kRadixThreads) before[tile * BINS + d] = (uint16_t)sum_of(d);
        __syncthreads();
        if (full) {
#pragma unroll
            for (int i = 0; i < kRadixItems; ++i) atomicAdd(&mine[(k[i] >> shift) & mask], 1u);
        } else {
            for (int64_t i = tile0 + t; i < N; i += kRadixThreads) atomicAdd(&mine[(src.key(i) >> shift) & mask], 1u);
        }
        // at the loop's end: at its head the compiler was seen to leave out the
        // wait for the atomics of the iteration before
        __syncthreads();
    }
    for (int d = t; d < BINS; d += kRadixThreads) counts[(int64_t)blockIdx.x * BINS + d] = sum_of(d);
}

// counts[c][d] -> elements with digit d in chunks before c; totals[d].  A
// block takes kColDigits digits, its 1024 threads that many digits in
// 1024 / kColDigits ranges of rows.
constexpr int kColDigits = 16;
constexpr int kColParts = 1024 / kColDigits;

template <int BITS>
static __global__ __launch_bounds__(1024) void radix_colscan(uint32_t *__restrict__ counts, int64_t rows,
                                                             uint32_t *__restrict__ totals)
{
    constexpr int BINS = 1 << BITS;
    constexpr int kBatch = 8;  // loads in flight per thread
    __shared__ uint32_t s_part[kColParts][kColDigits];
    const int c = threadIdx.x % kColDigits, p = threadIdx.x / kColDigits;
    uint32_t *col = counts + (int64_t)blockIdx.x * kColDigits + c;
    const int64_t per = (rows + kColParts - 1) / kColParts;
    const int64_t r0 = p * per < rows ? p * per : rows, r1 = r0 + per < rows ? r0 + per : rows;
    uint32_t acc = 0;
    for (int64_t r = r0; r < r1; r += kBatch) {
        uint32_t v[kBatch];
#pragma unroll
        for (int i = 0; i < kBatch; ++i) v[i] = r + i < r1 ? col[(r + i) * BINS] : 0u;
#pragma unroll
        for (int i = 0; i < kBatch; ++i) acc += v[i];
    }
    s_part[p][c] = acc;
    __syncthreads();
    if (threadIdx.x < kColDigits) {
        uint32_t run = 0;
        for (int q = 0; q < kColParts; ++q) {
            const uint32_t x = s_part[q][threadIdx.x];
            s_part[q][threadIdx.x] = run;
            run += x;
        }
        totals[blockIdx.x * kColDigits + threadIdx.x] = run;
    }
    __syncthreads();
    uint32_t run = s_part[p][c];
    for (int64_t r = r0; r < r1; r += kBatch) {
        uint32_t v[kBatch];
#pragma unroll
        for (int i = 0; i < kBatch; ++i) v[i] = r + i < r1 ? col[(r + i) * BINS] : 0u;
#pragma unroll
        for (int i = 0; i < kBatch; ++i)
            if (r + i < r1) {
                col[(r + i) * BINS] = run;
                run += v[i];
            }
    }
}

// Exclusive prefix of v over the block's threads; s_w holds one word per wave.
__device__ __forceinline__ uint32_t radix_block_excl(uint32_t v, uint32_t *s_w)
{
    const int lane = lane_id(), w = threadIdx.x / kWave;
    uint32_t incl = v;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t o = __shfl_up(incl, d, kWave);
        if (lane >= d) incl += o;
    }
    if (lane == kWave - 1) s_w[w] = incl;
    __syncthreads();
    uint32_t pre = 0;
#pragma unroll
    for (int ww = 0; ww < kRadixWaves; ++ww)
        if (ww < w) pre += s_w[ww];
    return pre + incl - v;
}

// a & ~(bal ^ bit), one instruction (left to itself the compiler takes two)
__device__ __forceinline__ uint32_t lanes_alike(uint32_t a, uint32_t bal, uint32_t bit)
{
    return (uint32_t)__builtin_amdgcn_bitop3_b32((int)a, (int)bal, (int)bit, 0x90);
}

template <int BITS, typename Src, typename Dst>
static __global__ __launch_bounds__(kRadixThreads, 4) void radix_scatter(Src src, Dst dst, int64_t N, int chunk,
                                                                         int shift, uint32_t mask,
                                                                         const uint16_t *__restrict__ before,
                                                                         const uint32_t *__restrict__ counts,
                                                                         const uint32_t *__restrict__ totals)
{
    constexpr int BINS = 1 << BITS;
    // digits per thread in the per-digit phases: 4 consecutive ones, the first
    // BINS / 4 threads (their 16-bit counters are one 8-byte word per wave)
    constexpr int kPer = 4;
    constexpr int kDigitThreads = BINS / kPer;
    static_assert(kDigitThreads <= kRadixThreads, "every digit has its thread");
    __shared__ uint2 s_cnt2[kRadixWaves][BINS / 4];  // per-wave digit counts, then positions (16 bits each)
    __shared__ uint32_t s_buf[kRadixTile];
    __shared__ uint32_t s_delta[BINS];  // output position less position in the tile, per digit
    __shared__ uint32_t s_w[2][kRadixWaves];

    const int t = threadIdx.x, lane = lane_id();
    const int w = __builtin_amdgcn_readfirstlane(t / kWave);
    const int64_t tile = xcd_tile(blockIdx.x, gridDim.x);
    typedef uint16_t __attribute__((may_alias)) u16;  // single digits of the words above
    u16 *const cnt = reinterpret_cast<u16 *>(s_cnt2[w]);

    const int64_t tile0 = tile * kRadixTile;
    const int tile_n = (int)(N - tile0 < kRadixTile ? N - tile0 : kRadixTile);
    // element i of this lane: position w0 + i * kWave of the tile
    const int w0 = w * kRadixWaveSpan + lane;
    uint32_t key[kRadixItems], val[kRadixItems];
    uint32_t pos[kRadixItems / 2] = {0};  // ranks, then positions in the tile, 16 bits each
    if (tile_n == kRadixTile) {
#pragma unroll
        for (int i = 0; i < kRadixItems; ++i) src.load(tile0 + w0 + i * kWave, key[i], val[i]);
    } else {
#pragma unroll
        for (int i = 0; i < kRadixItems; ++i) {
            key[i] = val[i] = 0u;
            if (w0 + i * kWave < tile_n) src.load(tile0 + w0 + i * kWave, key[i], val[i]);
        }
    }
#pragma unroll
    for (int j = 0; j < BINS / 4; j += kWave) s_cnt2[w][j + lane] = make_uint2(0u, 0u);
    // the digits' first output positions for this tile
    uint32_t goff[kPer] = {0};
    {
        uint32_t x[kPer] = {0}, sum = 0;
        if (t < kDigitThreads) {
            const uint4 tt = reinterpret_cast<const uint4 *>(totals)[t];
            const uint4 cc = reinterpret_cast<const uint4 *>(counts + tile / chunk * BINS)[t];
            const uint2 bb = reinterpret_cast<const uint2 *>(before + tile * BINS)[t];
            x[0] = tt.x, x[1] = tt.y, x[2] = tt.z, x[3] = tt.w;
            goff[0] = cc.x + (bb.x & 0xFFFFu);
            goff[1] = cc.y + (bb.x >> 16);
            goff[2] = cc.z + (bb.y & 0xFFFFu);
            goff[3] = cc.w + (bb.y >> 16);
#pragma unroll
            for (int j = 0; j < kPer; ++j) sum += x[j];
        }
        uint32_t run = radix_block_excl(sum, s_w[0]);
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            goff[j] += run;
            run += x[j];
        }
    }
    src.check(key);
    // Stable rank inside the wave's elements: the lanes holding the same
    // digit are found with a ballot per bit (a lane keeps the ballot's lanes
    // or the others: ~(ballot ^ its own bit spread over the word)), the
    // lowest of them moves the wave's counter on.  One wave's LDS operations
    // are in order, so no barrier until the counts meet.
#pragma unroll
    for (int i = 0; i < kRadixItems; ++i) {
        const bool ok = w0 + i * kWave < tile_n;
        // an opaque copy: the ballots of later elements would otherwise be
        // computed ahead and held in registers
        uint32_t k = key[i];
        asm volatile("" : "+v"(k));
        const uint32_t dig = (k >> shift) & mask;
        const uint64_t act = __ballot(ok);
        uint32_t plo = (uint32_t)act, phi = (uint32_t)(act >> 32);
#pragma unroll
        for (int b = 0; b < BITS; ++b) {
            int32_t bit = ((int32_t)(dig << (31 - b))) >> 31;  // 0 or -1
            asm("" : "+v"(bit));  // one field extract, then compared as it is
            const uint64_t bal = __ballot(bit != 0);
            plo = lanes_alike(plo, (uint32_t)bal, (uint32_t)bit);
            phi = lanes_alike(phi, (uint32_t)(bal >> 32), (uint32_t)bit);
        }
        const uint32_t below = __builtin_amdgcn_mbcnt_hi(phi, __builtin_amdgcn_mbcnt_lo(plo, 0u));
        const uint32_t base = cnt[dig];
        if (ok && below == 0) cnt[dig] = (u16)(base + (uint32_t)(__popc(plo) + __popc(phi)));
        pos[i / 2] |= (base + below) << (16 * (i & 1));
    }
    __syncthreads();
    // per digit: the waves' counts become positions in the tile
    uint2 run[kRadixWaves], tot = make_uint2(0u, 0u);
    if (t < kDigitThreads) {
#pragma unroll
        for (int ww = 0; ww < kRadixWaves; ++ww) {
            const uint2 x = s_cnt2[ww][t];
            run[ww] = tot;
            tot.x += x.x;  // two 16-bit sums at once: a tile's sums stay below 2^16
            tot.y += x.y;
        }
    }
    const uint32_t d0 = tot.x & 0xFFFFu, d1 = tot.x >> 16, d2 = tot.y & 0xFFFFu, d3 = tot.y >> 16;
    const uint32_t st = radix_block_excl(d0 + d1 + d2 + d3, s_w[1]);
    if (t < kDigitThreads) {
        const uint32_t st1 = st + d0, st2 = st1 + d1, st3 = st2 + d2;
#pragma unroll
        for (int ww = 0; ww < kRadixWaves; ++ww)
            s_cnt2[ww][t] = make_uint2(run[ww].x + (st | (st1 << 16)), run[ww].y + (st2 | (st3 << 16)));
        reinterpret_cast<uint4 *>(s_delta)[t] = make_uint4(goff[0] - st, goff[1] - st1, goff[2] - st2, goff[3] - st3);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kRadixItems; ++i) {
        const uint32_t dig = (key[i] >> shift) & mask;
        pos[i / 2] += (uint32_t)cnt[dig] << (16 * (i & 1));
        if (w0 + i * kWave < tile_n) s_buf[(pos[i / 2] >> (16 * (i & 1))) & 0xFFFFu] = key[i];
    }
    __syncthreads();
    uint32_t out[kRadixItems];
#pragma unroll
    for (int i = 0; i < kRadixItems; ++i) {
        const int p = i * kRadixThreads + t;
        const uint32_t k = s_buf[p];  // past tile_n: whatever the buffer holds, not used
        out[i] = s_delta[(k >> shift) & mask] + (uint32_t)p;
        if (Dst::kKeys && p < tile_n) dst.key(out[i], k);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kRadixItems; ++i)
        if (w0 + i * kWave < tile_n) s_buf[(pos[i / 2] >> (16 * (i & 1))) & 0xFFFFu] = val[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kRadixItems; ++i) {
        const int p = i * kRadixThreads + t;
        if (p < tile_n) dst.val(out[i], s_buf[p]);
    }
}

// Device scratch of a pass over N or fewer elements: the digit totals, the
// chunks' counts, the tiles' counts before them.
inline size_t radix_scratch_bytes(int64_t N)
{
    const int64_t tiles = radix_tiles(N);
    const int64_t chunks = std::min<int64_t>(tiles, std::max<int64_t>(2 * kRadixFill, tiles / kRadixChunk + 1));
    return ((size_t)(1 + chunks) * sizeof(uint32_t) + (size_t)tiles * sizeof(uint16_t)) << kRadixBits;
}

// The passes over keys of `bits` bits: as few as 11-bit digits allow, of
// nearly equal width.
struct RadixDigits {
    int passes, width;
    explicit RadixDigits(int bits)
        : passes(std::max(1, (bits + kRadixBits - 1) / kRadixBits)), width((std::max(bits, 1) + passes - 1) / passes)
    {
    }
};

// Names of a sort's timed scopes.
struct RadixNames {
    std::string hist, scan, scat;
    explicit RadixNames(const char *name)
        : hist(std::string(name) + ".histogram"), scan(std::string(name) + ".count_scan"),
          scat(std::string(name) + ".scatter")
    {
    }
};

// One pass by the digit (key >> shift) of `width` bits; 0 < N < 2^32.  Digits
// of up to 8 bits have kernels of their own (fewer ballots, less LDS).
template <int BITS, typename Src, typename Dst>
pm_status radix_pass_bits(const RadixNames &nm, const Src &src, const Dst &dst, int64_t N, int shift, int width,
                          void *scratch, hipStream_t s)
{
    const uint32_t mask = (1u << width) - 1u;
    const int64_t tiles = radix_tiles(N);
    const int chunk = radix_chunk(tiles);
    const int64_t chunks = (tiles + chunk - 1) / chunk;
    uint32_t *totals = (uint32_t *)scratch, *counts = totals + (1 << kRadixBits);
    uint16_t *before = (uint16_t *)(counts + (chunks << BITS));
    {
        ProfScope prof(nm.hist.c_str(), s);
        hipLaunchKernelGGL((radix_histogram<BITS, Src>), dim3((unsigned)chunks), dim3(kRadixThreads), 0, s, src, N,
                           tiles, chunk, shift, mask, before, counts);
        PM_HIP(hipGetLastError());
    }
    {
        ProfScope prof(nm.scan.c_str(), s);
        hipLaunchKernelGGL(radix_colscan<BITS>, dim3((1 << BITS) / kColDigits), dim3(1024), 0, s, counts, chunks,
                           totals);
        PM_HIP(hipGetLastError());
    }
    ProfScope prof(nm.scat.c_str(), s);
    hipLaunchKernelGGL((radix_scatter<BITS, Src, Dst>), dim3((unsigned)tiles), dim3(kRadixThreads), 0, s, src, dst, N,
                       chunk, shift, mask, before, counts, totals);
    PM_HIP(hipGetLastError());
    return PM_OK;
}

template <typename Src, typename Dst>
pm_status radix_pass(const RadixNames &nm, const Src &src, const Dst &dst, int64_t N, int shift, int width,
                     void *scratch, hipStream_t s)
{
    return width <= 8 ? radix_pass_bits<8>(nm, src, dst, N, shift, width, scratch, s)
                      : radix_pass_bits<kRadixBits>(nm, src, dst, N, shift, width, scratch, s);
}

// Elements in a key array with the position as value, or in two arrays.
struct RadixKeys {
    const uint32_t *k;
    __device__ __forceinline__ uint32_t key(int64_t i) const { return k[i]; }
    __device__ __forceinline__ void load(int64_t i, uint32_t &kk, uint32_t &vv) const
    {
        kk = read_once(k + i);
        vv = (uint32_t)i;
    }
    __device__ __forceinline__ void check(const uint32_t (&)[kRadixItems]) const {}
};
struct RadixPairs {
    const uint32_t *k, *v;
    __device__ __forceinline__ uint32_t key(int64_t i) const { return k[i]; }
    __device__ __forceinline__ void load(int64_t i, uint32_t &kk, uint32_t &vv) const
    {
        kk = read_once(k + i);
        vv = read_once(v + i);
    }
    __device__ __forceinline__ void check(const uint32_t (&)[kRadixItems]) const {}
};
struct RadixToPairs {
    static constexpr bool kKeys = true;
    uint32_t *k, *v;
    __device__ __forceinline__ void key(uint32_t d, uint32_t x) const { k[d] = x; }
    __device__ __forceinline__ void val(uint32_t d, uint32_t x) const { v[d] = x; }
};
// The same with only the key bits that later passes sort by, as 16 bits
// (keys that the caller does not want): a quarter less to write and to read
// back, and half as much for the next histogram.
struct RadixNarrow {
    const uint16_t *k;
    const uint32_t *v;
    __device__ __forceinline__ uint32_t key(int64_t i) const { return k[i]; }
    __device__ __forceinline__ void load(int64_t i, uint32_t &kk, uint32_t &vv) const
    {
        kk = read_once(k + i);
        vv = read_once(v + i);
    }
    __device__ __forceinline__ void check(const uint32_t (&)[kRadixItems]) const {}
};
struct RadixToNarrow {
    static constexpr bool kKeys = true;
    uint16_t *k;
    uint32_t *v;
    int shift;
    __device__ __forceinline__ void key(uint32_t d, uint32_t x) const { k[d] = (uint16_t)(x >> shift); }
    __device__ __forceinline__ void val(uint32_t d, uint32_t x) const { v[d] = x; }
};
struct RadixToVals {
    static constexpr bool kKeys = false;
    uint32_t *v;
    __device__ __forceinline__ void key(uint32_t, uint32_t) const {}
    __device__ __forceinline__ void val(uint32_t d, uint32_t x) const { v[d] = x; }
};

// Sort the N < 2^32 elements of `first` stably by the low `bits` bits of their
// keys.  Passes write the buffer pairs (k0, v0) and (k1, v1) in turn; the
// first one may overwrite only what `first` does not read.  *out_k / *out_v
// point at the result (*out_k is null with keys_wanted false: the last pass
// then writes no keys).
template <typename Src>
pm_status radix_sort(const char *name, const Src &first, uint32_t *k0, uint32_t *v0, uint32_t *k1, uint32_t *v1,
                     int64_t N, int bits, void *scratch, hipStream_t s, uint32_t **out_k, uint32_t **out_v,
                     bool keys_wanted = true)
{
    *out_k = keys_wanted ? k0 : nullptr;
    *out_v = v0;
    if (N <= 0) return PM_OK;
    const RadixNames nm(name);
    const RadixDigits dg(bits);
    if (dg.passes == 2 && !keys_wanted) {  // bits - width <= 11 are left for the second pass
        uint16_t *kn = reinterpret_cast<uint16_t *>(k0);
        PM_TRY(radix_pass(nm, first, RadixToNarrow{kn, v0, dg.width}, N, 0, dg.width, scratch, s));
        *out_v = v1;
        return radix_pass(nm, RadixNarrow{kn, v0}, RadixToVals{v1}, N, 0, bits - dg.width, scratch, s);
    }
    const uint32_t *ki = nullptr, *vi = nullptr;
    uint32_t *ko = k0, *vo = v0;
    for (int p = 0; p < dg.passes; ++p) {
        const bool keys = p + 1 < dg.passes || keys_wanted;
        const int shift = p * dg.width, width = std::max(1, std::min(dg.width, bits - shift));
        if (p == 0 && keys)
            PM_TRY(radix_pass(nm, first, RadixToPairs{ko, vo}, N, shift, width, scratch, s));
        else if (p == 0)
            PM_TRY(radix_pass(nm, first, RadixToVals{vo}, N, shift, width, scratch, s));
        else if (keys)
            PM_TRY(radix_pass(nm, RadixPairs{ki, vi}, RadixToPairs{ko, vo}, N, shift, width, scratch, s));
        else
            PM_TRY(radix_pass(nm, RadixPairs{ki, vi}, RadixToVals{vo}, N, shift, width, scratch, s));
        *out_k = keys ? ko : nullptr;
        *out_v = vo;
        ki = ko;
        vi = vo;
        ko = (ko == k0) ? k1 : k0;
        vo = (vo == v0) ? v1 : v0;
    }
    return PM_OK;
}

}  // namespace pm
