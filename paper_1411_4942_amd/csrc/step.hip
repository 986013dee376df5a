// Draw-ordered steps (step.hpp).  A step's samples are bound by the lines they
// miss in L2: request by request in id order a sample of the graphs of up to
// 4e6 edges missed 6.8 of its 15 lines, at 5.4e10 misses a second, the rate of
// random lines of this memory.  Sorted by (graph, sampler, draw) the samples
// of all the requests on a graph sweep its slots once, together: 64 requests
// of 1.0e8 samples in all on 12 graphs went from 13.2 to 8.3 ms of steps, 1.4
// of them the sorts and the others 65 ps a sample; 64 graphs at 2e5 + 2e5
// samples from 2.82 to 2.34 ms a run (2.03 with the
// blocks of step.hpp).
#include "step.hpp"

#include <algorithm>
#include <cstring>
#include <new>

#include "drawsort.hpp"
#include "profile.hpp"
#include "sampler.hpp"

namespace pm {

static_assert(sizeof(StepChunk) == 32 && sizeof(StepGroup) == 24, "uploaded as they are");
static_assert(kSortedChunk <= 1u << kDrawKeyBits, "a rank is a sort key");

// The sort key of a position: its group's first position plus the rank its
// draw is expected to have inside the group, so the keys spread evenly over
// the part whatever the groups' sizes, and the sorted positions
// [begin, next group's begin) are exactly a group's.  The rank is monotone in
// the draw (each rounding is); draws a rounding apart may share one.
struct StepKey {
    const BatchGraph *graphs;
    const StepChunk *chunks;
    const StepGroup *groups;
    uint32_t nchunks;
    __device__ uint32_t operator()(int64_t i) const
    {
        const uint32_t p = (uint32_t)i;
        // the active lanes hold ascending positions: one search for the
        // first, then chunk after chunk, all from scalar loads
        const uint32_t p0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)p);
        uint32_t c = 0, hi = nchunks;  // last chunk with start <= p0
        while (hi - c > 1) {
            const uint32_t mid = (c + hi) >> 1;
            if (chunks[mid].start <= p0)
                c = mid;
            else
                hi = mid;
        }
        uint32_t key = 0;
        for (; c < nchunks; ++c) {
            const StepChunk C = chunks[c];
            const uint32_t end = chunks[c + 1].start;
            const StepGroup G = groups[C.group];
            const uint32_t n = groups[C.group + 1].begin - G.begin;
            if (p >= C.start && p < end) {
                const uint64_t r = draw_bounded(C.seed, G.tag, C.first + (p - C.start), graphs[G.graph].v[G.tag].R);
                const uint32_t rank = (uint32_t)((double)r * G.scale);
                key = G.begin + (rank < n ? rank : n - 1);
            }
            if (!__any(p >= end)) break;
        }
        return key;
    }
};

// The samples at the sorted positions ids[0, kc): whole waves step over them;
// a wave's positions lie in one group, or in a few taken one after another,
// so the graph is wave-uniform.  Each lane finds its request among the
// group's few chunks in LDS and counts its class there (the lanes' requests
// differ, so the wave keeps no counters of its own).
__global__ __launch_bounds__(kBlock) void k_sample_step(const BatchGraph *__restrict__ graphs,
                                                        const StepChunk *__restrict__ chunks,
                                                        const StepGroup *__restrict__ groups, uint32_t nchunks,
                                                        uint32_t ngroups, const uint32_t *__restrict__ ids,
                                                        uint32_t kc, uint32_t *__restrict__ counts)
{
    __shared__ uint32_t s_start[kStepChunks];
    __shared__ uint32_t s_cnt[kStepChunks * PM_NUM_TALLIES];
    for (uint32_t i = threadIdx.x; i < nchunks; i += kBlock) s_start[i] = chunks[i].start;
    for (uint32_t i = threadIdx.x; i < nchunks * PM_NUM_TALLIES; i += kBlock) s_cnt[i] = 0;
    __syncthreads();
    const uint64_t step = (uint64_t)gridDim.x * kBlock;
    uint32_t gi = 0;
    for (uint64_t base = wave_index(blockIdx.x) * kWave; base < kc; base += step) {  // wave-uniform
        const uint32_t j = (uint32_t)base + (uint32_t)lane_id();  // kc <= 2^24
        const uint32_t stop = (uint32_t)base + kWave < kc ? (uint32_t)base + kWave : kc;
        const uint32_t pos = j < kc ? ids[j] : 0u;
        while (gi + 1 < ngroups && groups[gi + 1].begin <= (uint32_t)base) ++gi;
        for (uint32_t at = (uint32_t)base, q = gi; at < stop && q < ngroups; ++q) {
            const StepGroup G = groups[q];
            const uint32_t end = groups[q + 1].begin, c1 = groups[q + 1].chunk0;
            if (j >= at && j < end && j < stop) {
                uint32_t c = G.chunk0, hi = c1;  // last chunk with start <= pos
                while (hi - c > 1) {
                    const uint32_t mid = (c + hi) >> 1;
                    if (s_start[mid] <= pos)
                        c = mid;
                    else
                        hi = mid;
                }
                const uint64_t id = chunks[c].first + (pos - s_start[c]), seed = chunks[c].seed;
                const uint32_t cls = G.tag == 0 ? sample_class<false>(graphs[G.graph].v[0], seed, id)
                                                : sample_class<true>(graphs[G.graph].v[1], seed, id);
                atomicAdd(&s_cnt[c * PM_NUM_TALLIES + cls], 1u);
            }
            at = end;
        }
    }
    __syncthreads();
    const uint32_t words = nchunks * PM_NUM_TALLIES;
    for (uint32_t i = threadIdx.x; i < words; i += kBlock) counts[(uint64_t)blockIdx.x * words + i] = s_cnt[i];
}

// Column sums of the blocks' counts, kWave columns (8 chunks) per block.
__global__ __launch_bounds__(1024) void k_step_sum(const uint32_t *__restrict__ counts, uint32_t rows,
                                                   const StepChunk *__restrict__ chunks,
                                                   const StepGroup *__restrict__ groups, uint32_t nchunks,
                                                   unsigned long long *__restrict__ tallies)
{
    constexpr uint32_t kRows = 1024 / kWave;
    __shared__ uint32_t s_sum[kRows][kWave];
    const uint32_t words = nchunks * PM_NUM_TALLIES, lane = threadIdx.x % kWave, q = threadIdx.x / kWave;
    const uint32_t w = blockIdx.x * kWave + lane;
    uint32_t v = 0;  // a part has at most 2^24 samples
    if (w < words)
        for (uint32_t r = q; r < rows; r += kRows) v += counts[(uint64_t)r * words + w];
    s_sum[q][lane] = v;
    __syncthreads();
    if (q == 0 && w < words) {
        for (uint32_t r = 1; r < kRows; ++r) v += s_sum[r][lane];
        const StepChunk C = chunks[w / PM_NUM_TALLIES];
        const uint64_t at = ((uint64_t)C.slot * 2 + groups[C.group].tag) * PM_NUM_TALLIES + w % PM_NUM_TALLIES;
        tallies[at] += v;  // a (slot, sampler) has one chunk in a part
    }
}

namespace {

// One part: its tables on the host.
struct HostPart {
    std::vector<StepChunk> chunks;
    std::vector<StepGroup> groups;
    uint32_t samples = 0;
};

void close_part(HostPart &p, const std::vector<uint64_t> &weights)
{
    p.groups.push_back(StepGroup{0.0, p.samples, (uint32_t)p.chunks.size(), 0, 0});
    p.chunks.push_back(StepChunk{0, 0, p.samples, 0, 0, 0});
    for (size_t i = 0; i + 1 < p.groups.size(); ++i)
        p.groups[i].scale = (double)(p.groups[i + 1].begin - p.groups[i].begin) / (double)weights[i];
}

// The items in group order cut into parts of equal size, or of kStepChunks
// chunks where that comes first.
std::vector<HostPart> cut_parts(std::vector<StepItem> &items, uint64_t samples)
{
    std::stable_sort(items.begin(), items.end(), [](const StepItem &a, const StepItem &b) {
        return a.graph != b.graph ? a.graph < b.graph : a.tag < b.tag;
    });
    const uint64_t parts = (samples + kSortedChunk - 1) / kSortedChunk, per = (samples + parts - 1) / parts;
    std::vector<HostPart> P;
    std::vector<uint64_t> weights;  // of the last part's groups
    for (const StepItem &it : items)
        for (uint64_t done = 0; done < it.count;) {
            if (P.empty() || P.back().samples == per || P.back().chunks.size() == kStepChunks) {
                if (!P.empty()) close_part(P.back(), weights);
                P.emplace_back();
                weights.clear();
            }
            HostPart &p = P.back();
            if (p.groups.empty() || p.groups.back().graph != it.graph || p.groups.back().tag != it.tag) {
                p.groups.push_back(StepGroup{0.0, p.samples, (uint32_t)p.chunks.size(), it.graph, it.tag});
                weights.push_back(it.R);
            }
            const uint64_t take = std::min<uint64_t>(it.count - done, per - p.samples);
            p.chunks.push_back(
                StepChunk{it.first + done, it.seed, p.samples, it.slot, (uint32_t)p.groups.size() - 1, 0});
            p.samples += (uint32_t)take;
            done += take;
        }
    close_part(P.back(), weights);
    return P;
}

size_t table_bytes(const HostPart &p)
{
    return p.chunks.size() * sizeof(StepChunk) + p.groups.size() * sizeof(StepGroup);
}

// words of the blocks' counts
constexpr size_t kCountWords = (size_t)kStepBlocks * kStepChunks * PM_NUM_TALLIES;

// One part whose tables lie at `tables`: sort its positions, run its samples,
// add their counts to the tallies.
pm_status launch_part(const BatchGraph *graphs, const HostPart &p, const char *tables, const DrawSortBufs &b,
                      uint32_t *counts, uint64_t *tallies, unsigned blocks, hipStream_t s)
{
    const StepChunk *chunks = reinterpret_cast<const StepChunk *>(tables);
    const StepGroup *groups = reinterpret_cast<const StepGroup *>(tables + p.chunks.size() * sizeof(StepChunk));
    const uint32_t nchunks = (uint32_t)p.chunks.size() - 1, ngroups = (uint32_t)p.groups.size() - 1;
    uint32_t *ids = nullptr;
    PM_TRY(draw_sort("step_sort", StepKey{graphs, chunks, groups, nchunks}, p.samples,
                     std::max(1, bits_for(p.samples - 1)), s, b, &ids));
    const unsigned nb = std::min(std::min(blocks, kStepBlocks), (p.samples + kBlock - 1) / kBlock);
    ProfScope prof("sample_step", s);
    hipLaunchKernelGGL(k_sample_step, dim3(nb), dim3(kBlock), 0, s, graphs, chunks, groups, nchunks, ngroups, ids,
                       p.samples, counts);
    hipLaunchKernelGGL(k_step_sum, dim3((nchunks * PM_NUM_TALLIES + kWave - 1) / kWave), dim3(1024), 0, s, counts, nb,
                       chunks, groups, nchunks, (unsigned long long *)tallies);
    PM_HIP(hipGetLastError());
    return PM_OK;
}

}  // namespace

// Room for the parts' tables; false when the device or the host has no memory.
bool StepRunner::grow(size_t bytes, hipStream_t s)
{
    if (bytes <= table_cap) return true;
    dev_free(d_tables, s);
    if (h_tables) (void)hipHostFree(h_tables);
    d_tables = h_tables = nullptr;
    table_cap = 0;
    if (dev_alloc((void **)&d_tables, 2 * bytes, s) != PM_OK) return false;
    if (hipHostMalloc((void **)&h_tables, 2 * bytes, hipHostMallocDefault) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    table_cap = 2 * bytes;
    return true;
}

void StepRunner::free(hipStream_t s)
{
    dev_free(d_tables, s);
    if (h_tables) (void)hipHostFree(h_tables);
    d_tables = h_tables = nullptr;
    table_cap = 0;
}

// Positions that the sort's buffers of a part are taken for: a power of two, so
// that steps of any size reuse few blocks of the library's cache.
static uint64_t order_positions(uint64_t part)
{
    uint64_t cap = 1ull << 20;
    while (cap < part) cap <<= 1;
    return cap;
}
static_assert((kSortedChunk & (kSortedChunk - 1)) == 0, "the largest part is a power of two");

// A step of one part pays from draw_order_min() samples on (64 graphs of up to
// 2e6 edges at 2.6e6 samples in all: 0.77 ms in id order, 0.44 ms ordered; one
// graph of 2.4e5 edges at 2e6: 0.18 ms either way).  Many small items cut a
// step into parts of kStepChunks chunks; below this size a part's launches
// (about 60 us) cost what the order saves.
constexpr uint64_t kStepPartMin = 1ull << 20;
// Above this (2^16 parts, minutes of sampling) a step is left to the id order
// too, which refuses what its tile table cannot hold: the parts' tables would
// grow with a budget of any size.
constexpr uint64_t kStepMax = kSortedChunk << 16;

pm_status StepRunner::run(const BatchGraph *graphs, std::vector<StepItem> &items, uint64_t *tallies, int64_t slots,
                          unsigned blocks, hipStream_t s, bool *done)
{
    *done = false;
    uint64_t samples = 0;
    for (const StepItem &it : items) {
        if (it.count > kStepMax - samples) return PM_OK;
        samples += it.count;
    }
    if (samples == 0 || !draw_order_enabled() || samples < draw_order_min()) return PM_OK;
    const auto too_small = [&](uint64_t parts) {
        return parts > 1 && samples / parts < std::min<uint64_t>(draw_order_min(), kStepPartMin);
    };
    // (the least there can be, before the work of cutting them)
    if (too_small((items.size() + kStepChunks - 1) / kStepChunks)) return PM_OK;
    bool enqueued = false;
    const auto step = [&]() -> pm_status {
        const std::vector<HostPart> parts = cut_parts(items, samples);
        if (too_small(parts.size()) || memory.skip()) return PM_OK;
        size_t bytes = 0;
        uint64_t largest = 0;
        for (const HostPart &p : parts) {
            bytes += table_bytes(p);
            largest = std::max<uint64_t>(largest, p.samples);
        }
        // the sort's buffers, then the blocks' counts: the library's cached
        // memory for the step, as pm_count's
        Temps tmp(s);
        const uint64_t cap = order_positions(largest);
        char *order = nullptr;
        if (!grow(bytes, s) || tmp.get(&order, draw_sort_bytes(cap) + 4 * kCountWords) != PM_OK) {
            memory.failed();
            return PM_OK;
        }
        memory.succeeded();
        size_t at = 0;
        for (const HostPart &p : parts) {  // (both tables are multiples of 8 bytes)
            const size_t c = p.chunks.size() * sizeof(StepChunk);
            std::memcpy(h_tables + at, p.chunks.data(), c);
            std::memcpy(h_tables + at + c, p.groups.data(), p.groups.size() * sizeof(StepGroup));
            at += table_bytes(p);
        }
        DrawSortBufs b{};
        draw_sort_carve(order, cap, &b);
        uint32_t *counts = reinterpret_cast<uint32_t *>(order + draw_sort_bytes(cap));
        enqueued = true;
        PM_HIP(hipMemcpyAsync(d_tables, h_tables, at, hipMemcpyHostToDevice, s));
        PM_TRY(fill_async<uint64_t>(tallies, 0ull, slots * 2 * PM_NUM_TALLIES, s));
        at = 0;
        for (const HostPart &p : parts) {
            PM_TRY(launch_part(graphs, p, d_tables + at, b, counts, tallies, blocks, s));
            at += table_bytes(p);
        }
        *done = true;
        return PM_OK;
    };
    pm_status st;
    try {
        st = step();
    } catch (const std::bad_alloc &) {
        if (!enqueued) return PM_OK;  // the id order needs no tables
        set_error("ordered step: no host memory");
        st = PM_ENOMEM;
    }
    // a step that failed midway has parts in flight: they read the tables, which
    // the next step writes, and the graphs, which the caller may then free
    if (st != PM_OK) (void)hipStreamSynchronize(s);
    return st;
}

}  // namespace pm
