// Edge-list ingest: the undirected simple graph of a list of vertex pairs, as
// CSR, built on the device.  Every pair stands for an undirected edge (both
// directions become slots), self-loops are dropped and repeated pairs merged
// -- the clean-up the paper applies to its input graphs before counting
// (Section 6: direction ignored, duplicates and self-loops removed).
//
// Only one direction of a pair, (low end, high end), is sorted; the other
// follows from the finished half:
//   1. stable radix sort by high end, then by low end (the first pass reads
//      the raw pairs): pairs ordered (low, high), repeats side by side
//   2. keep the first of each run of equal pairs (no loops): the upper half
//      of every row, in order
//   3. stable radix sort of the kept pairs by high end: the lower half of
//      every row, in order
//   4. rows are lower half, then upper half: each half's row starts, their
//      sums as offsets, and every column to its place
// Sorting both directions by column and by row instead moved twice the
// elements through as many passes: 1.3e8 raw R-MAT pairs took 11.3 ms against
// 6.75 ms here (the passes 4.6, duplicates 0.6, row starts and columns 1.1,
// and the caller's copy), 6.7e5 pairs 332 against 205 us.  Reading the pairs
// and writing the CSR alone is 0.34 ms.
#include "graph.hpp"
#include "profile.hpp"
#include "radix.hpp"
#include "rowstarts.hpp"
#include "scan.hpp"

namespace pm {

pm_status graph_create(const pm_csr_view *csr, uint32_t flags, hipStream_t s, pm_graph **out);

namespace {

enum : uint32_t { ING_RANGE = 1u };

// what the host reads back after step 2
struct IngestState {
    uint32_t err;
    uint32_t kept;
};

// The raw pairs as radix elements: key the high end, value the low end.  The
// scatter also checks the ends (the passes take any key).
struct RawPairs {
    const int32_t *a, *b;
    int64_t n;
    IngestState *st;
    __device__ __forceinline__ uint32_t key(int64_t i) const
    {
        const uint32_t x = (uint32_t)a[i], y = (uint32_t)b[i];
        return x < y ? y : x;
    }
    __device__ __forceinline__ void load(int64_t i, uint32_t &k, uint32_t &v) const
    {
        const uint32_t x = (uint32_t)read_once(a + i), y = (uint32_t)read_once(b + i);
        k = x < y ? y : x;
        v = x < y ? x : y;
    }
    __device__ __forceinline__ void check(const uint32_t (&k)[kRadixItems]) const
    {
        uint32_t top = 0;
#pragma unroll
        for (int i = 0; i < kRadixItems; ++i) top = top < k[i] ? k[i] : top;
        if ((int64_t)top > n - 1) atomicOr(&st->err, (uint32_t)ING_RANGE);  // a negative end is above n as unsigned
    }
};

// Steps 2's kept pairs, one wave per run of kKeepItems rows of 64 pairs: the
// kept ones of a row are a ballot, the pair before a lane's own comes from the
// lane below (the row's first from the row before).  WRITE stores the kept
// pairs from `first` (the tile's first position) on; without, only their
// number per tile is stored.
constexpr int kKeepItems = 16;
constexpr int64_t kKeepTile = (int64_t)kBlock * kKeepItems;

template <bool WRITE>
__global__ __launch_bounds__(kBlock) void k_keep(const uint32_t *__restrict__ lo, const uint32_t *__restrict__ hi,
                                                 int64_t M, uint32_t *__restrict__ tile_sums,
                                                 uint32_t *__restrict__ lo_out, uint32_t *__restrict__ hi_out)
{
    __shared__ uint32_t s_sum[kBlock / kWave];
    const int w = threadIdx.x / kWave, lane = lane_id();
    const int64_t base = (int64_t)blockIdx.x * kKeepTile + (int64_t)w * (kWave * kKeepItems);
    uint32_t a[kKeepItems], b[kKeepItems];
#pragma unroll
    for (int i = 0; i < kKeepItems; ++i) {
        const int64_t idx = base + i * kWave + lane;
        a[i] = idx < M ? lo[idx] : 0u;  // past the end: a loop, not kept
        b[i] = idx < M ? hi[idx] : 0u;
    }
    // the pair before the wave's first: none equals a loop that is not kept
    uint32_t pa = 0u, pb = 0u;
    if (base > 0 && base <= M) {
        pa = lo[base - 1];
        pb = hi[base - 1];
    }
    uint64_t keep[kKeepItems];
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < kKeepItems; ++i) {
        const uint32_t ua = __shfl_up(a[i], 1, kWave), ub = __shfl_up(b[i], 1, kWave);
        const uint32_t qa = lane ? ua : pa, qb = lane ? ub : pb;
        keep[i] = __ballot(a[i] != b[i] && (qa != a[i] || qb != b[i]));
        sum += (uint32_t)__popcll(keep[i]);
        pa = __shfl(a[i], kWave - 1, kWave);
        pb = __shfl(b[i], kWave - 1, kWave);
    }
    if (lane == 0) s_sum[w] = sum;
    __syncthreads();
    if (!WRITE) {
        if (threadIdx.x == 0) {
            uint32_t t = 0;
#pragma unroll
            for (int i = 0; i < kBlock / kWave; ++i) t += s_sum[i];
            tile_sums[blockIdx.x] = t;
        }
        return;
    }
    uint32_t run = tile_sums[blockIdx.x];
    for (int i = 0; i < w; ++i) run += s_sum[i];
#pragma unroll
    for (int i = 0; i < kKeepItems; ++i) {
        if ((keep[i] >> lane) & 1ull) {
            const uint32_t p = run + __builtin_amdgcn_mbcnt_hi((uint32_t)(keep[i] >> 32),
                                                               __builtin_amdgcn_mbcnt_lo((uint32_t)keep[i], 0u));
            lo_out[p] = a[i];
            hi_out[p] = b[i];
        }
        run += (uint32_t)__popcll(keep[i]);
    }
}

// Row starts of the sorted keys of K entries (rowstarts.hpp): entry i sets
// those of its span; a block fills its long spans together.  kEach entries per
// thread, their loads together.
constexpr uint32_t kGapAlone = 16;
constexpr int kEach = 4;

__global__ __launch_bounds__(kBlock) void k_row_starts(const uint32_t *__restrict__ key, int64_t K, int64_t n,
                                                       uint32_t *__restrict__ start)
{
    __shared__ uint32_t s_gap[kBlock * kEach][2];  // first row of the gap, the entry
    __shared__ uint32_t s_n;
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * (kBlock * kEach) + threadIdx.x;
    RowSpan r[kEach];
#pragma unroll
    for (int j = 0; j < kEach; ++j) r[j] = row_span(key, K, n, base + j * kBlock);
#pragma unroll
    for (int j = 0; j < kEach; ++j) {
        const int64_t i = base + j * kBlock;
        if (r[j].first > r[j].last || i > K) continue;
        if (r[j].last - r[j].first < kGapAlone) {
            for (uint32_t v = r[j].first; v <= r[j].last; ++v) start[v] = (uint32_t)i;
        } else {
            const uint32_t q = atomicAdd(&s_n, 1u);
            s_gap[q][0] = r[j].first;
            s_gap[q][1] = (uint32_t)i;
        }
    }
    __syncthreads();
    const uint32_t gaps = s_n;
    for (uint32_t q = 0; q < gaps; ++q) {
        const int64_t i = s_gap[q][1], end = i < K ? (int64_t)key[i] : n;
        for (int64_t v = (int64_t)s_gap[q][0] + threadIdx.x; v <= end; v += kBlock) start[v] = (uint32_t)i;
    }
}

// offsets of both halves together
__global__ __launch_bounds__(kBlock) void k_offsets(const uint32_t *__restrict__ up, const uint32_t *__restrict__ low,
                                                    int64_t n, int64_t *__restrict__ off)
{
    const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (v <= n) off[v] = (int64_t)up[v] + (int64_t)low[v];
}

// Every column to its slot.  Row v starts at up[v] + low[v] with its lower
// half: entry q of the lower half (row hi_s[q]) goes to q + up[row], entry i
// of the upper half (row lo_u[i]) to i + low[row + 1].
__global__ __launch_bounds__(kBlock) void k_place(const uint32_t *__restrict__ lo_u, const uint32_t *__restrict__ hi_u,
                                                  const uint32_t *__restrict__ hi_s, const uint32_t *__restrict__ lo_s,
                                                  const uint32_t *__restrict__ up, const uint32_t *__restrict__ low,
                                                  int64_t K, int32_t *__restrict__ col)
{
    const int64_t base = (int64_t)blockIdx.x * (kBlock * kEach) + threadIdx.x;
    uint32_t lu[kEach], hu[kEach], hs[kEach], ls[kEach], pu[kEach], ps[kEach];
#pragma unroll
    for (int j = 0; j < kEach; ++j) {
        const int64_t i = base + j * kBlock < K ? base + j * kBlock : K - 1;  // (past the end: not written)
        lu[j] = read_once(lo_u + i);
        hs[j] = read_once(hi_s + i);
        hu[j] = read_once(hi_u + i);
        ls[j] = read_once(lo_s + i);
    }
#pragma unroll
    for (int j = 0; j < kEach; ++j) {
        pu[j] = low[lu[j] + 1];
        ps[j] = up[hs[j]];
    }
#pragma unroll
    for (int j = 0; j < kEach; ++j) {
        const int64_t i = base + j * kBlock;
        if (i >= K) continue;
        col[(uint32_t)i + pu[j]] = (int32_t)hu[j];
        col[(uint32_t)i + ps[j]] = (int32_t)ls[j];
    }
}

// The CSR of the edge list into off[n+1] and col[capacity] (device).
pm_status csr_from_edges_impl(const pm_edge_view *ev, int64_t *off, int32_t *col, int64_t capacity, int64_t *slots_out,
                              hipStream_t s)
{
    const int64_t n = ev->n, E = ev->num_edges;
    Temps tmp(s);
    const int32_t *src = ev->src, *dst = ev->dst;
    if (!ev->on_device && E > 0) {
        int32_t *ds = nullptr, *dd = nullptr;
        PM_TRY(tmp.get(&ds, (size_t)E));
        PM_TRY(tmp.get(&dd, (size_t)E));
        PM_HIP(hipMemcpyAsync(ds, src, sizeof(int32_t) * E, hipMemcpyHostToDevice, s));
        PM_HIP(hipMemcpyAsync(dd, dst, sizeof(int32_t) * E, hipMemcpyHostToDevice, s));
        src = ds;
        dst = dd;
    }
    if (E == 0) {
        PM_TRY(fill_async<int64_t>(off, 0ll, n + 1, s));
        *slots_out = 0;
        return PM_OK;
    }
    const size_t ee = (size_t)E;
    const int bits = bits_for(n > 0 ? (uint64_t)(n - 1) : 0);
    IngestState *st = nullptr, hst{};
    char *scr = nullptr;
    uint32_t *k0, *v0, *k1, *v1, *sums = nullptr;
    const int64_t tiles = (E + kKeepTile - 1) / kKeepTile;
    // (all of it before the first kernel that reads the pairs: up to the read
    // back nothing returns for want of memory while the caller's arrays are read)
    PM_TRY(tmp.get(&st, 1));
    PM_TRY(fill_async<uint32_t>((uint32_t *)st, 0u, 2, s));
    PM_TRY(tmp.get(&sums, (size_t)tiles));
    PM_TRY(tmp.get(&scr, radix_scratch_bytes(E)));
    PM_TRY(tmp.get(&k0, ee));
    PM_TRY(tmp.get(&v0, ee));
    PM_TRY(tmp.get(&k1, ee));
    PM_TRY(tmp.get(&v1, ee));
    uint32_t *hi = nullptr, *lo = nullptr, *lo_s = nullptr, *hi_s = nullptr;
    PM_TRY(radix_sort("ingest.sort_high", RawPairs{src, dst, n, st}, k0, v0, k1, v1, E, bits, scr, s, &hi, &lo));
    // by low end, between the free pair and this one (either may be written:
    // a pass reads one pair and writes the other)
    uint32_t *kf = hi == k0 ? k1 : k0, *vf = hi == k0 ? v1 : v0;
    PM_TRY(radix_sort("ingest.sort_low", RadixPairs{lo, hi}, kf, vf, hi, lo, E, bits, scr, s, &lo_s, &hi_s));
    // the kept pairs into the other buffers
    uint32_t *lo_u = lo_s == kf ? hi : kf, *hi_u = hi_s == vf ? lo : vf;
    {
        ProfScope prof("ingest.dedup", s);
        hipLaunchKernelGGL(k_keep<false>, dim3((unsigned)tiles), dim3(kBlock), 0, s, lo_s, hi_s, E, sums, nullptr,
                           nullptr);
        hipLaunchKernelGGL((scan_tiles_kernel<uint32_t, SumOp<uint32_t>>), dim3(1), dim3(1024), 0, s, sums, tiles,
                           SumOp<uint32_t>(), 0u, &st->kept);
        hipLaunchKernelGGL(k_keep<true>, dim3((unsigned)tiles), dim3(kBlock), 0, s, lo_s, hi_s, E, sums, lo_u,
                           hi_u);
        PM_HIP(hipGetLastError());
    }
    PM_HIP(hipMemcpyAsync(&hst, st, sizeof(hst), hipMemcpyDeviceToHost, s));
    PM_HIP(hipStreamSynchronize(s));
    if (hst.err & ING_RANGE) {
        set_error("edge list: an endpoint is not a vertex id in [0, n)");
        return PM_EGRAPH;
    }
    const int64_t K = hst.kept, slots = 2 * K;
    if (slots > capacity) {
        set_error("edge list: the CSR needs " + std::to_string(slots) + " column slots, capacity is " +
                  std::to_string(capacity));
        return PM_EINVAL;
    }
    // the lower halves: the kept pairs by high end, between the sorted pairs'
    // buffers (no longer needed) and one more pair
    uint32_t *k2 = nullptr, *v2 = nullptr, *up = nullptr, *low = nullptr;
    PM_TRY(tmp.get(&k2, (size_t)std::max<int64_t>(K, 1)));
    PM_TRY(tmp.get(&v2, (size_t)std::max<int64_t>(K, 1)));
    PM_TRY(tmp.get(&up, (size_t)n + 1));
    PM_TRY(tmp.get(&low, (size_t)n + 1));
    uint32_t *hi_l = nullptr, *lo_l = nullptr;
    PM_TRY(radix_sort("ingest.sort_half", RadixPairs{hi_u, lo_u}, lo_s, hi_s, k2, v2, K, bits, scr, s, &hi_l, &lo_l));
    {
        ProfScope prof("ingest.place", s);
        const unsigned kb = (unsigned)(K / (kBlock * kEach) + 1);  // K + 1 entries
        hipLaunchKernelGGL(k_row_starts, dim3(kb), dim3(kBlock), 0, s, lo_u, K, n, up);
        hipLaunchKernelGGL(k_row_starts, dim3(kb), dim3(kBlock), 0, s, hi_l, K, n, low);
        hipLaunchKernelGGL(k_offsets, dim3((unsigned)(n / kBlock + 1)), dim3(kBlock), 0, s, up, low, n, off);
        if (K > 0)
            hipLaunchKernelGGL(k_place, dim3(kb), dim3(kBlock), 0, s, lo_u, hi_u, hi_l, lo_l, up, low, K, col);
        PM_HIP(hipGetLastError());
    }
    *slots_out = slots;
    return PM_OK;
}

pm_status check_edge_view(const pm_edge_view *ev)
{
    if (!ev || ev->n < 0 || ev->n > (int64_t)INT32_MAX - 1 || ev->num_edges < 0 ||
        (ev->num_edges > 0 && (!ev->src || !ev->dst)) || 2 * ev->num_edges >= (int64_t)UINT32_MAX) {
        set_error("edge list: n in [0, 2^31 - 1), 0 <= num_edges < 2^31, src and dst given");
        return PM_EINVAL;
    }
    return PM_OK;
}

}  // namespace

pm_status csr_from_edges(const pm_edge_view *ev, int64_t *off, int32_t *col, int64_t capacity, int64_t *slots_out,
                         hipStream_t s)
{
    PM_TRY(check_edge_view(ev));
    if (!off || !slots_out || capacity < 0 || (capacity > 0 && !col)) {
        set_error("edge list: null output or negative capacity");
        return PM_EINVAL;
    }
    ProfScope prof("ingest_total", s);
    return csr_from_edges_impl(ev, off, col, capacity, slots_out, s);
}

pm_status graph_from_edges(const pm_edge_view *ev, uint32_t flags, hipStream_t s, pm_graph **out)
{
    PM_TRY(check_edge_view(ev));
    if (!out) {
        set_error("edge list: null output");
        return PM_EINVAL;
    }
    *out = nullptr;
    Temps tmp(s);
    int64_t *off = nullptr;
    int32_t *col = nullptr;
    const int64_t cap = 2 * ev->num_edges;
    PM_TRY(tmp.get(&off, (size_t)(ev->n + 1)));
    PM_TRY(tmp.get(&col, (size_t)(cap > 0 ? cap : 1)));
    int64_t slots = 0;
    {
        ProfScope prof("ingest_total", s);
        PM_TRY(csr_from_edges_impl(ev, off, col, cap, &slots, s));
    }
    pm_csr_view v;
    v.n = ev->n;
    v.row_offsets = off;
    v.cols = col;
    v.on_device = 1;
    return graph_create(&v, flags, s, out);
}

}  // namespace pm
