// Exact induced 4-vertex counts on the device: ground truth at sizes the
// sampler runs at, split the way the paper describes its enumeration code
// (Section 6): the cycle-based subgraph counts by enumeration under the
// degree order, the others by formulas, then Eq. 1 solved for the induced
// counts.
//
// On the prepared graph vertex ids are ranks of the degree order and every
// row is ascending, so N+(x) (neighbours of higher rank) is the row suffix
// after position split[x] and the lower neighbours are the prefix.
//   N_1 = sum_v C(d_v, 3)                  (already in the prepared graph)
//   N_2 = W - 3T                           3-paths (W from the tau total)
//   N_3 = sum_v t_v (d_v - 2) = 1/2 sum_e t_e (d_u + d_v - 4)
//   N_4 = 4-cycles: at each cycle's highest vertex x, pairs of lower wedge
//         middles between x and each lower opposite vertex y
//   N_5 = sum_e C(t_e, 2)                  diamonds
//   N_6 = 4-cliques, counted at their lowest vertex u without listing them:
//         the graph induced on N+(u) as bit rows, a clique {u, v, w, x}
//         being a bit of row(v) & row(w) for an edge (v, w) inside N+(u)
// t_e = triangles on edge e (each found once, from its lowest vertex).
#include <algorithm>
#include <cstring>

#include "graph.hpp"
#include "profile.hpp"
#include "rowhash.hpp"

namespace pm {

pm_status check_device(const pm_graph *g);
int sampler_cu_count(int dev);

namespace {

struct ExactAcc {
    unsigned long long tri;           // triangles (each once)
    unsigned long long k4;            // 4-cliques (each once)
    unsigned long long n3_lo, n3_hi;  // 2 N_3
    unsigned long long n5_lo, n5_hi;  // N_5
    unsigned long long n4_lo, n4_hi;  // N_4
};

// 128-bit accumulation from per-block partial sums
__device__ void add128(unsigned long long *lo, unsigned long long *hi, unsigned __int128 v)
{
    const unsigned long long l = (unsigned long long)v, h = (unsigned long long)(v >> 64);
    const unsigned long long old = atomicAdd(lo, l);
    const unsigned long long carry = (old + l < old) ? 1ull : 0ull;
    if (h + carry) atomicAdd(hi, h + carry);
}

// Sum of one 128-bit value per thread over the block, valid in thread 0.
// Every thread of the block must call it.
template <int THREADS>
__device__ unsigned __int128 block_sum128(unsigned __int128 v)
{
    __shared__ unsigned long long s_lo[THREADS], s_hi[THREADS];
    __syncthreads();  // a previous call's readers are done with the arrays
    s_lo[threadIdx.x] = (unsigned long long)v;
    s_hi[threadIdx.x] = (unsigned long long)(v >> 64);
    __syncthreads();
    for (int d = THREADS / 2; d > 0; d >>= 1) {
        if ((int)threadIdx.x < d) {
            const unsigned __int128 a = (unsigned __int128)s_lo[threadIdx.x] |
                                        ((unsigned __int128)s_hi[threadIdx.x] << 64);
            const unsigned __int128 b = (unsigned __int128)s_lo[threadIdx.x + d] |
                                        ((unsigned __int128)s_hi[threadIdx.x + d] << 64);
            const unsigned __int128 c = a + b;
            s_lo[threadIdx.x] = (unsigned long long)c;
            s_hi[threadIdx.x] = (unsigned long long)(c >> 64);
        }
        __syncthreads();
    }
    return (unsigned __int128)s_lo[0] | ((unsigned __int128)s_hi[0] << 64);
}

// Sum of one 64-bit value per lane over the wave, valid in lane 0.
__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v)
{
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) v += __shfl_down(v, d, kWave);
    return v;
}

// Sum of one 128-bit value per lane over the wave, valid in lane 0.
__device__ __forceinline__ unsigned __int128 wave_sum128(unsigned __int128 v)
{
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) {
        const unsigned long long lo = __shfl_down((unsigned long long)v, d, kWave);
        const unsigned long long hi = __shfl_down((unsigned long long)(v >> 64), d, kWave);
        v += (unsigned __int128)lo | ((unsigned __int128)hi << 64);
    }
    return v;
}

// One value per thread summed over the block and added to *dst, one atomic per
// block (an atomic per wave on these few words cost 5.9 ns each).  Every
// thread of the block calls it; s_w holds THREADS / kWave words.
template <int THREADS>
__device__ __forceinline__ void block_add(unsigned long long v, unsigned long long *s_w, unsigned long long *dst)
{
    v = wave_sum_u64(v);
    __syncthreads();  // s_w may still be read by an earlier call
    if (lane_id() == 0) s_w[threadIdx.x / kWave] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0;
        for (int w = 0; w < THREADS / kWave; ++w) t += s_w[w];
        if (t) atomicAdd(dst, t);
    }
}

constexpr uint32_t kNoId = 0xFFFFFFFFu;  // not a vertex id (they are below 2^31): an empty member-hash slot

// The vertices by the kernels that handle them.  Triangles and 4-cliques:
// classes by forward degree D.  4-cycles: classes by S, the sum of the degrees
// of x's lower neighbours (at least the wedges counted at x), which bounds the
// distinct ids a table must hold.
enum : int { kCl64, kCl256, kCl1024, kClMore, kC4Wave, kC4Block, kC4Big, kC4Bits, kC4Ranges, kExactClasses };
constexpr uint32_t kC4WaveMax = 384;    // wedges: tables of 512, 4096 and 16384 slots, at most 3/4 full
constexpr uint32_t kC4BlockMax = 3072;
constexpr uint32_t kC4BigMax = 12288;
// above, where the ranges of k_four_cycles would be many: a bitmap of the ids
// (spans of kC4Span) and a table of the repeated ones
constexpr uint32_t kC4BitsMax = 60000;
constexpr uint32_t kC4BitsFrom = 1u << 18;  // x from here on: 4 ranges of ids or more
constexpr uint32_t kC4Span = 1u << 20;
constexpr uint32_t kC4Spans = 4;            // each span walks the rows again

// Counters on lines of their own, and the largest forward degree.
struct ExactLists {
    struct alignas(128) Line {
        uint32_t n;
    };
    Line count[kExactClasses];
    Line dmax;
};

// Class c's list lies in array c / 2 of n words: even classes from the front,
// odd ones from the back (a vertex is in at most one class of each pair; the
// last class has an array of its own, since a vertex of kC4Bits can join it).
constexpr int kExactArrays = (kExactClasses + 1) / 2;
__device__ __forceinline__ uint32_t list_at(const uint32_t *__restrict__ lists, int64_t n, int c, uint32_t i)
{
    const uint32_t *a = lists + (int64_t)(c / 2) * n;
    return c & 1 ? a[n - 1 - i] : a[i];
}

// split[x] = number of neighbours of x below x (rows ascending), and the
// lists.  A block takes kBlock vertices, highest ids (the heaviest) first:
// 16 lanes per vertex find its split and sum its lower neighbours' degrees,
// highest first, until they pass kC4BitsMax; then a thread per vertex appends
// it, one atomic per class and block.
constexpr int kClassLanes = 16;

__global__ __launch_bounds__(kBlock) void k_classify(const uint32_t *__restrict__ off, const uint32_t *__restrict__ col,
                                                     int64_t n, uint32_t *__restrict__ split,
                                                     uint32_t *__restrict__ lists, ExactLists *L)
{
    __shared__ uint32_t s_split[kBlock], s_deg[kBlock], s_sum[kBlock];
    __shared__ uint32_t s_n[kExactClasses], s_base[kExactClasses];
    __shared__ uint32_t s_dmax;
    const int t = threadIdx.x, sub = t & (kClassLanes - 1);
    if (t < kExactClasses) s_n[t] = 0;
    if (t == 0) s_dmax = 0;
    for (int r = 0; r < kClassLanes; ++r) {
        const int q = r * (kBlock / kClassLanes) + t / kClassLanes;
        const int64_t x = n - 1 - ((int64_t)blockIdx.x * kBlock + q);
        uint32_t sp = 0, d = 0, sum = 0;
        if (x >= 0) {
            const uint32_t a = off[x], e = off[x + 1];
            d = e - a;
            uint32_t lo = a, hi = e;
            while (lo < hi) {  // the same steps in all of the vertex's lanes
                const uint32_t mid = lo + (hi - lo) / 2;
                if (col[mid] < (uint32_t)x)
                    lo = mid + 1;
                else
                    hi = mid;
            }
            sp = lo - a;
            for (uint32_t k = 0; k < sp && sum <= kC4BitsMax; k += 4 * kClassLanes) {
                uint32_t w[4], dw = 0;  // four reads in flight
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t i = k + j * kClassLanes + sub;
                    w[j] = i < sp ? col[a + sp - 1 - i] : kNoId;
                }
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (w[j] != kNoId) {
                        const uint32_t dj = off[w[j] + 1] - off[w[j]];
                        dw += dj > kC4BitsMax ? kC4BitsMax + 1 : dj;
                    }
#pragma unroll
                for (int o = kClassLanes / 2; o > 0; o >>= 1) dw += __shfl_xor(dw, o, kClassLanes);
                sum += dw;
            }
        }
        if (sub == 0) {
            s_split[q] = sp;
            s_deg[q] = d;
            s_sum[q] = sum;
        }
    }
    __syncthreads();
    const int64_t x = n - 1 - ((int64_t)blockIdx.x * kBlock + t);
    int cl = -1, c4 = -1;
    uint32_t icl = 0, ic4 = 0;
    if (x >= 0) {
        const uint32_t sp = s_split[t], D = s_deg[t] - sp, S = s_sum[t];
        split[x] = sp;
        if (D >= 2) cl = D <= 64 ? kCl64 : D <= 256 ? kCl256 : D <= 1024 ? kCl1024 : kClMore;
        if (sp >= 2)
            c4 = S <= kC4WaveMax    ? kC4Wave
                 : S <= kC4BlockMax ? kC4Block
                 : S <= kC4BigMax   ? kC4Big
                 : S <= kC4BitsMax && sp < 4095 && x >= kC4BitsFrom && n <= (int64_t)kC4Spans * kC4Span ? kC4Bits
                                                                                                        : kC4Ranges;
        if (cl >= 0) icl = atomicAdd(&s_n[cl], 1u);
        if (c4 >= 0) ic4 = atomicAdd(&s_n[c4], 1u);
        if (D >= 2) atomicMax(&s_dmax, D);
    }
    __syncthreads();
    if (t < kExactClasses && s_n[t]) s_base[t] = atomicAdd(&L->count[t].n, s_n[t]);
    if (t == kExactClasses && s_dmax) atomicMax(&L->dmax.n, s_dmax);
    __syncthreads();
    const auto put = [&](int c, uint32_t i) {
        uint32_t *a = lists + (int64_t)(c / 2) * n;
        a[c & 1 ? n - 1 - i : (int64_t)i] = (uint32_t)x;
    };
    if (cl >= 0) put(cl, s_base[cl] + icl);
    if (c4 >= 0) put(c4, s_base[c4] + ic4);
}

// Triangles and 4-cliques at their lowest vertex u, one u per block at a time
// (a class's vertices, d+(u) <= 32 W; W words of 32 bits per row).  Row i of
// the graph induced on N+(u) = {ids[0] < ids[1] < ...} has bit j when
// ids[i] ~ ids[j], j > i (only forward neighbours are looked up).
//  - Each bit is a triangle {u, v_i, v_j}, found once.  It adds one to t_e
//    of its three edges: (v_i, v_j) at the forward slot p of row v_i where
//    the lookup found v_j, and (u, v_i), (u, v_j) at u's own forward slots
//    (counted per member in the block, then added once per slot).
//  - A clique {u, v_i, v_j, v_k} (i < j < k) is bit k of row i & row j for
//    each bit j of row i, so each is counted once, by whole words.
// Rows and member counters live in LDS (`scratch` null) or, for long forward
// rows, in the block's slice of a global scratch array.  A member is found
// in an LDS hash of N+(u) (id -> index, at most half full: one or two
// reads) in the LDS classes, by binary search in the global one.
template <int W, bool GLOBAL, int THREADS>
__global__ __launch_bounds__(THREADS) void k_cliques(const uint32_t *__restrict__ off,
                                                    const uint32_t *__restrict__ col,
                                                    const uint32_t *__restrict__ split, int64_t n,
                                                    const uint32_t *__restrict__ lists, int cls, uint32_t count,
                                                    uint32_t hi_d, uint32_t *__restrict__ scratch, uint32_t gslots,
                                                    uint32_t *__restrict__ t_e, ExactAcc *acc)
{
    constexpr int kLdsIds = GLOBAL ? 1 : 32 * W;
    constexpr int kLdsRows = GLOBAL ? 1 : 32 * W * W;
    constexpr uint32_t kSlots = GLOBAL ? 1 : 64 * W;  // member hash: twice the members
    __shared__ uint32_t s_ids[kLdsIds];
    __shared__ uint32_t s_tri[kLdsIds];  // triangles on (u, ids[i])
    __shared__ uint32_t s_rows[kLdsRows];
    __shared__ uint32_t h_key[kSlots];   // member id, or kNoId
    __shared__ uint16_t h_idx[kSlots];   // its index in ids
    __shared__ unsigned long long s_sum[THREADS / kWave];
    // GLOBAL with gslots > 0: ids, their counters and a member hash of gslots
    // slots (a power of two >= 2 hi_d) in dynamic LDS; gslots = 0: ids and
    // counters in the block's global slice, members found by binary search
    extern __shared__ uint32_t dyn[];
    const uint32_t wd = GLOBAL ? (hi_d + 31) / 32 : (uint32_t)W;  // words per row
    const uint32_t slots = GLOBAL ? gslots : kSlots;
    uint32_t *const slice = GLOBAL ? scratch + (uint64_t)blockIdx.x * ((uint64_t)hi_d * wd + 2ull * hi_d) : nullptr;
    uint32_t *ids = GLOBAL ? (gslots ? dyn : slice) : s_ids;
    uint32_t *tri_u = GLOBAL ? ids + hi_d : s_tri;
    uint32_t *rows = GLOBAL ? slice + 2ull * hi_d : s_rows;
    uint32_t *hkey = GLOBAL ? dyn + 2ull * hi_d : h_key;
    uint16_t *hidx = GLOBAL ? reinterpret_cast<uint16_t *>(dyn + 2ull * hi_d + gslots) : h_idx;
    const int wv = threadIdx.x / kWave, lane = lane_id(), nwv = THREADS / kWave;
    unsigned long long k4 = 0, tri = 0;
    for (uint32_t k = blockIdx.x; k < count; k += gridDim.x) {
        const uint32_t u = list_at(lists, n, cls, k);
        const uint32_t beg = off[u] + split[u], D = off[u + 1] - beg;  // <= hi_d by the class
        for (uint32_t i = threadIdx.x; i < D; i += THREADS) {
            ids[i] = col[beg + i];
            tri_u[i] = 0;
        }
        for (uint64_t i = threadIdx.x; i < (uint64_t)D * wd; i += THREADS) rows[i] = 0;
        if (GLOBAL) __threadfence();  // the cleared rows, before the atomics below
        if (slots) {
            for (uint32_t i = threadIdx.x; i < slots; i += THREADS) hkey[i] = kNoId;
            __syncthreads();
            for (uint32_t i = threadIdx.x; i < D; i += THREADS) {  // D <= slots / 2: a free slot is always found
                const uint32_t key = ids[i];
                for (uint32_t h = hash_mix32(key) & (slots - 1);; h = (h + 1) & (slots - 1))
                    if (atomicCAS(&hkey[h], kNoId, key) == kNoId) {
                        hidx[h] = (uint16_t)i;
                        break;
                    }
            }
        }
        __syncthreads();
        // rows: each wave takes a member v_i and looks its forward neighbours up
        for (uint32_t i = wv; i < D; i += nwv) {
            const uint32_t v = ids[i];
            const uint32_t vb = off[v] + split[v], ve = off[v + 1];
            for (uint32_t p = vb + lane; p < ve; p += kWave) {
                const uint32_t x = col[p];
                uint32_t lo = D;  // x's index in ids (> i: x > v = ids[i]), D if absent
                if (!slots) {
                    uint32_t hi = D;
                    lo = i + 1;
                    while (lo < hi) {
                        const uint32_t mid = (lo + hi) >> 1;
                        if (ids[mid] < x)
                            lo = mid + 1;
                        else
                            hi = mid;
                    }
                    if (lo < D && ids[lo] != x) lo = D;
                } else {
                    for (uint32_t h = hash_mix32(x) & (slots - 1);; h = (h + 1) & (slots - 1)) {
                        const uint32_t k = hkey[h];
                        if (k == x) {
                            lo = hidx[h];
                            break;
                        }
                        if (k == kNoId) break;
                    }
                }
                if (lo < D) {  // the triangle {u, v, x}
                    atomicOr(&rows[(uint64_t)i * wd + (lo >> 5)], 1u << (lo & 31));
                    ++tri;
                    atomicAdd(&t_e[p], 1u);  // (v, x)
                    atomicAdd(&tri_u[i], 1u);
                    atomicAdd(&tri_u[lo], 1u);
                }
            }
        }
        if (GLOBAL) __threadfence();  // the finished rows, before they are read back
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < D; i += THREADS)  // (u, ids[i]): other lowest vertices add here too
            if (tri_u[i]) atomicAdd(&t_e[beg + i], tri_u[i]);
        for (uint32_t i = threadIdx.x; i < D; i += THREADS) {
            const uint32_t *ri = rows + (uint64_t)i * wd;
            for (uint32_t wj = 0; wj < wd; ++wj) {
                uint32_t bits = ri[wj];
                while (bits) {
                    const uint32_t j = wj * 32 + (uint32_t)__builtin_ctz(bits);
                    bits &= bits - 1;
                    const uint32_t *rj = rows + (uint64_t)j * wd;
                    for (uint32_t w = j >> 5; w < wd; ++w) k4 += (unsigned long long)__popc(ri[w] & rj[w]);
                }
            }
        }
        __syncthreads();  // the rows are rebuilt for the next u
    }
    block_add<THREADS>(k4, s_sum, &acc->k4);
    block_add<THREADS>(tri, s_sum, &acc->tri);
}

// The same for vertices of at most 64 forward neighbours, a wave each: a row
// is one 64-bit word, and no barrier is needed.  Four members at a time are
// looked up, 16 lanes walking the forward row of each.  What bounds it is the
// chain of dependent reads per vertex (its offsets, its row, the members'
// offsets, their rows), so many waves run at once (7 KiB of LDS per block of
// four).  A block per vertex, four barriers each, took 2.36 ms on a graph of
// 1e6 vertices and 1e7 edges, where this takes 1.23 ms.
constexpr int kClSlots = 128;  // member hash: at most half full

__global__ __launch_bounds__(kBlock) void k_cliques_wave(const uint32_t *__restrict__ off,
                                                         const uint32_t *__restrict__ col,
                                                         const uint32_t *__restrict__ split, int64_t n,
                                                         const uint32_t *__restrict__ lists, uint32_t count,
                                                         uint32_t *__restrict__ t_e, ExactAcc *acc)
{
    constexpr int kWaves = kBlock / kWave;
    __shared__ uint32_t s_key[kWaves][kClSlots];
    __shared__ uint32_t s_idx[kWaves][kClSlots];
    __shared__ uint32_t s_row[kWaves][kWave][2];
    __shared__ uint32_t s_tri[kWaves][kWave];
    __shared__ unsigned long long s_sum[kWaves];
    const int w = threadIdx.x / kWave, lane = lane_id();
    uint32_t *key = s_key[w], *idx = s_idx[w], *tri_u = s_tri[w];
    uint32_t(*row)[2] = s_row[w];
    const int grp = lane / 16, sub = lane & 15;
    unsigned long long k4 = 0, tri = 0;
    for (uint32_t k = blockIdx.x * kWaves + w; k < count; k += gridDim.x * kWaves) {  // wave-uniform
        const uint32_t u = list_at(lists, n, kCl64, k);
        const uint32_t beg = off[u] + split[u], D = off[u + 1] - beg;  // 2 .. 64
        uint32_t id = 0, vb = 0, ve = 0;
        if (lane < (int)D) {
            id = col[beg + lane];
            vb = off[id] + split[id];
            ve = off[id + 1];
        }
        key[lane] = kNoId;
        key[lane + kWave] = kNoId;
        row[lane][0] = row[lane][1] = 0;
        tri_u[lane] = 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (lane < (int)D)
            for (uint32_t h = hash_mix32(id) & (kClSlots - 1);; h = (h + 1) & (kClSlots - 1))
                if (atomicCAS(&key[h], kNoId, id) == kNoId) {
                    idx[h] = (uint32_t)lane;
                    break;
                }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        for (uint32_t i0 = 0; i0 < D; i0 += kWave / 16) {  // wave-uniform
            const uint32_t i = i0 + grp;
            const uint32_t b0 = __shfl(vb, (int)(i & 63u), kWave), e0 = __shfl(ve, (int)(i & 63u), kWave);
            const uint32_t b = i < D ? b0 : 0u, e = i < D ? e0 : 0u;
            for (uint32_t p = b + sub; p < e; p += 16) {
                const uint32_t x = col[p];
                uint32_t h = hash_mix32(x) & (kClSlots - 1), kk;
                while ((kk = key[h]) != x && kk != kNoId) h = (h + 1) & (kClSlots - 1);
                if (kk == x) {  // the triangle {u, ids[i], x}; x's index is above i
                    const uint32_t j = idx[h];
                    atomicOr(&row[i][j >> 5], 1u << (j & 31));
                    ++tri;
                    atomicAdd(&t_e[p], 1u);
                    atomicAdd(&tri_u[i], 1u);
                    atomicAdd(&tri_u[j], 1u);
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (tri_u[lane]) atomicAdd(&t_e[beg + lane], tri_u[lane]);  // 0 from D on
        const uint32_t r0 = row[lane][0], r1 = row[lane][1];
        uint64_t bits = (uint64_t)r0 | ((uint64_t)r1 << 32);
        while (bits) {
            const int j = __builtin_ctzll(bits);
            bits &= bits - 1;
            k4 += (unsigned long long)(__popc(r0 & row[j][0]) + __popc(r1 & row[j][1]));
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    block_add<kBlock>(k4, s_sum, &acc->k4);
    block_add<kBlock>(tri, s_sum, &acc->tri);
}

// Sums over forward slots: 2 N_3 = sum t_e (d_u + d_v - 4), N_5 = sum C(t_e, 2)
__global__ __launch_bounds__(kBlock) void k_edge_sums(const uint32_t *__restrict__ off,
                                                      const SlotRec *__restrict__ rec,
                                                      const uint32_t *__restrict__ t_e, int64_t slots,
                                                      ExactAcc *acc)
{
    unsigned __int128 n3 = 0, n5 = 0;
    for (int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; s < slots;
         s += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t t = t_e[s];
        if (t == 0) continue;  // and so at every backward slot
        const SlotRec e = rec[s];
        const uint32_t u = e.row;
        const uint64_t du = (uint64_t)(off[u + 1] - off[u]), dv = e.cdeg;
        n3 += (unsigned __int128)t * (du + dv - 4);  // t > 0 means both degrees >= 2
        n5 += (unsigned __int128)(t * (t - 1) / 2);
    }
    n3 = block_sum128<kBlock>(n3);
    n5 = block_sum128<kBlock>(n5);
    if (threadIdx.x == 0) {
        if (n3) add128(&acc->n3_lo, &acc->n3_hi, n3);
        if (n5) add128(&acc->n5_lo, &acc->n5_hi, n5);
    }
}

// 4-cycles by the highest vertex x.  For each lower neighbour w of x and
// each lower neighbour y of w below x, the pair (x, y) gains a wedge; a pair
// with c wedges closes C(c, 2) 4-cycles at x.  Counted per x in an LDS
// open-addressing table of the touched y (the classes whose S bounds the
// distinct y at 3/4 of it), or range of ids by range of ids (below).
constexpr uint32_t kC4Empty = 0xFFFFFFFFu;

template <uint32_t SLOTS>
__device__ __forceinline__ void wedge_add(uint32_t *keys, uint32_t *cnts, uint32_t y)
{
    for (uint32_t h = hash_mix32(y) & (SLOTS - 1);; h = (h + 1) & (SLOTS - 1)) {
        uint32_t k = keys[h];
        if (k == kC4Empty) k = atomicCAS(&keys[h], kC4Empty, y);
        if (k == kC4Empty || k == y) {
            atomicAdd(&cnts[h], 1u);
            return;
        }
    }
}

// A wave per vertex, S <= kC4WaveMax: the rows of 64 lower neighbours at a
// time are walked as one list (an entry's row by a search in their prefix
// lengths), so that short rows leave no lane idle.
__global__ __launch_bounds__(kBlock) void k_c4_wave(const uint32_t *__restrict__ off, const uint32_t *__restrict__ col,
                                                    const uint32_t *__restrict__ split, int64_t n,
                                                    const uint32_t *__restrict__ lists, uint32_t count, ExactAcc *acc)
{
    constexpr int kWaves = kBlock / kWave;
    constexpr uint32_t kSlots = 512;
    __shared__ uint32_t s_key[kWaves][kSlots];
    __shared__ uint32_t s_cnt[kWaves][kSlots];
    __shared__ uint32_t s_pre[kWaves][kWave];  // entries before the neighbour's row
    __shared__ uint32_t s_at[kWaves][kWave];   // its first slot less those
    __shared__ unsigned long long s_sum[kWaves];
    const int w_id = threadIdx.x / kWave, lane = lane_id();
    uint32_t *keys = s_key[w_id], *cnts = s_cnt[w_id], *pre = s_pre[w_id], *at = s_at[w_id];
#pragma unroll
    for (int q = 0; q < (int)kSlots / kWave; ++q) {
        keys[q * kWave + lane] = kC4Empty;
        cnts[q * kWave + lane] = 0;
    }
    unsigned long long n4 = 0;
    for (uint32_t i = blockIdx.x * kWaves + w_id; i < count; i += gridDim.x * kWaves) {  // wave-uniform
        const uint32_t x = list_at(lists, n, kC4Wave, i);
        const uint32_t lo = off[x], D = split[x];
        for (uint32_t base = 0; base < D; base += kWave) {
            const uint32_t j = base + lane;
            uint32_t r0 = 0, len = 0;
            if (j < D) {
                const uint32_t w = col[lo + j];
                r0 = off[w];
                len = off[w + 1] - r0;
            }
            uint32_t incl = len;
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) {
                const uint32_t o = __shfl_up(incl, d, kWave);
                if (lane >= d) incl += o;
            }
            const uint32_t total = __shfl(incl, kWave - 1, kWave);
            pre[lane] = incl - len;
            at[lane] = r0 - (incl - len);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            for (uint32_t e = lane; e < total; e += kWave) {
                uint32_t k = 0;  // the last neighbour with pre[k] <= e (no row is empty)
#pragma unroll
                for (uint32_t step = kWave / 2; step > 0; step >>= 1)
                    if (pre[k + step] <= e) k += step;
                const uint32_t y = col[at[k] + e];
                if (y < x) wedge_add<kSlots>(keys, cnts, y);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
#pragma unroll
        for (int q = 0; q < (int)kSlots / kWave; ++q) {
            const uint64_t c = cnts[q * kWave + lane];
            if (c == 0) continue;
            n4 += c * (c - 1) / 2;
            keys[q * kWave + lane] = kC4Empty;
            cnts[q * kWave + lane] = 0;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    n4 = wave_sum_u64(n4);
    __syncthreads();
    if (lane == 0) s_sum[w_id] = n4;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned __int128 t = 0;
        for (int q = 0; q < kWaves; ++q) t += s_sum[q];
        if (t) add128(&acc->n4_lo, &acc->n4_hi, t);
    }
}

// A block per vertex, 16 lanes walking each lower neighbour's row: classes of
// S <= 3/4 SLOTS.  (A thread's sum stays below 2^64: a vertex adds at most
// C(S, 2) < 2^27.)
template <int THREADS, uint32_t SLOTS>
__global__ __launch_bounds__(THREADS) void k_c4_block(const uint32_t *__restrict__ off,
                                                      const uint32_t *__restrict__ col,
                                                      const uint32_t *__restrict__ split, int64_t n,
                                                      const uint32_t *__restrict__ lists, int cls, uint32_t count,
                                                      ExactAcc *acc)
{
    __shared__ uint32_t keys[SLOTS];
    __shared__ uint32_t cnts[SLOTS];
    __shared__ unsigned long long s_sum[THREADS / kWave];
    const int grp = threadIdx.x / 16, sub = threadIdx.x & 15;
    for (uint32_t h = threadIdx.x; h < SLOTS; h += THREADS) {
        keys[h] = kC4Empty;
        cnts[h] = 0;
    }
    __syncthreads();
    unsigned long long n4 = 0;
    for (uint32_t i = blockIdx.x; i < count; i += gridDim.x) {  // block-uniform
        const uint32_t x = list_at(lists, n, cls, i);
        const uint32_t lo = off[x], D = split[x];
        for (uint32_t j = grp; j < D; j += THREADS / 16) {
            const uint32_t w = col[lo + j], r1 = off[w + 1];
            for (uint32_t q = off[w] + sub; q < r1; q += 16) {
                const uint32_t y = col[q];
                if (y >= x) break;  // rows ascend: the rest are higher too
                wedge_add<SLOTS>(keys, cnts, y);
            }
        }
        __syncthreads();
        for (uint32_t h = threadIdx.x; h < SLOTS; h += THREADS) {
            const uint64_t c = cnts[h];
            if (c == 0) continue;
            n4 += c * (c - 1) / 2;
            keys[h] = kC4Empty;
            cnts[h] = 0;
        }
        __syncthreads();  // the table is clear before the next x
    }
    n4 = wave_sum_u64(n4);
    if (lane_id() == 0) s_sum[threadIdx.x / kWave] = n4;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned __int128 t = 0;
        for (int q = 0; q < THREADS / kWave; ++q) t += s_sum[q];
        if (t) add128(&acc->n4_lo, &acc->n4_hi, t);
    }
}

// A block per vertex x of more wedges than a table holds, most of them to ids
// y reached once (a Chung-Lu graph of 1e6 vertices: 45K wedges to 41K ids):
// a bitmap of one span of ids shows which wedges repeat, and only those are
// counted, in a small table (id in the span << 12 | repeats; a pair's count
// is at most D < 4095).  A y of r repeats has r + 1 wedges, C(r + 1, 2)
// cycles.  A vertex whose table fills joins the last class.
// With it the vertices of 12288 < S <= 60000 took 0.53 ms on Chung-Lu 1e7
// edges, range by range (below) 1.7.
constexpr int kC4BitsThreads = 1024;
constexpr uint32_t kC4BitsSlots = 6144;
constexpr uint32_t kC4BitsFull = kC4BitsSlots * 4 / 5;

__global__ __launch_bounds__(kC4BitsThreads) void k_c4_bits(const uint32_t *__restrict__ off,
                                                            const uint32_t *__restrict__ col,
                                                            const uint32_t *__restrict__ split, int64_t n,
                                                            uint32_t *__restrict__ lists, uint32_t count,
                                                            ExactLists *L, ExactAcc *acc)
{
    __shared__ uint4 s_bits4[kC4Span / 128];
    __shared__ uint32_t s_tab[kC4BitsSlots];
    __shared__ uint32_t s_used;
    __shared__ unsigned long long s_sum[kC4BitsThreads / kWave];
    const int tid = threadIdx.x, grp = tid / 16, sub = tid & 15;
    for (uint32_t j = tid; j < kC4Span / 128; j += kC4BitsThreads) s_bits4[j] = make_uint4(0u, 0u, 0u, 0u);
    for (uint32_t j = tid; j < kC4BitsSlots; j += kC4BitsThreads) s_tab[j] = kC4Empty;
    if (tid == 0) s_used = 0;
    __syncthreads();
    unsigned int *const bits = reinterpret_cast<unsigned int *>(s_bits4);
    // one more repeat of id r0 + o; a full table is noted in s_used
    const auto repeat = [&](uint32_t o) {
        uint32_t h = hash_home(o, kC4BitsSlots);
        for (uint32_t probe = 0; probe < kC4BitsSlots; ++probe) {
            uint32_t k = s_tab[h];
            if (k == kC4Empty) {
                k = atomicCAS(&s_tab[h], kC4Empty, o << 12 | 1u);
                if (k == kC4Empty) {
                    atomicAdd(&s_used, 1u);
                    return;
                }
            }
            if (k >> 12 == o) {
                atomicAdd(&s_tab[h], 1u);
                return;
            }
            h = h + 1 == kC4BitsSlots ? 0u : h + 1;
        }
        atomicAdd(&s_used, kC4BitsSlots);
    };
    unsigned long long n4 = 0;
    for (uint32_t i = blockIdx.x; i < count; i += gridDim.x) {  // block-uniform
        const uint32_t x = list_at(lists, n, kC4Bits, i);
        const uint32_t lo = off[x], D = split[x];
        unsigned long long part = 0;
        bool full = false;
        for (uint32_t r0 = 0; r0 < x && !full; r0 += kC4Span) {  // block-uniform
            const uint32_t E = x - r0 < kC4Span ? x : r0 + kC4Span;
            for (uint32_t j = grp; j < D; j += kC4BitsThreads / 16) {
                if (s_used > kC4BitsFull) break;
                const uint32_t w = col[lo + j], r1 = off[w + 1];
                for (uint32_t q = off[w] + sub; q < r1; q += 16) {
                    const uint32_t y = col[q];
                    if (y >= E) break;  // rows ascend: the rest are higher too
                    if (y < r0) continue;
                    const uint32_t o = y - r0, bit = 1u << (o & 31);
                    if (atomicOr(&bits[o >> 5], bit) & bit) repeat(o);
                }
            }
            __syncthreads();
            full = s_used > kC4BitsFull;
            __syncthreads();  // read by all before it is cleared
            if (tid == 0) s_used = 0;
            for (uint32_t j = tid; j < kC4BitsSlots; j += kC4BitsThreads) {
                const uint32_t k = s_tab[j];
                if (k == kC4Empty) continue;
                const uint64_t r = k & 4095u;
                part += r * (r + 1) / 2;
                s_tab[j] = kC4Empty;
            }
            for (uint32_t j = tid; j < kC4Span / 128; j += kC4BitsThreads) s_bits4[j] = make_uint4(0u, 0u, 0u, 0u);
            __syncthreads();  // clear before the next span
        }
        if (!full)
            n4 += part;
        else if (tid == 0)
            lists[(int64_t)(kC4Ranges / 2) * n + atomicAdd(&L->count[kC4Ranges].n, 1u)] = x;
    }
    n4 = wave_sum_u64(n4);
    if (lane_id() == 0) s_sum[tid / kWave] = n4;
    __syncthreads();
    if (tid == 0) {
        unsigned __int128 t = 0;
        for (int q = 0; q < kC4BitsThreads / kWave; ++q) t += s_sum[q];
        if (t) add128(&acc->n4_lo, &acc->n4_hi, t);
    }
}

// The vertices of the last class, about the highest ids first;
// blocks take the next one from a queue, so the hubs' unequal work spreads
// over the blocks as it comes.  The opposite vertices y < x are
// counted one range of ids at a time in LDS: kC4Range 32-bit counters, or
// twice as many 16-bit ones when x has fewer than 2^16 lower neighbours (a
// pair's count never exceeds them).  Each lower neighbour w of x keeps a
// cursor into its row (rows ascend, so the entries of one range follow
// those of the range before): per range the four lanes that stand for w read
// the cursor and the id it points at (the next w's while this one is walked),
// and walk the row's segment inside the range only when that id lies in it,
// kC4In entries per lane at once.  What bounds it is the latency of those
// reads with one block's 16 waves per CU (the counters fill its LDS).  A lane
// per w, 4 entries at once and long segments queued to whole waves, took
// 2.83 ms on Chung-Lu 1e7 edges (1.5 ms here), 1.30 on R-MAT scale 16 (0.36)
// and 516 on R-MAT scale 22 (289); 4 or 16 entries per lane measured up to 10%
// slower.
constexpr int kC4Threads = 1024;
constexpr uint32_t kC4Range = 40448;  // LDS counters per range (nearly all of a 160 KB LDS)
constexpr int kC4Lanes = 4;           // per lower neighbour
constexpr int kC4In = 8;              // entries of its row that a lane reads at once
constexpr uint32_t kC4Inf = 0xFFFFFFFFu;
static_assert(kC4Range % 4 == 0, "the counters are read 16 bytes at a time");

// state[i] of the i-th lower neighbour w of the current x: {cursor into row
// w, end of row w, id at the cursor (kC4Inf past the end), unused}
__global__ __launch_bounds__(kC4Threads) void k_four_cycles(const uint32_t *__restrict__ off,
                                                            const uint32_t *__restrict__ col,
                                                            const uint32_t *__restrict__ split, int64_t n,
                                                            const uint32_t *__restrict__ lists,
                                                            const ExactLists *__restrict__ L,
                                                            uint4 *__restrict__ state_all, uint64_t cap,
                                                            uint32_t *queue, ExactAcc *acc)
{
    __shared__ __align__(16) uint32_t cnt[kC4Range];
    __shared__ uint32_t s_b;
    uint4 *state = state_all + (uint64_t)blockIdx.x * cap;
    const int tid = threadIdx.x, lane = lane_id();
    const uint32_t sub = tid & (kC4Lanes - 1);
    const uint32_t total = L->count[kC4Ranges].n;
    for (uint32_t i = tid; i < kC4Range; i += kC4Threads) cnt[i] = 0;
    unsigned __int128 n4 = 0;
    for (;;) {
        if (tid == 0) s_b = atomicAdd(queue, 1u);
        __syncthreads();
        const uint32_t b = s_b;
        __syncthreads();  // every thread has read s_b before thread 0 writes it again
        if (b >= total) break;  // block-uniform
        const uint32_t x = list_at(lists, n, kC4Ranges, b);
        const uint32_t lo = off[x], D = split[x];  // N-(x) = col[lo, lo + D)
        for (uint32_t i = tid; i < D; i += kC4Threads) {
            const uint32_t w = col[lo + i], c = off[w], e = off[w + 1];
            state[i] = make_uint4(c, e, c < e ? col[c] : kC4Inf, 0u);
        }
        // a pair's count is at most D: below 2^16, two 16-bit counters share a
        // word and a range spans twice the ids
        const bool half = D < 65536u;
        const uint32_t span = half ? 2 * kC4Range : kC4Range;
        const auto bump = [&](uint32_t y, uint32_t r0) {
            const uint32_t o = y - r0;
            if (half)
                atomicAdd(&cnt[o >> 1], 1u << ((o & 1u) << 4));
            else
                atomicAdd(&cnt[o], 1u);
        };
        __syncthreads();  // the state and the cleared counters are in place
        for (uint32_t r0 = 0; r0 < x; r0 += span) {
            const uint32_t E = x - r0 < span ? x : r0 + span;  // this range: ids [r0, E)
            uint4 st = make_uint4(0u, 0u, kC4Inf, 0u);
            uint32_t i = (uint32_t)tid / kC4Lanes;
            if (i < D) st = state[i];
            for (; i < D; i += kC4Threads / kC4Lanes) {
                uint4 ahead = make_uint4(0u, 0u, kC4Inf, 0u);
                if (i + kC4Threads / kC4Lanes < D) ahead = state[i + kC4Threads / kC4Lanes];
                if (st.z < E) {
                    uint32_t p = st.x, nxt, in;
                    do {
                        uint32_t v[kC4In];
#pragma unroll
                        for (int j = 0; j < kC4In; ++j) {
                            const uint32_t q = p + j * kC4Lanes + sub;
                            v[j] = q < st.y ? col[q] : kC4Inf;
                        }
                        // the entries in the range are the first ones read
                        // (rows ascend), the smallest other one is the next
                        in = 0;
                        nxt = kC4Inf;
#pragma unroll
                        for (int j = 0; j < kC4In; ++j) {
                            if (v[j] < E) {
                                bump(v[j], r0);
                                ++in;
                            } else {
                                nxt = v[j] < nxt ? v[j] : nxt;
                            }
                        }
#pragma unroll
                        for (int o = kC4Lanes / 2; o > 0; o >>= 1) {
                            in += __shfl_xor(in, o, kC4Lanes);
                            const uint32_t other = __shfl_xor(nxt, o, kC4Lanes);
                            nxt = other < nxt ? other : nxt;
                        }
                        p += in;
                    } while (in == kC4Lanes * kC4In);  // the same in the four lanes
                    if (sub == 0) state[i] = make_uint4(p, st.y, nxt, 0u);
                }
                st = ahead;
            }
            __syncthreads();
            // whole 16-byte words of the counters (kC4Range is a multiple of 4
            // words); a range's sum per thread: below 2^32 words of 2^63
            const uint32_t words = half ? (E - r0 + 1) / 2 : E - r0;
            unsigned __int128 part = 0;
            for (uint32_t j = tid * 4; j < words; j += kC4Threads * 4) {
                const uint4 wv = *reinterpret_cast<const uint4 *>(cnt + j);
                if ((wv.x | wv.y | wv.z | wv.w) == 0) continue;
                const uint32_t v4[4] = {wv.x, wv.y, wv.z, wv.w};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (half) {  // two products below 2^31
                        const uint32_t c0 = v4[q] & 0xFFFFu, c1 = v4[q] >> 16;
                        part += (uint64_t)(c0 * (c0 - 1) / 2) + (uint64_t)(c1 * (c1 - 1) / 2);
                    } else {
                        const uint64_t c = v4[q];
                        part += c * (c - 1) / 2;
                    }
                }
                *reinterpret_cast<uint4 *>(cnt + j) = make_uint4(0u, 0u, 0u, 0u);
            }
            n4 += part;
            // at the loop's end: at its head the compiler leaves out the wait
            // for the stores above
            __syncthreads();
        }
    }
    n4 = wave_sum128(n4);
    if (lane == 0 && n4) add128(&acc->n4_lo, &acc->n4_hi, n4);
}

}  // namespace

pm_status exact_counts(const pm_graph *g, pm_exact *out, hipStream_t s)
{
    if (!g || !out) {
        set_error("exact_counts: null argument");
        return PM_EINVAL;
    }
    PM_TRY(check_device(g));
    std::memset(out, 0, sizeof(*out));
    const int64_t n = g->n, slots = g->slots;
    Temps tmp(s);
    ExactAcc *acc = nullptr;
    PM_TRY(tmp.get(&acc, 1));
    PM_TRY(fill_async<unsigned char>((unsigned char *)acc, 0, (int64_t)sizeof(ExactAcc), s));
    ProfScope prof_total("exact_total", s);
    if (slots > 0) {
        uint32_t *split = nullptr, *t_e = nullptr, *lists = nullptr;
        ExactLists *L = nullptr, hl;
        PM_TRY(tmp.get(&split, (size_t)n));
        PM_TRY(tmp.get(&t_e, (size_t)slots));
        PM_TRY(tmp.get(&lists, (size_t)n * kExactArrays));
        PM_TRY(tmp.get(&L, 1));
        PM_TRY(fill_async<uint32_t>((uint32_t *)L, 0u, sizeof(ExactLists) / 4, s));
        {
            ProfScope prof("exact.classify", s);
            hipLaunchKernelGGL(k_classify, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, g->off,
                               g->col, n, split, lists, L);
            PM_HIP(hipGetLastError());
        }
        PM_HIP(hipMemcpyAsync(&hl, L, sizeof(hl), hipMemcpyDeviceToHost, s));
        PM_TRY(fill_async<uint32_t>(t_e, 0u, slots, s));
        PM_HIP(hipStreamSynchronize(s));
        const unsigned cus = (unsigned)sampler_cu_count(g->device);
        const auto blocks_for = [&](int c, unsigned per_block, unsigned cap) {
            return dim3(std::min<unsigned>((hl.count[c].n + per_block - 1) / per_block, cap));
        };
        {
            // triangles (with t_e) and 4-cliques by forward degree class:
            // rows in LDS up to 1024 members, in a global slice per block above
            ProfScope prof("exact.triangles_cliques", s);
            if (hl.count[kCl64].n) {
                ProfScope pc("exact.cliques.64", s);
                hipLaunchKernelGGL(k_cliques_wave, blocks_for(kCl64, kBlock / kWave, cus * 8), dim3(kBlock), 0, s,
                                   g->off, g->col, split, n, lists, hl.count[kCl64].n, t_e, acc);
            }
            if (hl.count[kCl256].n) {
                ProfScope pc("exact.cliques.256", s);
                hipLaunchKernelGGL((k_cliques<8, false, kBlock>), blocks_for(kCl256, 1, cus * 8), dim3(kBlock), 0, s,
                                   g->off, g->col, split, n, lists, kCl256, hl.count[kCl256].n, 256u, nullptr, 0u,
                                   t_e, acc);
            }
            if (hl.count[kCl1024].n) {
                ProfScope pc("exact.cliques.1024", s);
                hipLaunchKernelGGL((k_cliques<32, false, 1024>), blocks_for(kCl1024, 1, 8192), dim3(1024), 0, s,
                                   g->off, g->col, split, n, lists, kCl1024, hl.count[kCl1024].n, 1024u, nullptr, 0u,
                                   t_e, acc);
            }
            if (hl.count[kClMore].n) {
                ProfScope pc("exact.cliques.global", s);
                const uint32_t dmax = hl.dmax.n, wd = (dmax + 31) / 32;
                const uint64_t slice = ((uint64_t)dmax * wd + 2ull * dmax) * sizeof(uint32_t);
                // blocks with a slice each, at most 1 GiB of slices
                const unsigned gb = (unsigned)std::max<uint64_t>(1, std::min<uint64_t>(256, (1ull << 30) / slice));
                uint32_t *scr = nullptr;
                PM_TRY(tmp.get(&scr, (size_t)gb * ((size_t)dmax * wd + 2ull * dmax)));
                // ids, counters and the member hash in LDS when they fit in 64 KB
                uint32_t gslots = 1;
                while (gslots < 2 * dmax) gslots <<= 1;
                const size_t dyn = (2ull * dmax + gslots) * sizeof(uint32_t) + gslots * sizeof(uint16_t);
                const bool in_lds = dmax < 65536 && dyn <= (64u << 10);
                hipLaunchKernelGGL((k_cliques<1, true, 1024>), blocks_for(kClMore, 1, gb), dim3(1024),
                                   in_lds ? dyn : 0, s, g->off, g->col, split, n, lists, kClMore,
                                   hl.count[kClMore].n, dmax, scr, in_lds ? gslots : 0u, t_e, acc);
            }
            hipLaunchKernelGGL(k_edge_sums, dim3(grid_for(slots, kBlock, 1024)), dim3(kBlock), 0, s, g->off, g->rec,
                               t_e, slots, acc);
            PM_HIP(hipGetLastError());
            tmp.release(t_e);
        }
        // 4-cycles: by the class's table, or range by range in LDS
        ProfScope prof("exact.four_cycles", s);
        if (hl.count[kC4Bits].n) {
            ProfScope pc("exact.four_cycles.bits", s);
            hipLaunchKernelGGL(k_c4_bits, blocks_for(kC4Bits, 1, cus), dim3(kC4BitsThreads), 0, s, g->off, g->col,
                               split, n, lists, hl.count[kC4Bits].n, L, acc);
        }
        if (hl.count[kC4Ranges].n + hl.count[kC4Bits].n) {  // and those whose repeats filled their table
            ProfScope pc("exact.four_cycles.ranges", s);
            // one cursor state (16 bytes) per lower neighbour of the block's
            // current vertex: at most dmax, within a 4 GiB budget of blocks
            const uint64_t cap = (uint64_t)std::max<int64_t>(g->dmax, 1);
            const unsigned blocks = (unsigned)std::max<uint64_t>(
                1, std::min<uint64_t>(std::min<uint64_t>(256, (uint64_t)hl.count[kC4Ranges].n + hl.count[kC4Bits].n),
                                      (4ull << 30) / (cap * sizeof(uint4))));
            uint4 *state = nullptr;
            uint32_t *queue = nullptr;
            PM_TRY(tmp.get(&state, (size_t)blocks * (size_t)cap));
            PM_TRY(tmp.get(&queue, 1));
            PM_TRY(fill_async<uint32_t>(queue, 0u, 1, s));
            hipLaunchKernelGGL(k_four_cycles, dim3(blocks), dim3(kC4Threads), 0, s, g->off, g->col, split, n, lists, L,
                               state, cap, queue, acc);
        }
        if (hl.count[kC4Big].n) {
            ProfScope pc("exact.four_cycles.16384", s);
            hipLaunchKernelGGL((k_c4_block<1024, 16384>), blocks_for(kC4Big, 1, cus), dim3(1024), 0, s, g->off, g->col,
                               split, n, lists, kC4Big, hl.count[kC4Big].n, acc);
        }
        if (hl.count[kC4Block].n) {
            ProfScope pc("exact.four_cycles.4096", s);
            hipLaunchKernelGGL((k_c4_block<kBlock, 4096>), blocks_for(kC4Block, 1, cus * 4), dim3(kBlock), 0, s, g->off,
                               g->col, split, n, lists, kC4Block, hl.count[kC4Block].n, acc);
        }
        if (hl.count[kC4Wave].n) {
            ProfScope pc("exact.four_cycles.512", s);
            hipLaunchKernelGGL(k_c4_wave, blocks_for(kC4Wave, kBlock / kWave, cus * 8), dim3(kBlock), 0, s, g->off,
                               g->col, split, n, lists, hl.count[kC4Wave].n, acc);
        }
        PM_HIP(hipGetLastError());
    }
    ExactAcc h;
    PM_HIP(hipMemcpyAsync(&h, acc, sizeof(h), hipMemcpyDeviceToHost, s));
    PM_HIP(hipStreamSynchronize(s));

    typedef __int128 i128;
    typedef unsigned __int128 u128;
    const u128 n3x2 = (u128)h.n3_lo | ((u128)h.n3_hi << 64);
    const u128 n5 = (u128)h.n5_lo | ((u128)h.n5_hi << 64);
    const u128 n4 = (u128)h.n4_lo | ((u128)h.n4_hi << 64);
    const i128 N1 = (i128)g->N1, N2 = (i128)(g->R_tau / 2) - 3 * (i128)h.tri, N3 = (i128)(n3x2 / 2),
               N4 = (i128)n4, N5 = (i128)n5, N6 = (i128)h.k4;
    // Eq. 1 (N = A C) is upper triangular with unit diagonal; entry (i, j) is
    // the number of copies of motif i inside motif j
    const i128 c6 = N6;
    const i128 c5 = N5 - 6 * c6;
    const i128 c4 = N4 - c5 - 3 * c6;
    const i128 c3 = N3 - 4 * c5 - 12 * c6;
    const i128 c2 = N2 - 2 * c3 - 4 * c4 - 6 * c5 - 12 * c6;
    const i128 c1 = N1 - c3 - 2 * c5 - 4 * c6;
    const i128 Ns[7] = {0, N1, N2, N3, N4, N5, N6};
    const i128 Cs[7] = {0, c1, c2, c3, c4, c5, c6};
    for (int i = 1; i <= 6; ++i) {
        if (Cs[i] < 0 || Cs[i] >= ((i128)1 << 64) || Ns[i] < 0 || Ns[i] >= ((i128)1 << 64)) {
            set_error("exact_counts: a count does not fit in 64 bits");
            return PM_EOVERFLOW;
        }
        out->C[i] = (uint64_t)Cs[i];
        out->N[i] = (uint64_t)Ns[i];
    }
    out->triangles = h.tri;
    return PM_OK;
}

}  // namespace pm
