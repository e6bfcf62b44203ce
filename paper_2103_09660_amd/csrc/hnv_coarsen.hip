// Coarsening of one level on the GPU (Section 3.1, Algorithm 1).  The
// featureless form has the same reading as the host coarsening in
// hnv_host.cpp and the same maps bit for bit:
//   1. every hyperedge gets a rank in the order (weight descending, size
//      ascending, id ascending): a stable counting sort of the sizes, then, with
//      weights, a stable radix sort of that order by the inverted weight bits;
//   2. a node's choice c(v) is its incident hyperedge of least rank: an
//      atomic minimum, which does not depend on the order of the updates;
//   3. a group's coarse id follows its smallest node: a node starts a group
//      if it has no hyperedge or is the smallest node that chose c(v); an
//      exclusive scan over those flags numbers the groups in node order;
//   4. the coarse member lists: every member mapped through rep(), sorted and
//      made distinct by the thread, wavefront or workgroup that read it; a
//      hyperedge is removed iff its list is one node whose group chose it;
//   5. one scan over the hyperedges' counts of distinct members and of kept
//      hyperedges gives the offsets and numbers, and the lists are copied there.
// The passes over incidences walk windows of hyperedges with all lanes
// (walk_window), so none needs an incidence -> hyperedge map in memory.
// Integer work only (the key compares FP32 weights through their bit
// patterns, which order like the values for positive finite floats).
//
// With node features (bag-of-words counts), step 2 instead takes, per node,
// the hyperedge of largest cosine between the hyperedge feature (the mean of
// its members' rows) and the node's row, equal scores going to the least
// rank of step 1; the coarse node's row is the sum of its fine nodes' rows.
// The member sums, the dot products and the squared norms are exact
// integers, and the score d|d|/|s_e|^2 is one IEEE FP64 product and one
// quotient, so the choice does not depend on summation order.
#include <hip/hip_runtime.h>

#include "hnv_binsort.h"
#include "hnv_prim.h"

#include <climits>
#include <string>

#include "hnv_grid.h"
#include "hnv_internal.h"
#include "hnv_level_check.h"

namespace hnv {
namespace {

// The order of the hyperedges: by size first, then (with weights) a stable
// radix sort of that order by the complemented weight bits: weight descending,
// size ascending, id ascending.  The size order is a stable counting sort
// (sizes of kSizeBins - 1 members and more share the last bin, which k_big_rank
// puts in order), whose digit offsets also tell where each size begins: the
// passes over longer member lists take them from there.  A level that can hold
// more than kBigMax hyperedges of the last bin (by its incidences) sorts the
// sizes by radix instead.  (As one radix sort of 64-bit keys of weight and
// size: 119 us for the 1.5M sizes, where this takes 60.)
constexpr int kSizeBins = kBinsMax;
constexpr int64_t kBigMax = 1 << 15;

inline int64_t max_last_bin(int64_t n_nodes, int64_t nnz)
{
    return n_nodes < kSizeBins - 1 ? 0 : nnz / (kSizeBins - 1);
}

// The last bin's hyperedges, in id order at the end of `order` (offs: the
// scanned digit counts; the last bin's start is its first tile's): each one's
// place among them by (size, id), counted against all of them, into tmp
// (place -> hyperedge) and, when there are no weights, rank.  At most kBigMax
// hyperedges, a few hundred as a rule.
__global__ __launch_bounds__(kThreads) void k_big_rank(const int32_t *__restrict__ ptr,
                                                       const int32_t *__restrict__ order,
                                                       const int32_t *__restrict__ offs, int64_t n_tiles,
                                                       int64_t n_edges, int32_t *__restrict__ tmp,
                                                       int32_t *__restrict__ rank, const int *__restrict__ bad)
{
    if (*bad)   // the last bin may hold more than the grid's bound then
        return;
    const int64_t start = offs[(int64_t)(kSizeBins - 1) * n_tiles];
    const int64_t n = n_edges - start, i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if ((int64_t)blockIdx.x * kThreads >= n)
        return;
    __shared__ __align__(16) int32_t sizes[kThreads];
    const int32_t e = i < n ? order[start + i] : 0;
    const int32_t size = i < n ? ptr[e + 1] - ptr[e] : 0;
    int32_t place = 0;
    for (int64_t t = 0; t < n; t += kThreads) {
        __syncthreads();
        int32_t s = INT_MAX;   // past the end: before nothing
        if (t + threadIdx.x < n) {
            const int32_t f = order[start + t + threadIdx.x];
            s = ptr[f + 1] - ptr[f];
        }
        sizes[threadIdx.x] = s;
        __syncthreads();
        const int32_t equal_until = (int32_t)min<int64_t>(max<int64_t>(i - t, 0), kThreads);
#pragma unroll 8
        for (int c = 0; c < kThreads; c += 4) {
            const int4 x = *reinterpret_cast<const int4 *>(sizes + c);
            place += x.x < size + (c < equal_until);
            place += x.y < size + (c + 1 < equal_until);
            place += x.z < size + (c + 2 < equal_until);
            place += x.w < size + (c + 3 < equal_until);
        }
    }
    if (i < n) {
        tmp[place] = e;
        if (rank)
            rank[e] = (int32_t)(start + place);
    }
}

__global__ __launch_bounds__(kThreads) void k_big_order(const int32_t *__restrict__ tmp,
                                                        const int32_t *__restrict__ offs, int64_t n_tiles,
                                                        int64_t n_edges, int32_t *__restrict__ order,
                                                        const int *__restrict__ bad)
{
    if (*bad)
        return;
    const int64_t start = offs[(int64_t)(kSizeBins - 1) * n_tiles];
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n_edges - start)
        order[start + i] = tmp[i];
}

// key of the i-th hyperedge in size order: its complemented weight bits (the
// sign bit of a valid weight is clear, so the lower 31 decide)
__global__ __launch_bounds__(kThreads) void k_weight_keys(const int32_t *__restrict__ order,
                                                          const float *__restrict__ w, int64_t n_edges,
                                                          uint32_t *__restrict__ keys)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n_edges)
        keys[i] = ~__float_as_uint(w[order[i]]);
}

// each hyperedge's size (at most n_nodes) and id, for the radix sort of sizes
__global__ __launch_bounds__(kThreads) void k_size_keys(const int32_t *__restrict__ ptr, int64_t n_edges,
                                                        uint32_t *__restrict__ keys, int32_t *__restrict__ ids)
{
    const int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (e >= n_edges)
        return;
    keys[e] = (uint32_t)(ptr[e + 1] - ptr[e]);
    ids[e] = (int32_t)e;
}

// rank[order[i]] = i
__global__ __launch_bounds__(kThreads) void k_rank(const int32_t *__restrict__ order, int64_t n_edges,
                                                   int32_t *__restrict__ rank)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n_edges)
        rank[order[i]] = (int32_t)i;
}

// best[v] = least rank over the hyperedges containing v
__global__ __launch_bounds__(kThreads) void k_best(const int32_t *__restrict__ ptr, const int32_t *__restrict__ idx,
                                                   const int32_t *__restrict__ rank, int per, int64_t n_edges, int64_t nnz,
                                                   int32_t *__restrict__ best, const int *__restrict__ bad)
{
    __shared__ WalkLds lds;
    const int64_t e0 = window_start(per);
    if (*bad || e0 >= n_edges)   // the step's input failed its checks
        return;
    const int64_t e = e0 + threadIdx.x % kWave;
    const int32_t r = threadIdx.x % kWave < per && e < n_edges ? rank[e] : 0;
    // The minimum only decreases, so any value read earlier (even a stale
    // cached one) bounds the final one from above: a rank not below it
    // cannot win and needs no atomic.
    walk_window<kWalk>(
        window_of(ptr, e0, per, n_edges, nnz), lds, [&](uint32_t j, int, bool ok) { return ok ? idx[j] : -1; },
        [&](uint32_t, int l, bool ok, bool, int32_t v) {
            const int32_t lr = __shfl(r, l, kWave);
            if (ok && lr < best[v])
                atomicMin(best + v, lr);
        });
}

// The same minima without global atomics, for large levels: the incidences'
// (node, rank) pairs are partitioned by the node's high bits (one stable radix
// pass, node >> shift), then one workgroup per bucket of 2^shift nodes takes
// the minima in LDS and writes the bucket's best[] once.  A bucket's chain of
// loads bounds it (the hubs of coarse levels lie in the first buckets), so eight
// are in flight per thread, and a rank that cannot win skips the LDS atomic: with
// one at a time the 2M-node hierarchy takes 4.91 ms where this takes 4.74, the
// whole method at 700K nodes 11.97 and 11.73.  With
// k_best's global atomics up to 2^23 incidences instead of 2^20 it takes 12.12.
constexpr int kBucketShiftMax = 13;   // 8192 nodes, 32 KB of LDS per bucket
constexpr int kBucketThreads = 1024;

bool bucketed_best(int64_t n_nodes, int64_t nnz) { return nnz >= (int64_t(1) << 20) && bits_for(n_nodes) > 8; }

int bucket_shift(int64_t n_nodes) { return std::min(bits_for(n_nodes) - 8, kBucketShiftMax); }

int64_t bucket_count(int64_t n_nodes) { return ((n_nodes - 1) >> bucket_shift(n_nodes)) + 1; }

// the hyperedge rank of every incidence
__global__ __launch_bounds__(kThreads) void k_inc_rank(const int32_t *__restrict__ ptr,
                                                       const int32_t *__restrict__ rank, int per, int64_t n_edges,
                                                       int64_t nnz, int32_t *__restrict__ out, const int *__restrict__ bad)
{
    __shared__ WalkLds lds;
    const int64_t e0 = window_start(per);
    if (*bad || e0 >= n_edges)   // the step's input failed its checks
        return;
    const int64_t e = e0 + threadIdx.x % kWave;
    const int32_t r = threadIdx.x % kWave < per && e < n_edges ? rank[e] : 0;
    walk_window<kWalk>(
        window_of(ptr, e0, per, n_edges, nnz), lds, [&](uint32_t, int l, bool) { return __shfl(r, l, kWave); },
        [&](uint32_t j, int, bool ok, bool, int32_t lr) {
            if (ok)
                out[j] = lr;
        });
}

// start[b] = the first position of bucket b in node ids sorted on their bits
// from `shift` up (b in [0, n_buckets]; start[n_buckets] = n)
__global__ __launch_bounds__(kThreads) void k_bucket_starts(const uint32_t *__restrict__ keys, int64_t n,
                                                            int shift, int64_t n_buckets,
                                                            int64_t *__restrict__ start)
{
    const int64_t b = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (b > n_buckets)
        return;
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = (lo + hi) / 2;
        if ((int64_t)(keys[mid] >> shift) < b)
            lo = mid + 1;
        else
            hi = mid;
    }
    start[b] = lo;
}

__global__ __launch_bounds__(kBucketThreads) void k_bucket_min(const uint32_t *__restrict__ keys,
                                                               const int32_t *__restrict__ vals,
                                                               const int64_t *__restrict__ start, int shift,
                                                               int64_t n_nodes, int32_t *__restrict__ best,
                                                               const int *__restrict__ bad)
{
    __shared__ int32_t m[1 << kBucketShiftMax];
    const int span = 1 << shift;
    const int64_t base = (int64_t)blockIdx.x << shift;
    for (int t = threadIdx.x; t < span; t += kBucketThreads)
        m[t] = INT_MAX;
    __syncthreads();
    // (no incidences of a step whose input failed its checks)
    const int64_t a = start[blockIdx.x], b = *bad ? a : start[blockIdx.x + 1];
    constexpr int U = 8;   // loads in flight
    for (int64_t i = a + threadIdx.x; i < b; i += U * kBucketThreads) {
        int32_t at[U], x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t j = i + u * kBucketThreads < b ? i + u * kBucketThreads : i;
            at[u] = (int32_t)((int64_t)keys[j] - base);
            x[u] = vals[j];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (x[u] < m[at[u]])   // (an earlier read bounds the minimum from above)
                atomicMin(&m[at[u]], x[u]);
    }
    __syncthreads();
    for (int t = threadIdx.x; t < span && base + t < n_nodes; t += kBucketThreads)
        best[base + t] = m[t];
}

// choice, and per hyperedge the smallest node that chose it
__global__ __launch_bounds__(kThreads) void k_choice(const int32_t *__restrict__ best,
                                                     const int32_t *__restrict__ order, int64_t n_nodes,
                                                     int32_t *__restrict__ choice, int32_t *__restrict__ first)
{
    const int64_t v = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (v >= n_nodes)
        return;
    const int32_t b = best[v];
    const int32_t c = (b == INT_MAX) ? -1 : order[b];
    choice[v] = c;
    if (c >= 0 && (int32_t)v < first[c])   // an earlier read bounds the minimum from above
        atomicMin(first + c, (int32_t)v);
}

__global__ __launch_bounds__(kThreads) void k_group_flags(const int32_t *__restrict__ choice,
                                                          const int32_t *__restrict__ first, int64_t n_nodes,
                                                          int32_t *__restrict__ flag)
{
    const int64_t v = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (v >= n_nodes)
        return;
    const int32_t c = choice[v];
    flag[v] = (c < 0 || first[c] == (int32_t)v) ? 1 : 0;
}

__global__ __launch_bounds__(kThreads) void k_node_rep(const int32_t *__restrict__ choice,
                                                       const int32_t *__restrict__ first,
                                                       const int32_t *__restrict__ gid, int64_t n_nodes,
                                                       int32_t *__restrict__ node_rep, int64_t *__restrict__ sizes,
                                                       const int *__restrict__ bad)
{
    if (*bad)   // the step's input failed its checks
        return;
    const int64_t v = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (v >= n_nodes)
        return;
    const int32_t c = choice[v];
    node_rep[v] = (c < 0) ? gid[v] : gid[first[c]];
    if (v == n_nodes - 1)   // the coarse nodes: the groups before v and, when v starts one, v's
        sizes[0] = gid[v] + (c < 0 || first[c] == (int32_t)v ? 1 : 0);
}

// ---------------------------------------------------------------------------
// Coarse member lists.  A hyperedge's members are mapped through rep(), sorted
// and their distinct values written to the start of its segment, all by the
// thread, wavefront or workgroup that read them: lists of at most kSortThread
// members by one thread in registers (a network of 8, or of 16 above 8
// members); of at most kSortMid by one wavefront (a bitonic network over 64
// lanes x up to 4 registers); of at most kSortLong by a workgroup's registers
// and of at most kSortBlock by a workgroup in LDS; the few longer ones (none in most hypergraphs) by the library's segmented sort
// over a list of them.  Each list's result is the same whatever order the
// lists are taken in.  Bound by the random 4-byte reads of rep(); as separate
// passes (map, sort, distinct flags, kept flags) a step of the 2M-node
// hypergraph took 255 us here, and a scan and an emit of 13M flags after it,
// where this takes 155 us and a scan of 1.5M counts.
//
// A hyperedge is removed iff every member chose it.  Then all members lie in
// one group, so its list has one value; and members of one group made the same
// choice, so it is enough that the first member's choice is this hyperedge:
// its best rank is the hyperedge's own.
// ---------------------------------------------------------------------------

constexpr int kSortThread = 16;
constexpr int kSortMid = 256;
constexpr int kSortLong = 2048;
constexpr int kSortBlock = 32768;
constexpr int kSortBlockThreads = 1024;

// per hyperedge: distinct coarse members (0 when removed) and whether it is kept
struct EdgeCount {
    int32_t members, kept;
};
struct EdgeCountPlus {
    __host__ __device__ EdgeCount operator()(const EdgeCount &x, const EdgeCount &y) const
    {
        return EdgeCount{x.members + y.members, x.kept + y.kept};
    }
};

__device__ __forceinline__ EdgeCount edge_count(int32_t distinct, bool first_chose_it)
{
    return distinct == 1 && first_chose_it ? EdgeCount{0, 0} : EdgeCount{distinct, 1};
}

// The hyperedges of at least `size` members (at most kSizeBins - 1) are the
// entries [first_of(..), n_edges) of the size order.
struct SizeOrder {
    const int32_t *by_size;   // [n_edges]
    const int32_t *offs;      // scanned size counts, size b of tile t at b * n_tiles + t
    int64_t n_tiles, n_edges;
    __device__ int64_t first_of(int size) const { return offs[size * n_tiles]; }
};

// Bitonic sorting network over the N registers of one thread (N a power of
// two; every index is a compile-time constant).
template <int N>
__device__ __forceinline__ void thread_bitonic(int32_t (&v)[N])
{
#pragma unroll
    for (int k = 2; k <= N; k <<= 1) {
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int l = i ^ j;
                if (l > i) {
                    const int32_t a = v[i], b = v[l];
                    const bool up = (i & k) == 0;
                    v[i] = up ? min(a, b) : max(a, b);
                    v[l] = up ? max(a, b) : min(a, b);
                }
            }
        }
    }
}

// Sorts the N mapped members of a thread's list (n of them, INT_MAX past the
// end, which is above every coarse node) and writes the distinct ones to out.
template <int N, typename Sort>
__device__ __forceinline__ int32_t thread_list(const int32_t *__restrict__ idx, const int32_t *__restrict__ node_rep,
                                               int32_t s, int32_t n, int32_t *__restrict__ out, Sort sort)
{
    int32_t v[N];
#pragma unroll
    for (int i = 0; i < N; ++i)
        v[i] = (i < n) ? idx[s + i] : -1;
#pragma unroll
    for (int i = 0; i < N; ++i)
        v[i] = (i < n) ? node_rep[v[i]] : INT_MAX;
    sort(v);
    int32_t c = 0;
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (i < n && (i == 0 || v[i] != v[i - 1]))
            out[s + c++] = v[i];
    return c;
}

// One thread per hyperedge: a list of at most 8 members is sorted here with
// Batcher's odd-even merge network of 19 comparators, one of 9 to
// kSortThread members with a bitonic network of 16.  Longer lists are left to
// the kernels below.
__global__ __launch_bounds__(kThreads) void k_list_short(const int32_t *__restrict__ ptr,
                                                         const int32_t *__restrict__ idx,
                                                         const int32_t *__restrict__ node_rep,
                                                         const int32_t *__restrict__ best,
                                                         const int32_t *__restrict__ rank, int64_t n_edges,
                                                         int32_t *__restrict__ out, EdgeCount *__restrict__ count,
                                                         const int *__restrict__ bad)
{
    const int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (*bad || e >= n_edges)   // the step's input failed its checks
        return;
    const int32_t s = ptr[e], n = ptr[e + 1] - s;
    if (n <= kSortThread) {
        const bool chose = best[idx[s]] == rank[e];
        int32_t c;
        if (n <= 8)
            c = thread_list<8>(idx, node_rep, s, n, out, [](int32_t(&v)[8]) {
                constexpr int net[19][2] = {{0, 1}, {2, 3}, {4, 5}, {6, 7}, {0, 2}, {1, 3}, {4, 6}, {5, 7}, {1, 2}, {5, 6},
                                            {0, 4}, {3, 7}, {1, 5}, {2, 6}, {1, 4}, {3, 6}, {2, 4}, {3, 5}, {3, 4}};
#pragma unroll
                for (int i = 0; i < 19; ++i) {
                    const int32_t x = v[net[i][0]], y = v[net[i][1]];
                    v[net[i][0]] = min(x, y);
                    v[net[i][1]] = max(x, y);
                }
            });
        else
            c = thread_list<16>(idx, node_rep, s, n, out, [](int32_t(&v)[16]) { thread_bitonic<16>(v); });
        count[e] = edge_count(c, chose);
    }
}

// Compare step of lane i's key x with lane i ^ X's: the smaller one where the
// lane's bit of the distance is clear, the larger one elsewhere.  All on the
// vector unit: with every exchange through the LDS crossbar the sorts of 2,048
// keys took 132 us at the 2M-node level instead of 72.  A row is 16 lanes.
template <int X>
__device__ __forceinline__ int32_t row_xor(int32_t x)   // lane ^ X within a row
{
    if constexpr (X == 1)
        return __builtin_amdgcn_mov_dpp(x, 0xB1, 0xf, 0xf, false);    // quad_perm [1, 0, 3, 2]
    else if constexpr (X == 2)
        return __builtin_amdgcn_mov_dpp(x, 0x4E, 0xf, 0xf, false);    // quad_perm [2, 3, 0, 1]
    else if constexpr (X == 3)
        return __builtin_amdgcn_mov_dpp(x, 0x1B, 0xf, 0xf, false);    // quad_perm [3, 2, 1, 0]
    else if constexpr (X == 4) {
        const int32_t up = __builtin_amdgcn_update_dpp(x, x, 0x104, 0xf, 0x5, false);   // row_shl 4 into quads 0, 2
        return __builtin_amdgcn_update_dpp(up, x, 0x114, 0xf, 0xa, false);              // row_shr 4 into quads 1, 3
    } else if constexpr (X == 7)
        return __builtin_amdgcn_mov_dpp(x, 0x141, 0xf, 0xf, false);   // row_half_mirror
    else if constexpr (X == 8)
        return __builtin_amdgcn_mov_dpp(x, 0x128, 0xf, 0xf, false);   // row_ror 8
    else
        return __builtin_amdgcn_mov_dpp(x, 0x140, 0xf, 0xf, false);   // row_mirror (15)
}

// Both keys of the pair of lanes i and i ^ 16 (and i ^ 32), in either order.
__device__ __forceinline__ void pair16(int32_t x, int32_t &a, int32_t &b)
{
    const auto p = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    a = (int32_t)p[0];
    b = (int32_t)p[1];
}
__device__ __forceinline__ void pair32(int32_t x, int32_t &a, int32_t &b)
{
    const auto p = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    a = (int32_t)p[0];
    b = (int32_t)p[1];
}

// lane ^ 31's and lane ^ 63's key
__device__ __forceinline__ int32_t mirror32(int32_t x, int lane)
{
    int32_t a, b;
    pair16(row_xor<15>(x), a, b);
    return (lane & 16) ? a : b;
}
__device__ __forceinline__ int32_t mirror64(int32_t x, int lane)
{
    int32_t a, b;
    pair32(mirror32(x, lane), a, b);
    return (lane & 32) ? a : b;
}

template <int K, int X>
__device__ __forceinline__ void lane_step(int32_t (&v)[K], int lane)
{
    constexpr int bit = X == 1 ? 1 : X <= 3 ? 2 : X <= 7 ? 4 : X <= 15 ? 8 : X <= 31 ? 16 : 32;
    const bool low = (lane & bit) == 0;
#pragma unroll
    for (int r = 0; r < K; ++r) {
        int32_t a = v[r], b;
        if constexpr (X < 16)
            b = row_xor<X>(a);
        else if constexpr (X == 16)
            pair16(v[r], a, b);
        else if constexpr (X == 31)
            b = mirror32(a, lane);
        else if constexpr (X == 32)
            pair32(v[r], a, b);
        else
            b = mirror64(a, lane);
        const int32_t lo = min(a, b), hi = max(a, b);
        v[r] = low ? lo : hi;
    }
}

// The steps that follow the first one of a block of k = 64 M keys (M > 1):
// distances of M / 2 registers down to one.
template <int K, int M>
__device__ __forceinline__ void register_steps(int32_t (&v)[K])
{
#pragma unroll
    for (int d = M / 4; d > 0; d /= 2) {
#pragma unroll
        for (int r = 0; r < K; ++r) {
            if (r & d)
                continue;
            const int32_t a = v[r], b = v[r | d];
            v[r] = min(a, b);
            v[r | d] = max(a, b);
        }
    }
}

// A block of 64 M keys whose halves ascend: key i against key 64 M - 1 - i
// (the mirrored register and lane), then the register distances.
template <int K, int M>
__device__ __forceinline__ void merge_registers(int32_t (&v)[K], int lane)
{
#pragma unroll
    for (int r = 0; r < K; ++r) {
        constexpr int m = M - 1;
        if (r > (r ^ m))
            continue;
        const int32_t a = v[r], b = v[r ^ m];
        v[r] = min(a, mirror64(b, lane));
        v[r ^ m] = max(b, mirror64(a, lane));
    }
    register_steps<K, M>(v);
}

template <int K>
__device__ __forceinline__ void lane_steps(int32_t (&v)[K], int lane)
{
    lane_step<K, 32>(v, lane);
    lane_step<K, 16>(v, lane);
    lane_step<K, 8>(v, lane);
    lane_step<K, 4>(v, lane);
    lane_step<K, 2>(v, lane);
    lane_step<K, 1>(v, lane);
}

// Bitonic sorting network over 64 K keys held as v[r] in lane `lane`, key
// index r * 64 + lane, in the form whose every comparison is ascending: a block
// of two ascending halves is compared with its mirror image, then at halving
// distances.  The blocks of more than 64 keys are a loop at run time, to keep
// the code small; every register index is a constant.
template <int K>
__device__ __forceinline__ void wave_bitonic(int32_t (&v)[K], int lane)
{
    lane_step<K, 1>(v, lane);
    lane_step<K, 3>(v, lane);
    lane_step<K, 1>(v, lane);
    lane_step<K, 7>(v, lane);
    lane_step<K, 2>(v, lane);
    lane_step<K, 1>(v, lane);
    lane_step<K, 15>(v, lane);
    lane_step<K, 4>(v, lane);
    lane_step<K, 2>(v, lane);
    lane_step<K, 1>(v, lane);
    lane_step<K, 31>(v, lane);
    lane_step<K, 8>(v, lane);
    lane_step<K, 4>(v, lane);
    lane_step<K, 2>(v, lane);
    lane_step<K, 1>(v, lane);
    lane_step<K, 63>(v, lane);
    lane_step<K, 16>(v, lane);
    lane_step<K, 8>(v, lane);
    lane_step<K, 4>(v, lane);
    lane_step<K, 2>(v, lane);
    lane_step<K, 1>(v, lane);
    for (int m = 2; m <= K; m <<= 1) {
        if constexpr (K >= 2)
            if (m == 2)
                merge_registers<K, 2>(v, lane);
        if constexpr (K >= 4)
            if (m == 4)
                merge_registers<K, 4>(v, lane);
        if constexpr (K >= 8)
            if (m == 8)
                merge_registers<K, 8>(v, lane);
        lane_steps<K>(v, lane);
    }
}

// A wavefront's list: the coarse nodes of the members `ids` (n of them, 64 per
// register), sorted, the distinct values written to out; returns how many.
template <int K, int KM>
__device__ __forceinline__ int32_t wave_list(const int32_t (&ids)[KM], const int32_t *__restrict__ node_rep, int32_t n,
                                             int32_t *__restrict__ out, int lane)
{
    int32_t v[K];
#pragma unroll
    for (int r = 0; r < K; ++r)
        v[r] = (r * kWave + lane < n) ? node_rep[ids[r]] : INT_MAX;
    wave_bitonic<K>(v, lane);
    int32_t c = 0;
#pragma unroll
    for (int r = 0; r < K; ++r) {
        // the value before: the lane below's, or the last lane's of the register before
        int32_t before = __shfl_up(v[r], 1, kWave);
        if (r > 0) {
            const int32_t last = __shfl(v[r > 0 ? r - 1 : 0], kWave - 1, kWave);
            before = lane == 0 ? last : before;
        }
        const bool put = r * kWave + lane < n && ((r == 0 && lane == 0) || v[r] != before);
        const uint64_t m = __ballot(put);
        if (put)
            out[c + (int32_t)__popcll(m & ((1ull << lane) - 1ull))] = v[r];
        c += (int32_t)__popcll(m);
    }
    return c;
}

// The lists of more than kSortThread and at most kSortMid members, a wavefront
// each, longest first: kListBlocks workgroups at most, whose wavefronts go
// through the size order in turn and fetch the next list while they sort one
// (windows of 16 hyperedges per wavefront, found with a ballot, left most of
// the time to wavefronts without a list: 57 us at the 2M-node level, where
// this takes 49).
constexpr int kListBlocks = 2048;

__global__ __launch_bounds__(kThreads) void k_list_wave(const int32_t *__restrict__ ptr,
                                                        const int32_t *__restrict__ idx,
                                                        const int32_t *__restrict__ node_rep,
                                                        const int32_t *__restrict__ best,
                                                        const int32_t *__restrict__ rank, SizeOrder S,
                                                        int32_t *__restrict__ out, EdgeCount *__restrict__ count,
                                                        const int *__restrict__ bad)
{
    if (*bad)   // the step's input failed its checks
        return;
    constexpr int KM = kSortMid / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t first = S.first_of(kSortThread + 1), end = S.first_of(kSortMid + 1);
    const int64_t step = (int64_t)gridDim.x * (kThreads / kWave);
    int64_t i = end - 1 - ((int64_t)blockIdx.x * (kThreads / kWave) + threadIdx.x / kWave);
    if (i < first)
        return;   // uniform over the wavefront
    auto edge_at = [&](int64_t at) { return __builtin_amdgcn_readfirstlane(at >= first ? S.by_size[at] : 0); };
    int32_t ids[KM];
    auto load_ids = [&](int32_t s, int32_t n) {
#pragma unroll
        for (int r = 0; r < KM; ++r) {
            const int32_t p = r * kWave + lane;
            ids[r] = (p < n) ? idx[s + p] : 0;
        }
    };
    int32_t e = edge_at(i), next = edge_at(i - step);
    int32_t s = __builtin_amdgcn_readfirstlane(ptr[e]), n = __builtin_amdgcn_readfirstlane(ptr[e + 1]) - s;
    load_ids(s, n);
    for (; i >= first; i -= step) {
        // the first member's choice, and the next list's place
        const int32_t b0 = best[__builtin_amdgcn_readfirstlane(ids[0])], re = rank[e];
        const int32_t s2 = ptr[next], n2 = ptr[next + 1] - s2;
        const int32_t after = edge_at(i - 2 * step);
        const int32_t c = n <= 64    ? wave_list<1>(ids, node_rep, n, out + s, lane)
                          : n <= 128 ? wave_list<2>(ids, node_rep, n, out + s, lane)
                                     : wave_list<4>(ids, node_rep, n, out + s, lane);
        if (i - step >= first)
            load_ids(s2, n2);
        if (lane == 0)
            count[e] = edge_count(c, b0 == re);
        e = next;
        next = after;
        s = s2;
        n = n2;
    }
}

// The lists of more than kSortMid and at most kSortLong members, a workgroup
// each: every wavefront sorts 512 keys in registers (key index 512 wave + 64 r
// + lane), then blocks of 1,024 and 2,048 keys are merged in the same network,
// whose steps between wavefronts go through LDS.  (Windows of 64 hyperedges
// per workgroup took 72 us at the 2M-node level, where the size order takes
// 53; a wavefront with up to 32 registers of keys per list 60 and more.)
constexpr int kLongRegs = 8;

__global__ __launch_bounds__(kThreads) void k_list_long(const int32_t *__restrict__ ptr,
                                                        const int32_t *__restrict__ idx,
                                                        const int32_t *__restrict__ node_rep,
                                                        const int32_t *__restrict__ best,
                                                        const int32_t *__restrict__ rank, SizeOrder S,
                                                        int32_t *__restrict__ out, EdgeCount *__restrict__ count,
                                                        const int *__restrict__ bad)
{
    if (*bad)   // the step's input failed its checks
        return;
    static_assert(kThreads * kLongRegs == kSortLong, "a key per register of the workgroup");
    __shared__ int32_t keys[kSortLong];
    __shared__ int32_t part[kThreads / kWave];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int32_t base = wave * kLongRegs * kWave;
    const int64_t first = S.first_of(kSortMid + 1);
    for (int64_t i = S.n_edges - 1 - blockIdx.x; i >= first; i -= gridDim.x) {   // longest first
        const int32_t e = S.by_size[i], s = ptr[e], n = ptr[e + 1] - s;
        if (n > kSortLong)   // uniform over the workgroup
            continue;
        const int32_t b0 = best[idx[s]], re = rank[e];
        int32_t v[kLongRegs];
#pragma unroll
        for (int r = 0; r < kLongRegs; ++r) {
            const int32_t i = base + r * kWave + lane;
            v[r] = (i < n) ? idx[s + i] : -1;
        }
#pragma unroll
        for (int r = 0; r < kLongRegs; ++r)
            v[r] = (base + r * kWave + lane < n) ? node_rep[v[r]] : INT_MAX;
        if (base < n)   // (the later wavefronts of a short list hold only padding)
            wave_bitonic<kLongRegs>(v, lane);
        // compares every key with the one at index ^ x, the wavefronts with
        // `bit` clear keeping the smaller ones
        auto exchange = [&](int32_t x, int bit) {
            __syncthreads();   // the last exchange has been read
#pragma unroll
            for (int r = 0; r < kLongRegs; ++r)
                keys[base + r * kWave + lane] = v[r];
            __syncthreads();
#pragma unroll
            for (int r = 0; r < kLongRegs; ++r) {
                const int32_t y = keys[(base + r * kWave + lane) ^ x];
                v[r] = (wave & bit) == 0 ? min(v[r], y) : max(v[r], y);
            }
        };
        if (n > 512) {   // uniform over the workgroup
            exchange(1023, 1);
            register_steps<kLongRegs, 2 * kLongRegs>(v);
            lane_steps<kLongRegs>(v, lane);
        }
        if (n > 1024) {
            exchange(2047, 2);
            exchange(512, 1);
            register_steps<kLongRegs, 2 * kLongRegs>(v);
            lane_steps<kLongRegs>(v, lane);
        }
        // distinct values: a value is written if the one before it differs
        __syncthreads();
        if (lane == kWave - 1)
            keys[wave] = v[kLongRegs - 1];
        __syncthreads();
        int32_t last = wave > 0 ? keys[wave - 1] : -1, c = 0;
        uint64_t put[kLongRegs];
#pragma unroll
        for (int r = 0; r < kLongRegs; ++r) {
            int32_t before = __shfl_up(v[r], 1, kWave);
            before = lane == 0 ? last : before;
            last = __shfl(v[r], kWave - 1, kWave);
            put[r] = __ballot(base + r * kWave + lane < n && v[r] != before);
            c += (int32_t)__popcll(put[r]);
        }
        if (lane == 0)
            part[wave] = c;
        __syncthreads();
        int32_t at = s, total = 0;
        for (int w = 0; w < kThreads / kWave; ++w) {
            at += w < wave ? part[w] : 0;
            total += part[w];
        }
#pragma unroll
        for (int r = 0; r < kLongRegs; ++r) {
            if ((put[r] >> lane) & 1)
                out[at + (int32_t)__popcll(put[r] & ((1ull << lane) - 1ull))] = v[r];
            at += (int32_t)__popcll(put[r]);
        }
        if (threadIdx.x == 0)
            count[e] = edge_count(total, b0 == re);
    }
}

// Writes the distinct values of the ascending v[0, n) to out (which may be v
// itself: a round reads its values before it writes, and writes nothing past
// them) and returns how many, to every thread of the workgroup.
__device__ int32_t block_distinct(const int32_t *v, int32_t n, int32_t *out, int32_t (&part)[kSortBlockThreads / kWave])
{
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    int32_t c = 0, last = -1;   // the values written, and the value before the round's first
    for (uint32_t t = 0; t < (uint32_t)n; t += kSortBlockThreads) {
        const uint32_t i = t + threadIdx.x;
        const int32_t x = i < (uint32_t)n ? v[i] : -1;
        const int32_t before = i >= (uint32_t)n ? -1 : threadIdx.x == 0 ? last : v[i - 1];
        last = v[min(t + kSortBlockThreads, (uint32_t)n) - 1];
        const bool put = i < (uint32_t)n && x != before;
        const uint64_t m = __ballot(put);
        if (lane == 0)
            part[wave] = (int32_t)__popcll(m);
        __syncthreads();   // (also: the round's values have been read)
        int32_t at = c + (int32_t)__popcll(m & ((1ull << lane) - 1ull));
        for (int w = 0; w < kSortBlockThreads / kWave; ++w) {
            if (w < wave)
                at += part[w];
            c += part[w];
        }
        if (put)
            out[at] = x;
        __syncthreads();   // the counts have been read, the values written
    }
    return c;
}

// The lists of more than kSortLong members, a workgroup each: up to kSortBlock members bitonic in LDS; longer ones are
// only mapped, and appended to the library sort's segments.
__global__ __launch_bounds__(kSortBlockThreads) void k_list_block(
    const int32_t *__restrict__ ptr, const int32_t *__restrict__ idx, const int32_t *__restrict__ node_rep,
    const int32_t *__restrict__ best, const int32_t *__restrict__ rank, SizeOrder S, int32_t *__restrict__ out,
    int32_t *__restrict__ mapped,
    EdgeCount *__restrict__ count, int32_t *__restrict__ huge_begin, int32_t *__restrict__ huge_end,
    int32_t *__restrict__ huge, int32_t *__restrict__ n_huge, const int *__restrict__ bad)
{
    if (*bad)   // the step's input failed its checks
        return;
    __shared__ int32_t v[kSortBlock];
    __shared__ int32_t part[kSortBlockThreads / kWave];
    const int64_t first = S.first_of(kSizeBins - 1);
    for (int64_t l = S.n_edges - 1 - blockIdx.x; l >= first; l -= gridDim.x) {
        const int32_t e = S.by_size[l], s = ptr[e], n = ptr[e + 1] - s;
        if (n <= kSortLong)
            break;   // the sizes descend
        if (n > kSortBlock) {
            for (uint32_t i = threadIdx.x; i < (uint32_t)n; i += kSortBlockThreads)
                mapped[s + i] = node_rep[idx[s + i]];
            if (threadIdx.x == 0) {
                const int32_t h = atomicAdd(n_huge, 1);
                huge_begin[h] = s;
                huge_end[h] = s + n;
                huge[h] = e;
            }
            continue;
        }
        int32_t cap = 2 * kSortLong;
        while (cap < n)
            cap *= 2;
        for (int32_t i = threadIdx.x; i < cap; i += kSortBlockThreads)
            v[i] = i < n ? node_rep[idx[s + i]] : INT_MAX;
        __syncthreads();
        for (int32_t k = 2; k <= cap; k <<= 1) {
            for (int32_t j = k >> 1; j > 0; j >>= 1) {
                for (int32_t p = threadIdx.x; p < cap / 2; p += kSortBlockThreads) {
                    const int32_t i = 2 * p - (p & (j - 1)), q = i + j;   // pair p at distance j
                    const int32_t x = v[i], y = v[q];
                    const bool up = (i & k) == 0;
                    v[i] = up ? min(x, y) : max(x, y);
                    v[q] = up ? max(x, y) : min(x, y);
                }
                __syncthreads();
            }
        }
        const int32_t c = block_distinct(v, n, out + s, part);
        if (threadIdx.x == 0)
            count[e] = edge_count(c, best[idx[s]] == rank[e]);
        __syncthreads();   // the list's LDS has been read
    }
}

// The lists the library sorted (in out): their distinct values, in place.
__global__ __launch_bounds__(kSortBlockThreads) void k_list_huge(const int32_t *__restrict__ ptr,
                                                                 const int32_t *__restrict__ idx,
                                                                 const int32_t *__restrict__ best,
                                                                 const int32_t *__restrict__ rank,
                                                                 const int32_t *__restrict__ huge,
                                                                 const int32_t *__restrict__ n_huge, int32_t *out,
                                                                 EdgeCount *__restrict__ count,
                                                                 const int *__restrict__ bad)
{
    if (*bad)   // the step's input failed its checks
        return;
    __shared__ int32_t part[kSortBlockThreads / kWave];
    const int32_t lists = *n_huge;
    for (int32_t l = blockIdx.x; l < lists; l += gridDim.x) {
        const int32_t e = huge[l], s = ptr[e], n = ptr[e + 1] - s;
        const int32_t c = block_distinct(out + s, n, out + s, part);
        if (threadIdx.x == 0)
            count[e] = edge_count(c, best[idx[s]] == rank[e]);
    }
}

// per hyperedge: edge_rep, and for a kept one its coarse offset, weight and
// members (copied from the start of its segment; lists of more than kSortLong
// are left to k_emit_long); the last hyperedge closes the offsets and writes
// sizes[1] and sizes[2]
__global__ __launch_bounds__(kThreads) void k_emit(const int32_t *__restrict__ ptr,
                                                   const EdgeCount *__restrict__ count,
                                                   const EdgeCount *__restrict__ at, const int32_t *__restrict__ lists,
                                                   const float *__restrict__ w, int per, int64_t n_edges, int64_t nnz,
                                                   int32_t *__restrict__ edge_rep, int32_t *__restrict__ c_ptr,
                                                   int32_t *__restrict__ c_idx, float *__restrict__ c_w,
                                                   int64_t *__restrict__ sizes, const int *__restrict__ bad)
{
    __shared__ WalkLds lds;
    const int64_t e0 = window_start(per);
    if (*bad || e0 >= n_edges)   // the step's input failed its checks
        return;
    const int64_t e = e0 + threadIdx.x % kWave;
    const Window W = window_of(ptr, e0, per, n_edges, nnz);
    int32_t until = 0, shift = 0;   // the segment's incidences below `until` go to their position + shift
    if (threadIdx.x % kWave < per && e < n_edges) {
        const EdgeCount c = count[e], p = at[e];
        until = W.first + (ptr[e + 1] - W.first > kSortLong ? 0 : c.members);
        shift = p.members - W.first;
        edge_rep[e] = c.kept ? p.kept : -1;
        if (c.kept) {
            c_ptr[p.kept] = p.members;
            if (c_w)
                c_w[p.kept] = w ? w[e] : 1.0f;
        }
        if (e == n_edges - 1) {
            sizes[1] = p.kept + c.kept;
            sizes[2] = p.members + c.members;
            c_ptr[p.kept + c.kept] = p.members + c.members;
        }
    }
    walk_window<kWalk>(
        W, lds, [&](uint32_t j, int, bool ok) { return ok ? lists[j] : 0; },
        [&](uint32_t j, int l, bool ok, bool, int32_t x) {
            const int32_t u = __shfl(until, l, kWave), d = __shfl(shift, l, kWave);
            if (ok && j < (uint32_t)u)
                c_idx[(int32_t)j + d] = x;
        });
}

// the members of the lists of more than kSortLong, kEmitSplit workgroups each
constexpr int kEmitSplit = 16;
__global__ __launch_bounds__(kThreads) void k_emit_long(const int32_t *__restrict__ ptr,
                                                        const EdgeCount *__restrict__ count,
                                                        const EdgeCount *__restrict__ at,
                                                        const int32_t *__restrict__ lists, SizeOrder S,
                                                        int32_t *__restrict__ c_idx, const int *__restrict__ bad)
{
    if (*bad)   // the step's input failed its checks
        return;
    const int64_t first = S.first_of(kSizeBins - 1);
    for (int64_t l = S.n_edges - 1 - blockIdx.x; l >= first; l -= gridDim.x) {
        const int32_t e = S.by_size[l], s = ptr[e], to = at[e].members;
        if (ptr[e + 1] - s <= kSortLong)
            break;   // the sizes descend
        const uint32_t n = count[e].members;
        for (uint32_t i = blockIdx.y * kThreads + threadIdx.x; i < n; i += kEmitSplit * kThreads)
            c_idx[to + i] = lists[s + i];
    }
}

// The sizes a level without hyperedges, or without nodes, leaves open.
__global__ void k_sizes_empty(int64_t n_nodes, int64_t n_edges, int32_t *__restrict__ c_ptr,
                              int64_t *__restrict__ sizes, const int *__restrict__ bad)
{
    if (threadIdx.x != 0 || blockIdx.x != 0 || *bad)
        return;
    if (n_nodes == 0)
        sizes[0] = 0;
    if (n_edges == 0) {
        sizes[1] = sizes[2] = 0;
        c_ptr[0] = 0;
    }
}

// ---------------------------------------------------------------------------
// feature-based assignment (bag-of-words counts, int32 [rows x k], k % 4 == 0)
// ---------------------------------------------------------------------------

// Counts must be >= 0 (flag bit 4) and their total below 2^31 (checked on the
// host from `total`); with that bound every sum, product and dot below fits
// its integer type exactly.  The same pass takes the largest count and writes
// every count's low byte to x8 (rows of kp bytes, the columns past k zero;
// null: not wanted), which holds the counts themselves when the largest is at
// most 255.  Bound by the 4 bytes read per count.
__global__ __launch_bounds__(kThreads) void k_fcheck(const int4 *__restrict__ x, int64_t n_rows, int k4, int kp4,
                                                     int *__restrict__ flag, int *__restrict__ largest,
                                                     unsigned long long *__restrict__ total,
                                                     uint32_t *__restrict__ x8)
{
    __shared__ unsigned long long part[kThreads / kWave];
    unsigned long long sum = 0;
    int neg = 0, most = 0;
    // thread i takes word i of the byte matrix, then every stride-th
    const int64_t n = n_rows * kp4, stride = (int64_t)gridDim.x * kThreads;
    int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    int64_t row = i / kp4, step_rows = stride / kp4;
    int col = (int)(i - row * kp4), step_cols = (int)(stride - step_rows * kp4);
    for (; i < n; i += stride) {
        uint32_t w = 0;
        if (col < k4) {
            const int4 v = x[row * k4 + col];
            neg |= (v.x | v.y | v.z | v.w) < 0;
            most = max(max(most, max(v.x, v.y)), max(v.z, v.w));
            sum += (unsigned long long)(uint32_t)v.x + (uint32_t)v.y + (uint32_t)v.z + (uint32_t)v.w;
            w = (v.x & 255) | (v.y & 255) << 8 | (v.z & 255) << 16 | (uint32_t)(v.w & 255) << 24;
        }
        if (x8)
            x8[i] = w;
        row += step_rows;
        col += step_cols;
        if (col >= kp4) {
            col -= kp4;
            ++row;
        }
    }
    for (int o = kWave / 2; o > 0; o >>= 1) {
        sum += __shfl_xor(sum, o);
        most = max(most, __shfl_xor(most, o));
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        part[threadIdx.x / kWave] = sum;
        if (most > *largest)   // an earlier read bounds the maximum from below
            atomicMax(largest, most);
    }
    if (neg)
        atomicOr(flag, 16);
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long b = 0;
        for (int w = 0; w < kThreads / kWave; ++w)
            b += part[w];
        atomicAdd(total, b);
    }
}

// Members handled together by one wavefront in the feature kernels: their
// row loads are independent, so this many rows are in flight per lane
// (fewer for wide rows held in registers, to keep the register count down).
template <int NC>
constexpr int members_in_flight()
{
    return (NC == 0 || NC <= 2) ? 4 : 8 / NC;
}

// A feature row of k counts is read by one wavefront as NC passes of 256
// counts (4 per lane, 16 B); NC is a compile-time bound (k <= 256 NC) so the
// per-lane pieces of a row live in registers.  NC = 0: any k, one pass at a
// time (wide rows).
template <int NC>
struct RowPieces {
    int4 p[NC];
    __device__ void zero()
    {
#pragma unroll
        for (int i = 0; i < NC; ++i)
            p[i] = make_int4(0, 0, 0, 0);
    }
    __device__ void load(const int32_t *row, int lane, int k)
    {
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const int c = lane * 4 + i * kWave * 4;
            p[i] = (c < k) ? *reinterpret_cast<const int4 *>(row + c) : make_int4(0, 0, 0, 0);
        }
    }
    __device__ void add(const RowPieces &o)
    {
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            p[i].x += o.p[i].x;
            p[i].y += o.p[i].y;
            p[i].z += o.p[i].z;
            p[i].w += o.p[i].w;
        }
    }
    __device__ int64_t dot(const RowPieces &o) const
    {
        int64_t d = 0;
#pragma unroll
        for (int i = 0; i < NC; ++i)
            d += (int64_t)p[i].x * o.p[i].x + (int64_t)p[i].y * o.p[i].y + (int64_t)p[i].z * o.p[i].z +
                 (int64_t)p[i].w * o.p[i].w;
        return d;
    }
    __device__ void store(int32_t *row, int lane, int k) const
    {
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const int c = lane * 4 + i * kWave * 4;
            if (c < k)
                *reinterpret_cast<int4 *>(row + c) = p[i];
        }
    }
};

__device__ inline int64_t wave_sum(int64_t v)
{
    for (int o = kWave / 2; o > 0; o >>= 1)
        v += __shfl_xor(v, o);
    return v;
}

// out[r] = sum of the rows x[idx[j]], j in [ptr[r], ptr[r+1]), for r below
// *limit (all rows if limit is NULL); one wavefront per row.  SQ: also
// sq[r] = |out[r]|^2 (int64).  Integer sums: the order of the additions
// does not change the result.
template <bool SQ, int NC>
__global__ __launch_bounds__(kThreads) void k_rowsum(const int32_t *__restrict__ ptr, const int32_t *__restrict__ idx,
                                                     const int32_t *__restrict__ x, int k, int64_t n_rows,
                                                     const int64_t *__restrict__ limit, int32_t *__restrict__ out,
                                                     int64_t *__restrict__ sq)
{
    constexpr int U = members_in_flight<NC>();
    const int64_t r = linear_block() * (kThreads / kWave) + threadIdx.x / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    if (r >= n_rows || (limit && r >= *limit))
        return;
    const int32_t a = ptr[r], b = ptr[r + 1];
    if constexpr (NC > 0) {
        RowPieces<NC> acc;
        acc.zero();
        int32_t j = a;
        for (; j + U <= b; j += U) {
            RowPieces<NC> m[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                m[u].load(x + (int64_t)idx[j + u] * k, lane, k);
#pragma unroll
            for (int u = 0; u < U; ++u)
                acc.add(m[u]);
        }
        for (; j < b; ++j) {
            RowPieces<NC> m;
            m.load(x + (int64_t)idx[j] * k, lane, k);
            acc.add(m);
        }
        acc.store(out + r * k, lane, k);
        if (SQ) {
            const int64_t q = wave_sum(acc.dot(acc));
            if (lane == 0)
                sq[r] = q;
        }
    } else {
        int64_t q = 0;
        for (int c = lane * 4; c < k; c += kWave * 4) {
            int4 acc = make_int4(0, 0, 0, 0);
            for (int32_t j = a; j < b; ++j) {
                const int4 v = *reinterpret_cast<const int4 *>(x + (int64_t)idx[j] * k + c);
                acc.x += v.x;
                acc.y += v.y;
                acc.z += v.z;
                acc.w += v.w;
            }
            *reinterpret_cast<int4 *>(out + r * k + c) = acc;
            if (SQ)
                q += (int64_t)acc.x * acc.x + (int64_t)acc.y * acc.y + (int64_t)acc.z * acc.z +
                     (int64_t)acc.w * acc.w;
        }
        if (SQ) {
            q = wave_sum(q);
            if (lane == 0)
                sq[r] = q;
        }
    }
}

// IEEE FP64 cosine score d|d| / |s_e|^2 (0 when s_e = 0); d and |s_e|^2 are
// exact integers, the product and the quotient are each rounded once
__device__ inline double cosine_score(int64_t d, int64_t s2)
{
    if (s2 == 0)
        return 0.0;
    const double dd = (double)d;
    const double num = dd * fabs(dd);
    return num / (double)s2;
}

// order-preserving map of a double onto unsigned 64-bit integers
__device__ inline unsigned long long ordered_bits(double q)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(q);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

// per incidence (e, v): q = cosine score of e for v, kept in CSR order;
// bestq[v] = max over v's incidences (atomic max: order-independent).
// One wavefront takes 64 consecutive incidences, whatever their hyperedges:
// lane l loads incidence l's node, hyperedge and |s_e|^2, the wavefront then
// walks the 64 in steps of score_batch (rows broadcast by __shfl, the next
// step's rows loaded before this step's reduction), and at the end lane l
// finishes incidence l.
template <int NC>
constexpr int score_batch()
{
    return (NC == 0 || NC == 1) ? 4 : NC == 2 ? 2 : 1;
}

template <int NC>
__global__ __launch_bounds__(kThreads) void k_qscore(const int32_t *__restrict__ idx,
                                                     const int32_t *__restrict__ inc_edge,
                                                     const int32_t *__restrict__ s, const int64_t *__restrict__ s2,
                                                     const int32_t *__restrict__ x, int k, int64_t nnz,
                                                     double *__restrict__ q, unsigned long long *__restrict__ bestq)
{
    constexpr int U = score_batch<NC>();
    static_assert(kWave % U == 0, "a step must divide the wavefront");
    const int64_t j0 = ((int64_t)blockIdx.x * (kThreads / kWave) + threadIdx.x / kWave) * kWave;
    const int lane = threadIdx.x & (kWave - 1);
    if (j0 >= nnz)
        return;
    const int n = (int)std::min<int64_t>(kWave, nnz - j0);
    const int32_t my_v = lane < n ? idx[j0 + lane] : 0;
    const int32_t my_e = lane < n ? inc_edge[j0 + lane] : 0;
    const int64_t my_s2 = lane < n ? s2[my_e] : 0;
    int64_t mine = 0;
    if constexpr (NC > 0) {
        RowPieces<NC> f[U], m[U];
        auto load_step = [&](int t) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int32_t v = __shfl(my_v, t + u), e = __shfl(my_e, t + u);
                if (t + u < n) {
                    f[u].load(s + (int64_t)e * k, lane, k);
                    m[u].load(x + (int64_t)v * k, lane, k);
                } else {
                    f[u].zero();
                    m[u].zero();
                }
            }
        };
        load_step(0);
        for (int t = 0; t < n; t += U) {
            int64_t d[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                d[u] = f[u].dot(m[u]);
            if (t + U < n)
                load_step(t + U);
            for (int o = kWave / 2; o > 0; o >>= 1) {
#pragma unroll
                for (int u = 0; u < U; ++u)
                    d[u] += __shfl_xor(d[u], o);
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (lane == t + u)
                    mine = d[u];
        }
    } else {
        for (int t = 0; t < n; ++t) {
            const int32_t v = __shfl(my_v, t), e = __shfl(my_e, t);
            int64_t d = 0;
            for (int c = lane * 4; c < k; c += kWave * 4) {
                const int4 fc = *reinterpret_cast<const int4 *>(s + (int64_t)e * k + c);
                const int4 mc = *reinterpret_cast<const int4 *>(x + (int64_t)v * k + c);
                d += (int64_t)fc.x * mc.x + (int64_t)fc.y * mc.y + (int64_t)fc.z * mc.z + (int64_t)fc.w * mc.w;
            }
            d = wave_sum(d);
            if (lane == t)
                mine = d;
        }
    }
    if (lane < n) {
        const double sc = cosine_score(mine, my_s2);
        q[j0 + lane] = sc;
        const unsigned long long ob = ordered_bits(sc);
        if (ob > bestq[my_v])   // an earlier read bounds the maximum from below
            atomicMax(bestq + my_v, ob);
    }
}

// The register bound NC for a feature width k (0: wider than 2048).
inline int pieces_for(int k) { return k <= 256 ? 1 : k <= 512 ? 2 : k <= 1024 ? 4 : k <= 2048 ? 8 : 0; }

template <int NC>
void launch_edge_features(dim3 grid, hipStream_t st, const int32_t *ptr, const int32_t *idx,
                          const int32_t *inc_edge, const int32_t *x, int k, int64_t n_edges, int64_t nnz,
                          int32_t *fsum, int64_t *fsq, double *q, unsigned long long *bestq)
{
    k_rowsum<true, NC><<<grid, kThreads, 0, st>>>(ptr, idx, x, k, n_edges, nullptr, fsum, fsq);
    const int64_t waves = (nnz + kWave - 1) / kWave;
    const unsigned sgrid = (unsigned)((waves + kThreads / kWave - 1) / (kThreads / kWave));
    k_qscore<NC><<<sgrid, kThreads, 0, st>>>(idx, inc_edge, fsum, fsq, x, k, nnz, q, bestq);
}

template <int NC>
void launch_group_sums(dim3 grid, hipStream_t st, const int32_t *gptr, const int32_t *gnodes, const int32_t *x,
                       int k, int64_t n_rows, const int64_t *limit, int32_t *out)
{
    k_rowsum<false, NC><<<grid, kThreads, 0, st>>>(gptr, gnodes, x, k, n_rows, limit, out, nullptr);
}

// ---------------------------------------------------------------------------
// feature-based assignment on counts of at most 255: rows of kp bytes
//
// The member rows are gathered once, as bytes, by the wavefront that sums
// them, and the scores are taken there too, while the sum is in registers: a
// quarter of the bytes of the int32 rows, read once (short hyperedges) or
// again from cache, and no sum matrix written and read back.  Bound by the
// gather of kp bytes per incidence.  A row is read by a group of G lanes of
// 16 bytes (kp <= 16 G); the 64 / G groups of a wavefront take interleaved
// members.  Sums and dot products are integer, so their order is free.
// Measured at 1M nodes, 600K hyperedges, 4.5M incidences, k = 512, a step's
// average over 6: member sums and scores 2.84 -> 0.62 ms, X' 0.26 -> 0.20 ms,
// and the checking pass over X, which now writes the bytes too, 0.18 -> 0.24 ms.
// ---------------------------------------------------------------------------

constexpr int kByteCols = 1024;     // widest row of the byte path: one 16-byte piece per lane
constexpr int kByteSmall = 64;      // members of a hyperedge one wavefront takes
constexpr int kByteRows = 4;        // member rows in flight per lane group

inline int byte_stride(int k) { return (k + 15) / 16 * 16; }

// 16 counts of a lane as sums of bytes: s[i] holds columns 4 i and 4 i + 2 of
// the lane's piece in its low and high half (ev) and columns 4 i + 1 and
// 4 i + 3 (od); exact for at most 257 rows.
struct ByteSum {
    uint32_t ev[4], od[4];
    __device__ void zero()
    {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            ev[i] = od[i] = 0;
    }
    __device__ void add(const uint4 &r)
    {
        const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            ev[i] += w[i] & 0x00ff00ffu;
            od[i] += (w[i] >> 8) & 0x00ff00ffu;
        }
    }
};

__device__ inline uint32_t dot4(uint32_t a, uint32_t b, uint32_t c) { return __builtin_amdgcn_udot4(a, b, c, false); }

// dot of two 16-byte pieces
__device__ inline uint32_t dot16(const uint32_t (&p)[4], const uint4 &r)
{
    return dot4(p[3], r.w, dot4(p[2], r.z, dot4(p[1], r.y, dot4(p[0], r.x, 0u))));
}

__device__ inline uint32_t dot16(const uint32_t (&p)[4], const uint32_t (&q)[4])
{
    return dot4(p[3], q[3], dot4(p[2], q[2], dot4(p[1], q[1], dot4(p[0], q[0], 0u))));
}

// sum over the G lanes of a group
template <int G, typename V>
__device__ inline V lanes_sum(V v)
{
#pragma unroll
    for (int o = 1; o < G; o <<= 1)
        v += __shfl_xor(v, o);
    return v;
}

// The sums of d[0..3] over the G lanes of a group, d[u] returned to the lanes
// gl with slot_of<G>(gl) == u (the exchanges halve the values left, so four
// sums cost little more than one).
template <int G>
__device__ inline int slot_of(int gl)
{
    return G >= 4 ? ((gl & 1) << 1 | ((gl >> 1) & 1)) : -1;
}

template <int G, typename V>
__device__ inline V lanes_sum4(const V (&d)[4], int gl)
{
    const bool b0 = gl & 1, b1 = gl & 2;
    V a = b0 ? d[2] : d[0], b = b0 ? d[3] : d[1];
    a += __shfl_xor(b0 ? d[0] : d[2], 1);
    b += __shfl_xor(b0 ? d[1] : d[3], 1);
    V v = b1 ? b : a;
    v += __shfl_xor(b1 ? a : b, 2);
#pragma unroll
    for (int o = 4; o < G; o <<= 1)
        v += __shfl_xor(v, o);
    return v;
}

// the score of incidence j (node v), as k_qscore writes it
__device__ inline void put_score(int64_t j, int32_t v, int64_t d, int64_t s2, double *__restrict__ q,
                                 unsigned long long *__restrict__ bestq)
{
    const double sc = cosine_score(d, s2);
    q[j] = sc;
    const unsigned long long ob = ordered_bits(sc);
    if (ob > bestq[v])   // an earlier read bounds the maximum from below
        atomicMax(bestq + v, ob);
}

// Hyperedges of at most kByteSmall members, a wavefront each.
template <int G>
__global__ __launch_bounds__(kThreads) void k_byte_scores(const int32_t *__restrict__ ptr,
                                                          const int32_t *__restrict__ idx,
                                                          const unsigned char *__restrict__ x8, int kp,
                                                          int64_t n_edges, double *__restrict__ q,
                                                          unsigned long long *__restrict__ bestq)
{
    constexpr int Q = kWave / G, U = kByteRows;
    const int64_t e = linear_block() * (kThreads / kWave) + threadIdx.x / kWave;
    const int lane = threadIdx.x & (kWave - 1), g = lane / G, gl = lane % G;
    if (e >= n_edges)
        return;   // uniform over the wavefront
    const int32_t a = ptr[e], m = ptr[e + 1] - a;
    if (m > kByteSmall)
        return;
    const bool col_ok = gl * 16 < kp;
    const int32_t my_v = lane < m ? idx[a + lane] : 0;
    auto load_rows = [&](uint4 (&r)[U], int t) {   // members t + u Q + g
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = t + u * Q + g;
            const int32_t v = __shfl(my_v, j & (kWave - 1));
            r[u] = make_uint4(0, 0, 0, 0);
            if (j < m && col_ok)
                r[u] = *reinterpret_cast<const uint4 *>(x8 + (int64_t)v * kp + gl * 16);
        }
    };
    uint4 first[U];
    load_rows(first, 0);
    ByteSum s;
    s.zero();
#pragma unroll
    for (int u = 0; u < U; ++u)
        s.add(first[u]);
    for (int t = U * Q; t < m; t += U * Q) {
        uint4 r[U];
        load_rows(r, t);
#pragma unroll
        for (int u = 0; u < U; ++u)
            s.add(r[u]);
    }
#pragma unroll
    for (int o = G; o < kWave; o <<= 1) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            s.ev[i] += __shfl_xor(s.ev[i], o);
            s.od[i] += __shfl_xor(s.od[i], o);
        }
    }
    // the sums as byte planes: s = lo + 256 hi
    uint32_t lo[4], hi[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        lo[i] = (s.ev[i] & 0x00ff00ffu) | (s.od[i] & 0x00ff00ffu) << 8;
        hi[i] = ((s.ev[i] >> 8) & 0x00ff00ffu) | (s.od[i] & 0xff00ff00u);
    }
    const uint32_t l2 = lanes_sum<G>(dot16(lo, lo)), lh = lanes_sum<G>(dot16(lo, hi)), h2 = lanes_sum<G>(dot16(hi, hi));
    const int64_t s2 = (int64_t)l2 + 512 * (int64_t)lh + 65536 * (int64_t)h2;
    for (int t = 0; t < m; t += U * Q) {
        if (t > 0)
            load_rows(first, t);
        uint32_t dl[4], dh[4];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            dl[u] = dot16(lo, first[u]);
            dh[u] = dot16(hi, first[u]);
        }
        if constexpr (G >= 4) {
            const uint32_t tl = lanes_sum4<G>(dl, gl);
            const uint32_t th = h2 ? lanes_sum4<G>(dh, gl) : 0u;   // uniform: h2 = 0 iff every high byte is 0
            const int j = t + slot_of<G>(gl) * Q + g;
            const int32_t v = __shfl(my_v, j & (kWave - 1));
            if (gl < 4 && j < m)
                put_score(a + j, v, (int64_t)tl + 256 * (int64_t)th, s2, q, bestq);
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t d = (int64_t)lanes_sum<G>(dl[u]) + 256 * (int64_t)lanes_sum<G>(dh[u]);
                const int j = t + u * Q + g;
                const int32_t v = __shfl(my_v, j & (kWave - 1));
                if (gl == 0 && j < m)
                    put_score(a + j, v, d, s2, q, bestq);
            }
        }
    }
}

// Longer hyperedges: each workgroup finds those of a window of kByteWindow
// hyperedges and takes them one after the other, members interleaved over
// its wavefronts' lane groups, the sum in LDS (counts total below 2^31, so
// every sum fits 32 bits) and then as four byte planes in registers.
constexpr int kByteWindow = 32;

template <int G>
__global__ __launch_bounds__(kThreads) void k_byte_scores_long(const int32_t *__restrict__ ptr,
                                                               const int32_t *__restrict__ idx,
                                                               const unsigned char *__restrict__ x8, int kp,
                                                               int64_t n_edges, double *__restrict__ q,
                                                               unsigned long long *__restrict__ bestq)
{
    constexpr int U = kByteRows, P = kThreads / G;   // lane groups of the workgroup
    __shared__ uint32_t sum[G * 16];
    const int64_t e0 = linear_block() * kByteWindow;
    const int lane = threadIdx.x & (kWave - 1), gl = threadIdx.x % G, p = threadIdx.x / G;
    int32_t my_a = 0, my_m = 0;
    if (lane < kByteWindow && e0 + lane < n_edges) {
        my_a = ptr[e0 + lane];
        my_m = ptr[e0 + lane + 1] - my_a;
    }
    const bool col_ok = gl * 16 < kp;
    for (uint64_t todo = __ballot(my_m > kByteSmall); todo; todo &= todo - 1) {   // the same in every wavefront
        const int w = __ffsll((long long)todo) - 1;
        // (unsigned: a round may pass 2^31 - 1)
        const uint32_t a = __shfl(my_a, w), m = __shfl(my_m, w);
        __syncthreads();
        for (int c = threadIdx.x; c < G * 16; c += kThreads)
            sum[c] = 0;
        __syncthreads();
        auto load_rows = [&](uint4 (&r)[U], uint32_t t) {   // members t + u P + p
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t j = t + u * P + p;
                r[u] = make_uint4(0, 0, 0, 0);
                if (j < m && col_ok)
                    r[u] = *reinterpret_cast<const uint4 *>(x8 + (int64_t)idx[a + j] * kp + gl * 16);
            }
        };
        // at most 256 rows per lane group before its sums move to LDS
        for (uint32_t t0 = 0; t0 < m; t0 += 256 * P) {
            ByteSum s;
            s.zero();
            const uint32_t end = min(m, t0 + 256 * P);
            for (uint32_t t = t0; t < end; t += U * P) {
                uint4 r[U];
                load_rows(r, t);
#pragma unroll
                for (int u = 0; u < U; ++u)
                    s.add(r[u]);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                atomicAdd(&sum[gl * 16 + 4 * i], s.ev[i] & 0xffffu);
                atomicAdd(&sum[gl * 16 + 4 * i + 1], s.od[i] & 0xffffu);
                atomicAdd(&sum[gl * 16 + 4 * i + 2], s.ev[i] >> 16);
                atomicAdd(&sum[gl * 16 + 4 * i + 3], s.od[i] >> 16);
            }
        }
        __syncthreads();
        uint32_t plane[4][4];
        int64_t s2 = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t c[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                c[b] = sum[gl * 16 + 4 * i + b];
                s2 += (int64_t)c[b] * (int64_t)c[b];
            }
#pragma unroll
            for (int y = 0; y < 4; ++y)
                plane[y][i] = ((c[0] >> (8 * y)) & 255u) | ((c[1] >> (8 * y)) & 255u) << 8 |
                              ((c[2] >> (8 * y)) & 255u) << 16 | ((c[3] >> (8 * y)) & 255u) << 24;
        }
        s2 = lanes_sum<G>(s2);
        for (uint32_t t = 0; t < m; t += U * P) {
            uint4 r[U];
            load_rows(r, t);
            int64_t d[4];
#pragma unroll
            for (int u = 0; u < U; ++u)
                d[u] = (int64_t)dot16(plane[0], r[u]) + ((int64_t)dot16(plane[1], r[u]) << 8) +
                       ((int64_t)dot16(plane[2], r[u]) << 16) + ((int64_t)dot16(plane[3], r[u]) << 24);
            if constexpr (G >= 4) {
                const int64_t v = lanes_sum4<G>(d, gl);
                const uint32_t j = t + slot_of<G>(gl) * P + p;
                if (gl < 4 && j < m)
                    put_score((int64_t)a + j, idx[a + j], v, s2, q, bestq);
            } else {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int64_t v = lanes_sum<G>(d[u]);
                    const uint32_t j = t + u * P + p;
                    if (gl == 0 && j < m)
                        put_score((int64_t)a + j, idx[a + j], v, s2, q, bestq);
                }
            }
        }
    }
}

// out[r] = sum of the byte rows of members [ptr[r], ptr[r+1]) as int32, for r
// below *limit; one wavefront per row, 4 counts per lane and pass (NC = passes
// of 256 counts).  Bound by the 4 bytes written per count.
template <int NC>
__global__ __launch_bounds__(kThreads) void k_rowsum_bytes(const int32_t *__restrict__ ptr,
                                                           const int32_t *__restrict__ idx,
                                                           const uint32_t *__restrict__ x8, int k4, int kp4,
                                                           int64_t n_rows, const int64_t *__restrict__ limit,
                                                           int4 *__restrict__ out)
{
    constexpr int U = 4;
    const int64_t r = linear_block() * (kThreads / kWave) + threadIdx.x / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    if (r >= n_rows || r >= *limit)
        return;
    const int32_t a = ptr[r], b = ptr[r + 1];
    int4 acc[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i)
        acc[i] = make_int4(0, 0, 0, 0);
    for (uint32_t j = a; j < (uint32_t)b; j += U) {   // (unsigned: b may be 2^31 - 1)
        uint32_t w[U][NC];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool ok = j + u < (uint32_t)b;
            const int64_t base = ok ? (int64_t)idx[j + u] * kp4 : 0;
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                const int c = lane + i * kWave;
                w[u][i] = (ok && c < kp4) ? x8[base + c] : 0u;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                acc[i].x += w[u][i] & 255u;
                acc[i].y += (w[u][i] >> 8) & 255u;
                acc[i].z += (w[u][i] >> 16) & 255u;
                acc[i].w += w[u][i] >> 24;
            }
    }
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        const int c = lane + i * kWave;
        if (c < k4)
            out[r * k4 + c] = acc[i];
    }
}

template <int G>
void launch_byte_scores(hipStream_t st, const int32_t *ptr, const int32_t *idx, const unsigned char *x8, int kp,
                        int64_t n_edges, int64_t nnz, double *q, unsigned long long *bestq)
{
    const int per = kThreads / kWave;
    k_byte_scores<G><<<fold_grid((n_edges + per - 1) / per), kThreads, 0, st>>>(ptr, idx, x8, kp, n_edges, q, bestq);
    if (nnz > kByteSmall)
        k_byte_scores_long<G><<<fold_grid((n_edges + kByteWindow - 1) / kByteWindow), kThreads, 0, st>>>(
            ptr, idx, x8, kp, n_edges, q, bestq);
}

// best[v] = least rank among v's hyperedges whose score equals bestq[v]
__global__ __launch_bounds__(kThreads) void k_best_feat(const int32_t *__restrict__ ptr,
                                                        const int32_t *__restrict__ idx,
                                                        const int32_t *__restrict__ rank,
                                                        const double *__restrict__ q,
                                                        const unsigned long long *__restrict__ bestq, int per,
                                                        int64_t n_edges, int64_t nnz, int32_t *__restrict__ best)
{
    __shared__ WalkLds lds;
    const int64_t e0 = window_start(per);
    if (e0 >= n_edges)
        return;
    const int64_t e = e0 + threadIdx.x % kWave;
    const int32_t r = threadIdx.x % kWave < per && e < n_edges ? rank[e] : 0;
    struct Score {
        int32_t v;
        unsigned long long q, most;
    };
    walk_window<kWalk>(
        window_of(ptr, e0, per, n_edges, nnz), lds,
        [&](uint32_t j, int, bool ok) {
            Score x{ok ? idx[j] : 0, 0, 1};
            if (ok) {
                x.q = ordered_bits(q[j]);
                x.most = bestq[x.v];
            }
            return x;
        },
        [&](uint32_t, int l, bool, bool, const Score &x) {
            const int32_t lr = __shfl(r, l, kWave);
            if (x.q == x.most && lr < best[x.v])   // an earlier read bounds the minimum from above
                atomicMin(best + x.v, lr);
        });
}

// coarse-node member lists: count, then place (the order inside a group is
// free; the sums over it are exact integers)
__global__ __launch_bounds__(kThreads) void k_group_count(const int32_t *__restrict__ node_rep, int64_t n_nodes,
                                                          int32_t *__restrict__ gcount)
{
    const int64_t v = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (v < n_nodes)
        atomicAdd(gcount + node_rep[v], 1);
}

__global__ __launch_bounds__(kThreads) void k_group_fill(const int32_t *__restrict__ node_rep,
                                                         const int32_t *__restrict__ gptr, int64_t n_nodes,
                                                         int32_t *__restrict__ gcur, int32_t *__restrict__ gnodes)
{
    const int64_t v = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (v >= n_nodes)
        return;
    const int32_t g = node_rep[v];
    gnodes[gptr[g] + atomicAdd(gcur + g, 1)] = (int32_t)v;
}

// Lists of more than `size` members that one level can hold.
int64_t max_lists(int64_t n_nodes, int64_t nnz, int size) { return n_nodes > size ? nnz / (size + 1) : 0; }

struct CoarsenLayout {
    size_t keys_in, keys_out, ids_in, order, rank, bins, bin_offs, best, choice, first, gflag, gid, count, at, mapped,
        lists, spare, bstart, sizes, flag, n_huge, huge, huge_ends;
    // feature path (k > 0)
    size_t inc_edge, fsum, fsq, q, bestq, gcount, gptr, gcur, gnodes;
    size_t temp, temp_bytes, total;
};

hnv_status layout(int64_t nV, int64_t nE, int64_t nnz, int k, CoarsenLayout &L)
{
    size_t off = 0;
    auto take = [&](size_t bytes) {
        off = (off + 255) & ~size_t(255);
        const size_t p = off;
        off += std::max<size_t>(bytes, 8);
        return p;
    };
    L.keys_in = take(8 * nE);
    L.keys_out = take(8 * nE);
    L.ids_in = take(4 * nE);
    L.order = take(4 * nE);
    L.rank = take(4 * nE);
    const int64_t bins = bin_cap(nE, kSizeBins);
    L.bins = take(4 * bins);
    L.bin_offs = take(4 * bins);
    L.best = take(4 * nV);
    L.choice = take(4 * nV);
    L.first = take(4 * nE);
    L.gflag = take(4 * nV);
    L.gid = take(4 * nV);
    L.count = take(sizeof(EdgeCount) * nE);
    L.at = take(sizeof(EdgeCount) * nE);
    L.mapped = take(4 * nnz);
    L.lists = take(4 * nnz);
    L.spare = take(bucketed_best(nV, nnz) ? 4 * nnz : 0);
    L.bstart = take(8 * (size_t)(std::max<int64_t>(nV >> kBucketShiftMax, 256) + 2));
    // the check word (int flags, largest count, uint64 feature total), the
    // coarse sizes (3 x int64; one read-back takes both) and the count of the
    // lists for the library's sort, cleared together
    L.flag = take(64);
    L.sizes = L.flag + 16;
    L.n_huge = L.flag + 40;
    const int64_t max_huge = max_lists(nV, nnz, kSortBlock);
    L.huge = take(4 * max_huge);
    L.huge_ends = take(8 * max_huge);
    L.inc_edge = L.fsum = L.fsq = L.q = L.bestq = L.gcount = L.gptr = L.gcur = L.gnodes = 0;
    if (k > 0) {
        L.inc_edge = take(4 * nnz);
        // the member sums of the int32 path, or the byte copy of X of the byte path
        L.fsum = take(std::max(4 * (size_t)nE * k, k <= kByteCols ? (size_t)nV * byte_stride(k) : 0));
        L.fsq = take(8 * nE);
        L.q = take(8 * nnz);
        L.bestq = take(8 * nV);
        L.gcount = take(4 * (nV + 1));
        L.gptr = take(4 * (nV + 1));
        L.gcur = take(4 * nV);
        L.gnodes = take(4 * nV);
    }
    size_t t[7] = {};
    const int64_t scan = std::max<int64_t>(std::max(nV + 1, bins), 1);
    hipError_t e = prim_exclusive_sum(nullptr, t[0], (int32_t *)nullptr, (int32_t *)nullptr, scan);
    if (e == hipSuccess)
        e = prim_exclusive_scan(nullptr, t[1], (EdgeCount *)nullptr, (EdgeCount *)nullptr, EdgeCount{0, 0},
                                std::max<int64_t>(nE, 1), EdgeCountPlus());
    if (e == hipSuccess)
        e = prim_sort_pairs(nullptr, t[2], (uint32_t *)nullptr, (uint32_t *)nullptr, (int32_t *)nullptr,
                            (int32_t *)nullptr, std::max<int64_t>(nE, 1), 0, 31);
    if (e == hipSuccess && max_last_bin(nV, nnz) > kBigMax)
        e = prim_sort_pairs(nullptr, t[3], (uint32_t *)nullptr, (uint32_t *)nullptr, (int32_t *)nullptr,
                            (int32_t *)nullptr, std::max<int64_t>(nE, 1), 0, bits_for(nV + 1));
    if (e == hipSuccess && max_huge > 0)
        e = prim_segmented_sort_keys(nullptr, t[4], (uint32_t *)nullptr, (uint32_t *)nullptr, nnz, max_huge,
                                     (int32_t *)nullptr, (int32_t *)nullptr, 0, bits_for(nV));
    if (e == hipSuccess && bucketed_best(nV, nnz))
        e = prim_sort_pairs(nullptr, t[5], (uint32_t *)nullptr, (uint32_t *)nullptr, (int32_t *)nullptr,
                            (int32_t *)nullptr, nnz, bucket_shift(nV), bits_for(nV));
    if (e != hipSuccess)
        return fail(HNV_EDEVICE, std::string("sort / scan storage query (needs a visible GPU): ") +
                                     hipGetErrorString(e));
    L.temp_bytes = *std::max_element(t, t + 7);
    L.temp = take(L.temp_bytes);
    L.total = (off + 255) & ~size_t(255);
    return HNV_OK;
}

hnv_status check_sizes(int64_t n_nodes, int64_t n_edges, int64_t nnz, int k)
{
    if (n_nodes < 0 || n_edges < 0 || nnz < 0 || k < 0)
        return fail(HNV_EINVAL, "negative size");
    if (n_nodes >= INT_MAX || n_edges >= INT_MAX || nnz >= INT_MAX)
        return fail(HNV_EUNSUPPORTED, "sizes must be below 2^31");
    if (k % 4 != 0 || k > (1 << 16) || (int64_t)n_edges * k >= INT64_MAX / 8)
        return fail(HNV_EUNSUPPORTED, "feature width k must be a multiple of 4 up to 65536");
    return HNV_OK;
}

// One coarsening step; featureless when x is NULL (k = 0), else on the
// cosine of bag-of-words features with X' summed into c_x.
hnv_status coarsen_device(int64_t n_nodes, int64_t n_edges, int64_t nnz, const int32_t *edge_ptr,
                          const int32_t *edge_idx, const float *edge_w, const int32_t *x, int k, int32_t *node_rep,
                          int32_t *edge_rep, int32_t *c_edge_ptr, int32_t *c_edge_idx, float *c_edge_w,
                          int32_t *c_x, int64_t *c_sizes, void *workspace, size_t ws_bytes, void *stream)
{
    clear_error();
    hnv_status st = check_sizes(n_nodes, n_edges, nnz, k);
    if (st != HNV_OK)
        return st;
    if (!c_sizes || !edge_ptr || !c_edge_ptr || (nnz > 0 && (!edge_idx || !c_edge_idx)) ||
        (n_nodes > 0 && !node_rep) || (n_edges > 0 && !edge_rep))
        return fail(HNV_EINVAL, "a required pointer is NULL");
    const bool feat = k > 0;
    if (feat && n_nodes > 0 && (!x || !c_x))
        return fail(HNV_EINVAL, "features: x and c_x are required");
    if (feat && ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(c_x)) & 15))
        return fail(HNV_EINVAL, "features: x and c_x must be 16-byte aligned");
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255))
        return fail(HNV_EWORKSPACE, "workspace must be non-NULL and 256-byte aligned");
    CoarsenLayout L;
    if ((st = layout(n_nodes, n_edges, nnz, k, L)) != HNV_OK)
        return st;
    if (L.total > ws_bytes)
        return fail(HNV_EWORKSPACE, "workspace of " + std::to_string(ws_bytes) + " bytes, need " +
                                        std::to_string(L.total));
    char *base = static_cast<char *>(workspace);
    auto at = [&](size_t off) { return reinterpret_cast<int32_t *>(base + off); };
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const int nV = (int)n_nodes, nE = (int)n_edges, nz = (int)nnz;
    const int per = window_size(n_edges);
    const unsigned wgrid = window_grid(n_edges);
    auto sync_read = [&](void *dst, const void *src, size_t n) -> hnv_status {
        hipError_t e = hipMemcpyAsync(dst, src, n, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess)
            e = hipStreamSynchronize(s);
        return e == hipSuccess ? HNV_OK : fail(HNV_EDEVICE, std::string("read-back: ") + hipGetErrorString(e));
    };

    // 0. input check (every later kernel trusts offsets, member ids, counts)
    int *flag = reinterpret_cast<int *>(base + L.flag);
    unsigned long long *total = reinterpret_cast<unsigned long long *>(base + L.flag + 8);
    k_fill<<<1, kThreads, 0, s>>>(flag, 12, 0);
    int32_t *first = at(L.first);
    uint32_t *size_key = reinterpret_cast<uint32_t *>(base + L.keys_in);
    if (nE > 0)
        k_check_level<<<wgrid, kThreads, 0, s>>>(edge_ptr, edge_idx, edge_w, n_nodes, per, n_edges, nnz, 1, nullptr,
                                                        size_key, kSizeBins - 1, first, flag);
    if (feat && nV > 0) {
        const int kp4 = (k <= kByteCols ? byte_stride(k) : k) / 4;
        k_fcheck<<<(unsigned)std::min<int64_t>(grid_for((int64_t)nV * kp4), 2048), kThreads, 0, s>>>(
            reinterpret_cast<const int4 *>(x), n_nodes, k / 4, kp4, flag, flag + 1, total,
            k <= kByteCols ? reinterpret_cast<uint32_t *>(at(L.fsum)) : nullptr);
    }
    if ((st = dev_check("coarsening input check")) != HNV_OK)
        return st;
    // The checks' result: read here on the feature path; on the featureless
    // path with the coarse sizes at the end (every kernel there that follows
    // offsets or member ids, or writes an output, first reads the check
    // word and does nothing when it is set).
    struct {
        int bad, largest;   // check bits; the largest count
        unsigned long long total;
    } chk{};
    auto report = [&]() -> hnv_status {
        if (nE == 0) {
            int32_t p0 = 0;
            if (hnv_status r = sync_read(&p0, edge_ptr, 4); r != HNV_OK)
                return r;
            if (p0 != 0 || nz != 0)
                chk.bad |= 1;
        }
        if (chk.bad & 1)
            return fail(HNV_EINVAL, "edge_ptr: offsets must start at 0, increase, end at nnz, no empty hyperedge");
        if (chk.bad & 2)
            return fail(HNV_ERANGE, "a member id is outside [0, n_nodes)");
        if (chk.bad & 4)
            return fail(HNV_EUNSORTED, "member lists must be strictly ascending");
        if (chk.bad & 8)
            return fail(HNV_EINVAL, "weights must be finite and > 0");
        if ((chk.bad & 16) || chk.total >= (1ull << 31))
            return fail(HNV_EINVAL, "features must be counts >= 0 with a total below 2^31");
        return HNV_OK;
    };
    if (feat) {
        if ((st = sync_read(&chk, flag, sizeof(chk))) != HNV_OK || (st = report()) != HNV_OK)
            return st;
    }
    // counts that fit a byte, in rows of one 16-byte piece per lane: the byte path
    const bool bytes = feat && k <= kByteCols && chk.largest <= 255;

    int32_t *order = at(L.order), *rank = at(L.rank), *best = at(L.best), *choice = at(L.choice);
    int32_t *gflag = at(L.gflag), *gid = at(L.gid);
    int32_t *mapped = at(L.mapped), *lists = at(L.lists);
    EdgeCount *count = reinterpret_cast<EdgeCount *>(base + L.count);
    EdgeCount *place = reinterpret_cast<EdgeCount *>(base + L.at);
    int64_t *sizes = reinterpret_cast<int64_t *>(base + L.sizes);
    void *temp = base + L.temp;
    size_t tb = L.temp_bytes;
    SizeOrder S{};
    if (nE > 0) {
        // 1. ranks in the order (weight descending, size ascending, id
        // ascending): the size order, which is the whole order without weights
        int32_t *bins = at(L.bins), *offs = at(L.bin_offs);
        int32_t *by_size = edge_w ? at(L.ids_in) : order, *size_rank = edge_w ? nullptr : rank;
        const int rounds = bin_rounds(n_edges);
        const int64_t tiles = bin_tiles(n_edges), last_bin = max_last_bin(n_nodes, nnz);
        S = SizeOrder{by_size, offs, tiles, n_edges};
        k_bin_count<<<(unsigned)tiles, kThreads, 0, s>>>(size_key, n_edges, nullptr, kSizeBins, rounds, tiles, bins);
        if (prim_exclusive_sum(temp, tb, bins, offs, tiles * kSizeBins, s) != hipSuccess)
            return fail(HNV_EDEVICE, "scan of the size counts");
        if (last_bin <= kBigMax) {
            k_bin_scatter<<<(unsigned)tiles, kThreads, 0, s>>>(size_key, nullptr, n_edges, nullptr, kSizeBins,
                                                               bits_for(kSizeBins), rounds, tiles, offs, nullptr,
                                                               by_size, size_rank);
            if (last_bin > 0) {
                int32_t *tmp = at(L.keys_out);
                k_big_rank<<<grid_for(last_bin), kThreads, 0, s>>>(edge_ptr, by_size, offs, tiles, n_edges, tmp,
                                                                   size_rank, flag);
                k_big_order<<<grid_for(last_bin), kThreads, 0, s>>>(tmp, offs, tiles, n_edges, by_size, flag);
            }
        } else {
            uint32_t *kin = reinterpret_cast<uint32_t *>(base + L.keys_in);
            uint32_t *kout = reinterpret_cast<uint32_t *>(base + L.keys_out);
            int32_t *ids = reinterpret_cast<int32_t *>(kin + n_edges);
            k_size_keys<<<grid_for(nE), kThreads, 0, s>>>(edge_ptr, n_edges, kin, ids);
            tb = L.temp_bytes;
            if (prim_sort_pairs(temp, tb, kin, kout, ids, by_size, nE, 0, bits_for(n_nodes + 1), s) != hipSuccess)
                return fail(HNV_EDEVICE, "radix sort of hyperedge sizes");
            if (!edge_w)
                k_rank<<<grid_for(nE), kThreads, 0, s>>>(by_size, n_edges, rank);
        }
        if (edge_w) {
            uint32_t *kin = reinterpret_cast<uint32_t *>(base + L.keys_in);
            uint32_t *kout = reinterpret_cast<uint32_t *>(base + L.keys_out);
            k_weight_keys<<<grid_for(nE), kThreads, 0, s>>>(by_size, edge_w, n_edges, kin);
            tb = L.temp_bytes;
            if (prim_sort_pairs(temp, tb, kin, kout, by_size, order, nE, 0, 31, s) != hipSuccess)
                return fail(HNV_EDEVICE, "radix sort of hyperedge weights");
            k_rank<<<grid_for(nE), kThreads, 0, s>>>(order, n_edges, rank);
        }
    }
    if (nV > 0) {
        // 2. choices: the least rank, or (features) the least rank among the
        // hyperedges of best cosine score
        const bool buckets = nE > 0 && !feat && bucketed_best(n_nodes, nnz);
        if (!buckets)
            k_fill<<<grid_for(nV), kThreads, 0, s>>>(best, n_nodes, INT_MAX);
        if (nE > 0 && !feat) {
            if (buckets) {
                // (mapped and lists are free until step 5)
                int32_t *pr = mapped, *pr_sorted = at(L.spare);
                uint32_t *nodes_sorted = reinterpret_cast<uint32_t *>(lists);
                const int shift = bucket_shift(n_nodes);
                const int64_t nb = bucket_count(n_nodes);
                int64_t *bstart = reinterpret_cast<int64_t *>(base + L.bstart);
                k_inc_rank<<<wgrid, kThreads, 0, s>>>(edge_ptr, rank, per, n_edges, nnz, pr, flag);
                tb = L.temp_bytes;
                if (prim_sort_pairs(temp, tb, reinterpret_cast<const uint32_t *>(edge_idx), nodes_sorted, pr,
                                    pr_sorted, nz, shift, bits_for(n_nodes), s) != hipSuccess)
                    return fail(HNV_EDEVICE, "partition of incidences by node");
                k_bucket_starts<<<grid_for(nb + 1), kThreads, 0, s>>>(nodes_sorted, nnz, shift, nb, bstart);
                k_bucket_min<<<(unsigned)nb, kBucketThreads, 0, s>>>(nodes_sorted, pr_sorted, bstart, shift, n_nodes,
                                                                     best, flag);
            } else {
                k_best<<<wgrid, kThreads, 0, s>>>(edge_ptr, edge_idx, rank, per, n_edges, nnz, best, flag);
            }
        }
        if (nE > 0 && feat) {
            int32_t *fsum = at(L.fsum);
            int64_t *fsq = reinterpret_cast<int64_t *>(base + L.fsq);
            double *q = reinterpret_cast<double *>(base + L.q);
            unsigned long long *bestq = reinterpret_cast<unsigned long long *>(base + L.bestq);
            const dim3 wave_grid = fold_grid((n_edges + kThreads / kWave - 1) / (kThreads / kWave));
            k_fill<<<grid_for(2 * (int64_t)nV), kThreads, 0, s>>>(reinterpret_cast<int32_t *>(bestq),
                                                                   2 * (int64_t)nV, 0);
            if (bytes) {
                const unsigned char *x8 = reinterpret_cast<const unsigned char *>(fsum);
                const int kp = byte_stride(k);
#define HNV_BYTES(GG) launch_byte_scores<GG>(s, edge_ptr, edge_idx, x8, kp, n_edges, nnz, q, bestq)
                if (kp <= 16) HNV_BYTES(1);
                else if (kp <= 32) HNV_BYTES(2);
                else if (kp <= 64) HNV_BYTES(4);
                else if (kp <= 128) HNV_BYTES(8);
                else if (kp <= 256) HNV_BYTES(16);
                else if (kp <= 512) HNV_BYTES(32);
                else HNV_BYTES(64);
#undef HNV_BYTES
            } else {
                int32_t *inc_edge = at(L.inc_edge);
                k_inc_edge<<<wgrid, kThreads, 0, s>>>(edge_ptr, per, n_edges, nnz, inc_edge);
                switch (pieces_for(k)) {
                case 1: launch_edge_features<1>(wave_grid, s, edge_ptr, edge_idx, inc_edge, x, k, n_edges, nnz, fsum, fsq, q, bestq); break;
                case 2: launch_edge_features<2>(wave_grid, s, edge_ptr, edge_idx, inc_edge, x, k, n_edges, nnz, fsum, fsq, q, bestq); break;
                case 4: launch_edge_features<4>(wave_grid, s, edge_ptr, edge_idx, inc_edge, x, k, n_edges, nnz, fsum, fsq, q, bestq); break;
                case 8: launch_edge_features<8>(wave_grid, s, edge_ptr, edge_idx, inc_edge, x, k, n_edges, nnz, fsum, fsq, q, bestq); break;
                default: launch_edge_features<0>(wave_grid, s, edge_ptr, edge_idx, inc_edge, x, k, n_edges, nnz, fsum, fsq, q, bestq);
                }
            }
            k_best_feat<<<wgrid, kThreads, 0, s>>>(edge_ptr, edge_idx, rank, q, bestq, per, n_edges, nnz, best);
        }
        k_choice<<<grid_for(nV), kThreads, 0, s>>>(best, order, n_nodes, choice, first);
        // 3. group numbering by smallest node
        k_group_flags<<<grid_for(nV), kThreads, 0, s>>>(choice, first, n_nodes, gflag);
        tb = L.temp_bytes;
        if (prim_exclusive_sum(temp, tb, gflag, gid, nV, s) != hipSuccess)
            return fail(HNV_EDEVICE, "scan of group flags");
        k_node_rep<<<grid_for(nV), kThreads, 0, s>>>(choice, first, gid, n_nodes, node_rep, sizes, flag);
    }
    if (nE > 0) {
        // 4. coarse member lists, and with them the removed hyperedges
        const int64_t max_big = max_lists(n_nodes, nnz, kSortLong), max_huge = max_lists(n_nodes, nnz, kSortBlock);
        int32_t *huge = at(L.huge), *huge_begin = at(L.huge_ends), *huge_end = huge_begin + max_huge;
        int32_t *n_huge = at(L.n_huge);
        auto blocks = [&](int longer_than, int per_block, int most) {   // for the lists of more than `longer_than`
            return (unsigned)std::min<int64_t>(max_lists(n_nodes, nnz, longer_than) / per_block + 1, most);
        };
        k_list_short<<<grid_for(nE), kThreads, 0, s>>>(edge_ptr, edge_idx, node_rep, best, rank, n_edges, lists, count,
                                                       flag);
        if (max_lists(n_nodes, nnz, kSortThread) > 0)
            k_list_wave<<<blocks(kSortThread, kThreads / kWave, kListBlocks), kThreads, 0, s>>>(
                edge_ptr, edge_idx, node_rep, best, rank, S, lists, count, flag);
        if (max_lists(n_nodes, nnz, kSortMid) > 0)
            k_list_long<<<blocks(kSortMid, 1, kListBlocks), kThreads, 0, s>>>(edge_ptr, edge_idx, node_rep, best, rank, S,
                                                                              lists, count, flag);
        if (max_huge > 0)   // unused segments are empty
            k_fill<<<grid_for(2 * max_huge), kThreads, 0, s>>>(huge_begin, 2 * max_huge, 0);
        if (max_big > 0)
            k_list_block<<<blocks(kSortLong, 1, 512), kSortBlockThreads, 0, s>>>(
                edge_ptr, edge_idx, node_rep, best, rank, S, lists, mapped, count, huge_begin, huge_end, huge, n_huge,
                flag);
        if (max_huge > 0) {
            tb = L.temp_bytes;
            // non-negative ids below n_nodes: sorted as unsigned so only the low bits count
            if (prim_segmented_sort_keys(temp, tb, reinterpret_cast<const uint32_t *>(mapped),
                                         reinterpret_cast<uint32_t *>(lists), nz, max_huge, huge_begin, huge_end, 0,
                                         bits_for(n_nodes), s) != hipSuccess)
                return fail(HNV_EDEVICE, "segmented sort of very long coarse member lists");
            k_list_huge<<<(unsigned)std::min<int64_t>(max_huge, 512), kSortBlockThreads, 0, s>>>(
                edge_ptr, edge_idx, best, rank, huge, n_huge, lists, count, flag);
        }
        // 5. the kept hyperedges' numbers and offsets, and the coarse arrays
        tb = L.temp_bytes;
        if (prim_exclusive_scan(temp, tb, count, place, EdgeCount{0, 0}, nE, EdgeCountPlus(), s) != hipSuccess)
            return fail(HNV_EDEVICE, "scan of the coarse member counts");
        k_emit<<<wgrid, kThreads, 0, s>>>(edge_ptr, count, place, lists, edge_w, per, n_edges, nnz, edge_rep,
                                                 c_edge_ptr, c_edge_idx, c_edge_w, sizes, flag);
        if (max_big > 0)
            k_emit_long<<<dim3(blocks(kSortLong, 1, 256), kEmitSplit), kThreads, 0, s>>>(edge_ptr, count, place, lists, S,
                                                                                         c_edge_idx, flag);
    }
    if (nV == 0 || nE == 0)
        k_sizes_empty<<<1, 64, 0, s>>>(n_nodes, n_edges, c_edge_ptr, sizes, flag);
    if (feat && nV > 0) {
        // 6. X': each coarse node's row is the sum of its fine nodes' rows
        int32_t *gcount = at(L.gcount), *gptr = at(L.gptr), *gcur = at(L.gcur), *gnodes = at(L.gnodes);
        k_fill<<<grid_for(nV + 1), kThreads, 0, s>>>(gcount, n_nodes + 1, 0);
        k_fill<<<grid_for(nV), kThreads, 0, s>>>(gcur, n_nodes, 0);
        k_group_count<<<grid_for(nV), kThreads, 0, s>>>(node_rep, n_nodes, gcount);
        tb = L.temp_bytes;
        if (prim_exclusive_sum(temp, tb, gcount, gptr, nV + 1, s) != hipSuccess)
            return fail(HNV_EDEVICE, "scan of group sizes");
        k_group_fill<<<grid_for(nV), kThreads, 0, s>>>(node_rep, gptr, n_nodes, gcur, gnodes);
        const dim3 wave_grid = fold_grid((n_nodes + kThreads / kWave - 1) / (kThreads / kWave));
        if (bytes) {
            const uint32_t *x8 = reinterpret_cast<const uint32_t *>(at(L.fsum));
            const int kp4 = byte_stride(k) / 4;
            int4 *out = reinterpret_cast<int4 *>(c_x);
#define HNV_BYTES(NC) \
    k_rowsum_bytes<NC><<<wave_grid, kThreads, 0, s>>>(gptr, gnodes, x8, k / 4, kp4, n_nodes, sizes, out)
            if (kp4 <= 64) HNV_BYTES(1);
            else if (kp4 <= 128) HNV_BYTES(2);
            else HNV_BYTES(4);
#undef HNV_BYTES
        } else switch (pieces_for(k)) {
        case 1: launch_group_sums<1>(wave_grid, s, gptr, gnodes, x, k, n_nodes, sizes, c_x); break;
        case 2: launch_group_sums<2>(wave_grid, s, gptr, gnodes, x, k, n_nodes, sizes, c_x); break;
        case 4: launch_group_sums<4>(wave_grid, s, gptr, gnodes, x, k, n_nodes, sizes, c_x); break;
        case 8: launch_group_sums<8>(wave_grid, s, gptr, gnodes, x, k, n_nodes, sizes, c_x); break;
        default: launch_group_sums<0>(wave_grid, s, gptr, gnodes, x, k, n_nodes, sizes, c_x);
        }
    }
    if ((st = dev_check("coarsening kernels")) != HNV_OK)
        return st;
    if (feat)
        return sync_read(c_sizes, sizes, 3 * sizeof(int64_t));
    struct {
        int bad, pad;
        unsigned long long total;
        int64_t sizes[3];
    } back{};
    static_assert(sizeof(back) == 16 + 3 * sizeof(int64_t), "check word and sizes are read as one block");
    if ((st = sync_read(&back, flag, sizeof(back))) != HNV_OK)
        return st;
    chk.bad = back.bad;
    chk.total = back.total;
    if ((st = report()) != HNV_OK)
        return st;
    std::memcpy(c_sizes, back.sizes, sizeof(back.sizes));
    return HNV_OK;
}

}  // namespace
}  // namespace hnv

using namespace hnv;

extern "C" hnv_status hnv_coarsen_workspace_bytes(int64_t n_nodes, int64_t n_edges, int64_t nnz, size_t *bytes)
{
    return hnv_coarsen_features_workspace_bytes(n_nodes, n_edges, nnz, 0, bytes);
}

extern "C" hnv_status hnv_coarsen_features_workspace_bytes(int64_t n_nodes, int64_t n_edges, int64_t nnz, int k,
                                                           size_t *bytes)
{
    clear_error();
    if (!bytes)
        return fail(HNV_EINVAL, "bytes is NULL");
    hnv_status st = check_sizes(n_nodes, n_edges, nnz, k);
    if (st != HNV_OK)
        return st;
    CoarsenLayout L;
    if ((st = layout(n_nodes, n_edges, nnz, k, L)) == HNV_OK)
        *bytes = L.total;
    return st;
}

extern "C" hnv_status hnv_coarsen_level_device(int64_t n_nodes, int64_t n_edges, int64_t nnz,
                                               const int32_t *edge_ptr, const int32_t *edge_idx,
                                               const float *edge_w, int32_t *node_rep, int32_t *edge_rep,
                                               int32_t *c_edge_ptr, int32_t *c_edge_idx, float *c_edge_w,
                                               int64_t *c_sizes, void *workspace, size_t ws_bytes, void *stream)
{
    return coarsen_device(n_nodes, n_edges, nnz, edge_ptr, edge_idx, edge_w, nullptr, 0, node_rep, edge_rep,
                          c_edge_ptr, c_edge_idx, c_edge_w, nullptr, c_sizes, workspace, ws_bytes, stream);
}

extern "C" hnv_status hnv_coarsen_level_features_device(int64_t n_nodes, int64_t n_edges, int64_t nnz,
                                                        const int32_t *edge_ptr, const int32_t *edge_idx,
                                                        const float *edge_w, const int32_t *x, int k,
                                                        int32_t *node_rep, int32_t *edge_rep, int32_t *c_edge_ptr,
                                                        int32_t *c_edge_idx, float *c_edge_w, int32_t *c_x,
                                                        int64_t *c_sizes, void *workspace, size_t ws_bytes,
                                                        void *stream)
{
    if (k <= 0) {
        clear_error();
        return fail(HNV_EUNSUPPORTED, "feature width k must be a multiple of 4 up to 65536");
    }
    return coarsen_device(n_nodes, n_edges, nnz, edge_ptr, edge_idx, edge_w, x, k, node_rep, edge_rep, c_edge_ptr,
                          c_edge_idx, c_edge_w, c_x, c_sizes, workspace, ws_bytes, stream);
}
