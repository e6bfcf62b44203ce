// Device-side checks of a level given as device arrays (int32 offsets), and
// small helpers shared by the GPU coarsening and the device-built plan.
// Included by the .hip sources only; every symbol has internal linkage.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace hnv {
namespace {

constexpr int kThreads = 256;

inline unsigned grid_for(int64_t n) { return (unsigned)((n + kThreads - 1) / kThreads); }

// Bits that hold every value in [0, n).
inline int bits_for(int64_t n)
{
    int b = 1;
    while (b < 32 && (int64_t(1) << b) < n)
        ++b;
    return b;
}

__global__ __launch_bounds__(kThreads) void k_fill(int32_t *__restrict__ p, int64_t n, int32_t v)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n)
        p[i] = v;
}

// A wavefront's window of `per` (at most 64) consecutive hyperedges, one per
// lane: the incidences [begin, end) of the window are walked 64 at a time
// whatever their hyperedges, so that reads and writes per incidence are in
// order and lists of any length keep all lanes busy.  The first incidences of
// the hyperedges are bits of 64-bit words in LDS, one word per 64 incidences:
// an incidence's hyperedge is the number of bits up to it (its place among
// the window's hyperedges with members; `lane_of` gives their lanes where
// some have none).  load(j, l, ok) and use(j, l, ok, value) get the incidence,
// its hyperedge's lane and whether j < end (when not, nothing may be
// accessed), and use also whether it is its hyperedge's first; every lane
// calls them together, so they may shuffle; U loads are in flight.  Of
// offsets that do not ascend some incidence gets a wrong lane below 64.
//
// Measured: walking each list by its own thread, and those of more than 32 by
// the wavefront, took 51 us where this takes 31 for the checks of 13.1M
// incidences; finding the hyperedge by a binary search over the lanes (six
// shuffles per 64 incidences) 43 us.
struct Window {
    int32_t first;        // this lane's hyperedge's first incidence (end past the last hyperedge)
    int32_t begin, end;   // the window's incidences, clamped to [0, nnz]
    bool some;            // the hyperedge has members
};

constexpr int kWalk = 4;            // incidences in flight per lane
constexpr int kWalkWords = 64;      // words of start bits per wavefront: 4096 incidences at a time

struct WalkLds {
    unsigned long long bits[kThreads / 64][kWalkWords];
    int32_t lane_of[kThreads / 64][64];
};

// Hyperedges per window: 64, or fewer where a launch would not fill the chip
// otherwise (at 8K hyperedges and 50K incidences the least ranks took 25 us
// with windows of 64, 11 with 4).
inline int window_size(int64_t n_edges)
{
    int per = 4;
    while (per < 64 && n_edges / per > 8192)
        per *= 2;
    return per;
}
inline unsigned window_grid(int64_t n_edges)
{
    const int64_t per_block = (int64_t)window_size(n_edges) * (kThreads / 64);
    return (unsigned)((n_edges + per_block - 1) / per_block);
}

// The first hyperedge of this wavefront's window.
__device__ __forceinline__ int64_t window_start(int per)
{
    return ((int64_t)blockIdx.x * (kThreads / 64) + threadIdx.x / 64) * per;
}

__device__ __forceinline__ Window window_of(const int32_t *__restrict__ ptr, int64_t e0, int per, int64_t n_edges,
                                            int64_t nnz)
{
    const int lane = threadIdx.x % 64;
    const int64_t e1 = e0 + per < n_edges ? e0 + per : n_edges;
    Window W;
    W.begin = (int32_t)max<int64_t>(0, min<int64_t>(ptr[e0], nnz));
    W.end = (int32_t)max<int64_t>(W.begin, min<int64_t>(ptr[e1], nnz));
    const int32_t next = e0 + lane < e1 ? ptr[e0 + lane + 1] : 0;
    W.first = e0 + lane < e1 ? ptr[e0 + lane] : W.end;
    W.some = e0 + lane < e1 && next > W.first;
    return W;
}

// Orders this wavefront's LDS accesses (it shares the words with no other).
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <int U, typename L, typename C>
__device__ __forceinline__ void walk_window(const Window &W, WalkLds &lds, L load, C use)
{
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    unsigned long long *bits = lds.bits[wave];
    const unsigned long long with = __ballot(W.some), upto = ~0ull >> (63 - lane);
    // all hyperedges with members in the first lanes: a hyperedge's place is its lane
    const bool gaps = (with & (with + 1)) != 0;
    if (gaps && W.some)
        lds.lane_of[wave][__popcll(with & (upto >> 1))] = lane;
    const uint32_t end = (uint32_t)W.end, span = kWalkWords * 64;   // (unsigned: end may be close to 2^31)
    int before = -1;   // place of the last hyperedge that starts before the next word
    for (uint32_t s0 = (uint32_t)W.begin; s0 < end; s0 += span) {
        wave_lds_fence();   // the last span's words have been read
        bits[lane] = 0;
        wave_lds_fence();
        const uint32_t at = (uint32_t)W.first - s0;
        if (W.some && (uint32_t)W.first >= s0 && at < span)
            atomicOr(&bits[at / 64], 1ull << (at % 64));
        wave_lds_fence();
        const uint32_t s1 = end - s0 < span ? end : s0 + span;
        for (uint32_t j0 = s0; j0 < s1; j0 += 64 * U) {
            int l[U];
            bool starts[U], ok[U];
            decltype(load(0u, 0, false)) x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t j = j0 + 64 * u + lane;
                const uint32_t word = (j0 - s0) / 64 + u;
                const unsigned long long m = word < kWalkWords ? bits[word] : 0;   // uniform
                int p = before + (int)__popcll(m & upto);
                before += (int)__popcll(m);
                p = p < 0 ? 0 : p & 63;   // (in range with any offsets)
                l[u] = gaps ? lds.lane_of[wave][p] & 63 : p;
                starts[u] = (m >> lane) & 1;
                ok[u] = j < s1;
                x[u] = load(j, l[u], ok[u]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                use(j0 + 64 * u + lane, l[u], ok[u], starts[u], x[u]);
        }
    }
}

// inc_edge[j] = the hyperedge of incidence j (the offsets are valid).
__global__ __launch_bounds__(kThreads) void k_inc_edge(const int32_t *__restrict__ ptr, int per, int64_t n_edges,
                                                       int64_t nnz, int32_t *__restrict__ inc_edge)
{
    __shared__ WalkLds lds;
    const int64_t e0 = window_start(per);
    if (e0 >= n_edges)
        return;   // uniform over the wavefront
    walk_window<kWalk>(
        window_of(ptr, e0, per, n_edges, nnz), lds, [](uint32_t, int, bool) { return 0; },
        [&](uint32_t j, int l, bool ok, bool, int) {
            if (ok)
                inc_edge[j] = (int32_t)(e0 + l);
        });
}

// Flag bits of the checks: 0 offsets, 1 member range, 2 member order,
// 3 weights.  All checks of a level in one pass over its hyperedges: the offsets
// (start at 0, end at nnz, never decrease, stay in [0, nnz]) and every member's
// range; with `full` also no empty hyperedge, ascending members, and weights
// finite and > 0.  Every
// access stays in the arrays whatever the offsets are; members that no window
// reaches are not looked at, but then the offsets are bad.  With inc_edge also
// the hyperedge of every incidence (gaps and wrong ones with bad offsets); with
// key and first the coarsening's start: each size, at most key_max, and
// INT_MAX.  Bound by the 4 bytes read per incidence (and 4 written): 31 us
// at 13.1M incidences and 1.5M hyperedges, where a pass per incidence over a
// stored incidence map and the passes that wrote the map took 78.
__global__ __launch_bounds__(kThreads) void k_check_level(const int32_t *__restrict__ ptr,
                                                          const int32_t *__restrict__ idx,
                                                          const float *__restrict__ w, int64_t n_nodes,
                                                          int per, int64_t n_edges, int64_t nnz, int full,
                                                          int32_t *__restrict__ inc_edge, uint32_t *__restrict__ key,
                                                          int key_max, int32_t *__restrict__ first,
                                                          int *__restrict__ flag)
{
    __shared__ WalkLds lds;
    const int64_t e0 = window_start(per);
    if (e0 >= n_edges)
        return;   // uniform over the wavefront
    const int64_t e = e0 + threadIdx.x % 64;
    int bad = 0;
    if (threadIdx.x % 64 < per && e < n_edges) {
        const int64_t a = ptr[e], b = ptr[e + 1];
        if (a < 0 || b < a || b > nnz || (e == 0 && a != 0) || (e == n_edges - 1 && b != nnz) || (full && a == b))
            bad |= 1;
        if (full && w && !(w[e] > 0.0f && w[e] < INFINITY))
            bad |= 8;
        if (key)
            key[e] = (uint32_t)max<int64_t>(0, min<int64_t>(b - a, key_max));
        if (first)
            first[e] = 0x7fffffff;
    }
    const Window W = window_of(ptr, e0, per, n_edges, nnz);
    struct Member {
        int32_t v, before;
    };
    walk_window<kWalk>(
        W, lds,
        [&](uint32_t j, int, bool ok) {
            return Member{ok ? idx[j] : 0, ok && j > (uint32_t)W.begin ? idx[j - 1] : -1};
        },
        [&](uint32_t j, int l, bool ok, bool starts, const Member &m) {
            if (!ok)
                return;
            if (m.v < 0 || m.v >= n_nodes)
                bad |= 2;
            else if (full && !starts && m.before >= m.v)
                bad |= 4;
            if (inc_edge)
                inc_edge[j] = (int32_t)(e0 + l);
        });
    if (bad)
        atomicOr(flag, bad);
}

}  // namespace
}  // namespace hnv
