// Stable counting sort by keys of at most kBinsMax values, shared by the GPU
// coarsening and the device-built plan.
// Included by the .hip sources only; every symbol has internal linkage.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "hnv_internal.h"
#include "hnv_level_check.h"

namespace hnv {
namespace {

// A stable counting sort of (key, value) pairs by the key, which is below
// n_bins <= kBinsMax: per-tile counts of every key, an exclusive scan of the
// counts laid out key-major (key b of tile t at b * n_tiles + t), and a scatter
// in which each tile places its elements in input order.  It sorts the degree
// tiers of both sides (2 (small_max + 3) keys), the wavefront tier's items
// (2 chunk_keys, at most 1,024) and the coarsening's hyperedge sizes; the result
// equals a stable radix sort's.  The number of pairs is n_max, or *n_dev when that is given (the
// grid is sized for n_max).  Without input values a value is the element's
// index; either output may be absent (null); pos_out (or null): each input
// element's sorted position.
//
// A tile is `rounds` rounds of 64 elements per wavefront, a wavefront's rounds
// consecutive.  The scatter counts its tile once more, per wavefront, and then
// every wavefront places its own elements without waiting for the others (one
// round of the whole workgroup at a time, with three barriers and a walk over
// all bins per round, took 22 us where this takes 15, on average over the
// sorts of levels of 0.3M to 1.2M rows).  Short inputs take short tiles, so
// that their few elements spread over the chip.
constexpr int kBinsMax = 1024;
constexpr int kBinWaves = kThreads / kWave;

inline int bin_rounds(int64_t n) { return n <= (int64_t(1) << 18) ? 4 : 16; }
inline int64_t bin_tiles(int64_t n)
{
    const int64_t tile = (int64_t)kThreads * bin_rounds(n);
    return (n + tile - 1) / tile;
}
// entries of the digit counts of a sort of up to n pairs (a shorter input may
// have more tiles than a longer one)
inline int64_t bin_cap(int64_t n, int n_bins)
{
    return n_bins * std::max<int64_t>(bin_tiles(n), std::min<int64_t>(n, int64_t(1) << 18) / (4 * kThreads) + 1);
}

__device__ inline int64_t pairs_of(int64_t n_max, const int64_t *n_dev)
{
    return n_dev ? min(n_max, *n_dev) : n_max;
}

__global__ __launch_bounds__(kThreads) void k_bin_count(const uint32_t *__restrict__ key, int64_t n_max,
                                                        const int64_t *__restrict__ n_dev, int n_bins, int rounds,
                                                        int64_t n_tiles,
                                                        int32_t *__restrict__ counts)
{
    __shared__ int32_t h[kBinsMax];
    for (int b = threadIdx.x; b < n_bins; b += kThreads)
        h[b] = 0;
    __syncthreads();
    const int64_t n = pairs_of(n_max, n_dev);
    const int64_t base = (int64_t)blockIdx.x * kThreads * rounds;
    for (int k = 0; k < rounds; ++k) {
        const int64_t i = base + (int64_t)k * kThreads + threadIdx.x;
        if (i < n)
            atomicAdd(&h[key[i]], 1);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < n_bins; b += kThreads)
        counts[(int64_t)b * n_tiles + blockIdx.x] = h[b];
}

// The lanes of the wavefront that hold the same key (active lanes only):
// one ballot per key bit.  Every lane of the wavefront must call it.
__device__ inline uint64_t same_key_lanes(uint32_t key, int bits, bool active)
{
    uint64_t m = __ballot(active);
    for (int b = 0; b < bits; ++b) {
        const bool one = (key >> b) & 1u;
        const uint64_t ones = __ballot(active && one);
        m &= one ? ones : ~ones;
    }
    return m;
}

__global__ __launch_bounds__(kThreads) void k_bin_scatter(const uint32_t *__restrict__ key,
                                                          const int32_t *__restrict__ val, int64_t n_max,
                                                          const int64_t *__restrict__ n_dev, int n_bins, int bits,
                                                          int rounds,
                                                          int64_t n_tiles, const int32_t *__restrict__ offs,
                                                          uint32_t *__restrict__ key_out,
                                                          int32_t *__restrict__ val_out,
                                                          int32_t *__restrict__ pos_out)
{
    __shared__ int32_t next[kBinWaves][kBinsMax];   // counts, then the next free position, per wavefront
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    for (int b = threadIdx.x; b < n_bins; b += kThreads)
        for (int w = 0; w < kBinWaves; ++w)
            next[w][b] = 0;
    __syncthreads();
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
    const int64_t n = pairs_of(n_max, n_dev);
    const int64_t first = ((int64_t)blockIdx.x * kBinWaves + wave) * rounds * kWave + lane;
    for (int k = 0; k < rounds; ++k) {
        const int64_t i = first + (int64_t)k * kWave;
        if (i < n)
            atomicAdd(&next[wave][key[i]], 1);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < n_bins; b += kThreads) {
        int32_t at = offs[(int64_t)b * n_tiles + blockIdx.x];
        for (int w = 0; w < kBinWaves; ++w) {
            const int32_t c = next[w][b];
            next[w][b] = at;
            at += c;
        }
    }
    __syncthreads();
    for (int k = 0; k < rounds; ++k) {   // no barrier inside: wavefronts may stop early
        const int64_t i = first + (int64_t)k * kWave;
        const bool act = i < n;
        if (__ballot(act) == 0)
            break;
        const uint32_t kv = act ? key[i] : 0u;
        const uint64_t peers = same_key_lanes(kv, bits, act);
        const int leader = peers ? __ffsll((long long)peers) - 1 : lane;
        int32_t at = 0;
        if (act && lane == leader)
            at = atomicAdd(&next[wave][kv], (int32_t)__popcll(peers));
        at = __shfl(at, leader, kWave);
        if (act) {
            const int32_t pos = at + (int32_t)__popcll(peers & below);
            if (key_out)
                key_out[pos] = kv;
            if (val_out)
                val_out[pos] = val ? val[i] : (int32_t)i;
            if (pos_out)
                pos_out[i] = pos;
        }
    }
}

}  // namespace
}  // namespace hnv
