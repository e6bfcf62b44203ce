// A lane's share of the weights of a node's star edges (plain C++, also for the host).
#pragma once

#include <cstdint>

#include "hnv_internal.h"

namespace hnv {

// The weights of the star edges j, j + step, .. below end: written to wn, and
// their sum, U gathers in flight.  Positions are unsigned: a list may end at
// 2^31 - 1, and the last round passes it by up to U * step.
template <int U>
HNV_HD inline double sum_weights(const int32_t *idx, const float *w, int64_t n_nodes, uint32_t j, uint32_t end,
                                 uint32_t step, float *wn)
{
    double t = 0.0;
    for (; j < end; j += U * step) {
        float x[U];
#pragma unroll
        for (int k = 0; k < U; ++k)
            x[k] = j + k * step < end ? w[idx[j + k * step] - n_nodes] : 0.0f;
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (j + k * step < end) {
                wn[j + k * step] = x[k];
                t += (double)x[k];
            }
    }
    return t;
}

}  // namespace hnv
