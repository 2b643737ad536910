// The placement step of the blocks that are graphs (pms_graph.h), shared by
// the reductions of matrices and of Vietoris-Rips filtrations.
#pragma once

#include "pms_common.h"

namespace pms {

constexpr unsigned long long kGraphEmpty = ~0ull;
constexpr int32_t kGraphOut = 0x7FFFFFFF;  // the node beyond a boundary face (top block)

__device__ inline unsigned long long graph_load(const unsigned long long *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Places the edge (node pair u, v) of pivot order `ord`.  kTop: the node to
// reduce is the smaller end and the other end grows (kGraphOut last), else
// the larger end and the other end shrinks (-1, no vertex, last).  Long walks
// shorten the pivots they pass (adding to a pivot an earlier one), so that a
// path is walked in full only once.
template <bool kTop>
__device__ inline void graph_place(unsigned long long *P, uint32_t ord, int32_t u, int32_t v)
{
    for (int step = 0; u != v; step++) {
        if (kTop ? u > v : u < v) {
            const int32_t t = u;
            u = v;
            v = t;
        }
        // u is the node to reduce, v the other end
        unsigned long long key = ((unsigned long long)ord << 32) | (uint32_t)(kTop ? v : v + 1);
        unsigned long long cur = graph_load(&P[u]);
        if (cur >= key) {
            cur = atomicMin(&P[u], key);
            if (cur == kGraphEmpty) return;
            if (cur > key) {  // placed; the displaced pivot plus this one: (its other end, v)
                ord = (uint32_t)(cur >> 32);
                u = (int32_t)(uint32_t)cur - (kTop ? 0 : 1);
                continue;
            }
        }
        const int32_t w = (int32_t)(uint32_t)cur - (kTop ? 0 : 1);
        if (step >= 16 && w != (kTop ? kGraphOut : -1)) {
            const unsigned long long nx = graph_load(&P[w]);
            if ((uint32_t)(nx >> 32) < (uint32_t)(cur >> 32))  // an earlier pivot (kGraphEmpty is later)
                atomicMin(&P[u], (cur & 0xFFFFFFFF00000000ull) | (uint32_t)nx);
        }
        u = w;
    }
}

}  // namespace pms
