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

// A node's word: the pivot's order above its other end.  The other end is
// coded so that walking on makes it smaller in both blocks (in the top one it
// grows), and atomicMin can store a shortened word.
template <bool kTop>
__host__ __device__ inline uint32_t graph_code(int32_t v)
{
    return (uint32_t)(kTop ? kGraphOut - v : v + 1);
}
template <bool kTop>
__host__ __device__ inline int32_t graph_end(unsigned long long word)
{
    return kTop ? kGraphOut - (int32_t)(uint32_t)word : (int32_t)(uint32_t)word - 1;
}

// Places the edge (node pair u, v) of pivot order `ord`.  kTop: the node to
// reduce is the smaller end and the other end grows (kGraphOut last), else
// the larger end and the other end shrinks (-1, no vertex, last).  Long walks
// shorten the pivots they pass by adding to a pivot the next one, where that is
// earlier: each walk of such a path halves it for the next (pms_selftest).
// Returns the steps taken.  (With the other end of the top block uncoded, no
// shortened word was ever stored: k_graph_top_walk of a 128^3 field 2.04 ms,
// now 1.04; of a 64^3 field 263 us, now 155.)
template <bool kTop>
__device__ inline int graph_place(unsigned long long *P, uint32_t ord, int32_t u, int32_t v)
{
    int step = 0;
    for (; u != v; step++) {
        if (kTop ? u > v : u < v) {
            const int32_t t = u;
            u = v;
            v = t;
        }
        // u is the node to reduce, v the other end
        unsigned long long key = ((unsigned long long)ord << 32) | graph_code<kTop>(v);
        unsigned long long cur = graph_load(&P[u]);
        if (cur >= key) {
            cur = atomicMin(&P[u], key);
            if (cur == kGraphEmpty) return step;
            if (cur > key) {  // placed; the displaced pivot plus this one: (its other end, v)
                ord = (uint32_t)(cur >> 32);
                u = graph_end<kTop>(cur);
                continue;
            }
        }
        const int32_t w = graph_end<kTop>(cur);
        if (step >= 16 && w != (kTop ? kGraphOut : -1)) {
            const unsigned long long nx = graph_load(&P[w]);
            if ((uint32_t)(nx >> 32) < (uint32_t)(cur >> 32))  // an earlier pivot (kGraphEmpty is later)
                atomicMin(&P[u], (cur & 0xFFFFFFFF00000000ull) | (uint32_t)nx);
        }
        u = w;
    }
    return step;
}

}  // namespace pms
