// The blocks of the boundary matrix that are graphs, reduced without columns
// (included by pms_reduce.hip after the reduction's device state).
//
// The rows of dimension b and the columns of dimension b + 1 form a block of
// d; the blocks' pairs are found independently (Sec. 2.3: low* is a property
// of the complex).  Two kinds of block have at most two non-zeros on one side
// and are graphs:
//
//   block 0    an edge's column holds its (at most) two vertices;
//   top block  on a triangulated volume a top simplex meets each face from at
//              most two sides: a face's row holds at most two columns.
//
// In block 0 the reduced column of an edge is again a pair of vertices
// (additions replace one end), so the whole state is, per vertex, the pivot
// edge and its other end.  The top block is reduced from its rows: the same
// pairs come from the anti-transposed matrix (rows as columns, in decreasing
// order, each reduced to its smallest entry), where a face's column holds its
// two cofaces.  One 64-bit word per node holds the pivot, in the order of the
// reduction (block 0: the edge; top: the face, larger first), above the other
// end, and one atomicMin both compares and places it: a loser continues from
// the winner's other end, a displaced pivot is carried on by the thread that
// displaced it.  Every interleaving ends in the same words (the reduced
// matrix's lows are unique), and no other memory is shared, so no fences.
//
// What this replaces: on a smooth 64^3 field a tetrahedron's column adds up
// to 11 758 pivots one after the other (each addition about 1 us in k_chain),
// while the longest walk from the triangles' side is 78 nodes.  Measured:
// build + reduce + backward of 64^3 fields 42.0 -> 4.8 ms, build + reduce of
// 128^3 399 -> 41.9 ms, of 32^3 white noise 9.3 -> 3.9 ms.  The kernels here
// are bound by scattered 4- and 8-byte accesses (a node's word, a face's two
// cofaces), not by the walks.
#pragma once

constexpr unsigned long long kGraphEmpty = ~0ull;
constexpr int32_t kGraphOut = 0x7FFFFFFF;  // the node beyond a boundary face (top block)
constexpr int32_t kNotGraph0 = 1, kNotGraphTop = 2;

// Columns per dimension (7: that dimension and above).
__global__ void __launch_bounds__(kBlock) k_dim_count(Dev d)
{
    __shared__ int32_t s_n[8];
    if (threadIdx.x < 8) s_n[threadIdx.x] = 0;
    __syncthreads();
    int32_t n[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int64_t j = blockIdx.x * (int64_t)kBlock + threadIdx.x; j < d.m; j += (int64_t)gridDim.x * kBlock) {
        const int dj = min((int)d.dim[j], 7);
#pragma unroll
        for (int k = 0; k < 8; k++) n[k] += dj == k;
    }
#pragma unroll
    for (int k = 0; k < 8; k++) {
        const int32_t t = wave_sum_dpp(n[k]);
        if ((threadIdx.x & (kWave - 1)) == 0 && t) atomicAdd(&s_n[k], t);
    }
    __syncthreads();
    if (threadIdx.x < 8 && s_n[threadIdx.x]) atomicAdd(&d.cnt->n_dim[threadIdx.x], s_n[threadIdx.x]);
}

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

// The rows of edge j as nodes (a missing one: -1); false when it has more than two.
__device__ inline bool graph_edge(const Dev &d, int64_t j, int32_t *u, int32_t *v)
{
    const int32_t n = d.len[j];
    const int64_t s = d.col_ptr[j];
    *u = n > 0 ? d.rows[s] : -1;
    *v = n > 1 ? d.rows[s + 1] : -1;
    return n <= 2;
}

// The last row of column j, -1 when empty.
__device__ inline int32_t last_row(const Dev &d, int32_t j)
{
    const int32_t n = d.len[j];
    return n > 0 ? d.rows[d.col_ptr[j] + n - 1] : -1;
}

// Block 0, edges whose larger vertex has no earlier edge: pivots as they are.
// Also counts the pivots known from beta (every dimension): the columns whose
// low, after the rows of columns with beta are dropped, is beta.
__global__ void __launch_bounds__(kBlock) k_graph0_seed(Dev d)
{
    int32_t nb = 0;
    for (int64_t j = blockIdx.x * (int64_t)kBlock + threadIdx.x; j < d.m; j += (int64_t)gridDim.x * kBlock) {
        const int32_t b = d.beta[j];
        if (b >= 0) {
            const int32_t *c = d.rows + d.col_ptr[j];
            int32_t n = d.len[j];
            while (n > 0 && is_neg(d.neg, c[n - 1])) n--;
            nb += n > 0 && c[n - 1] == b;
        }
        if (d.dim[j] != 1) continue;
        int32_t u, v;
        if (!graph_edge(d, j, &u, &v)) {
            atomicOr(&d.cnt->not_graph, kNotGraph0);
            continue;
        }
        const int32_t hi = max(u, v), lo = min(u, v);
        if (hi >= 0 && d.left[hi] == (int32_t)j) d.T[hi] = ((unsigned long long)j << 32) | (uint32_t)(lo + 1);
    }
    const int64_t t = block_sum64(nb);
    if (threadIdx.x == 0) stat_add(d, S_BETAPIV, (unsigned long long)t, blockIdx.x);
}

// Block 0, the others: walked to their places, except the births of the
// pairs (i, left(i)) with i the last row of its first coface (they are
// positive: their columns reduce to zero).
__global__ void __launch_bounds__(kBlock) k_graph0_walk(Dev d)
{
    if (d.cnt->not_graph & kNotGraph0) return;
    for (int64_t j = blockIdx.x * (int64_t)kBlock + threadIdx.x; j < d.m; j += (int64_t)gridDim.x * kBlock) {
        if (d.dim[j] != 1) continue;
        const int32_t t = d.left[j];
        if (t != 0x7FFFFFFF && last_row(d, t) == (int32_t)j) continue;
        int32_t u, v;
        graph_edge(d, j, &u, &v);
        const int32_t hi = max(u, v);
        if (hi < 0 || d.left[hi] == (int32_t)j) continue;
        graph_place<false>(d.T, (uint32_t)j, u, v);
    }
}

// Top block: number of cofaces (from bit 40 up) and the sum of their indices
// of every face; more than two cofaces leave a count above two, whatever the
// sum carries into it.
__global__ void __launch_bounds__(kBlock) k_cof_sum(Dev d, unsigned long long *S, int32_t top)
{
    for (int64_t j = blockIdx.x * (int64_t)kBlock + threadIdx.x; j < d.m; j += (int64_t)gridDim.x * kBlock) {
        if (d.dim[j] != top) continue;
        const int32_t n = d.len[j];
        const int64_t s = d.col_ptr[j];
        for (int32_t k = 0; k < n; k++) atomicAdd(&S[d.rows[s + k]], (1ull << 40) + (unsigned long long)j);
    }
}

// The cofaces of face i (a missing one: kGraphOut); false when it has more than two.
__device__ inline bool graph_face(const Dev &d, const unsigned long long *S, int64_t i, int32_t *t0, int32_t *t1)
{
    const unsigned long long x = S[i];
    const int32_t n = (int32_t)(x >> 40);
    *t0 = n > 0 ? d.left[i] : kGraphOut;
    *t1 = n > 1 ? (int32_t)((x & ((1ull << 40) - 1)) - (unsigned long long)*t0) : kGraphOut;
    return n <= 2;
}

__global__ void __launch_bounds__(kBlock) k_graph_top_seed(Dev d, const unsigned long long *S, int32_t top)
{
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < d.m; i += (int64_t)gridDim.x * kBlock) {
        if (d.dim[i] != top - 1) continue;
        int32_t t0, t1;
        if (!graph_face(d, S, i, &t0, &t1)) {
            atomicOr(&d.cnt->not_graph, kNotGraphTop);
            continue;
        }
        if (t0 != kGraphOut && last_row(d, t0) == (int32_t)i)
            d.T[t0] = ((unsigned long long)(0x7FFFFFFFu - (uint32_t)i) << 32) | (uint32_t)t1;
    }
}

// (faces with beta defined are negative: their rows hold no birth)
__global__ void __launch_bounds__(kBlock) k_graph_top_walk(Dev d, const unsigned long long *S, int32_t top)
{
    if (d.cnt->not_graph & kNotGraphTop) return;
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < d.m; i += (int64_t)gridDim.x * kBlock) {
        if (d.dim[i] != top - 1 || d.beta[i] >= 0) continue;
        int32_t t0, t1;
        graph_face(d, S, i, &t0, &t1);
        if (t0 == kGraphOut || last_row(d, t0) == (int32_t)i) continue;
        graph_place<true>(d.T, 0x7FFFFFFFu - (uint32_t)i, t0, t1);
    }
}

// The pairs of the solved blocks into the reduction's state: low* and piv;
// deaths of block 0 known negative (their rows leave every column); births of
// the top block cleared.
__global__ void __launch_bounds__(kBlock) k_graph_apply(Dev d, int32_t top, int do_top, int compression)
{
    const int32_t bad = d.cnt->not_graph;
    const bool g0 = !(bad & kNotGraph0), gt = do_top && !(bad & kNotGraphTop);
    for (int64_t j = blockIdx.x * (int64_t)kBlock + threadIdx.x; j < d.m; j += (int64_t)gridDim.x * kBlock) {
        const int dj = d.dim[j];
        if (dj == 0) {
            const unsigned long long x = d.T[j];
            if (x == kGraphEmpty) continue;
            if (!g0) {  // the rounds' table starts empty
                d.T[j] = kGraphEmpty;
                continue;
            }
            const int32_t e = (int32_t)(x >> 32);
            d.piv[j] = e;
            d.low_star[e] = (int32_t)j;
            if (compression) {
                d.prec[e].k = -1;
                atomicOr(&d.neg[e >> 5], 1u << (e & 31));
            }
        } else if (dj == top && gt) {
            const unsigned long long x = d.T[j];
            if (x == kGraphEmpty) continue;
            const int32_t i = (int32_t)(0x7FFFFFFFu - (uint32_t)(x >> 32));
            d.piv[i] = (int32_t)j;
            d.low_star[j] = i;
            d.state[i] = ST_ZERO;
            d.len[i] = 0;
        }
    }
}

// The first active list: live columns of the dimensions no graph has solved.
__device__ inline bool mix_keep(const Dev &d, int64_t j, int32_t top, bool g0, bool gt)
{
    const int dj = d.dim[j];
    return d.state[j] == ST_ACTIVE && !(dj == 1 && g0) && !(dj == top && gt);
}

__global__ void __launch_bounds__(kBlock) k_mix_count(Dev d, int32_t *keep_cnt, int32_t top, int do_top)
{
    const int32_t bad = d.cnt->not_graph;
    const bool g0 = !(bad & kNotGraph0), gt = do_top && !(bad & kNotGraphTop);
    const int64_t tiles = (d.m + kBlock - 1) / kBlock;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t j = tile * kBlock + threadIdx.x;
        int32_t tk;
        block_excl_sum32(j < d.m && mix_keep(d, j, top, g0, gt) ? 1 : 0, &tk);
        if (threadIdx.x == 0) keep_cnt[tile] = tk;
    }
}

__global__ void __launch_bounds__(kBlock) k_mix_compact(Dev d, const int32_t *keep_off, int32_t *act, int32_t top,
                                                        int do_top)
{
    const int32_t bad = d.cnt->not_graph;
    const bool g0 = !(bad & kNotGraph0), gt = do_top && !(bad & kNotGraphTop);
    const int64_t tiles = (d.m + kBlock - 1) / kBlock;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t j = tile * kBlock + threadIdx.x;
        const int keep = j < d.m && mix_keep(d, j, top, g0, gt);
        int32_t tot;
        const int32_t pos = block_excl_sum32(keep, &tot);
        if (keep) act[keep_off[tile] + pos] = (int32_t)j;
    }
}

// The reduction starts from that list; with the top block solved the
// dimension below is the one whose columns nothing clears any more.
__global__ void k_mix_start(Dev d, int32_t top, int do_top)
{
    d.cnt->n_cur = d.cnt->n_next;
    d.cnt->beta_counted = 1;
    d.cnt->topdim = do_top && !(d.cnt->not_graph & kNotGraphTop) ? top - 1 : top;
}
