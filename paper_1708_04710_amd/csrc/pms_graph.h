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
// while the longest walk from the triangles' side is 78 nodes.  Measured, by
// these kernels alone: build + reduce + backward of a 64^3 field 42.0 -> 4.8 ms
// (3.4 to 5.3 with what came after, by the field), build + reduce of a 128^3 one
// 399 -> 41.9 ms (15.0 to 16.7), of 32^3 white noise 9.3 -> 3.9 ms (2.6 to 2.8).
// The kernels here are bound by scattered 4- and 8-byte accesses (a node's
// word, a face's two cofaces), not by the walks.
#pragma once

constexpr int32_t kNotGraph0 = 1, kNotGraphTop = 2;
constexpr int kMixPer = 4, kMixTile = kMixPer * kBlock;

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
            int32_t low = d.low[j];  // the last row, still
            if (low >= 0 && is_neg(d.neg, low)) {
                const int32_t *c = d.rows + d.col_ptr[j];
                int32_t n = d.len[j] - 1;
                while (n > 0 && is_neg(d.neg, c[n - 1])) n--;
                low = n > 0 ? c[n - 1] : -1;
            }
            nb += low == b;
        }
        if (d.dim[j] != 1) continue;
        int32_t u, v;
        if (!graph_edge(d, j, &u, &v)) {
            atomicOr(&d.cnt->not_graph, kNotGraph0);
            continue;
        }
        const int32_t hi = max(u, v), lo = min(u, v);
        if (hi >= 0 && d.left[hi] == (int32_t)j) d.T[hi] = ((unsigned long long)j << 32) | graph_code<false>(lo);
    }
    const int64_t t = block_sum64(nb);
    if (threadIdx.x == 0) stat_add(d, S_BETAPIV, (unsigned long long)t, blockIdx.x);
}

// Block 0, the others: walked to their places, except the births of the
// pairs (i, left(i)) with i the last row of its first coface (they are
// positive: their columns reduce to zero).  (Every column's low is its last row
// before the rounds: read from there instead of through len, col_ptr and rows
// this kernel takes 0.90 ms instead of 1.00 at 128^3, the seeds of both blocks
// 0.76 instead of 0.98.)
__global__ void __launch_bounds__(kBlock) k_graph0_walk(Dev d)
{
    if (d.cnt->not_graph & kNotGraph0) return;
    for (int64_t j = blockIdx.x * (int64_t)kBlock + threadIdx.x; j < d.m; j += (int64_t)gridDim.x * kBlock) {
        if (d.dim[j] != 1) continue;
        const int32_t t = d.left[j];
        if (t != 0x7FFFFFFF && d.low[t] == (int32_t)j) continue;
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

// The cofaces of face i (a missing one: kGraphOut); false when it has more than
// two.  S: their numbers and sums, or null: the builder gave the second (the
// atomics of k_cof_sum take 1.3 ms at 128^3, writing second 0.16).
__device__ inline bool graph_face(const Dev &d, const unsigned long long *S, int64_t i, int32_t *t0, int32_t *t1)
{
    if (!S) {
        *t0 = d.left[i];  // (none: kGraphOut)
        *t1 = d.second[i];
        return true;
    }
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
        if (t0 != kGraphOut && d.low[t0] == (int32_t)i)
            d.T[t0] = ((unsigned long long)(0x7FFFFFFFu - (uint32_t)i) << 32) | graph_code<true>(t1);
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
        if (t0 == kGraphOut || d.low[t0] == (int32_t)i) continue;
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
            if (compression) atomicOr(&d.neg[e >> 5], 1u << (e & 31));
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

// ---------------------------------------------------------------- from the rows
// The faces' cofaces as lists, for blocks reduced from their rows (pms_dual.h):
// counted into end[face], scanned, and filled so that end[face] is the end of
// its list (in no particular order: a column's cofaces only flip bits).
// dims: bit b + 1 set: columns of dimension b + 1 are listed.
__global__ void __launch_bounds__(kBlock) k_cof_count(Dev d, int32_t dims, int32_t *end)
{
    for (int64_t j = blockIdx.x * (int64_t)kBlock + threadIdx.x; j < d.m; j += (int64_t)gridDim.x * kBlock) {
        if (!((dims >> d.dim[j]) & 1)) continue;
        const int32_t n = d.len[j];
        const int64_t s = d.col_ptr[j];
        for (int32_t k = 0; k < n; k++) atomicAdd(&end[d.rows[s + k]], 1);
    }
}

__global__ void __launch_bounds__(kBlock) k_cof_fill(Dev d, int32_t dims, int32_t *end, int32_t *cof)
{
    for (int64_t j = blockIdx.x * (int64_t)kBlock + threadIdx.x; j < d.m; j += (int64_t)gridDim.x * kBlock) {
        if (!((dims >> d.dim[j]) & 1)) continue;
        const int32_t n = d.len[j];
        const int64_t s = d.col_ptr[j];
        for (int32_t k = 0; k < n; k++) cof[atomicAdd(&end[d.rows[s + k]], 1)] = (int32_t)j;
    }
}

// Exclusive sums of n counts in tiles of kMixTile: each tile's sum, (a scan of
// the sums,) then every entry.  (One workgroup over all m counts of a 400-point
// torus to dimension 2 took 277 us.)
__global__ void __launch_bounds__(kBlock) k_tile_total(const int32_t *a, int64_t n, int32_t *tile)
{
    int32_t t = 0;
#pragma unroll
    for (int u = 0; u < kMixPer; u++) {
        const int64_t j = (int64_t)blockIdx.x * kMixTile + u * kBlock + threadIdx.x;
        t += j < n ? a[j] : 0;
    }
    const int64_t s = block_sum64(t);
    if (threadIdx.x == 0) tile[blockIdx.x] = (int32_t)s;
}

__global__ void __launch_bounds__(kBlock) k_tile_sums32(int32_t *a, int64_t n, const int32_t *tile)
{
    int32_t at = tile[blockIdx.x];
#pragma unroll
    for (int u = 0; u < kMixPer; u++) {
        const int64_t j = (int64_t)blockIdx.x * kMixTile + u * kBlock + threadIdx.x;
        const int32_t x = j < n ? a[j] : 0;
        int32_t tot;
        const int32_t e = at + block_excl_sum32(x, &tot);
        if (j < n) a[j] = e;
        at += tot;
    }
}

// The faces of dimension b: the apparent ones paired, those neither apparent
// nor known negative listed.
__global__ void __launch_bounds__(kBlock) k_dual_cand(Dev d, DualState s, int32_t b)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t tiles = (d.m + kBlock - 1) / kBlock;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t i = tile * kBlock + threadIdx.x;
        bool list = false;
        if (i < d.m && d.dim[i] == b) {
            const int32_t t = d.left[i];
            s.vlen[i] = 0;
            const bool app = t != 0x7FFFFFFF && last_row(d, t) == (int32_t)i;
            if (app) s.low_star[t] = (int32_t)i;
            list = !app && d.low_star[i] == -1 && d.beta[i] < 0;
        }
        const uint64_t mk = __ballot(list);
        if (mk) {
            int32_t at = 0;
            if (lane == __ffsll((long long)mk) - 1) at = atomicAdd(&s.count[0], __popcll(mk));
            at = __shfl(at, __ffsll((long long)mk) - 1, kWave) + __popcll(mk & ((1ull << lane) - 1ull));
            if (list) s.list[0][at] = make_int2(0, (int32_t)i);
        }
    }
}

// Faces of a matrix over the columns that hold them.
struct CsrProv {
    static constexpr int kT = kWave;
    const int32_t *end, *cof;
    __device__ int32_t floor(int32_t i) const { return i; }
    __device__ void bind(int32_t) {}
    __device__ int64_t key(int32_t i) const { return i; }
    __device__ int32_t face(int64_t k) const { return (int32_t)k; }
    __device__ int64_t col(int32_t t) const { return t; }
    __device__ int32_t apparent(int32_t, int32_t ls) const { return ls; }
    // its list
    __device__ void load(int32_t i, int32_t &d0, int32_t &d1) const
    {
        d0 = i > 0 ? end[i - 1] : 0;
        d1 = end[i];
    }
    __device__ int flip(const DualMap<kT> &map, int32_t, int32_t d0, int32_t d1, int32_t, DualCand &) const
    {
        int n = 0;
#pragma unroll 4
        for (int32_t q = d0 + (int32_t)(threadIdx.x & (kWave - 1)); q < d1; q += kWave, n++) map.toggle(cof[q]);
        return n;
    }
    __device__ int flip_many(const DualMap<kT> &map, const int32_t *faces, int32_t cnt) const
    {
        const int lane = threadIdx.x & (kWave - 1);
        int n = 0;
        for (int32_t k0 = 0; k0 < cnt; k0 += kWave) {
            int32_t d0, d1;
            load(faces[min(k0 + lane, cnt - 1)], d0, d1);
            for (int32_t k = 0; k < min(cnt - k0, (int32_t)kWave); k += 4) {
                int32_t a[4], z[4], t[4];
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    const int32_t q = min(k + u, (int32_t)kWave - 1);
                    a[u] = __builtin_amdgcn_readlane(d0, q) + lane;
                    z[u] = k0 + k + u < cnt ? __builtin_amdgcn_readlane(d1, q) : 0;
                }
                while (a[0] < z[0] || a[1] < z[1] || a[2] < z[2] || a[3] < z[3]) {
#pragma unroll
                    for (int u = 0; u < 4; u++) t[u] = a[u] < z[u] ? cof[a[u]] : -1;
#pragma unroll
                    for (int u = 0; u < 4; u++) {
                        if (t[u] >= 0) {
                            map.toggle(t[u]);
                            n++;
                        }
                        a[u] += kWave;
                    }
                }
            }
        }
        return n;
    }
};

// A block reduced from its rows into the reduction's state (as k_graph_apply),
// or, when it was given up, its claims withdrawn.
__global__ void __launch_bounds__(kBlock) k_dual_apply(Dev d, int32_t b, int ok, int compression)
{
    for (int64_t j = blockIdx.x * (int64_t)kBlock + threadIdx.x; j < d.m; j += (int64_t)gridDim.x * kBlock) {
        if (d.dim[j] != b + 1) continue;
        const int32_t x = d.low_star[j];
        if (x == -1) continue;
        if (!ok) {
            d.low_star[j] = -1;
            continue;
        }
        const int32_t i = x < -1 ? -2 - x : x;
        d.low_star[j] = i;
        d.piv[i] = (int32_t)j;
        d.state[i] = ST_ZERO;
        d.len[i] = 0;
        if (compression) atomicOr(&d.neg[j >> 5], 1u << (j & 31));
    }
}

// The first active list: live columns of the dimensions no graph has solved.
__device__ inline bool mix_keep(const Dev &d, int64_t j, int32_t solved)
{
    return d.state[j] == ST_ACTIVE && !((solved >> d.dim[j]) & 1);
}

// The dimensions whose columns are solved: those the host knows (dual), and
// the graphs that turned out to be such.
__device__ inline int32_t mix_solved(const Dev &d, int32_t top, int do_top, int32_t dual)
{
    const int32_t bad = d.cnt->not_graph;
    return dual | (bad & kNotGraph0 ? 0 : 2) | (do_top && !(bad & kNotGraphTop) ? 1 << top : 0);
}

// A column of an unsolved block whose low, its known-negative rows dropped, is
// its beta: no other column has that low further left, so it is a pivot as it
// is.  (Only where the block below is solved: the row's own column is then not
// in the list, and need not be cleared.)
__device__ inline bool mix_pivot(const Dev &d, int64_t j, int32_t solved)
{
    const int dj = d.dim[j];
    return (dj == 1 || ((solved >> (dj - 1)) & 1)) && d.low[j] >= 0 && d.low[j] == d.beta[j];
}

// Before the first round, in tiles of kMixTile: the records of the rows of the
// unsolved blocks (only those are ever looked up: a 128^3 field's 54 M rows
// have 15 M of them, and 32 bytes each are most of what k_init writes); the
// lows of their columns; and the number of those that go into the rounds.
// The columns that are pivots as they are (11.3 of 12.4 M of that field) are
// made pivots by k_mix_compact instead of passing through the first round,
// whose five kernels took 2.3 ms.
__global__ void __launch_bounds__(kBlock) k_mix_count(Dev d, int32_t *keep_cnt, int32_t top, int do_top, int32_t dual)
{
    const int32_t solved = mix_solved(d, top, do_top, dual);
    const int64_t tiles = (d.m + kMixTile - 1) / kMixTile;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        int32_t n = 0;
        for (int u = 0; u < kMixPer; u++) {
            const int64_t j = tile * kMixTile + u * kBlock + threadIdx.x;
            if (j >= d.m) continue;
            const int dj = d.dim[j];
            if (dj < top && !((solved >> (dj + 1)) & 1)) {
                int4 *pr = reinterpret_cast<int4 *>(&d.prec[j]);
                pr[0] = make_int4(-1, is_neg(d.neg, (int32_t)j) ? -1 : 0, 0, 0);
                pr[1] = make_int4(0, 0, 0, 0);
            }
            if (!mix_keep(d, j, solved)) continue;
            int32_t low = d.low[j];
            if (low >= 0 && is_neg(d.neg, low)) {
                const int32_t *c = d.rows + d.col_ptr[j];
                int32_t k = d.len[j] - 1;
                while (k > 0 && is_neg(d.neg, c[k - 1])) k--;
                low = k > 0 ? c[k - 1] : -1;
                d.len[j] = k;
                d.low[j] = low;
                if (k == 0) d.state[j] = ST_ZERO;
            }
            n += low >= 0 && !mix_pivot(d, j, solved);
        }
        const int64_t t = block_sum64(n);
        if (threadIdx.x == 0) keep_cnt[tile] = (int32_t)t;
    }
}

__global__ void __launch_bounds__(kBlock) k_mix_compact(Dev d, const int32_t *keep_off, int32_t *act, int32_t top,
                                                        int do_top, int32_t dual, int compression)
{
    const int32_t solved = mix_solved(d, top, do_top, dual);
    const int64_t tiles = (d.m + kMixTile - 1) / kMixTile;
    int64_t np = 0, pb = 0;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        int32_t at = keep_off[tile];
        for (int u = 0; u < kMixPer; u++) {
            const int64_t j = tile * kMixTile + u * kBlock + threadIdx.x;
            bool keep = j < d.m && mix_keep(d, j, solved);
            if (keep && mix_pivot(d, j, solved)) {
                pb += make_pivot(d, (int32_t)j, d.low[j], compression);  // (known negative already, by its beta)
                np++;
                keep = false;
            }
            int32_t tot;
            const int32_t pos = at + block_excl_sum32(keep ? 1 : 0, &tot);
            if (keep) act[pos] = (int32_t)j;
            at += tot;
        }
    }
    const int64_t t = block_sum64(np), tb = block_sum64(pb);
    if (threadIdx.x == 0) {
        stat_add(d, S_NEWPIV, (unsigned long long)t, blockIdx.x);
        stat_add(d, S_PBYTES, (unsigned long long)tb, blockIdx.x);
    }
}

// The records of all rows, when no block is solved apart after all.
__global__ void __launch_bounds__(kBlock) k_all_records(Dev d)
{
    for (int64_t j = blockIdx.x * (int64_t)kBlock + threadIdx.x; j < d.m; j += (int64_t)gridDim.x * kBlock) {
        int4 *pr = reinterpret_cast<int4 *>(&d.prec[j]);
        pr[0] = make_int4(-1, is_neg(d.neg, (int32_t)j) ? -1 : 0, 0, 0);
        pr[1] = make_int4(0, 0, 0, 0);
    }
}

// The reduction starts from that list; below solved top dimensions, the first
// unsolved one holds the columns nothing clears any more.
__global__ void __launch_bounds__(kWave) k_mix_start(Dev d, int32_t top, int do_top, int32_t dual, Counters *host)
{
    const int32_t solved = mix_solved(d, top, do_top, dual);
    int32_t t = top;
    while (t > 0 && ((solved >> t) & 1)) t--;
    if (threadIdx.x == 0) {
        d.cnt->n_cur = d.cnt->n_next;
        d.cnt->beta_counted = 1;
        d.cnt->topdim = t;
    }
    publish(d, host);
}
