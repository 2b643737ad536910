// Lower-star filtration of the Freudenthal triangulation of a 3-D vertex
// grid, built on the GPU.
//
// The simplices of the triangulation are the chains v0 < v1 < ... < vk of
// grid vertices whose successive steps are non-zero 0/1 vectors with
// disjoint supports (k <= 3).  A simplex is stored as (anchor v0, shape),
// where the shape is the sequence of steps: 1 shape of dimension 0, 7 of
// dimension 1, 12 of dimension 2 and 6 of dimension 3.  Its value is the
// largest vertex value (lower-star filtration), and the filtration order is
// compatible (Sec. 2.2): by value, then dimension, then the lexicographic
// order of the ascending vertex tuple.  Because a simplex's vertices are the
// anchor plus fixed offsets, the lexicographic order is (anchor, rank of the
// shape's offset tuple).
//
// Only the vertices are sorted (by value, then id).  Every simplex belongs to
// its last vertex in that order, and a vertex is in 75 simplices at most, of
// its 14 neighbours: one comparison a neighbour tells which of them are its
// own (a 75-bit mask), counts over the sorted vertices give where they start,
// and within a vertex they are numbered by the fixed order (dimension, anchor,
// rank).  Vertices of one value share a run, ordered likewise: up to kLsTies of
// them each counts the others' simplices before its own.  More (plateaus,
// small integers) take a stable radix sort of all simplices, generated in the
// order of dimension, anchor and rank, by their value's place.  A 64^3
// field of 256 levels takes 720 us that way (870 by sorting all simplices by
// one 64-bit key).
//
// The boundary matrix (eq. "def:boundary_matrix") follows from a dense
// (anchor, shape) -> filtration index table: the facets of (v, s) are
// (v + delta, s') with delta and s' read from a per-shape table.  The same
// table read the other way gives each simplex's cofaces, so the builder also
// returns left (Def. "left": the first column holding a row, the first
// coface in the order) and beta (Def. "beta": the largest row of a column
// whose left is that column), which the reduction would otherwise compute
// with one atomic per nonzero.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <new>
#include <vector>

#include "pms_common.h"
#include "pms_build.h"
#include "pms_sort.h"

namespace pms {

constexpr int kShapes = 26;

struct ShapeTab {
    int32_t nx, ny, nz;
    int8_t dim[kShapes];
    int8_t ext[kShapes];      // OR of the steps: axes the shape advances along
    int8_t rank[kShapes];     // lexicographic rank within its dimension
    int32_t cum[kShapes][4];  // vertex offsets from the anchor (cum[0] = 0)
    int8_t mask[kShapes][4];  // the same as axis masks
    int8_t by_rank[4][16];    // shape id of (dim, rank)
    int8_t facet[kShapes][4]; // facet shape id after removing vertex k
    int32_t fdelta[kShapes][4];  // anchor shift of that facet
    // cofaces: the shapes one dimension up with this shape as a facet, and the
    // step (axis mask, 0: none) from their anchor to this one
    int8_t ncof[kShapes];
    int8_t cof_s[kShapes][14];
    int8_t cof_e[kShapes][14];
};

// A vertex's simplices in the order (dimension, anchor, rank): the shape, the
// steps from the anchor to the vertex (axis mask), the neighbours needed (bit
// e - 1: the vertex minus step e, bit 6 + e: plus step e).
constexpr int kCand = 75;
constexpr int kLsTies = 8;
constexpr int64_t kLsManyV = 1 << 18;  // vertices at which tiles of kBlock fill the chip four times over
struct CandTab {
    uint32_t c[kCand];            // need | shape << 14 | step mask << 19 | dimension << 22
    int32_t step[8];              // vertex offset of each axis mask
    int32_t nx, ny, nz;
    unsigned long long dim_lo[4], dim_hi[4];  // the candidates of each dimension
};
__device__ inline int cand_shape(uint32_t c) { return (c >> 14) & 31; }
__device__ inline int cand_step(uint32_t c) { return (c >> 19) & 7; }
__device__ inline int cand_dim(uint32_t c) { return (c >> 22) & 3; }

__device__ inline uint32_t f32_order_bits(float x)
{
    if (x == 0.0f) x = 0.0f;  // -0 and +0 are one value
    const uint32_t b = __float_as_uint(x);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

__device__ inline float f32_from_order_bits(uint32_t u)
{
    const uint32_t b = (u & 0x80000000u) ? (u & 0x7FFFFFFFu) : ~u;
    return __uint_as_float(b);
}

__global__ void __launch_bounds__(kBlock) k_ls_vkeys(const float *__restrict__ grid, int32_t nv, uint32_t *key, uint32_t *id,
                                                     int32_t *err)
{
    for (int32_t v = blockIdx.x * kBlock + threadIdx.x; v < nv; v += gridDim.x * kBlock) {
        const float x = grid[v];
        if (x != x) atomicExch(err, 1);  // NaN has no place in an order
        key[v] = f32_order_bits(x);
        id[v] = (uint32_t)v;
    }
}

// Each vertex's place; err[1]: a value has more than kLsTies vertices.
__global__ void __launch_bounds__(kBlock) k_ls_rank(const uint32_t *__restrict__ key, const uint32_t *__restrict__ id,
                                                    int32_t nv, int32_t *rk, int32_t *err)
{
    bool big = false;
    for (int32_t p = blockIdx.x * kBlock + threadIdx.x; p < nv; p += gridDim.x * kBlock) {
        rk[id[p]] = p;
        big = big || (p >= kLsTies && key[p] == key[p - kLsTies]);
    }
    if (__ballot(big) != 0 && (threadIdx.x & (kWave - 1)) == 0) err[1] = 1;  // (any writer writes the same)
}

// Each vertex's mask, at its place.  One thread a vertex in id order, so that
// the 14 neighbours' places are read coalesced.
__global__ void __launch_bounds__(kBlock) k_ls_masks(CandTab t, int32_t nv, const int32_t *__restrict__ rk,
                                                     ulonglong2 *mask, const int32_t *__restrict__ err)
{
    if (err[0] || err[1]) return;
    const int32_t nx = t.nx, nxy = t.nx * t.ny;
    for (int32_t v = blockIdx.x * kBlock + threadIdx.x; v < nv; v += gridDim.x * kBlock) {
        const int32_t z = v / nxy, r = v - z * nxy, y = r / nx, x = r - y * nx;
        const int back = (x > 0 ? 1 : 0) | (y > 0 ? 2 : 0) | (z > 0 ? 4 : 0);
        const int fwd = (x + 1 < nx ? 1 : 0) | (y + 1 < t.ny ? 2 : 0) | (z + 1 < t.nz ? 4 : 0);
        const int32_t own = rk[v];
        int32_t nb[14];
#pragma unroll
        for (int e = 1; e < 8; e++) {
            nb[e - 1] = rk[(e & ~back) ? v : v - t.step[e]];
            nb[e + 6] = rk[(e & ~fwd) ? v : v + t.step[e]];
        }
        uint32_t low = 0;
#pragma unroll
        for (int e = 0; e < 14; e++) low |= (uint32_t)(nb[e] < own) << e;  // (itself is not)
        unsigned long long lo = 0, hi = 0;
#pragma unroll
        for (int c = 0; c < kCand; c++) {
            const unsigned long long has = (t.c[c] & 0x3FFFu & ~low) == 0;
            if (c < 64) lo |= has << c;
            else hi |= has << (c - 64);
        }
        mask[own] = make_ulonglong2(lo, hi);
    }
}

// A mask's simplices below dimension d: their number and that of their facets,
// packed (the first in the upper 31 bits).
constexpr int kLsPack = 33;
__device__ inline unsigned long long ls_below(const CandTab &t, const ulonglong2 m, int d)
{
    unsigned long long n = 0;
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const unsigned long long c = (unsigned long long)(__popcll(m.x & t.dim_lo[k]) + __popcll(m.y & t.dim_hi[k]));
        if (k < d) n += (c << kLsPack) + c * (k ? k + 1 : 0);
    }
    return n;
}

// Sums over tiles of kV (32 or kBlock) vertices.
template <int kV>
__global__ void __launch_bounds__(kBlock) k_ls_sums(CandTab t, int32_t nv, const ulonglong2 *__restrict__ mask,
                                                    int64_t *tile_sum, const int32_t *__restrict__ err)
{
    if (err[0] || err[1]) return;
    const int32_t p = blockIdx.x * kBlock + threadIdx.x;
    int64_t n = p < nv ? (int64_t)ls_below(t, mask[p], 4) : 0;
    if constexpr (kV == kBlock) {
        n = block_sum64(n);
        if (threadIdx.x == 0) tile_sum[blockIdx.x] = n;
    } else {
        static_assert(kV == 32, "half a wavefront");
#pragma unroll
        for (int o = kV / 2; o > 0; o >>= 1) n += __shfl_xor(n, o, kWave);
        if (threadIdx.x % kV == 0 && p < nv) tile_sum[p / kV] = n;
    }
}

// the n-th set bit (n from 0) of a mask with more than n
__device__ inline int ls_select(const ulonglong2 m, int n)
{
    const int nl = __popcll(m.x);
    unsigned long long w = n < nl ? m.x : m.y;
    int k = n < nl ? n : n - nl, at = n < nl ? 0 : 64;
#pragma unroll
    for (int h = 32; h > 0; h >>= 1) {
        const int c = __popcll(w & ((1ull << h) - 1));
        if (k >= c) {
            k -= c;
            at += h;
            w >>= h;
        }
    }
    return at;
}

// The simplices of kV vertices in the sorted order, one thread a simplex:
// neighbouring threads write neighbouring places (but for the index table, and
// where vertices share a value).  Bound by those writes: 53.7 M simplices of a
// 128^3 field take 0.98 ms, of which the scattered index table is most; the 64-bit
// sort of all simplices and its decoding took 4.8.  Fields of few vertices
// take tiles of 32: the last vertices in the order have up to 75 simplices
// each, and a tile of 256 of them holds the launch (32^3 noise: 79 us, 32 in the small tiles).
template <int kV>
__global__ void __launch_bounds__(kBlock) k_ls_emit(ShapeTab t, CandTab ct,
                                                    const uint32_t *__restrict__ key, const uint32_t *__restrict__ id,
                                                    const ulonglong2 *__restrict__ mask, int32_t nv, int64_t m,
                                                    const int64_t *__restrict__ tile_off, int32_t *idx_tab, int32_t *code,
                                                    int8_t *dim, float *value, int32_t *crit, int32_t *verts,
                                                    int64_t *col_ptr, int32_t *err)
{
    __shared__ uint32_t s_c[kCand];
    __shared__ int32_t s_cum[kShapes][4];
    __shared__ int8_t s_rank[kShapes];
    __shared__ ulonglong2 s_mask[kV];
    __shared__ int64_t s_start[kV];
    __shared__ int32_t s_first[kV + 1];
    __shared__ int32_t s_id[kV];
    __shared__ float s_val[kV];
    __shared__ uint8_t s_tie[kV];  // vertices of the value before this one, and after it (4 bits each)
    if (err[0] || err[1]) return;
    for (int k = threadIdx.x; k < kCand; k += kBlock) s_c[k] = ct.c[k];
    for (int k = threadIdx.x; k < kShapes * 4; k += kBlock) s_cum[k / 4][k % 4] = t.cum[k / 4][k % 4];
    if (threadIdx.x < kShapes) s_rank[threadIdx.x] = t.rank[threadIdx.x];
    const int32_t p0 = blockIdx.x * kV, p = p0 + (int32_t)threadIdx.x;
    const bool in = threadIdx.x < kV && p < nv;
    const ulonglong2 mk = in ? mask[p] : make_ulonglong2(0, 0);
    const int64_t n = in ? (int64_t)ls_below(ct, mk, 4) : 0;
    const int64_t start = tile_off[blockIdx.x] + block_excl_sum64(n);
    const int32_t first = (int32_t)((unsigned long long)start >> kLsPack) -
                          (int32_t)((unsigned long long)tile_off[blockIdx.x] >> kLsPack);
    if (threadIdx.x < kV) {
        s_mask[threadIdx.x] = mk;
        s_start[threadIdx.x] = start;
        s_first[threadIdx.x] = first;
        if (threadIdx.x == kV - 1) s_first[kV] = first + (int32_t)((unsigned long long)n >> kLsPack);
    }
    int tie = 0;
    if (in) {
        const uint32_t k0 = key[p];
        const int32_t v = (int32_t)id[p];
        s_id[threadIdx.x] = v;
        s_val[threadIdx.x] = f32_from_order_bits(k0);
        int b = 0, a = 0;
        while (b < kLsTies && p - b > 0 && key[p - b - 1] == k0) b++;
        while (a < kLsTies && p + a + 1 < nv && key[p + a + 1] == k0) a++;
        tie = b | a << 4;
    }
    if (threadIdx.x < kV) s_tie[threadIdx.x] = (uint8_t)tie;
    __syncthreads();
    const int32_t total = s_first[kV];
    for (int32_t o = threadIdx.x; o < total; o += kBlock) {
        int lo = 0;  // the last vertex whose first simplex is at or before o (each has one: itself)
#pragma unroll
        for (int h = kV / 2; h > 0; h >>= 1)
            if (s_first[lo + h] <= o) lo += h;
        const ulonglong2 mw = s_mask[lo];
        const int c = ls_select(mw, o - s_first[lo]);
        const uint32_t cd = s_c[c];
        const int s = cand_shape(cd), d = cand_dim(cd);
        const int32_t vc = s_id[lo], v = vc - ct.step[cand_step(cd)];
        unsigned long long at = (unsigned long long)s_start[lo];
        int32_t q = o - s_first[lo];  // simplices before this one
        const int tw = s_tie[lo];
        if (tw == 0) {
            const unsigned long long bl = ls_below(ct, mw, d);
            const int32_t same = q - (int32_t)(bl >> kLsPack);  // of its dimension
            at += bl + ((unsigned long long)same << kLsPack) + (unsigned long long)(same * (d ? d + 1 : 0));
        } else {
            // all of the value below dimension d, then those of dimension d with a
            // smaller (anchor, rank)
            const int32_t pw = p0 + lo, g0 = pw - (tw & 15), g1 = pw + (tw >> 4);
            int32_t same = 0;
            for (int32_t w = g0; w <= g1; w++) {
                const ulonglong2 mo = mask[w];
                if (w < pw) at -= ls_below(ct, mo, 4);
                at += ls_below(ct, mo, d);
                const int32_t delta = v - (int32_t)id[w];
                const unsigned long long xl = mo.x & ct.dim_lo[d], xh = mo.y & ct.dim_hi[d];
                if (delta > 0) {  // its anchors are all smaller
                    same += __popcll(xl) + __popcll(xh);
                } else if (delta >= -ct.step[7]) {
                    for (int k = 0; k < kCand; k++) {
                        if (!((k < 64 ? xl >> k : xh >> (k - 64)) & 1ull)) continue;
                        const int32_t dk = -ct.step[cand_step(s_c[k])];
                        same += dk < delta || (dk == delta && s_rank[cand_shape(s_c[k])] < s_rank[s]) ? 1 : 0;
                    }
                }
            }
            at += ((unsigned long long)same << kLsPack) + (unsigned long long)(same * (d ? d + 1 : 0));
        }
        const int64_t pos = (int64_t)(at >> kLsPack), cp = (int64_t)(at & ((1ull << kLsPack) - 1));
        if (pos >= m) {
            atomicExch(err, 2);
            continue;
        }
        const int32_t u1 = v + s_cum[s][1], u2 = v + s_cum[s][2], u3 = v + s_cum[s][3];
        idx_tab[(int64_t)v * kShapes + s] = (int32_t)pos;
        code[pos] = v * kShapes + s;
        dim[pos] = (int8_t)d;
        value[pos] = s_val[lo];
        reinterpret_cast<int2 *>(crit)[pos] = make_int2(vc, -1);
        if (verts)
            reinterpret_cast<int4 *>(verts)[pos] = make_int4(v, d >= 1 ? u1 : -1, d >= 2 ? u2 : -1, d >= 3 ? u3 : -1);
        col_ptr[pos] = cp;
        if (pos == m - 1) col_ptr[m] = cp + (d ? d + 1 : 0);
    }
}

// ---- values of many vertices: all simplices sorted by their value's place
// The place of each vertex's value: the first of the sorted vertices with it.
__global__ void __launch_bounds__(kBlock) k_ls_first(const uint32_t *__restrict__ key, const uint32_t *__restrict__ id,
                                                     int32_t nv, uint32_t *place, int32_t *err)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) err[1] = 0;  // seen by the host
    for (int32_t p = blockIdx.x * kBlock + threadIdx.x; p < nv; p += gridDim.x * kBlock) {
        const uint32_t k0 = key[p];
        int32_t lo = 0, hi = p;
        while (lo < hi) {
            const int32_t mid = (lo + hi) >> 1;
            if (key[mid] < k0) lo = mid + 1;
            else hi = mid;
        }
        place[id[p]] = (uint32_t)lo;
    }
}

// Every (dimension, anchor, rank) in that order: the largest place of its
// vertices (nv when it leaves the grid: sorted last) and its code.
__global__ void __launch_bounds__(kBlock) k_ls_keys(ShapeTab t, const uint32_t *__restrict__ place, int64_t nv,
                                                    uint32_t *keys, uint32_t *code)
{
    __shared__ int32_t s_cum[kShapes][4];
    __shared__ int8_t s_ext[kShapes], s_shape[4][16];
    for (int k = threadIdx.x; k < kShapes * 4; k += kBlock) s_cum[k / 4][k % 4] = t.cum[k / 4][k % 4];
    if (threadIdx.x < kShapes) s_ext[threadIdx.x] = t.ext[threadIdx.x];
    if (threadIdx.x < 64) s_shape[threadIdx.x / 16][threadIdx.x % 16] = t.by_rank[threadIdx.x / 16][threadIdx.x % 16];
    __syncthreads();
    const uint32_t n = (uint32_t)(nv * kShapes), n1 = (uint32_t)nv, nx = (uint32_t)t.nx, nxy = (uint32_t)(t.nx * t.ny);
    for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
        const int dm = i < n1 ? 0 : i < 8 * n1 ? 1 : i < 20 * n1 ? 2 : 3;
        const uint32_t per = dm == 0 ? 1 : dm == 1 ? 7 : dm == 2 ? 12 : 6;
        const uint32_t q = i - (dm == 0 ? 0 : dm == 1 ? n1 : dm == 2 ? 8 * n1 : 20 * n1);
        const uint32_t v = q / per;
        const int s = s_shape[dm][q - v * per], e = s_ext[s];
        const uint32_t z = v / nxy, r = v - z * nxy, y = r / nx, x = r - y * nx;
        uint32_t k0 = (uint32_t)nv;
        if (!((e & 1) && x + 1 >= nx) && !((e & 2) && y + 1 >= (uint32_t)t.ny) && !((e & 4) && z + 1 >= (uint32_t)t.nz)) {
            uint32_t g[4];
#pragma unroll
            for (int k = 0; k < 4; k++) g[k] = place[v + (k <= dm ? s_cum[s][k] : 0)];
            k0 = max(max(g[0], g[1]), max(g[2], g[3]));  // (k > dm: the anchor again)
        }
        keys[i] = k0;
        code[i] = v * kShapes + (uint32_t)s;
    }
}

// The sorted simplices: index table, dimension, value, critical vertex, vertex
// tuple, and the per-tile facet counts for col_ptr.
__global__ void __launch_bounds__(kBlock) k_ls_index(ShapeTab t, const float *__restrict__ grid,
                                                     const uint32_t *__restrict__ keys, const uint32_t *__restrict__ code,
                                                     int64_t m, int64_t nv, int32_t *idx_tab, int8_t *dim, float *value,
                                                     int32_t *crit, int32_t *verts, int64_t *tile_sum, int32_t *err)
{
    // the shape tables in LDS: neighbouring simplices have different shapes
    __shared__ int32_t s_cum[kShapes][4];
    __shared__ int8_t s_dim[kShapes];
    for (int k = threadIdx.x; k < kShapes * 4; k += kBlock) s_cum[k / 4][k % 4] = t.cum[k / 4][k % 4];
    if (threadIdx.x < kShapes) s_dim[threadIdx.x] = t.dim[threadIdx.x];
    __syncthreads();
    const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    int64_t nf = 0;
    if (p < m && (int64_t)keys[p] >= nv) atomicExch(err, 2);
    else if (p < m) {
        const int32_t v = (int32_t)(code[p] / kShapes), s = (int32_t)(code[p] - (uint32_t)v * kShapes);
        const int dm = s_dim[s];
        idx_tab[code[p]] = (int32_t)p;
        dim[p] = (int8_t)dm;
        // the vertices (k > dm: the anchor again), their values read together
        int32_t u[4];
        float gu[4];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            u[k] = v + (k <= dm ? s_cum[s][k] : 0);
            gu[k] = grid[u[k]];
        }
        // argmax vertex by (value, id): the vertex whose value the simplex takes
        int32_t best = v;
        float bv = gu[0];
#pragma unroll
        for (int k = 1; k < 4; k++)
            if (k <= dm && (gu[k] > bv || (gu[k] == bv && u[k] > best))) { best = u[k]; bv = gu[k]; }
        value[p] = f32_from_order_bits(f32_order_bits(bv));
        reinterpret_cast<int2 *>(crit)[p] = make_int2(best, -1);
        if (verts)
            reinterpret_cast<int4 *>(verts)[p] =
                make_int4(u[0], dm >= 1 ? u[1] : -1, dm >= 2 ? u[2] : -1, dm >= 3 ? u[3] : -1);
        nf = dm > 0 ? dm + 1 : 0;
    }
    const int64_t tot = block_sum64(nf);
    if (threadIdx.x == 0) tile_sum[blockIdx.x] = tot;
}

__global__ void __launch_bounds__(kBlock) k_ls_colptr(const int8_t *__restrict__ dim, int64_t m,
                                                      const int64_t *__restrict__ tile_off, int64_t *col_ptr)
{
    const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t nf = p < m && dim[p] > 0 ? dim[p] + 1 : 0;
    const int64_t start = tile_off[blockIdx.x] + block_excl_sum64(nf);
    if (p < m) col_ptr[p] = start;
    if (p == m - 1) col_ptr[m] = start + nf;
}

__global__ void __launch_bounds__(kBlock) k_ls_rows(ShapeTab t, const int32_t *__restrict__ code, int64_t m,
                                                    int64_t nnz, const int32_t *__restrict__ idx_tab,
                                                    const int64_t *__restrict__ col_ptr, int32_t *rows,
                                                    const int32_t *__restrict__ left, int32_t *beta,
                                                    const int32_t *__restrict__ err)
{
    // the shape tables in LDS: neighbouring simplices have different shapes
    __shared__ int32_t s_fdelta[kShapes][4];
    __shared__ int8_t s_facet[kShapes][4], s_dim[kShapes];
    if (err[0] || err[1]) return;
    for (int k = threadIdx.x; k < kShapes * 4; k += kBlock) {
        s_fdelta[k / 4][k % 4] = t.fdelta[k / 4][k % 4];
        s_facet[k / 4][k % 4] = t.facet[k / 4][k % 4];
    }
    if (threadIdx.x < kShapes) s_dim[threadIdx.x] = t.dim[threadIdx.x];
    __syncthreads();
    const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (p >= m) return;
    const int32_t cd = code[p], v = cd / kShapes, s = cd - v * kShapes, dm = s_dim[s];
    const int nf = dm > 0 ? dm + 1 : 0;
    const int64_t start = col_ptr[p];
    if (start + nf <= nnz) {
        // the facets' indices, read together (k >= nf: the simplex's own entry)
        int32_t r[4];
#pragma unroll
        for (int k = 0; k < 4; k++)
            r[k] = idx_tab[k < nf ? (int64_t)(v + s_fdelta[s][k]) * kShapes + s_facet[s][k]
                                  : (int64_t)v * kShapes + s];
        for (int a = 1; a < nf; a++) {  // ascending rows
            const int32_t x = r[a];
            int b = a - 1;
            while (b >= 0 && r[b] > x) { r[b + 1] = r[b]; b--; }
            r[b + 1] = x;
        }
        for (int k = 0; k < nf; k++) rows[start + k] = r[k];
        // beta: the largest row whose first column is this one (loads together, then the scan)
        int32_t lf[4];
#pragma unroll
        for (int k = 0; k < 4; k++) lf[k] = left[k < nf ? r[k] : 0];
        int32_t b = -1;
#pragma unroll
        for (int k = 0; k < 4; k++)
            if (k < nf && lf[k] == (int32_t)p) b = r[k];  // rows ascending: the last hit is the largest
        beta[p] = b;
    }
}

// left of every simplex (Def. "left"): the smallest filtration index among
// its cofaces (none: 2^31 - 1).  A coface of (v, s) is anchored at v minus a
// step e (a subset of the axes), so a workgroup that handles the anchors
// v0 .. v0 + kLeftV - 1 needs the index-table rows of four planes, v - b and
// v - b - 1 for b in {0, nx, nx ny, nx ny + nx}: it stages them into LDS with
// coalesced loads (rows padded to an odd stride), then takes its (anchor,
// shape) pairs shape-major, so a wavefront holds one shape and reads the
// coface tables as scalars.  The one scattered access is the write of left at
// the simplex's filtration index.
constexpr int kLeftV = 64;                                  // anchors per tile
constexpr int kLeftRow = kShapes + 1;                       // LDS row stride
constexpr int kLeftPlane = (kLeftV + 1) * kShapes;          // staged entries per plane
constexpr int kLeftPer = (kLeftPlane + kBlock - 1) / kBlock;

// The smallest staged index among the cofaces of (v0 + vl, s), kN >= the
// shape's coface count (a vertex has 14, an edge at most 6, a triangle 2);
// *second: the largest of two and more (2^31 - 1: fewer).  The LDS reads are
// issued together.
template <int kN>
__device__ inline int32_t ls_first_coface(const ShapeTab &t, int s, int vl, int back, int fwd,
                                          const int32_t (*seg)[(kLeftV + 1) * kLeftRow], int32_t *second)
{
    const int nc = t.ncof[s];
    int32_t got[kN];
    bool ok[kN];
#pragma unroll
    for (int c = 0; c < kN; c++) {
        const int sp = c < nc ? t.cof_s[s][c] : s;
        const int e = c < nc ? t.cof_e[s][c] : 0;
        // the coface's anchor v - e is on the grid, and the coface fits there
        ok[c] = c < nc && !(e & ~back) && !(t.ext[sp] & ~e & ~fwd);
        got[c] = seg[(e >> 1) & 3][(vl + 1 - (e & 1)) * kLeftRow + sp];
    }
    int32_t best = 0x7FFFFFFF, last = -1;
#pragma unroll
    for (int c = 0; c < kN; c++)
        if (ok[c]) {
            best = min(best, got[c]);
            last = max(last, got[c]);
        }
    *second = last > best ? last : 0x7FFFFFFF;  // (best stays 2^31 - 1 without a coface)
    return best;
}

__global__ void __launch_bounds__(kBlock) k_ls_left(ShapeTab t, int64_t nv, int64_t m,
                                                    const int32_t *__restrict__ idx_tab, int32_t *left,
                                                    int32_t *second, int face_dim, const int32_t *__restrict__ err)
{
    if (err[0] || err[1]) return;
    static_assert(kLeftV == 64 && kBlock % kLeftV == 0, "one shape per wavefront");
    __shared__ int32_t seg[4][(kLeftV + 1) * kLeftRow];
    __shared__ uint8_t nb[kLeftV];  // back | fwd << 3: axes with a grid neighbour below / above
    const int32_t nx = t.nx, ny = t.ny, nz = t.nz, nxy = nx * ny;
    for (int64_t v0 = (int64_t)blockIdx.x * kLeftV; v0 < nv; v0 += (int64_t)gridDim.x * kLeftV) {
        // plane g holds the kLeftV + 1 rows from v0 - b_g - 1 on: one
        // contiguous run of the table starting at a uniform entry
        int32_t val[4][kLeftPer];
#pragma unroll
        for (int g = 0; g < 4; g++) {
            const int64_t start = (v0 - ((g & 1 ? nx : 0) + (g & 2 ? nxy : 0)) - 1) * kShapes;
#pragma unroll
            for (int q = 0; q < kLeftPer; q++) {
                const int r = q * kBlock + (int)threadIdx.x;
                const int64_t e = start + r;
                const bool in = r < kLeftPlane && e >= 0 && e < nv * kShapes;
                val[g][q] = idx_tab[in ? e : 0];
                if (!in) val[g][q] = -1;
            }
        }
#pragma unroll
        for (int g = 0; g < 4; g++)
#pragma unroll
            for (int q = 0; q < kLeftPer; q++) {
                const int r = q * kBlock + (int)threadIdx.x;
                const int j = r / kShapes;
                if (r < kLeftPlane) seg[g][j * kLeftRow + (r - j * kShapes)] = val[g][q];
            }
        if (threadIdx.x < kLeftV) {
            const int64_t v = v0 + threadIdx.x;
            const int32_t z = (int32_t)(v / nxy), rem = (int32_t)(v - (int64_t)z * nxy), y = rem / nx, x = rem - y * nx;
            const int fwd = (x + 1 < nx ? 1 : 0) | (y + 1 < ny ? 2 : 0) | (z + 1 < nz ? 4 : 0);
            const int back = (x > 0 ? 1 : 0) | (y > 0 ? 2 : 0) | (z > 0 ? 4 : 0);
            nb[threadIdx.x] = (uint8_t)(back | fwd << 3);
        }
        __syncthreads();
        for (int k = threadIdx.x; k < kShapes * kLeftV; k += kBlock) {
            const int s = __builtin_amdgcn_readfirstlane(k / kLeftV);  // k / 64 is one value per wavefront
            const int vl = k % kLeftV;
            const int bits = nb[vl], back = bits & 7, fwd = bits >> 3;
            if (v0 + vl >= nv || (t.ext[s] & ~fwd)) continue;  // past the end, or the shape leaves the grid
            const int32_t p = seg[0][(vl + 1) * kLeftRow + s];
            int32_t best = 0x7FFFFFFF, other = 0x7FFFFFFF;
            switch (t.dim[s]) {
            case 0: best = ls_first_coface<14>(t, s, vl, back, fwd, seg, &other); break;
            case 1: best = ls_first_coface<6>(t, s, vl, back, fwd, seg, &other); break;
            case 2: best = ls_first_coface<2>(t, s, vl, back, fwd, seg, &other); break;
            default: break;
            }
            if ((uint64_t)(uint32_t)p < (uint64_t)m) {
                left[p] = best;
                if (t.dim[s] == face_dim) second[p] = other;
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------- host
static int step_offset(int e, int nx, int ny)
{
    return (e & 1) + ((e >> 1) & 1) * nx + ((e >> 2) & 1) * nx * ny;
}

static void make_tables(ShapeTab &t, int nx, int ny, int nz)
{
    t.nx = nx;
    t.ny = ny;
    t.nz = nz;
    std::vector<std::vector<int>> shapes;
    shapes.push_back({});
    for (int e = 1; e < 8; e++) shapes.push_back({e});
    for (int e1 = 1; e1 < 8; e1++)
        for (int e2 = 1; e2 < 8; e2++)
            if (!(e1 & e2)) shapes.push_back({e1, e2});
    const int perm[6][3] = {{1, 2, 4}, {1, 4, 2}, {2, 1, 4}, {2, 4, 1}, {4, 1, 2}, {4, 2, 1}};
    for (auto &p : perm) shapes.push_back({p[0], p[1], p[2]});
    auto find = [&](const std::vector<int> &st) {
        for (size_t i = 0; i < shapes.size(); i++)
            if (shapes[i] == st) return (int)i;
        return -1;
    };
    for (int s = 0; s < kShapes; s++) {
        const auto &st = shapes[s];
        t.dim[s] = (int8_t)st.size();
        int e = 0, c = 0;
        t.cum[s][0] = 0;
        for (int k = 0; k < 4; k++) t.mask[s][k] = 0;
        for (size_t k = 0; k < st.size(); k++) {
            e |= st[k];
            c += step_offset(st[k], nx, ny);
            t.cum[s][k + 1] = c;
            t.mask[s][k + 1] = (int8_t)e;
        }
        for (size_t k = st.size() + 1; k < 4; k++) t.cum[s][k] = 0;
        t.ext[s] = (int8_t)e;
        for (int k = 0; k < 4; k++) { t.facet[s][k] = 0; t.fdelta[s][k] = 0; }
        const int d = (int)st.size();
        if (d >= 1)
            for (int k = 0; k <= d; k++) {
                std::vector<int> f;
                int delta = 0;
                if (k == 0) {
                    f.assign(st.begin() + 1, st.end());
                    delta = step_offset(st[0], nx, ny);
                } else if (k < d) {
                    for (int q = 0; q < d; q++) {
                        if (q == k - 1) f.push_back(st[q] | st[q + 1]);
                        else if (q != k) f.push_back(st[q]);
                    }
                } else {
                    f.assign(st.begin(), st.end() - 1);
                }
                t.facet[s][k] = (int8_t)find(f);
                t.fdelta[s][k] = delta;
            }
    }
    // lexicographic rank of the offset tuple within each dimension
    for (int d = 0; d < 4; d++) {
        std::vector<int> ids;
        for (int s = 0; s < kShapes; s++)
            if (t.dim[s] == d) ids.push_back(s);
        std::stable_sort(ids.begin(), ids.end(), [&](int a, int b) {
            for (int k = 1; k <= d; k++)
                if (t.cum[a][k] != t.cum[b][k]) return t.cum[a][k] < t.cum[b][k];
            return false;
        });
        for (int r = 0; r < 16; r++) t.by_rank[d][r] = 0;
        for (size_t r = 0; r < ids.size(); r++) {
            t.rank[ids[r]] = (int8_t)r;
            t.by_rank[d][r] = (int8_t)ids[r];
        }
    }
    // cofaces: facet k of (v', s') is (v' + step, facet[s'][k]), the step being
    // the shape's first step when k = 0 and none otherwise
    for (int s = 0; s < kShapes; s++) t.ncof[s] = 0;
    for (int sp = 0; sp < kShapes; sp++) {
        const int d = t.dim[sp];
        for (int k = 0; d >= 1 && k <= d; k++) {
            const int f = t.facet[sp][k];
            const int n = t.ncof[f]++;
            t.cof_s[f][n] = (int8_t)sp;
            t.cof_e[f][n] = (int8_t)(k == 0 ? shapes[sp][0] : 0);
        }
    }
}

// The simplices of a vertex: each shape of each dimension, the vertex at each
// of its places.
static void make_candidates(CandTab &ct, const ShapeTab &t)
{
    ct.nx = t.nx;
    ct.ny = t.ny;
    ct.nz = t.nz;
    for (int e = 0; e < 8; e++) ct.step[e] = step_offset(e, t.nx, t.ny);
    struct Cand { int dim, off, rank; uint32_t code; };
    std::vector<Cand> all;
    for (int s = 0; s < kShapes; s++) {
        const int8_t *at = t.mask[s];
        for (int k = 0; k <= t.dim[s]; k++) {
            uint32_t need = 0;
            for (int q = 0; q <= t.dim[s]; q++) {
                if (q < k) need |= 1u << ((at[k] ^ at[q]) - 1);
                if (q > k) need |= 1u << ((at[q] ^ at[k]) + 6);
            }
            all.push_back({t.dim[s], -ct.step[at[k]], t.rank[s],
                           need | (uint32_t)s << 14 | (uint32_t)at[k] << 19 | (uint32_t)t.dim[s] << 22});
        }
    }
    std::sort(all.begin(), all.end(), [](const Cand &a, const Cand &b) {
        return a.dim != b.dim ? a.dim < b.dim : a.off != b.off ? a.off < b.off : a.rank < b.rank;
    });
    for (int d = 0; d < 4; d++) ct.dim_lo[d] = ct.dim_hi[d] = 0;
    for (int c = 0; c < kCand; c++) {
        ct.c[c] = all[c].code;
        (c < 64 ? ct.dim_lo : ct.dim_hi)[all[c].dim] |= 1ull << (c & 63);
    }
}

// Number of simplices and facets (closed form: a shape fits at an anchor iff
// every axis it advances along has room).
static void ls_sizes(const ShapeTab &t, int64_t *m, int64_t *nnz)
{
    int64_t M = 0, Z = 0;
    for (int mask = 0; mask < 8; mask++) {
        int64_t anchors = 1;
        const int32_t ext[3] = {t.nx, t.ny, t.nz};
        for (int a = 0; a < 3; a++) anchors *= (mask >> a & 1) ? (int64_t)(ext[a] - 1) : 1;
        if (anchors <= 0) continue;
        for (int s = 0; s < kShapes; s++) {
            if ((t.ext[s] & ~mask) != 0) continue;
            // anchors whose availability mask is exactly `mask`
            M += anchors;
            Z += anchors * (t.dim[s] > 0 ? t.dim[s] + 1 : 0);
        }
    }
    *m = M;
    *nnz = Z;
}

pms_status build_lowerstar(Ctx *c, const float *grid, int32_t nx, int32_t ny, int32_t nz, Filtration **out)
{
    if (!grid || !out || nx < 1 || ny < 1 || nz < 1) return set_err(c, PMS_ERR_INVALID_ARG, "bad grid arguments");
    const int64_t nv = (int64_t)nx * ny * nz;
    if (nv >= (1ll << 26)) return set_err(c, PMS_ERR_INVALID_ARG, "grid too large for the 26-bit anchor field");
    ShapeTab t;
    make_tables(t, nx, ny, nz);
    int64_t m = 0, nnz = 0;
    ls_sizes(t, &m, &nnz);
    Filtration *f = *out;
    pms_status st = filtration_reserve(c, &f, m, nnz, /*f32*/ 1);
    if (st != PMS_OK) return st;
    *out = f;
    hipStream_t s = c->stream;
    const int64_t nk = nv * kShapes;
    const int64_t tiles = (m + kBlock - 1) / kBlock, kV = nv >= kLsManyV ? kBlock : 32,
                  vtiles = (nv + kV - 1) / kV;
    CandTab ct;
    make_candidates(ct, t);
    uint32_t *vkey = (uint32_t *)grow_scratch(c, B_BUILD0, nv * 16);  // the vertices' values and ids, twice
    ulonglong2 *mask = (ulonglong2 *)grow_scratch(c, B_BUILD1, nv * 16);
    int32_t *idx = (int32_t *)grow_scratch(c, B_BUILD2, nk * 4);
    // sums per tile of vertices, or (many vertices of one value) of simplices: a flat
    // grid has 6 simplices a vertex, fewer tiles of kBlock than of 32 vertices
    int64_t *tsum = (int64_t *)grow_scratch(c, B_BUILD3, (std::max(tiles, vtiles) + 1) * 8);
    int32_t *err = (int32_t *)grow_scratch(c, B_BUILD4, 64);
    uint32_t *code = (uint32_t *)grow_scratch(c, B_BUILD7, nk * 4);
    int32_t *rk = (int32_t *)grow_scratch(c, B_BUILD8, nv * 4);
    if (!vkey || !mask || !idx || !tsum || !err || !code || !rk) return set_err(c, PMS_ERR_OOM, "builder scratch");
    uint32_t *vkey2 = vkey + nv, *vid = vkey2 + nv, *vid2 = vid + nv;
    const unsigned gv = grid_for(nv, kBlock, 1u << 16);
    PMS_HIP(hipMemsetAsync(err, 0, 8, s));
    PMS_LAUNCH(c, K_LS_KEYS, 12.0 * nv, k_ls_vkeys, gv, kBlock, grid, (int32_t)nv, vkey, vid, err);
    auto sort = [&](uint32_t *&a, uint32_t *&b, uint32_t *&va, uint32_t *&vb, int64_t n, int bits) -> pms_status {
        hipEvent_t e0 = nullptr;
        if (c->prof_on) { e0 = prof_event(c); (void)hipEventRecord(e0, s); }
        bool in_b = false;
        const pms_status ss = radix_sort<uint32_t, uint32_t>(c, a, b, va, vb, n, bits, B_BUILD5, B_BUILD6, &in_b);
        if (ss != PMS_OK) return ss;
        if (in_b) {  // a, va: the sorted keys and values
            std::swap(a, b);
            std::swap(va, vb);
        }
        if (c->prof_on) {
            hipEvent_t e1 = prof_event(c);
            (void)hipEventRecord(e1, s);
            c->pend.push_back({K_SORT, e0, e1, 16.0 * n});
        }
        return PMS_OK;
    };
    st = sort(vkey, vkey2, vid, vid2, nv, 32);
    if (st != PMS_OK) return st;
    PMS_LAUNCH(c, K_LS_KEYS, 12.0 * nv, k_ls_rank, gv, kBlock, vkey, vid, (int32_t)nv, rk, err);
    PMS_LAUNCH(c, K_LS_KEYS, 20.0 * nv, k_ls_masks, gv, kBlock, ct, (int32_t)nv, rk, mask, err);
    const unsigned gs = (unsigned)((nv + kBlock - 1) / kBlock);
    if (kV == kBlock) PMS_LAUNCH(c, K_LS_INDEX, 16.0 * nv, k_ls_sums<kBlock>, gs, kBlock, ct, (int32_t)nv, mask, tsum, err);
    else PMS_LAUNCH(c, K_LS_INDEX, 16.0 * nv, k_ls_sums<32>, gs, kBlock, ct, (int32_t)nv, mask, tsum, err);
    PMS_LAUNCH(c, K_BUILD_SCAN, 16.0 * vtiles, k_scan_i64, 1, 1024, tsum, vtiles);
    // index table, code, dimension, value, critical vertex, vertices, column
    if (kV == kBlock)
        PMS_LAUNCH(c, K_LS_INDEX, 24.0 * nv + 45.0 * m, k_ls_emit<kBlock>, (unsigned)vtiles, kBlock, t, ct, vkey, vid, mask,
                   (int32_t)nv, m, tsum, idx, (int32_t *)code, f->dim, (float *)f->value, f->crit, f->verts, f->col_ptr,
                   err);
    else
        PMS_LAUNCH(c, K_LS_INDEX, 24.0 * nv + 45.0 * m, k_ls_emit<32>, (unsigned)vtiles, kBlock, t, ct, vkey, vid, mask,
                   (int32_t)nv, m, tsum, idx, (int32_t *)code, f->dim, (float *)f->value, f->crit, f->verts, f->col_ptr,
                   err);
    // the dimension of the top simplices' faces: at most two cofaces each
    const int face_dim = (nx > 1) + (ny > 1) + (nz > 1) - 1;
    auto rest = [&](const uint32_t *cd) {
        // the simplex's and its cofaces' table entries, left out
        PMS_LAUNCH(c, K_LS_LEFT, 4.0 * m + 4.0 * nnz + 4.0 * m, k_ls_left, grid_for(nv, kLeftV, 65536), kBlock, t, nv, m,
                   idx, f->left, f->second, face_dim, err);
        // + the facets' left, beta out
        PMS_LAUNCH(c, K_LS_ROWS, 12.0 * m + 4.0 * nnz + 4.0 * nnz + 4.0 * nnz + 4.0 * m, k_ls_rows, (unsigned)tiles,
                   kBlock, t, (const int32_t *)cd, m, nnz, idx, f->col_ptr, f->rows, f->left, f->beta, err);
    };
    rest(code);
    PMS_HIP(hipGetLastError());
    int32_t *herr = (int32_t *)c->host_pinned;
    PMS_HIP(hipMemcpyAsync(herr, err, 8, hipMemcpyDeviceToHost, s));
    PMS_HIP(hipStreamSynchronize(s));
    if (!herr[0] && herr[1]) {  // many vertices of one value: nothing was built
        uint32_t *code2 = (uint32_t *)grow_scratch(c, B_BUILD9, nk * 4);
        uint32_t *keys = (uint32_t *)grow_scratch(c, B_BUILD10, nk * 4);
        uint32_t *keys2 = (uint32_t *)grow_scratch(c, B_BUILD11, nk * 4);
        if (!code2 || !keys || !keys2) return set_err(c, PMS_ERR_OOM, "builder scratch");
        uint32_t *place = (uint32_t *)rk;
        int bits = 1;  // of places 0 .. nv
        while ((nv >> bits) != 0) bits++;
        PMS_LAUNCH(c, K_LS_KEYS, 16.0 * nv, k_ls_first, gv, kBlock, vkey, vid, (int32_t)nv, place, err);
        PMS_LAUNCH(c, K_LS_KEYS, 8.0 * nk + 4.0 * nv, k_ls_keys, grid_for(nk, kBlock, 1u << 16), kBlock, t, place, nv,
                   keys, code);
        st = sort(keys, keys2, code, code2, nk, bits);
        if (st != PMS_OK) return st;
        PMS_LAUNCH(c, K_LS_INDEX, 8.0 * m + 33.0 * m, k_ls_index, (unsigned)tiles, kBlock, t, grid, keys, code, m, nv,
                   idx, f->dim, (float *)f->value, f->crit, f->verts, tsum, err);
        PMS_LAUNCH(c, K_BUILD_SCAN, 16.0 * tiles, k_scan_i64, 1, 1024, tsum, tiles);
        PMS_LAUNCH(c, K_BUILD_SCAN, 9.0 * m, k_ls_colptr, (unsigned)tiles, kBlock, f->dim, m, tsum, f->col_ptr);
        rest(code);
        PMS_HIP(hipGetLastError());
        PMS_HIP(hipMemcpyAsync(herr, err, 8, hipMemcpyDeviceToHost, s));
        PMS_HIP(hipStreamSynchronize(s));
    }
    if (c->prof_on) prof_flush(c);
    if (herr[0] == 1) return set_err(c, PMS_ERR_INVALID_ARG, "grid holds NaN");
    if (herr[0]) return set_err(c, PMS_ERR_HIP, "internal: simplex count mismatch in the lower-star builder");
    f->m = m;
    f->nnz = nnz;
    f->value_is_f32 = 1;
    f->has_left_beta = f->has_second = 1;
    return PMS_OK;
}

}  // namespace pms
