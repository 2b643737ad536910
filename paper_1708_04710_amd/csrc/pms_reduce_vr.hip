// The reduction of a Vietoris-Rips filtration built by edge order: block 0 as
// a graph, the blocks above from the faces' side (pms_dual.h), with the
// cofaces of a face computed from the edges' ranks instead of read: nothing of
// the size of the matrix is touched but low* and the outputs.
//
//   k_vr_fill    low* empty, counters and birth bits clear
//   k_vr_h0      one workgroup per cloud: its edges in order placed in a table
//                of vertices in LDS (pms_graph_place.h) until it is connected; then
//                the apparent triangles, and the list of the edges that are left
//   k_vr_cocycle edges over triangles; k_vr_cand, k_dual triangles over tetrahedra
//   k_vr_count, k_vr_scan, k_vr_scatter, k_vr_inst   pairs and essentials
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "pms_build.h"
#include "pms_common.h"
#include "pms_dual.h"
#include "pms_graph_place.h"
#include "pms_vr_edges.h"

namespace pms {

// Edges (by rank within their cloud) over triangles, for the claims.
struct VrEdgeProv {
    VeView v;
    VeCloud I;
    __device__ void bind(int32_t b) { I = v.cl[b]; }
    __device__ int64_t key(int32_t e) const { return I.eoff + e; }
    __device__ int32_t face(int64_t k) const { return (int32_t)(k - I.eoff); }
    __device__ int64_t col(int32_t t) const { return I.col_base + t; }
};

// The edges' columns as cochains.  A column is the coboundary of the set V of
// edges it is the sum of, and is non-zero at a triangle when an odd number of
// its edges is in V.  Reducing it by apparent pairs means: going through the
// edges l in order, the triangle l is apparent with fixes whether l joins V,
// and the first of l's other triangles that this leaves odd is the column's
// low.  With V as a symmetric bit matrix in LDS all triangles of latest edge
// l = (a, b) are tested at once, (V[a] ^ V[b]) & mask(l), and 64 edges at a
// time, one per lane, repeated until none changes (an edge depends on earlier
// ones only; two rounds are the rule).
//
// The same additions one after the other (a bitmap over the triangles, as
// k_dual) took 0.41 us each, and a column up to 4 000 of them: 64 circles of
// 128 points 3.5 ms, 512 clouds 14.4 ms.  Here a column costs a pass over the
// later edges, (E / 64) steps of a few hundred cycles, whatever it adds.
//
// Ties: triangles of a tie group interleave, so the group's edges (at most 64)
// are brought into one step, a step that ends inside a group being cut before
// it, and the low is the smallest index among their odd triangles; edges whose
// apparent triangle lies beyond it stay as they were, and a column that goes on
// from there takes the whole group again.
//
// A step is a chain of a load from L2, LDS reads and ballots: the next step's
// edges are loaded during this one (kM words of masks a lane, or 0: their words
// when needed), and the wavefront waits for nothing else.  (Waiting for every
// load at each of its five synchronisations: 512 clouds 1.93 ms, 64 circles
// 0.23, 400 points 0.82; now 1.62, 0.17, 0.65, bound by the instructions of a step.)
template <int kM>
__global__ void __launch_bounds__(kWave) k_vr_cocycle(VeView v, DualState s, int32_t *kedge, int round)
{
    constexpr int kW = kM ? kM : 1;
    extern __shared__ uint64_t s_v[];  // [n][M]
    const int32_t nq = s.count[round];
    if ((int32_t)blockIdx.x >= nq || *s.fail) return;
    const int lane = threadIdx.x;
    unsigned long long adds = 0, entries = 0;
    for (;;) {
        int32_t q = 0;
        if (lane == 0) q = atomicAdd(&s.head[round], 1);
        q = bcast_first(q);
        if (q >= nq) break;
        const int2 it = s.list[round & 1][q];
        const VeCloud &I = v.cl[bcast_first(it.x)];
        const int32_t face = bcast_first(it.y), n = I.n, M = I.M, E = I.E;
        const int64_t eoff = I.eoff, key = eoff + face;
        const uint32_t *ev = v.ev + eoff;
        const uint64_t *mask = v.mask + I.moff;
        const bool ties = I.gmax > 1;
        auto toggle = [&](uint32_t ab) __attribute__((always_inline)) {
            const int a = (int)(ab >> 16), b = (int)(ab & 0xFFFFu);
            atomicXor((unsigned long long *)&s_v[a * M + (b >> 6)], 1ull << (b & 63));
            atomicXor((unsigned long long *)&s_v[b * M + (a >> 6)], 1ull << (a & 63));
        };
        // what a lane needs of its edge of a step
        struct Step {
            uint32_t ab;
            int32_t c;
            uint64_t m[kW];
        };
        auto load = [&](int32_t l0) __attribute__((always_inline)) {
            const int32_t l = min(l0 + lane, E - 1);
            Step t;
            t.ab = ev[l];
            t.c = v.apc[eoff + l];
            if constexpr (kM > 0) {
#pragma unroll
                for (int w = 0; w < kM; w++) t.m[w] = mask[(int64_t)l * M + min(w, M - 1)];
            }
            return t;
        };
        for (int k = lane; k < n * M; k += kWave) s_v[k] = 0;
        wave_sync();
        const int32_t n0 = s.vlen[key];
        int32_t l0 = face;
        bool moved = n0 > 0;  // V is more than the face
        if (n0 == 0) {
            if (lane == 0) toggle(ev[face]);
        } else {
            const int32_t *a = s.arena + s.vstart[key];
            for (int32_t k = lane; k < n0; k += kWave) toggle((uint32_t)a[k]);
            l0 = kedge[key];
        }
        wave_sync();
        int32_t low = -1;
        bool full = false;
        Step cur = load(l0), ahead;
        int32_t have = l0;
        while (l0 < E) {
            const int32_t l = l0 + lane;
            const bool in = l < E;
            if (have != l0) cur = load(l0);
            ahead = load(l0 + kWave);
            const int32_t l1 = l0 + kWave;
            const uint32_t ab = cur.ab;
            const int c = cur.c;
            const int a = (int)(ab >> 16), b = (int)(ab & 0xFFFFu);
            const uint64_t *ra = s_v + a * M, *rb = s_v + b * M, *rm = mask + (int64_t)(in ? l : E - 1) * M;
            const bool was = (ra[b >> 6] >> (b & 63)) & 1;
            bool now = was;
            // which edges join, and the first triangle left odd
            uint64_t x[kW];
            for (;;) {
                bool want = now;
                if constexpr (kM > 0) {
                    uint64_t xc = 0;
#pragma unroll
                    for (int w = 0; w < kM; w++) {
                        const int q = min(w, M - 1);
                        x[w] = ra[q] ^ rb[q];
                        xc = (c >> 6) == w ? x[w] : xc;
                    }
                    if (in && c >= 0) want = (xc >> (c & 63)) & 1;
                } else if (in && c >= 0) {
                    want = ((ra[c >> 6] ^ rb[c >> 6]) >> (c & 63)) & 1;
                }
                const bool ch = in && want != now;
                wave_sync();
                if (__ballot(ch) == 0) break;
                if (ch) {
                    now = want;
                    toggle(ab);
                }
                wave_sync();
            }
            int first = -1;
            if (in) {
                if constexpr (kM > 0) {
#pragma unroll
                    for (int w = kM - 1; w >= 0; w--) {
                        const uint64_t y = w < M ? (x[w] & cur.m[w]) ^ (now ? cur.m[w] : 0ull) : 0ull;
                        first = y ? w * 64 + __ffsll((long long)y) - 1 : first;
                    }
                } else {
                    for (int w = 0; w < M && first < 0; w++) {
                        const uint64_t m = rm[w], y = ((ra[w] ^ rb[w]) & m) ^ (now ? m : 0ull);
                        if (y) first = w * 64 + __ffsll((long long)y) - 1;
                    }
                }
            }
            const uint64_t odd = __ballot(first >= 0);
            wave_sync();
            int32_t stop = kWave;  // lanes from here on stay as they were
            int32_t again = l0 + kWave;
            low = -1;
            if (odd) {
                const int f = __ffsll((long long)odd) - 1;
                const int32_t lf = l0 + f;
                const int32_t g1 = v.gend[eoff + lf];
                const int32_t g0 = v.gst[eoff + lf];
                if (g1 - g0 == 1) {
                    low = __builtin_amdgcn_readlane(in && first >= 0 ? ve_tri(v, I, l, first) : 0, f);
                    stop = f + 1;
                    again = lf;
                } else if (g1 > l0 + kWave && g0 > l0) {  // the group into one step
                    stop = g0 - l0;
                    again = g0;
                } else {
                    int32_t t = 0x7FFFFFFF;
                    if (first >= 0 && l < g1) t = ve_tri(v, I, l, first);
                    for (int o = kWave / 2; o > 0; o >>= 1) t = min(t, __shfl_xor(t, o, kWave));
                    low = bcast_first(t);
                    stop = g1 - l0;
                    again = g0;
                }
            } else if (ties && l0 + kWave < E) {  // (no group reaches past a step it starts)
                const int32_t g0 = v.gst[eoff + l0 + kWave];
                if (g0 > l0) {
                    stop = g0 - l0;
                    again = g0;
                }
            }
            const bool undo = now != was && (lane >= stop || (low >= 0 && v.app[eoff + (in ? l : E - 1)] > low));
            if (undo) toggle(ab);
            const uint64_t joined = __ballot(now != was && !undo);
            adds += __popcll(joined);
            moved = moved || joined;
            wave_sync();
            cur = ahead;
            have = l1;
            if (low < 0) {
                l0 = again;
                continue;
            }
            const int32_t ls = bcast_first(s.low_star[I.col_base + low]);  // (not written during a round)
            l0 = again;
            if (ls == -1) break;
            const int64_t ko = -2 - (int64_t)ls;
            if (ls >= 0) { full = true; break; }  // (never: an apparent triangle is even)
            if (ko < key) break;  // an owner further on: it gives way
            const int32_t no = s.vlen[ko];
            if (no > 0) {
                const int32_t *x = s.arena + s.vstart[ko];
                for (int32_t k = lane; k < no; k += kWave) toggle((uint32_t)x[k]);
            } else if (lane == 0) {
                toggle(v.ev[ko]);
            }
            entries += no > 0 ? no : 1;
            adds++;
            moved = true;
            low = -1;
            wave_sync();
        }
        // remember V as its edges (the face alone needs no list)
        if (!full && moved && low >= 0) {
            int32_t cnt = 0;
            for (int k = lane; k < n * M; k += kWave) {
                const int r = k / M, w = k - r * M;
                uint64_t x = s_v[k];
                if (w == (r >> 6)) x &= ~(2ull * (1ull << (r & 63)) - 1ull);  // columns after the row
                else if (w < (r >> 6)) x = 0;
                cnt += __popcll(x);
            }
            const int32_t inc = wave_incl_sum32(cnt), nv = bcast_lane(inc, kWave - 1);
            int32_t at = 0;
            if (lane == 0) at = atomicAdd(s.arena_top, nv);
            at = bcast_first(at);
            if (at < 0 || (int64_t)at + nv > s.arena_cap) full = true;
            else {
                int32_t *o = s.arena + at + inc - cnt;
                for (int k = lane; k < n * M; k += kWave) {
                    const int r = k / M, w = k - r * M;
                    uint64_t x = s_v[k];
                    if (w == (r >> 6)) x &= ~(2ull * (1ull << (r & 63)) - 1ull);
                    else if (w < (r >> 6)) x = 0;
                    for (; x; x &= x - 1) *o++ = (int32_t)((uint32_t)r << 16 | (uint32_t)(w * 64 + __ffsll((long long)x) - 1));
                }
                entries += nv;
                if (lane == 0) {
                    s.vstart[key] = at;
                    s.vlen[key] = nv;
                    kedge[key] = l0;
                }
            }
        } else if (lane == 0) {
            kedge[key] = face;
        }
        if (lane == 0) {
            s.klow[key] = low;
            if (full) *s.fail = 1;
        }
        wave_sync();
        if (full) break;
    }
    if (lane == 0) {
        if (adds) atomicAdd(s.adds, adds);
        if (entries) atomicAdd(s.entries, entries);
    }
}

// Triangles (by index within their cloud) over tetrahedra: eight wavefronts, a
// lane per fourth vertex (of the up to 512 at a time), so that an addition is
// three dependent loads whatever the cloud's size; lists a face per wavefront.
struct VrTriProv {
    static constexpr int kT = 512;
    VeView v;
    const int4 *verts;
    VeCloud I;
    __device__ void bind(int32_t b) { I = v.cl[b]; }
    __device__ int64_t key(int32_t p) const { return I.col_base + p; }
    __device__ int32_t face(int64_t k) const { return (int32_t)(k - I.col_base); }
    __device__ int64_t col(int32_t t) const { return I.col_base + t; }
    __device__ int32_t floor(int32_t p) const { return p; }
    __device__ int32_t apparent(int32_t, int32_t ls) const { return (int32_t)(ls - I.col_base); }
    // the triangle's vertices, 16 bits each
    __device__ void load(int32_t p, int32_t &d0, int32_t &d1) const
    {
        const int4 q = verts[I.col_base + p];
        d0 = (int32_t)((uint32_t)(q.x - I.pbase) << 16 | (uint32_t)(q.y - I.pbase));
        d1 = (int32_t)(q.z - I.pbase);
    }
    // the cofaces with d = first, first + step, ..
    __device__ int cofaces(const DualMap<kT> &map, int32_t d0, int32_t d1, int first, int step, int32_t cur,
                           DualCand &cand) const
    {
        const int x = (int)((uint32_t)d0 >> 16), y = (int)((uint32_t)d0 & 0xFFFFu), z = d1;
        const int32_t *R = v.erank + I.slot_base;
        const int32_t *rx = R + (int64_t)x * I.n, *ry = R + (int64_t)y * I.n, *rz = R + (int64_t)z * I.n;
        const int32_t xy = rx[y], xz = rx[z], yz = ry[z], xyz = max(max(xy, xz), yz);
        const int off = xyz == xy ? z : xyz == xz ? y : x;  // the vertex off the triangle's latest edge
        int n = 0;
        int32_t best = 0x7FFFFFFF, bl = 0;
        int bd = 0;
        constexpr int kAhead = 4;
        for (int e0 = first; e0 < I.n; e0 += kAhead * step) {
            int32_t xd[kAhead], yd[kAhead], zd[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; u++) {
                const int d = e0 + u * step < I.n ? e0 + u * step : x;  // (the diagonal is no edge)
                xd[u] = rx[d];
                yd[u] = ry[d];
                zd[u] = rz[d];
            }
            int32_t l[kAhead], p[kAhead];
            int s[kAhead], t[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; u++) {
                const int d = e0 + u * step;
                l[u] = -1;
                s[u] = off;
                t[u] = d;  // the two vertices off the latest edge
                if (xd[u] == kNoEdge || yd[u] == kNoEdge || zd[u] == kNoEdge) continue;
                l[u] = max(max(xyz, xd[u]), max(yd[u], zd[u]));
                if (l[u] != xyz) {
                    s[u] = l[u] == xd[u] ? y : x;
                    t[u] = l[u] == zd[u] ? y : z;
                }
            }
#pragma unroll
            for (int u = 0; u < kAhead; u++) p[u] = l[u] >= 0 ? ve_tet(v, I, l[u], min(s[u], t[u]), max(s[u], t[u])) : -1;
#pragma unroll
            for (int u = 0; u < kAhead; u++) {
                if (p[u] < 0) continue;
                map.toggle(p[u]);
                n++;
                if (p[u] > cur && p[u] < best) {
                    best = p[u];
                    bl = l[u];
                    bd = max(s[u], t[u]);
                }
            }
        }
        cand.t = best;
        cand.f = -1;
        if (best != 0x7FFFFFFF) {
            // an apparent tetrahedron's face is its last facet, without ties
            // that of the latest edge and the later of the other two vertices
            const int32_t p = ve_tri(v, I, bl, bd);
            const uint32_t ab = v.ev[I.eoff + bl];
            const int a = (int)(ab >> 16), b = (int)(ab & 0xFFFFu), lo = min(a, bd), hi = max(b, bd);
            cand.d0 = (int32_t)((uint32_t)lo << 16 | (uint32_t)(a + b + bd - lo - hi));
            cand.d1 = hi;
            if (v.appt[I.col_base + p] == best) cand.f = p;
        }
        return n;
    }
    __device__ int flip(const DualMap<kT> &map, int32_t, int32_t d0, int32_t d1, int32_t cur, DualCand &cand) const
    {
        return cofaces(map, d0, d1, (int)threadIdx.x, kT, cur, cand);
    }
    __device__ int flip_many(const DualMap<kT> &map, const int32_t *faces, int32_t cnt) const
    {
        int n = 0;
        DualCand unused;
        for (int32_t k = threadIdx.x / kWave; k < cnt; k += kT / kWave) {
            int32_t d0, d1;
            load(faces[k], d0, d1);
            n += cofaces(map, d0, d1, (int)(threadIdx.x & (kWave - 1)), kWave, 0x7FFFFFFE, unused);
        }
        return n;
    }
};

struct VrTotals {
    int32_t n_pairs, n_ess;
    int32_t apparent, pad;
    unsigned long long adds, entries;
};

constexpr int kFinTile = 1024;  // columns per workgroup of the output kernels

__global__ void __launch_bounds__(kBlock) k_vr_fill(int32_t *low_star, int64_t m, uint32_t *bits, int64_t nwords,
                                                    int32_t *tile_e, int64_t tiles, VrTotals *tot)
{
    const int64_t g = blockIdx.x * (int64_t)kBlock + threadIdx.x, st = (int64_t)gridDim.x * kBlock;
    for (int64_t j = g; j < m; j += st) low_star[j] = -1;
    for (int64_t j = g; j < nwords; j += st) bits[j] = 0u;
    for (int64_t j = g; j < tiles; j += st) tile_e[j] = 0;
    if (g == 0) *tot = VrTotals{0, 0, 0, 0, 0ull, 0ull};
}

__global__ void __launch_bounds__(1024) k_vr_h0(VeView v, DualState s, int maxdim, int32_t *face_col, VrTotals *tot)
{
    __shared__ unsigned long long P[1024];
    __shared__ int32_t s_left;
    const VeCloud I = v.cl[blockIdx.x];
    const int nt = blockDim.x, tid = threadIdx.x, lane = tid & (kWave - 1);
    for (int x = tid; x < I.n; x += nt) P[x] = kGraphEmpty;
    __syncthreads();
    for (int32_t e0 = 0; e0 < I.E; e0 += nt) {
        if (e0 + tid < I.E) {
            const uint32_t ab = v.ev[I.eoff + e0 + tid];
            graph_place<false>(P, (uint32_t)(e0 + tid), (int32_t)(ab >> 16), (int32_t)(ab & 0xFFFFu));
        }
        if (tid == 0) s_left = 0;
        __syncthreads();
        int32_t left = 0;
        for (int x = tid; x < I.n; x += nt) left += P[x] == kGraphEmpty;
        left = wave_sum_dpp(left);
        if (lane == 0 && left) atomicAdd(&s_left, left);
        __syncthreads();
        if (s_left == 1) break;  // connected: the later edges close cycles
        __syncthreads();
    }
    __syncthreads();
    const int32_t *ix = v.eidx + I.slot_base;
    for (int x = tid; x < I.n; x += nt) {
        if (P[x] == kGraphEmpty) continue;
        const uint32_t ab = v.ev[I.eoff + (int32_t)(P[x] >> 32)];
        s.low_star[I.col_base + ix[(int64_t)(ab >> 16) * I.n + (ab & 0xFFFFu)]] = (int32_t)I.col_base + x;
    }
    __syncthreads();
    int32_t napp = 0;
    for (int32_t e0 = 0; e0 < I.E; e0 += nt) {
        const int32_t e = e0 + tid;
        bool list = false;
        if (e < I.E) {
            const uint32_t ab = v.ev[I.eoff + e];
            const int32_t col = (int32_t)I.col_base + ix[(int64_t)(ab >> 16) * I.n + (ab & 0xFFFFu)];
            const int32_t t = v.app[I.eoff + e];
            face_col[I.eoff + e] = col;
            s.vlen[I.eoff + e] = 0;
            if (t >= 0) {
                s.low_star[I.col_base + t] = col;
                napp++;
            }
            list = maxdim >= 2 && t < 0 && s.low_star[col] == -1;
        }
        const uint64_t mk = __ballot(list);
        if (mk) {
            int32_t at = 0;
            if (lane == __ffsll((long long)mk) - 1) at = atomicAdd(&s.count[0], __popcll(mk));
            at = __shfl(at, __ffsll((long long)mk) - 1, kWave) + __popcll(mk & ((1ull << lane) - 1ull));
            if (list) s.list[0][at] = make_int2((int32_t)blockIdx.x, e);
        }
    }
    napp = wave_sum_dpp(napp);
    if (lane == 0 && napp) atomicAdd(&tot->apparent, napp);
}

// The triangles of one cloud: apparent ones paired, those that are neither
// apparent nor negative listed (dimension 3).
__global__ void __launch_bounds__(kBlock) k_vr_cand(VeView v, DualState s, const int8_t *dim, VrTotals *tot)
{
    const VeCloud I = v.cl[blockIdx.y];
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t mb = I.n + I.E + I.T + I.Q;
    int32_t napp = 0;
    for (int64_t p0 = (int64_t)blockIdx.x * kBlock; p0 < mb; p0 += (int64_t)gridDim.x * kBlock) {
        const int64_t p = p0 + threadIdx.x, g = I.col_base + p;
        bool list = false;
        if (p < mb && dim[g] == 2) {
            const int32_t q = v.appt[g];
            s.vlen[g] = 0;
            if (q >= 0) {
                s.low_star[I.col_base + q] = (int32_t)g;
                napp++;
            }
            list = q < 0 && s.low_star[g] == -1;
        }
        const uint64_t mk = __ballot(list);
        if (mk) {
            int32_t at = 0;
            if (lane == __ffsll((long long)mk) - 1) at = atomicAdd(&s.count[0], __popcll(mk));
            at = __shfl(at, __ffsll((long long)mk) - 1, kWave) + __popcll(mk & ((1ull << lane) - 1ull));
            if (list) s.list[0][at] = make_int2((int32_t)blockIdx.y, (int32_t)p);
        }
    }
    napp = wave_sum_dpp(napp);
    if (lane == 0 && napp) atomicAdd(&tot->apparent, napp);
}

// Claims into columns (an edge's key by its table, a triangle's is its
// column), births marked, deaths and essentials counted per tile.  Most births
// lie in the tile of their death: those are counted in registers (an atomic
// each: 28 M columns of 512 clouds 220 us, now 75; 100 points 25 and 6).
__global__ void __launch_bounds__(kBlock) k_vr_count(int32_t *low_star, int64_t m, const int8_t *dim,
                                                     const int32_t *face_col, uint32_t *bits, int32_t *tile_d,
                                                     int32_t *tile_e)
{
    const int64_t tiles = (m + kFinTile - 1) / kFinTile;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        int32_t nd = 0, nb = 0;  // deaths; births among this tile's columns
#pragma unroll
        for (int u = 0; u < kFinTile / kBlock; u++) {
            const int64_t j = tile * kFinTile + u * kBlock + threadIdx.x;
            if (j >= m) continue;
            int32_t x = low_star[j];
            if (x == -1) continue;
            if (x < -1) {
                const int64_t k = -2 - (int64_t)x;
                x = dim[j] == 2 ? face_col[k] : (int32_t)k;
                low_star[j] = x;
            }
            nd++;
            atomicOr(&bits[x >> 5], 1u << (x & 31));
            if (x / kFinTile == tile) nb++;
            else atomicSub(&tile_e[x / kFinTile], 1);
        }
        const int64_t t = block_sum64((int64_t)nd | (int64_t)nb << 32);
        if (threadIdx.x == 0) {
            tile_d[tile] = (int32_t)t;
            atomicAdd(&tile_e[tile], (int32_t)(min((int64_t)kFinTile, m - tile * kFinTile) - (t & 0xFFFFFFFF) - (t >> 32)));
        }
    }
}

__global__ void __launch_bounds__(1024) k_vr_scan(int32_t *tile_d, int32_t *tile_e, int64_t tiles, VrTotals *tot)
{
    const int32_t t = block_seg_scan(blockIdx.x ? tile_e : tile_d, tiles, 0, [](int32_t x, int32_t y) { return x + y; });
    if (threadIdx.x == 0) *(blockIdx.x ? &tot->n_ess : &tot->n_pairs) = t;
}

__global__ void __launch_bounds__(kBlock) k_vr_scatter(const int32_t *low_star, int64_t m, const uint32_t *bits,
                                                       const int32_t *tile_d, const int32_t *tile_e, int32_t *birth,
                                                       int32_t *death, int64_t cap_p, int32_t *ess, int64_t cap_e)
{
    constexpr int kPer = kFinTile / kBlock;
    const int64_t tiles = (m + kFinTile - 1) / kFinTile;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t j0 = tile * kFinTile + threadIdx.x * kPer;
        int32_t x[kPer];
        uint32_t b = 0;
        int32_t nd = 0, ne = 0;
        if (j0 < m) b = bits[j0 >> 5] >> (j0 & 31);
#pragma unroll
        for (int u = 0; u < kPer; u++) {
            x[u] = j0 + u < m ? low_star[j0 + u] : -2;
            nd += x[u] >= 0;
            ne += x[u] == -1 && !((b >> u) & 1u);
        }
        // both prefix sums in one scan: at most 1024 of each
        int32_t tot;
        const int32_t pre = block_excl_sum32(nd | ne << 16, &tot);
        int64_t pd = tile_d[tile] + (pre & 0xFFFF), pe = tile_e[tile] + (pre >> 16);
#pragma unroll
        for (int u = 0; u < kPer; u++) {
            if (x[u] >= 0) {
                if (birth && pd < cap_p) {
                    birth[pd] = x[u];
                    death[pd] = (int32_t)(j0 + u);
                }
                pd++;
            } else if (x[u] == -1 && !((b >> u) & 1u)) {
                if (ess && pe < cap_e) ess[pe] = (int32_t)(j0 + u);
                pe++;
            }
        }
    }
}

// Where the instances' pairs and essentials start, and every pair's instance.
__global__ void __launch_bounds__(kBlock) k_vr_inst(int32_t count, const int64_t *col_off, const VrTotals *tot,
                                                    const int32_t *death, const int32_t *ess, int64_t *pair_off,
                                                    int64_t *ess_off, int32_t *pair_inst)
{
    const int64_t g = blockIdx.x * (int64_t)kBlock + threadIdx.x, st = (int64_t)gridDim.x * kBlock;
    auto first_ge = [](const int32_t *a, int64_t n, int64_t x) {
        int64_t lo = 0, hi = n;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (a[mid] < x) lo = mid + 1;
            else hi = mid;
        }
        return lo;
    };
    for (int64_t b = g; b <= count; b += st) {
        if (pair_off) pair_off[b] = death ? first_ge(death, tot->n_pairs, col_off[b]) : 0;
        if (ess_off) ess_off[b] = ess ? first_ge(ess, tot->n_ess, col_off[b]) : 0;
    }
    if (pair_inst && death)
        for (int64_t k = g; k < tot->n_pairs; k += st) {
            const int64_t j = death[k];
            int32_t lo = 0, hi = count - 1;
            while (lo < hi) {
                const int32_t mid = (lo + hi + 1) >> 1;
                if (col_off[mid] <= j) lo = mid;
                else hi = mid - 1;
            }
            pair_inst[k] = lo;
        }
}

// *done = 0 (status PMS_OK): a list outgrew its room; nothing but scratch and
// unspecified outputs was written.
pms_status reduce_vr(Ctx *c, const Filtration *f, pms_result *res, int32_t count, const int64_t *inst_col_off,
                     int64_t *inst_pair_off, int64_t *inst_ess_off, int32_t *pair_inst, int *done)
{
    *done = 0;
    const int64_t m = f->m;
    const int32_t B = f->vr_count, maxdim = f->vr_maxdim;
    hipStream_t st = c->stream;
    const VeView v = filtration_vr_view(f);
    const int64_t tiles = (m + kFinTile - 1) / kFinTile, nwords = (m + 31) / 32;
    const int64_t nkey = std::max<int64_t>(f->vr_edges, maxdim >= 3 ? m : 0);

    DualState s{};
    // workgroups: as many as the CUs' LDS holds.  Edges: a bit matrix of the
    // points.  Triangles: a bitmap of the cloud, or of as much of it as fits,
    // moving on (what lies beyond waits in the overflow list).
    auto resident = [&](int64_t lds_bytes) {
        return 256 * std::max<int64_t>(1, std::min<int64_t>(16, 160 * 1024 / (lds_bytes + 512)));
    };
    unsigned blocks_of[2] = {1, 1};
    blocks_of[0] = (unsigned)std::min<int64_t>(resident((int64_t)f->vr_max_n * ((f->vr_max_n + 63) / 64) * 8),
                                               std::max<int64_t>(f->vr_edges, 1));
    const DualLimits &lim = c->dual;
    if (maxdim >= 3) {
        const int64_t bits = std::min<int64_t>(f->vr_max_m, lim.bits ? lim.bits : kDualLdsBits);
        s.nw0 = dual_words(bits);
        s.nw1 = dual_summary_words(bits);
        blocks_of[1] = (unsigned)std::min<int64_t>(std::min<int64_t>(resident((s.nw1 + s.nw0) * 4), 1024),
                                                   std::max<int64_t>(nkey, 1));
        if (f->vr_max_m > bits) s.ovf_cap = lim.beyond ? std::min(lim.beyond, 1 << 18) : 1 << 18;
    }
    const unsigned blocks = blocks_of[1];
    s.vcap = lim.sum ? std::min(lim.sum, 8192) : 8192;
    s.arena_cap = std::max<int64_t>(1 << 20, 16 * f->vr_edges);
    if (lim.arena) s.arena_cap = std::min<int64_t>(s.arena_cap, lim.arena);
    s.low_star = res->low_star;
    int32_t *cnt = (int32_t *)grow_scratch(c, B_DUAL0, (size_t)kDualCounters * 4 + sizeof(VrTotals));
    s.list[0] = (int2 *)grow_scratch(c, B_DUAL1, (size_t)nkey * 8);
    s.list[1] = (int2 *)grow_scratch(c, B_DUAL2, (size_t)nkey * 8);
    int32_t *keys = (int32_t *)grow_scratch(c, B_DUAL3, (size_t)nkey * 5 * 4);
    s.arena = (int32_t *)grow_scratch(c, B_DUAL4, (size_t)(s.arena_cap + (int64_t)blocks * s.vcap) * 4);
    uint32_t *bits = (uint32_t *)grow_scratch(c, B_NEG, (size_t)nwords * 4);
    int32_t *tile_d = (int32_t *)grow_scratch(c, B_AGG2, (size_t)tiles * 4);
    int32_t *tile_e = (int32_t *)grow_scratch(c, B_FLAGS, (size_t)tiles * 4);
    s.ovf = s.ovf_cap ? (int32_t *)grow_scratch(c, B_DUAL5, (size_t)blocks * s.ovf_cap * 4) : nullptr;
    if (!cnt || !s.list[0] || !s.list[1] || !keys || !s.arena || !bits || !tile_d || !tile_e || (s.ovf_cap && !s.ovf))
        return set_err(c, PMS_ERR_OOM, "scratch allocation failed");
    VrTotals *tot = (VrTotals *)cnt;
    dual_counters(s, cnt + sizeof(VrTotals) / 4);
    s.vstart = keys;
    s.vlen = keys + nkey;
    s.klow = keys + 2 * nkey;
    int32_t *face_col = keys + 3 * nkey, *kedge = keys + 4 * nkey;
    s.vtmp = s.arena + s.arena_cap;
    s.adds = &tot->adds;
    s.entries = &tot->entries;

    const double dm = (double)m;
    PMS_LAUNCH(c, K_FILL, 4 * dm + dm / 8, k_vr_fill, grid_for(m, kBlock * 4, 8192), kBlock, res->low_star, m, bits, nwords,
               tile_e, tiles, tot);
    PMS_LAUNCH(c, K_FILL, 0, k_dual_counters, 1, kBlock, s, 1, 0);
    PMS_LAUNCH(c, K_GRAPH, 24.0 * f->vr_edges, k_vr_h0, (unsigned)B, B >= 256 ? 256 : 1024, v, s, maxdim, face_col, tot);
    int32_t rounds = 0;
    int64_t active = 0;
    int ok = 1;
    if (maxdim >= 2) {
        const VrEdgeProv pe{v, {}};
        const size_t lds = (size_t)f->vr_max_n * ((f->vr_max_n + 63) / 64) * 8;
        const int words = (f->vr_max_n + 63) / 64;
        auto *fn = words <= 1 ? k_vr_cocycle<1> : words <= 2 ? k_vr_cocycle<2> : words <= 4 ? k_vr_cocycle<4> : words <= 8 ? k_vr_cocycle<8> : k_vr_cocycle<0>;
        PMS_ALLOW_LDS(fn, 1023 * 16 * 8);  // (the most points of a cloud)
        const pms_status sd = dual_rounds(
            c, pe, s, [&](int r) { fn<<<blocks_of[0], kWave, lds, st>>>(v, s, kedge, r); }, K_DUAL, &rounds, &active, &ok);
        if (sd != PMS_OK) return sd;
        if (!ok) return PMS_OK;
    }
    if (maxdim >= 3) {
        PMS_LAUNCH(c, K_FILL, 0, k_dual_counters, 1, kBlock, s, 1, 0);
        const unsigned gx = (unsigned)std::max<int64_t>(1, std::min<int64_t>((f->vr_max_m + kBlock - 1) / kBlock, std::max(16, 16384 / B)));
        PMS_LAUNCH(c, K_DUAL, 5 * dm, k_vr_cand, dim3(gx, (unsigned)B), kBlock, v, s, f->dim, tot);
        VrTriProv pt{v, (const int4 *)f->verts, {}};
        pms_status sd = dual_map_lds(c, pt);
        if (sd == PMS_OK)
            sd = dual_rounds(c, pt, s, [&](int r) { dual_launch(c, pt, s, blocks_of[1], r); }, K_DUAL, &rounds, &active, &ok);
        if (sd != PMS_OK) return sd;
        if (!ok) return PMS_OK;
    }
    const unsigned gt = grid_for(tiles, 1, 65536);
    const bool want_pairs = res->pair_birth && res->pair_death;
    const bool want_ess = res->essential != nullptr;
    PMS_LAUNCH(c, K_FINAL, 4 * dm, k_vr_count, gt, kBlock, res->low_star, m, f->dim, face_col, bits, tile_d, tile_e);
    PMS_LAUNCH(c, K_SCAN, 16.0 * tiles, k_vr_scan, 2, 1024, tile_d, tile_e, tiles, tot);
    if (want_pairs || want_ess)
        PMS_LAUNCH(c, K_FINAL, 8 * dm, k_vr_scatter, gt, kBlock, res->low_star, m, bits, tile_d, tile_e,
                   want_pairs ? res->pair_birth : nullptr, want_pairs ? res->pair_death : nullptr, res->cap_pairs,
                   want_ess ? res->essential : nullptr, res->cap_essential);
    VrTotals &h = *(VrTotals *)c->host_pinned;
    PMS_HIP(hipMemcpyAsync(&h, tot, sizeof(h), hipMemcpyDeviceToHost, st));
    std::vector<int64_t> off;
    if (inst_col_off) {
        // (a pair list too small for its pairs is not read beyond its end)
        const bool fits = res->cap_pairs >= m / 2 && (!want_ess || res->cap_essential >= m);
        if (!fits) {
            PMS_HIP(hipStreamSynchronize(st));
            if ((want_pairs && res->cap_pairs < h.n_pairs) || (want_ess && res->cap_essential < h.n_ess)) {
                res->n_pairs = h.n_pairs;
                res->n_essential = h.n_ess;
                *done = 1;
                return set_err(c, PMS_ERR_CAPACITY, "output capacity too small (n_pairs / n_essential hold the sizes)");
            }
        }
        if (inst_pair_off || inst_ess_off || pair_inst)
            PMS_LAUNCH(c, K_FINAL, 16.0 * count, k_vr_inst, grid_for(std::max<int64_t>(count + 1, m / 64), kBlock, 2048),
                       kBlock, count, inst_col_off, tot, want_pairs ? res->pair_death : nullptr, res->essential,
                       inst_pair_off, inst_ess_off, pair_inst);
        off.resize((size_t)count + 1);
        PMS_HIP(hipMemcpyAsync(off.data(), inst_col_off, off.size() * 8, hipMemcpyDeviceToHost, st));
    }
    PMS_HIP(hipGetLastError());
    PMS_HIP(hipStreamSynchronize(st));
    if (c->prof_on) prof_flush(c);
    *done = 1;
    if (inst_col_off) {
        bool good = off[0] == 0 && off[(size_t)count] == m;
        for (int32_t b = 0; good && b < count; b++) good = off[(size_t)b] <= off[(size_t)b + 1];
        if (!good)
            return set_err(c, PMS_ERR_INVALID_ARG, "inst_col_off must ascend from 0 to m (count + 1 entries)");
    }
    res->n_pairs = h.n_pairs;
    res->n_essential = h.n_ess;
    res->rounds = rounds + 1;  // (block 0 is one)
    res->phase0_pivots = h.apparent;
    res->additions = (int64_t)h.adds;
    res->xor_entries = (int64_t)h.entries;
    res->active_sum = active;
    res->addition_bytes = (int64_t)(8 * h.entries);  // (as k_dual's abytes)
    if ((want_pairs && res->cap_pairs < res->n_pairs) || (want_ess && res->cap_essential < res->n_essential))
        return set_err(c, PMS_ERR_CAPACITY, "output capacity too small (n_pairs / n_essential hold the sizes)");
    return PMS_OK;
}

}  // namespace pms
