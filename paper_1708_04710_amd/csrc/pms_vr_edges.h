// Vietoris-Rips filtrations by edge order: what the builder leaves behind for
// the reduction, and the index of a simplex from its vertices.
//
// A simplex enters with its latest edge, so a cloud's filtration is its edges
// in order (value, then lexicographic), each followed by the triangles, then
// the tetrahedra, whose latest edge it is.  With e = (a, b) fixed, the
// triangles (e, c) ascend with c and the tetrahedra (e, {c, d}) with (c, d):
// the lexicographic order of two sets of vertices of one size is decided by
// the smallest vertex of their symmetric difference, and {a, b} is common.
// So every index follows from the edges' ranks, a bitmask per edge and prefix
// counts, with no sort of the simplices.  Edges of equal value (a tie group)
// share their range: a triangle's place in it is the number of the group's
// triangles with a smaller vertex tuple, counted by one bound per edge.
#pragma once

#include "pms_common.h"

namespace pms {

constexpr int32_t kNoEdge = 0x7FFFFFFF;     // rank of a pair that is no edge (and of the diagonal)
// Edges of one value that the tie counting handles: a triangle's place costs
// one bound and W popcounts per edge of its group, a tetrahedron's as much
// per triangle of the group.  One cloud with a larger group (12 equal points
// have 66 edges of length 0) sends its whole batch to the sorted build and the
// reduction of its matrix: 64 full clouds of 100 points take 0.89 ms, 12.8 when 14
// points of each are equal, 16.9 when of one cloud (13.7 and 18.4 before there
// was a build by edge order).
constexpr int32_t kVeMaxTies = 64, kVeMaxTies3 = 8;
constexpr uint32_t kTied = 0x80000000u;     // rec.y of an edge in a tie group

struct VeCloud {
    int32_t n, D, W, M;         // points, coordinates, mask words of 32 and 64 per edge
    int32_t has_thr, pad;
    int64_t thr_i;
    float thr_f;
    int32_t E;                  // edges
    int64_t pt_off, pbase;      // first coordinate in pts; global id of point 0
    int64_t slot_base;          // start of its n x n matrices
    int64_t cap_off;            // start of its edges in the capacity-sized scratch
    int64_t eoff;               // start of its edges (E + 1 entries)
    int64_t woff, moff;         // start of its mask words of 32 and 64 (E W and E M entries)
    int64_t T, Q;               // triangles, tetrahedra
    int64_t col_base, nnz_base; // first column, first row entry
    int64_t toff;               // its first triangle among all clouds' (dimension 3)
    int64_t qfirst;             // q2 there
    int32_t gmax;               // edges of the largest tie group
    int32_t W2;                 // words per triangle in rec2 (one stride for the batch)
};

// Device arrays left with the filtration.
struct VeView {
    const VeCloud *cl;
    const uint32_t *ev;       // [edge] a << 16 | b, a < b
    const int32_t *erank;     // [slot] rank of edge (a, b), symmetric, kNoEdge when absent
    const int32_t *eidx;      // [slot] its index within the cloud
    const uint2 *rec;         // [edge W + c / 32] x: the c whose triangle (e, c) has latest edge e;
                              // y: index within the cloud of the first of them (kTied: tie group)
    const int32_t *gst, *gend;// [edge] its tie group's ranks [gst, gend)
    const int32_t *tscan;     // [edge, E + 1] triangles before it
    const int64_t *q2;        // [triangle, T + 1] all clouds' tetrahedra before its own (dimension 3)
    const uint64_t *mask;     // [moff + edge M + c / 64] rec's x in words of 64
    const int32_t *apc;       // [edge] the third vertex of that triangle, -1: none
    const int32_t *app;       // [edge] index of the triangle it forms an apparent pair with, -1: none
    const uint32_t *recd;     // [edge W + c / 32] dense number of the first triangle of the word (dimension 3)
    const uint2 *rec2;        // [(toff + dense) W2 + d / 32] like rec for the tetrahedra (e, c, d), d > c
    const int32_t *appt;      // [column] index of the tetrahedron a triangle is apparent with, -1: none
};

__device__ inline uint32_t below(int c) { return (1u << (c & 31)) - 1u; }

// The number of vertices c' with the sorted tuple (a, b, c') < (x, y, z), as
// a bound: c' < bound exactly when it is (a < b; c' not a or b).
__device__ inline int ve_bound(int a, int b, int x, int y, int z)
{
    // c' < a: (c', a, b)
    const bool eq1 = a < y || (a == y && b < z);
    int k = x + (eq1 ? 1 : 0);
    if (k <= a) return k;
    // a < c' < b: (a, c', b)
    if (a > x) return a;
    if (a == x) {
        const int k2 = y + (b < z ? 1 : 0);
        if (k2 <= a) return a;
        if (k2 <= b) return k2;
    }
    // c' > b: (a, b, c')
    if (a < x || (a == x && b < y)) return 0x7FFFFFFF;
    if (a == x && b == y) return z > b ? z : b;
    return b;
}

// A triangle's place among those of its tie group.
__device__ inline int32_t ve_tie_rank(const VeView &v, const VeCloud &I, int32_t e, int c)
{
    const uint32_t ab = v.ev[I.eoff + e];
    const int a = (int)(ab >> 16), b = (int)(ab & 0xFFFFu);
    const int x = min(a, c), z = max(b, c), y = a + b + c - x - z;
    int32_t r = 0;
    for (int32_t f = v.gst[I.eoff + e]; f < v.gend[I.eoff + e]; f++) {
        const uint32_t fg = v.ev[I.eoff + f];
        const int k = min(ve_bound((int)(fg >> 16), (int)(fg & 0xFFFFu), x, y, z), I.n);
        const uint2 *w = v.rec + I.woff + (int64_t)f * I.W;
        for (int q = 0; q * 32 < k; q++) r += __popc(k - q * 32 >= 32 ? w[q].x : w[q].x & below(k));
    }
    return r;
}

// Tetrahedra of the cloud before those of edge e (0 <= e <= E).
__device__ inline int32_t ve_q(const VeView &v, const VeCloud &I, int32_t e)
{
    return v.q2 ? (int32_t)(v.q2[I.toff + v.tscan[I.eoff + e]] - I.qfirst) : 0;
}

// First index (within the cloud) of the triangles of edge e's tie group.
__device__ inline int32_t ve_tri_first(const VeView &v, const VeCloud &I, int32_t e)
{
    const int32_t g = v.gst[I.eoff + e];
    return I.n + v.gend[I.eoff + e] + v.tscan[I.eoff + g] + ve_q(v, I, g);
}

// Index (within the cloud) of the triangle with latest edge e and third vertex c.
__device__ inline int32_t ve_tri(const VeView &v, const VeCloud &I, int32_t e, int c)
{
    const uint2 r = v.rec[I.woff + (int64_t)e * I.W + (c >> 5)];
    if (r.y & kTied) return ve_tri_first(v, I, e) + ve_tie_rank(v, I, e, c);
    return (int32_t)r.y + __popc(r.x & below(c));
}

// The number of vertices d with the sorted tuple of {f[0] < f[1] < f[2], d}
// below t, as a bound on d (the tuple grows with d).
__device__ inline int ve_bound4(const int f[3], const int t[4], int n)
{
    int lo = 0, hi = n;  // the first d whose tuple is not below t
    while (lo < hi) {
        const int d = (lo + hi) >> 1;
        const int x[4] = {min(f[0], d), max(f[0], min(f[1], d)), max(f[1], min(f[2], d)), max(f[2], d)};
        bool less = false, more = false;
        for (int k = 0; k < 4; k++) {
            less = less || (!more && x[k] < t[k]);
            more = more || (!less && x[k] > t[k]);
        }
        if (less) lo = d + 1;
        else hi = d;
    }
    return lo;
}

// A tetrahedron's place among those of edge e's tie group (its latest edge),
// t its ascending vertices.
__device__ inline int32_t ve_tie_rank4(const VeView &v, const VeCloud &I, int32_t e, const int t[4])
{
    int32_t r = 0;
    for (int32_t f = v.gst[I.eoff + e]; f < v.gend[I.eoff + e]; f++) {
        const uint32_t fg = v.ev[I.eoff + f];
        const int a = (int)(fg >> 16), b = (int)(fg & 0xFFFFu);
        int64_t dense = I.toff + v.tscan[I.eoff + f];
        for (int w = 0; w < I.W; w++) {
            uint32_t m = v.rec[I.woff + (int64_t)f * I.W + w].x;
            for (; m; m &= m - 1, dense++) {
                const int c = w * 32 + __ffs((int)m) - 1;
                const int x = min(a, c), z = max(b, c);
                const int tri[3] = {x, a + b + c - x - z, z};
                const int k = ve_bound4(tri, t, I.n);
                const uint2 *w2 = v.rec2 + dense * I.W2;
                for (int q = 0; q * 32 < k; q++) r += __popc(k - q * 32 >= 32 ? w2[q].x : w2[q].x & below(k));
            }
        }
    }
    return r;
}

// First index (within the cloud) of the tetrahedra of edge e's tie group.
__device__ inline int32_t ve_tet_first(const VeView &v, const VeCloud &I, int32_t e)
{
    const int32_t g0 = v.gst[I.eoff + e], g1 = v.gend[I.eoff + e];
    return I.n + g1 + v.tscan[I.eoff + g1] + ve_q(v, I, g0);
}

// Index (within the cloud) of the tetrahedron with latest edge e and the two
// other vertices c < d.
__device__ inline int32_t ve_tet(const VeView &v, const VeCloud &I, int32_t e, int c, int d)
{
    const int64_t o = I.woff + (int64_t)e * I.W + (c >> 5);
    const int64_t dense = I.toff + v.recd[o] + __popc(v.rec[o].x & below(c));
    const uint2 r = v.rec2[dense * I.W2 + (d >> 5)];
    if (!(r.y & kTied)) return (int32_t)r.y + __popc(r.x & below(d));
    const uint32_t ab = v.ev[I.eoff + e];
    const int a = (int)(ab >> 16), b = (int)(ab & 0xFFFFu), y0 = max(a, c), y1 = min(b, d);
    const int t[4] = {min(a, c), min(y0, y1), max(y0, y1), max(b, d)};
    return ve_tet_first(v, I, e) + ve_tie_rank4(v, I, e, t);
}

// Index (within the cloud) of the triangle x, y, z from its edges' ranks.
__device__ inline int32_t ve_tri_xyz(const VeView &v, const VeCloud &I, int x, int y, int z, int32_t xy, int32_t xz,
                                     int32_t yz)
{
    if (xy > xz && xy > yz) return ve_tri(v, I, xy, z);
    return xz > yz ? ve_tri(v, I, xz, y) : ve_tri(v, I, yz, x);
}

}  // namespace pms
