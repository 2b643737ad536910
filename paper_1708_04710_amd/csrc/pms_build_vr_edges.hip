// Vietoris-Rips filtrations (dimension <= 3) built from the order of the
// edges (pms_vr_edges.h): only the edges are sorted, and every triangle and
// tetrahedron is written straight to its place.
//
//   k_ve_edges   one workgroup per cloud: squared distances, threshold, the
//                present edges sorted by the workgroup (bitonic, keys (value, a, b)), ranks
//                and tie groups; clouds with more than kLdsEdges edges are
//                sorted by the device-wide radix sort instead (k_ve_keys, k_ve_ranks)
//   k_ve_masks   one wavefront per edge (a ballot per 64 points), or k_ve_masks_lds
//                one lane per edge: the third vertices whose two other edges come
//                earlier, its apparent triangle
//   k_ve_scan    one workgroup per cloud: prefix counts of the triangles
//   k_ve_emit    one lane per edge: its index, the first index of each mask word
//   k_ve_tris    one lane per triangle: its column; the vertices' and edges' columns
//   k_ve_tmasks, k_ve_tets, k_ve_appt   the same for tetrahedra (dimension 3)
//
// The sorted build wrote and read every simplex's 64-bit key 8 to 10 times;
// here a simplex is written once (49 bytes with FP32 values).  Lanes take
// simplices in order, whatever edge they belong to: with a wavefront per edge
// the lanes beyond an edge's triangles idle (11 on average in truncated
// clouds, 26 M simplices: 1.9 ms) and one edge of many tetrahedra holds up the
// launch (3.5 M tetrahedra: 3.0 ms).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cstring>
#include <type_traits>
#include <vector>

#include "pms_build.h"
#include "pms_common.h"
#include "pms_sort.h"
#include "pms_vr_edges.h"

namespace pms {

constexpr int kVeThreads = 1024;
constexpr int kLdsEdges = 16 * kVeThreads;  // 64-bit keys sorted in one workgroup's LDS (128 KB)
constexpr int kVeValueBitsF = 31, kVeValueBitsI = 35;

// Squared distance of points a, b (FP32: rounded step by step in coordinate
// order, bits of a non-negative float order like its value) and whether the
// edge is present; *bad: 1 not finite, 2 too large for its field.
template <bool F32>
__device__ inline unsigned long long ve_dist(const VeCloud &I, const void *pts, int a, int b, bool *present, int *bad)
{
    if (F32) {
        const float *p = (const float *)pts + I.pt_off;
        float s = 0.0f;
        for (int k = 0; k < I.D; k++) {
            const float dk = __fsub_rn(p[(int64_t)a * I.D + k], p[(int64_t)b * I.D + k]);
            s = __fadd_rn(s, __fmul_rn(dk, dk));
        }
        if (!(s >= 0.0f) || s == INFINITY) *bad = 1;
        *present = !I.has_thr || s <= I.thr_f;
        return __float_as_uint(s);
    }
    const int32_t *p = (const int32_t *)pts + I.pt_off;
    long long s = 0;
    for (int k = 0; k < I.D; k++) {
        const long long dk = (long long)p[(int64_t)a * I.D + k] - (long long)p[(int64_t)b * I.D + k];
        s += dk * dk;
    }
    if (s >= (1ll << kVeValueBitsI)) *bad = 2;
    *present = !I.has_thr || s <= I.thr_i;
    return (unsigned long long)s;
}

// The r-th edge of a cloud in order, from the sorted keys (the r-th is k[r]):
// its ends, value, ranks and tie group.
__device__ inline void ve_place(VeCloud *cl, const VeCloud &I, int lexb, const unsigned long long *k, int32_t E,
                                int32_t r, uint32_t *ev, unsigned long long *eval, int32_t *erank, int32_t *gst,
                                int32_t *gend)
{
    const unsigned long long key = k[r], val = key >> lexb;
    const uint32_t lex = (uint32_t)(key & ((1ull << lexb) - 1ull));
    const int a = (int)(lex / (uint32_t)I.n), b = (int)(lex % (uint32_t)I.n);
    int32_t g0 = r, g1 = r + 1;
    if (r > 0 && (k[r - 1] >> lexb) == val) {  // tied: the first key of this value
        int32_t lo = 0, hi = r - 1;
        while (lo < hi) {
            const int32_t mid = (lo + hi) >> 1;
            if ((k[mid] >> lexb) < val) lo = mid + 1;
            else hi = mid;
        }
        g0 = lo;
    }
    if (r + 1 < E && (k[r + 1] >> lexb) == val) {
        int32_t lo = r + 2, hi = E;
        while (lo < hi) {
            const int32_t mid = (lo + hi) >> 1;
            if ((k[mid] >> lexb) <= val) lo = mid + 1;
            else hi = mid;
        }
        g1 = lo;
    }
    if (g1 - g0 > 1 && r == g0) atomicMax(&cl->gmax, g1 - g0);
    ev[I.cap_off + r] = ((uint32_t)a << 16) | (uint32_t)b;
    // the value alone: a cloud field above it (device-wide sort) is dropped
    eval[I.cap_off + r] = val;
    gst[I.cap_off + r] = g0;
    gend[I.cap_off + r] = g1;
    erank[I.slot_base + (int64_t)a * I.n + b] = r;
    erank[I.slot_base + (int64_t)b * I.n + a] = r;
}

// x of the lane whose number differs in bit kM.
template <int kM>
__device__ inline unsigned long long lane_xor(unsigned long long x)
{
    uint32_t h[2] = {(uint32_t)x, (uint32_t)(x >> 32)};
#pragma unroll
    for (int k = 0; k < 2; k++) {
        if constexpr (kM == 1) h[k] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)h[k], 0xB1, 0xF, 0xF, true);  // quad_perm 1 0 3 2
        else if constexpr (kM == 2) h[k] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)h[k], 0x4E, 0xF, 0xF, true);  // quad_perm 2 3 0 1
        else if constexpr (kM == 8) h[k] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)h[k], 0x128, 0xF, 0xF, true);  // row_ror 8
        else h[k] = (uint32_t)__shfl_xor((int)h[k], kM, kWave);
    }
    return (unsigned long long)h[1] << 32 | h[0];
}

// E <= kE * kVeThreads keys sorted in place by the workgroup: bitonic, element
// t kE + r in thread t's register r.  Partners in the thread's own registers or
// in another lane of its wavefront need no barrier: of the 91 steps of 8 192
// keys 10 go through LDS (with all of them there k_ve_edges took 82 us for one cloud
// of 100 points, now 46; 512 clouds 368 and 274).
template <int kE>
__device__ inline void ve_sort(unsigned long long *key, int32_t E)
{
    const int t = threadIdx.x;
    unsigned long long v[kE];
#pragma unroll
    for (int r = 0; r < kE; r++) v[r] = r * kVeThreads + t < E ? key[r * kVeThreads + t] : ~0ull;
    auto own = [&](int r, int j, bool asc) {
        const unsigned long long x = v[r], y = v[r | j];
        const bool sw = (x > y) == asc;
        v[r] = sw ? y : x;
        v[r | j] = sw ? x : y;
    };
    auto other = [&](int r, unsigned long long y, bool least) {
        const bool sw = (v[r] > y) == least;
        v[r] = sw ? y : v[r];
    };
#pragma unroll
    for (int k = 2; k < kE; k <<= 1)
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1)
#pragma unroll
            for (int r = 0; r < kE; r++)
                if (!(r & j)) own(r, j, !(r & k));
    for (int k = kE < 2 ? 2 : kE; k <= kVeThreads * kE; k <<= 1) {
        const bool asc = ((t * kE) & k) == 0;
        for (int j = k >> 1; j >= kWave * kE; j >>= 1) {
            const int m = j / kE;
            __syncthreads();
#pragma unroll
            for (int r = 0; r < kE; r++) key[r * kVeThreads + t] = v[r];
            __syncthreads();
#pragma unroll
            for (int r = 0; r < kE; r++) other(r, key[r * kVeThreads + (t ^ m)], ((t & m) == 0) == asc);
        }
        auto lanes = [&](auto mask) {
            constexpr int kM = decltype(mask)::value;
            if (k < 2 * kM * kE) return;
            const bool least = ((t & kM) == 0) == asc;
#pragma unroll
            for (int r = 0; r < kE; r++) other(r, lane_xor<kM>(v[r]), least);
        };
        lanes(std::integral_constant<int, 32>());
        lanes(std::integral_constant<int, 16>());
        lanes(std::integral_constant<int, 8>());
        lanes(std::integral_constant<int, 4>());
        lanes(std::integral_constant<int, 2>());
        lanes(std::integral_constant<int, 1>());
#pragma unroll
        for (int j = kE >> 1; j > 0; j >>= 1)
#pragma unroll
            for (int r = 0; r < kE; r++)
                if (!(r & j)) own(r, j, asc);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kE; r++) key[t * kE + r] = v[r];
    __syncthreads();
}

template <bool F32>
__global__ void __launch_bounds__(kVeThreads) k_ve_edges(VeCloud *cl, const void *pts, int lexb, int32_t cap,
                                                         uint32_t *ev, unsigned long long *eval, int32_t *erank,
                                                         int32_t *gst, int32_t *gend, int32_t *err)
{
    extern __shared__ unsigned long long s_key[];
    __shared__ int32_t s_n;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const VeCloud I = cl[blockIdx.x];
    if (tid == 0) s_n = 0;
    const int32_t nn = I.n * I.n;
    for (int32_t i = tid; i < nn; i += kVeThreads) erank[I.slot_base + i] = kNoEdge;
    __syncthreads();
    for (int32_t i0 = 0; i0 < nn; i0 += kVeThreads) {
        const int32_t i = i0 + tid;
        const int a = i / I.n, b = i - a * I.n;
        bool in = false;
        unsigned long long v = 0;
        if (i < nn && a < b) {
            int bad = 0;
            v = ve_dist<F32>(I, pts, a, b, &in, &bad);
            if (bad) atomicExch(err, bad);
        }
        const uint64_t m = __ballot(in);
        if (m) {
            int32_t at = 0;
            if (lane == __ffsll((long long)m) - 1) at = atomicAdd(&s_n, __popcll(m));
            at = __shfl(at, __ffsll((long long)m) - 1, kWave) + __popcll(m & ((1ull << lane) - 1ull));
            if (in && at < cap) s_key[at] = (v << lexb) | (unsigned long long)i;
        }
    }
    __syncthreads();
    const int32_t E = s_n;
    if (tid == 0) {
        cl[blockIdx.x].E = E;
        cl[blockIdx.x].gmax = 1;
    }
    if (E > cap) return;  // the host takes the device-wide sort
    if (E <= kVeThreads) ve_sort<1>(s_key, E);
    else if (E <= 2 * kVeThreads) ve_sort<2>(s_key, E);
    else if (E <= 4 * kVeThreads) ve_sort<4>(s_key, E);
    else if (E <= 8 * kVeThreads) ve_sort<8>(s_key, E);
    else ve_sort<16>(s_key, E);
    for (int32_t r = tid; r < E; r += kVeThreads)
        ve_place(&cl[blockIdx.x], I, lexb, s_key, E, r, ev, eval, erank, gst, gend);
}

// Device-wide sort: keys (cloud, value, a, b) of every pair, all ones when
// it is no edge (sorted last), and the clouds' edge counts.
template <bool F32>
__global__ void __launch_bounds__(kBlock) k_ve_keys(VeCloud *cl, const void *pts, int lexb, int cshift,
                                                    unsigned long long *keys, int32_t *erank, int32_t *err)
{
    const VeCloud I = cl[blockIdx.y];
    int32_t cnt = 0;
    for (int32_t i = blockIdx.x * kBlock + threadIdx.x; i < I.n * I.n; i += gridDim.x * kBlock) {
        erank[I.slot_base + i] = kNoEdge;
        const int a = i / I.n, b = i - a * I.n;
        if (a >= b) continue;
        int bad = 0;
        bool in;
        const unsigned long long v = ve_dist<F32>(I, pts, a, b, &in, &bad);
        if (bad) atomicExch(err, bad);
        keys[I.cap_off + (int64_t)a * I.n - (int64_t)a * (a + 1) / 2 + (b - a - 1)] =
            in ? ((unsigned long long)blockIdx.y << cshift) | (v << lexb) | (unsigned long long)i : ~0ull;
        cnt += in;
    }
    const int64_t t = block_sum64(cnt);
    if (threadIdx.x == 0 && t) atomicAdd(&cl[blockIdx.y].E, (int32_t)t);
}

// (eoff: the cloud's first key in the sorted array)
__global__ void __launch_bounds__(kBlock) k_ve_ranks(VeCloud *cl, int lexb, int cshift, unsigned long long *keys,
                                                     uint32_t *ev, unsigned long long *eval, int32_t *erank,
                                                     int32_t *gst, int32_t *gend, const int64_t *first)
{
    const VeCloud I = cl[blockIdx.y];
    const unsigned long long *k = keys + first[blockIdx.y];
    const unsigned long long vm = (1ull << (cshift - lexb)) - 1ull;
    for (int32_t r = blockIdx.x * kBlock + threadIdx.x; r < I.E; r += gridDim.x * kBlock) {
        ve_place(&cl[blockIdx.y], I, lexb, k, I.E, r, ev, eval, erank, gst, gend);
        eval[I.cap_off + r] &= vm;  // without the cloud
    }
}

// Third vertices, apparent triangle, counts; the edge arrays from their
// capacity-sized scratch to the filtration's own.
__global__ void __launch_bounds__(kBlock) k_ve_masks(const VeCloud *cl, int maxdim, const uint32_t *ev_s,
                                                     const int32_t *gst_s, const int32_t *gend_s, const int32_t *erank,
                                                     uint32_t *ev, int32_t *gst, int32_t *gend, uint2 *rec,
                                                     uint64_t *mask, int32_t *tcnt, int32_t *apc)
{
    const VeCloud I = cl[blockIdx.y];
    const int lane = threadIdx.x & (kWave - 1);
    const int nw = maxdim >= 2 ? (I.n + 63) / 64 : 0;
    for (int32_t e = blockIdx.x * kWavesPerBlock + threadIdx.x / kWave; e < I.E; e += gridDim.x * kWavesPerBlock) {
        const uint32_t ab = ev_s[I.cap_off + e];
        const int32_t ge = gend_s[I.cap_off + e];
        const int32_t *ra = erank + I.slot_base + (int64_t)(ab >> 16) * I.n;
        const int32_t *rb = erank + I.slot_base + (int64_t)(ab & 0xFFFFu) * I.n;
        int32_t t = 0, first = -1;
        bool first_in = false;
        for (int w = 0; w < nw; w++) {
            const int c = w * 64 + lane;
            const int32_t x = c < I.n ? ra[c] : kNoEdge, y = c < I.n ? rb[c] : kNoEdge;
            const uint64_t m = __ballot(x < e && y < e);
            const uint64_t mv = __ballot(x < ge && y < ge);  // cofaces of the edge's own value
            if (first < 0 && mv) {
                first = w * 64 + __ffsll((long long)mv) - 1;
                first_in = (m >> (first & 63)) & 1;
            }
            if (lane == 0) {
                uint2 *r = rec + I.woff + (int64_t)e * I.W + 2 * w;
                r[0].x = (uint32_t)m;
                if (2 * w + 1 < I.W) r[1].x = (uint32_t)(m >> 32);
                mask[I.moff + (int64_t)e * I.M + w] = m;
            }
            t += __popcll(m);
        }
        if (lane == 0) {
            const int64_t o = I.eoff + e;
            ev[o] = ab;
            gst[o] = gst_s[I.cap_off + e];
            gend[o] = ge;
            tcnt[o] = t;
            apc[o] = first_in ? first : -1;
        }
    }
}

// The same with the cloud's ranks in LDS as pairs of 16-bit words (n <=
// kLdsPoints: at most 32 640 edges), one lane per edge going through its ends'
// rows: 3.5 instructions per 64 vertices and edge against 25 with a ballot, and
// rows of an odd number of words, so that different rows start in different
// banks.  Two rows per edge from L2, the kernel above takes 745 us for 512 clouds
// of 32 to 256 points (1.9 M edges); with ballots over LDS 505; this one 218 (64
// clouds of 128 points: 129, now 27).  Few edges leave most lanes idle and are
// bound by one lane's chain (100 points: 13 us, a wavefront an edge 4).
constexpr int kLdsPoints = 256, kVeMaskThreads = 1024;
constexpr int64_t kVeManyEdges = 1 << 16;
__host__ __device__ inline int ve_rank_row(int n) { return (n + 31) / 32 * 16 + 1; }

__global__ void __launch_bounds__(kVeMaskThreads) k_ve_masks_lds(const VeCloud *cl, int maxdim, const uint32_t *ev_s,
                                                                 const int32_t *gst_s, const int32_t *gend_s,
                                                                 const int32_t *erank, uint32_t *ev, int32_t *gst,
                                                                 int32_t *gend, uint2 *rec, uint64_t *mask,
                                                                 int32_t *tcnt, int32_t *apc)
{
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    extern __shared__ u16x2 s_rank[];
    const VeCloud I = cl[blockIdx.y];
    const int W = maxdim >= 2 ? I.W : 0, row = ve_rank_row(I.n);
    if ((int32_t)blockIdx.x * kVeMaskThreads >= I.E) return;
    if (W > 0) {
        // (columns past n: no edge)
        const int32_t words = I.n * row;
        for (int32_t i0 = threadIdx.x; i0 < words; i0 += 4 * kVeMaskThreads) {
            int32_t r[4][2];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int32_t i = min(i0 + u * kVeMaskThreads, words - 1), a = i / row, c = 2 * (i - a * row);
                const int32_t *ra = erank + I.slot_base + (int64_t)a * I.n;
                r[u][0] = c < I.n ? ra[c] : kNoEdge;
                r[u][1] = c + 1 < I.n ? ra[c + 1] : kNoEdge;
            }
#pragma unroll
            for (int u = 0; u < 4; u++)
                if (i0 + u * kVeMaskThreads < words)
                    s_rank[i0 + u * kVeMaskThreads] =
                        u16x2{(uint16_t)min(r[u][0], 0xFFFF), (uint16_t)min(r[u][1], 0xFFFF)};
        }
    }
    __syncthreads();
    for (int32_t e = (int32_t)blockIdx.x * kVeMaskThreads + (int32_t)threadIdx.x; e < I.E;
         e += (int32_t)gridDim.x * kVeMaskThreads) {
        const uint32_t ab = ev_s[I.cap_off + e];
        const int32_t ge = gend_s[I.cap_off + e];
        const u16x2 *ra = s_rank + (ab >> 16) * row, *rb = s_rank + (ab & 0xFFFFu) * row;
        uint2 *r = rec + I.woff + (int64_t)e * I.W;
        int32_t t = 0, first = -1;
        bool first_in = false;
        uint32_t even = 0;
        for (int w = 0; w < W; w++, ra += 16, rb += 16) {
            uint32_t m = 0;
#pragma unroll
            for (int k = 15; k >= 0; k--) {
                const u16x2 z = __builtin_elementwise_max(ra[k], rb[k]);
                m = m << 1 | (uint32_t)(z.y < e);
                m = m << 1 | (uint32_t)(z.x < e);
            }
            uint32_t mv = m;  // cofaces of the edge's own value
            if (ge - e > 1) {
                mv = 0;
                for (int k = 15; k >= 0; k--) {
                    const u16x2 z = __builtin_elementwise_max(ra[k], rb[k]);
                    mv = mv << 2 | (uint32_t)(z.y < ge) << 1 | (uint32_t)(z.x < ge);
                }
            }
            if (first < 0 && mv) {
                const int f = __ffs((int)mv) - 1;
                first = w * 32 + f;
                first_in = (m >> f) & 1u;
            }
            t += __popc(m);
            r[w].x = m;
            if (w & 1 || w == W - 1)
                mask[I.moff + (int64_t)e * I.M + (w >> 1)] = w & 1 ? (uint64_t)m << 32 | even : (uint64_t)m;
            even = m;
        }
        const int64_t o = I.eoff + e;
        ev[o] = ab;
        gst[o] = gst_s[I.cap_off + e];
        gend[o] = ge;
        tcnt[o] = t;
        apc[o] = first_in ? first : -1;
    }
}

__global__ void __launch_bounds__(1024) k_ve_scan(VeCloud *cl, int32_t *tcnt)
{
    const VeCloud I = cl[blockIdx.x];
    int32_t *t = tcnt + I.eoff;
    const int32_t T = block_seg_scan(t, (int64_t)I.E, 0, [](int32_t x, int32_t y) { return x + y; });
    if (threadIdx.x == 0) {
        t[I.E] = T;
        cl[blockIdx.x].T = T;
    }
}

struct VeOut {
    int64_t m, nnz;
    int64_t *col_ptr;
    int32_t *rows;
    int8_t *dim;
    void *value;
    int32_t *crit;
    int32_t *verts;
};

// Everything of column p but its rows.
template <bool F32>
__device__ inline void ve_put(const VeOut &o, int64_t p, int64_t cp, int nf, int dm, unsigned long long val, int2 crit,
                              int4 verts)
{
    o.col_ptr[p] = cp;
    if (p == o.m - 1) o.col_ptr[o.m] = cp + nf;
    o.dim[p] = (int8_t)dm;
    if (F32) ((float *)o.value)[p] = __uint_as_float((uint32_t)val);
    else ((int64_t *)o.value)[p] = (int64_t)val;
    reinterpret_cast<int2 *>(o.crit)[p] = crit;
    reinterpret_cast<int4 *>(o.verts)[p] = verts;
}

// The largest i in [lo, hi) with a[i] <= x (a[lo] <= x), by the whole wavefront:
// 64 probes a step.
template <typename T>
__device__ inline int64_t wave_last_le(const T *a, int64_t lo, int64_t hi, int64_t x)
{
    const int lane = threadIdx.x & (kWave - 1);
    while (hi - lo > 1) {
        const int64_t step = (hi - lo + kWave - 1) / kWave;
        const int64_t at = lo + lane * step;
        const uint64_t m = __ballot(at < hi && (int64_t)a[at < hi ? at : lo] <= x);
        const int64_t k = __popcll(m) - 1;  // (a ascends: a prefix of the lanes)
        hi = min(hi, lo + (k + 1) * step);
        lo += k * step;
    }
    return lo;
}

// The same by one lane.
template <typename T>
__device__ inline int64_t lane_last_le(const T *a, int64_t lo, int64_t hi, int64_t x)
{
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)a[mid] <= x) lo = mid;
        else hi = mid;
    }
    return lo;
}

// The k-th (from 0) vertex of a mask of W words.
__device__ inline int ve_select(const uint2 *w, int W, int k)
{
    int q = 0;
    uint32_t m = W > 0 ? w[0].x : 0u;
    while (q + 1 < W && __popc(m) <= k) {
        k -= __popc(m);
        m = w[++q].x;
    }
    while (k-- > 0) m &= m - 1;
    return q * 32 + __ffs((int)m) - 1;
}

// Edges of a workgroup of k_ve_emit and k_ve_tris: their mask words (32 each
// for 1 023 points, the most) pass through LDS.
// Few edges in all: 8 a workgroup (an edge of 100 points has up to 98 triangles;
// 64 of the last ones hold a launch of 4 950 edges for 27 us, 8 for 7.6).
constexpr int kVeTile = 64, kVeFewTile = 8, kTileWords = 32 * kVeTile;
inline int ve_tile(int64_t E) { return E >= kVeManyEdges ? kVeTile : kVeFewTile; }

// One lane per edge: its index, rec's indices.  The mask words are read and
// written by the whole workgroup in their order.
__global__ void __launch_bounds__(kBlock) k_ve_emit(VeView v, int maxdim, int per, int32_t *eidx, uint2 *rec, int32_t *app,
                                                    uint32_t *recd)
{
    __shared__ uint32_t s_w[kTileWords], s_run[kTileWords];
    const VeCloud I = v.cl[blockIdx.y];
    const int W = maxdim >= 2 ? I.W : 0;
    for (int32_t e0 = blockIdx.x * per; e0 < I.E; e0 += gridDim.x * per) {
        const int32_t ne = min(per, I.E - e0);
        uint2 *r0 = rec + I.woff + (int64_t)e0 * I.W;
        for (int32_t k = threadIdx.x; k < ne * W; k += kBlock) s_w[k] = r0[k].x;
        __syncthreads();
        if ((int32_t)threadIdx.x < ne) {
            const int32_t e = e0 + (int32_t)threadIdx.x;
            const int64_t oe = I.eoff + e;
            const uint32_t ab = v.ev[oe];
            const int a = (int)(ab >> 16), b = (int)(ab & 0xFFFFu);
            const int32_t g0 = v.gst[oe], g1 = v.gend[oe];
            const int32_t ts = v.tscan[I.eoff + g0], qs = ve_q(v, I, g0), own = v.tscan[oe];
            const bool tied = g1 - g0 > 1;
            const int32_t pe = I.n + e + ts + qs;
            const int32_t tb = I.n + g1 + ts + qs;
            eidx[I.slot_base + (int64_t)a * I.n + b] = pe;
            eidx[I.slot_base + (int64_t)b * I.n + a] = pe;
            const int apc = v.apc[oe];
            uint32_t *rd = recd ? recd + I.woff + (int64_t)e * I.W : nullptr;
            int32_t run = 0, at = -1;
            for (int w = 0; w < W; w++) {
                const uint32_t m = s_w[threadIdx.x * W + w];
                s_run[threadIdx.x * W + w] = tied ? kTied : (uint32_t)(tb + run);
                if (rd) rd[w] = (uint32_t)(own + run);
                if (apc >= 0 && (apc >> 5) == w) at = tb + run + __popc(m & below(apc));
                run += __popc(m);
            }
            app[oe] = apc >= 0 && tied ? tb + ve_tie_rank(v, I, e, apc) : at;
        }
        __syncthreads();
        for (int32_t k = threadIdx.x; k < ne * W; k += kBlock) r0[k].y = s_run[k];
        __syncthreads();
    }
}

// The columns of vertices, edges and triangles: one lane per triangle, in the
// order of (edge, third vertex), a workgroup the triangles of kVeTile edges, and
// the edges' own columns, which lie between them (written by a kernel of their
// own, 1.6 M edges' scattered pieces of lines took 0.3 ms).  Which edge and
// which vertex from the edges' counts and mask words in LDS.  Bound by the writes; the other edges' indices are
// gathered from one cloud's table and hit L2.  (The same look-ups from memory,
// a chain of up to twenty loads per triangle: 26 M triangles of 512 clouds 1.19
// ms, 22 M of 64 clouds 0.58; now 0.68 and 0.37, 2.5 TB/s of writes.)
template <bool F32>
__global__ void __launch_bounds__(kBlock) k_ve_tris(VeView v, VeOut o, int maxdim, int per, const unsigned long long *eval,
                                                    int32_t *appt)
{
    __shared__ uint32_t s_w[kTileWords];
    __shared__ int32_t s_ts[kVeTile + 1], s_ab[kVeTile], s_g0[kVeTile], s_g1[kVeTile], s_tg[kVeTile], s_qs[kVeTile];
    __shared__ unsigned long long s_val[kVeTile];
    const VeCloud I = v.cl[blockIdx.y];
    const int32_t pb = (int32_t)I.pbase, cb = (int32_t)I.col_base;
    const int32_t *ts = v.tscan + I.eoff;
    const int32_t *ix = v.eidx + I.slot_base;
    for (int32_t x = blockIdx.x * kBlock + threadIdx.x; x < I.n; x += gridDim.x * kBlock)
        ve_put<F32>(o, I.col_base + x, I.nnz_base, 0, 0, 0, make_int2(-1, -1), make_int4(pb + x, -1, -1, -1));
    const int W = maxdim >= 2 ? I.W : 0;
    for (int32_t e0 = blockIdx.x * per; e0 < I.E; e0 += gridDim.x * per) {
        const int32_t ne = min(per, I.E - e0);
        const uint2 *rec = v.rec + I.woff + (int64_t)e0 * W;
        if ((int32_t)threadIdx.x <= ne) s_ts[threadIdx.x] = ts[e0 + threadIdx.x];
        if ((int32_t)threadIdx.x < ne) {
            const int32_t e = e0 + (int32_t)threadIdx.x;
            const int64_t oe = I.eoff + e;
            const int32_t g0 = v.gst[oe], tg = ts[g0], qs = ve_q(v, I, g0);
            const uint32_t ab = v.ev[oe];
            const unsigned long long val = eval[I.cap_off + e];
            s_ab[threadIdx.x] = (int32_t)ab;
            s_g0[threadIdx.x] = g0;
            s_g1[threadIdx.x] = v.gend[oe];
            s_tg[threadIdx.x] = tg;
            s_qs[threadIdx.x] = qs;
            s_val[threadIdx.x] = val;
            const int a = (int)(ab >> 16), b = (int)(ab & 0xFFFFu);
            const int64_t cp = I.nnz_base + 2LL * e + 3LL * tg + 4LL * qs;
            ve_put<F32>(o, (int64_t)cb + I.n + e + tg + qs, cp, 2, 1, val, make_int2(pb + a, pb + b),
                        make_int4(pb + a, pb + b, -1, -1));
            o.rows[cp] = cb + a;
            o.rows[cp + 1] = cb + b;
        }
        for (int32_t k = threadIdx.x; k < ne * W; k += kBlock) s_w[k] = rec[k].x;
        __syncthreads();
        const int32_t t1 = s_ts[ne];
        for (int32_t t = s_ts[0] + (int32_t)threadIdx.x; t < t1; t += kBlock) {
            int i = 0, end = ne;  // the last edge with s_ts[i] <= t
            while (end - i > 1) {
                const int mid = (i + end) >> 1;
                if (s_ts[mid] <= t) i = mid;
                else end = mid;
            }
            const int32_t e = e0 + i;
            int k = t - s_ts[i], q = 0;
            uint32_t m = s_w[i * W];
            while (__popc(m) <= k) {  // (the edge has more than k)
                k -= __popc(m);
                q++;
                m = s_w[i * W + q];
            }
            int c = q * 32;  // the k-th bit of m
#pragma unroll
            for (int h = 16; h > 0; h >>= 1) {
                const int below_h = __popc(m & ((1u << h) - 1u));
                if (k >= below_h) {
                    k -= below_h;
                    c += h;
                    m >>= h;
                }
            }
            const uint32_t ab = (uint32_t)s_ab[i];
            const int a = (int)(ab >> 16), b = (int)(ab & 0xFFFFu);
            const int32_t ra = ix[(int64_t)a * I.n + c], rb = ix[(int64_t)b * I.n + c];
            const int32_t g1 = s_g1[i], tg = s_tg[i], qs = s_qs[i];
            const int32_t r = g1 - s_g0[i] > 1 ? ve_tie_rank(v, I, e, c) : t - tg;
            const int64_t p = (int64_t)cb + I.n + g1 + tg + qs + r;
            const int64_t cp = I.nnz_base + 2LL * g1 + 3LL * (tg + r) + 4LL * qs;
            const int x = min(a, c), z = max(b, c);
            ve_put<F32>(o, p, cp, 3, 2, s_val[i], make_int2(pb + a, pb + b),
                        make_int4(pb + x, pb + a + b + c - x - z, pb + z, -1));
            o.rows[cp] = cb + min(ra, rb);
            o.rows[cp + 1] = cb + max(ra, rb);
            o.rows[cp + 2] = cb + I.n + e + tg + qs;
            if (appt) appt[p] = -1;
        }
        __syncthreads();
    }
}

// The fourth vertices d > c of every triangle (e, c) whose tetrahedron has
// latest edge e: the masks of rec2 and their sizes (dimension 3).  One
// wavefront per kTriRun consecutive triangles.
constexpr int kTriRun = 8;
__global__ void __launch_bounds__(kBlock) k_ve_tmasks(VeView v, uint2 *rec2, uint2 *tri, int64_t *qcnt)
{
    const VeCloud I = v.cl[blockIdx.y];
    const int lane = threadIdx.x & (kWave - 1);
    const int32_t *ts = v.tscan + I.eoff;
    const int nw = (I.n + 63) / 64;
    const int32_t runs = (int32_t)((I.T + kTriRun - 1) / kTriRun);
    for (int32_t q = blockIdx.x * kWavesPerBlock + threadIdx.x / kWave; q < runs; q += gridDim.x * kWavesPerBlock) {
        const int32_t t0 = q * kTriRun, t1 = (int32_t)min((int64_t)t0 + kTriRun, I.T);
        int32_t e = (int32_t)wave_last_le(ts, 0, I.E, t0);
        for (int32_t t = t0; t < t1; t++) {
            while (ts[e + 1] <= t) e++;
            const uint2 *re = v.rec + I.woff + (int64_t)e * I.W;
            const int c = ve_select(re, I.W, t - ts[e]);
            const int32_t *rc = v.erank + I.slot_base + (int64_t)c * I.n;
            uint2 *r2 = rec2 + (I.toff + t) * I.W2;
            int32_t n = 0;
            for (int w = 0; w < nw; w++) {
                const int d = w * 64 + lane;
                const bool in = d > c && d < I.n && ((re[d < I.n ? d >> 5 : 0].x >> (d & 31)) & 1u) && rc[d] < e;
                const uint64_t mm = __ballot(in);
                n += __popcll(mm);
                if (lane == 0) {
                    r2[2 * w].x = (uint32_t)mm;
                    if (2 * w + 1 < I.W) r2[2 * w + 1].x = (uint32_t)(mm >> 32);
                }
            }
            if (lane == 0) {
                qcnt[I.toff + t] = n;
                tri[I.toff + t] = make_uint2((uint32_t)e, (uint32_t)c);
            }
        }
    }
}

// After the scan of the triangles' counts: the clouds' tetrahedra.
__global__ void k_ve_qbounds(VeCloud *cl, int32_t B, int64_t T, int64_t Q, int64_t *q2)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) q2[T] = Q;
    for (int b = blockIdx.x * blockDim.x + threadIdx.x; b < B; b += gridDim.x * blockDim.x) {
        const int64_t t0 = cl[b].toff, t1 = t0 + cl[b].T;
        const int64_t q0 = t0 < T ? q2[t0] : Q, q1 = t1 < T ? q2[t1] : Q;
        cl[b].qfirst = q0;
        cl[b].Q = q1 - q0;
    }
}

// One lane per triangle: rec2's indices and the first vertex of a coface of
// the triangle's value, which may make it apparent (k_ve_appt).
__global__ void __launch_bounds__(kBlock) k_ve_tindex(VeView v, const uint2 *tri, uint2 *rec2, int32_t *appt)
{
    const VeCloud I = v.cl[blockIdx.y];
    for (int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x; t < I.T; t += (int64_t)gridDim.x * kBlock) {
        const int32_t e = (int32_t)tri[I.toff + t].x;
        const int c = (int)tri[I.toff + t].y;
        const int64_t oe = I.eoff + e;
        const int32_t g1 = v.gend[oe];
        const bool tied = g1 - v.gst[oe] > 1;
        uint32_t at = (uint32_t)(I.n + g1 + v.tscan[I.eoff + g1] + (int32_t)(v.q2[I.toff + t] - I.qfirst));
        uint2 *r2 = rec2 + (I.toff + t) * I.W2;
        for (int w = 0; w < I.W; w++) {
            r2[w].y = tied ? kTied : at;
            at += (uint32_t)__popc(r2[w].x);
        }
        // the cofaces of its value come by their vertices, so by the fourth one
        const uint32_t ab = v.ev[oe];
        const int32_t *R = v.erank + I.slot_base;
        const int32_t *ra = R + (int64_t)(ab >> 16) * I.n, *rb = R + (int64_t)(ab & 0xFFFFu) * I.n,
                      *rc = R + (int64_t)c * I.n;
        int first = -1;
        if (tied) {
            for (int d = 0; d < I.n && first < 0; d++)
                if (ra[d] < g1 && rb[d] < g1 && rc[d] < g1) first = d;
        } else {  // only one before c can make it apparent
            const uint2 *re = v.rec + I.woff + (int64_t)e * I.W;
            for (int w = 0; w <= (c >> 5) && first < 0; w++)
                for (uint32_t m = w == (c >> 5) ? re[w].x & below(c) : re[w].x; m && first < 0; m &= m - 1) {
                    const int d = w * 32 + __ffs((int)m) - 1;
                    if (rc[d] < e) first = d;
                }
        }
        if (first >= 0) appt[I.col_base + ve_tri(v, I, e, c)] = -2 - first;
    }
}

// One lane per tetrahedron, in the order of (triangle, fourth vertex).
template <bool F32>
__global__ void __launch_bounds__(kBlock) k_ve_tets(VeView v, VeOut o, const unsigned long long *eval, const uint2 *tri)
{
    const VeCloud I = v.cl[blockIdx.y];
    const int32_t pb = (int32_t)I.pbase, cb = (int32_t)I.col_base;
    const int64_t *q2 = v.q2 + I.toff;
    const int64_t tiles = (I.Q + kBlock - 1) / kBlock;
    const int64_t t0 = tiles * blockIdx.x / gridDim.x, t1 = tiles * (blockIdx.x + 1) / gridDim.x;
    int64_t lo = 0;
    for (int64_t tile = t0; tile < t1; tile++) {
        lo = wave_last_le(q2, lo, I.T, I.qfirst + tile * kBlock);
        const int64_t hi = wave_last_le(q2, lo, I.T, I.qfirst + tile * kBlock + kBlock - 1) + 1;
        const int64_t q = tile * kBlock + threadIdx.x;
        if (q >= I.Q) continue;
        const int64_t t = lane_last_le(q2, lo, hi, I.qfirst + q);
        const uint2 ec = tri[I.toff + t];
        const int32_t e = (int32_t)ec.x;
        const int c = (int)ec.y;
        const int d = ve_select(v.rec2 + (I.toff + t) * I.W2, I.W, (int)(I.qfirst + q - q2[t]));
        const int64_t oe = I.eoff + e;
        const uint32_t ab = v.ev[oe];
        const int a = (int)(ab >> 16), b = (int)(ab & 0xFFFFu);
        const int32_t g0 = v.gst[oe], g1 = v.gend[oe];
        const int32_t *R = v.erank + I.slot_base;
        const int32_t rac = R[(int64_t)a * I.n + c], rad = R[(int64_t)a * I.n + d], rbc = R[(int64_t)b * I.n + c],
                      rbd = R[(int64_t)b * I.n + d], rcd = R[(int64_t)c * I.n + d];
        // the middle two of {a, b, c, d}, a < b and c < d
        const int y0 = max(a, c), y1 = min(b, d);
        const int x[4] = {min(a, c), min(y0, y1), max(y0, y1), max(b, d)};
        const int32_t qs = ve_q(v, I, g0), ts1 = v.tscan[I.eoff + g1];
        const int32_t r = g1 - g0 > 1 ? ve_tie_rank4(v, I, e, x) : (int32_t)q - qs;
        const int64_t p = (int64_t)cb + I.n + g1 + ts1 + qs + r;
        const int64_t cp = I.nnz_base + 2LL * g1 + 3LL * ts1 + 4LL * (qs + r);
        int32_t f[4] = {ve_tri_xyz(v, I, a, c, d, rac, rad, rcd), ve_tri_xyz(v, I, b, c, d, rbc, rbd, rcd),
                        ve_tri(v, I, e, c), ve_tri(v, I, e, d)};
#pragma unroll
        for (int i = 1; i < 4; i++)
#pragma unroll
            for (int k = 3; k >= i; k--)
                if (f[k - 1] > f[k]) { const int32_t z = f[k]; f[k] = f[k - 1]; f[k - 1] = z; }
        ve_put<F32>(o, p, cp, 4, 3, eval[I.cap_off + e], make_int2(pb + a, pb + b),
                    make_int4(pb + x[0], pb + x[1], pb + x[2], pb + x[3]));
        for (int k = 0; k < 4; k++) o.rows[cp + k] = cb + f[k];
    }
}

// The triangles' first cofaces (a vertex, left by k_ve_tets) into the index of
// the apparent tetrahedron, -1 when the triangle is not its last facet.
__global__ void __launch_bounds__(kBlock) k_ve_appt(VeView v, const int32_t *verts, const int8_t *dim, int32_t *appt)
{
    const VeCloud I = v.cl[blockIdx.y];
    const int32_t mb = (int32_t)(I.n + I.E + I.T + I.Q);
    for (int32_t p = blockIdx.x * kBlock + threadIdx.x; p < mb; p += gridDim.x * kBlock) {
        const int64_t g = I.col_base + p;
        if (dim[g] != 2 || appt[g] == -1) continue;
        const int d = -2 - appt[g];
        const int4 q = reinterpret_cast<const int4 *>(verts)[g];
        const int x[4] = {q.x - (int)I.pbase, q.y - (int)I.pbase, q.z - (int)I.pbase, d};
        const int32_t *R = v.erank + I.slot_base;
        int32_t r[6], best = -1;  // pairs 01 02 03 12 13 23
        int bu = 0, bw = 1, k = 0;
        for (int u = 0; u < 4; u++)
            for (int w = u + 1; w < 4; w++, k++) {
                r[k] = R[(int64_t)x[u] * I.n + x[w]];
                if (r[k] > best) { best = r[k]; bu = u; bw = w; }
            }
        int rest[2], nr = 0;
        for (int u = 0; u < 4; u++)
            if (u != bu && u != bw) rest[nr++] = x[u];
        const int32_t last = max(ve_tri_xyz(v, I, x[0], x[1], x[3], r[0], r[2], r[4]),
                                 max(ve_tri_xyz(v, I, x[0], x[2], x[3], r[1], r[2], r[5]),
                                     ve_tri_xyz(v, I, x[1], x[2], x[3], r[3], r[4], r[5])));
        appt[g] = last < p ? ve_tet(v, I, best, min(rest[0], rest[1]), max(rest[0], rest[1])) : -1;
    }
}

// ---------------------------------------------------------------- host
// Builds *out from the edges' order.  *done = 0 (status PMS_OK): not
// applicable, the sorted build takes the batch: key fields too wide for one
// word, or a tie group beyond kVeMaxTies / kVeMaxTies3.
pms_status build_vr_edges(Ctx *c, const void *pts, bool f32, const int32_t *n, const int32_t *D, const int64_t *pt_off,
                          const void *thr, int32_t B, int32_t maxdim, Filtration **out, int64_t *inst_col_off,
                          int *done)
{
    *done = 0;
    struct {
        VeCloud *first;
        int32_t n;
        VeCloud *begin() const { return first; }
        VeCloud *end() const { return first + n; }
        VeCloud &operator[](size_t b) const { return first[b]; }
        VeCloud *data() const { return first; }
    } h{(VeCloud *)pinned_stage(c, (size_t)B * sizeof(VeCloud) + 64), B};
    if (!h.first) return set_err(c, PMS_ERR_OOM, "pinned host memory");
    int32_t &herr = *(int32_t *)(h.first + B);
    int64_t slots = 0, pairs = 0, pbase = 0, nmax = 1, maxpairs = 0;
    double work = 0, maxwork = 0;  // coordinates of all pairs' distances; of one cloud's
    for (int b = 0; b < B; b++) {
        VeCloud &I = h[(size_t)b];
        memset(&I, 0, sizeof(I));
        I.n = n[b];
        I.D = D[b];
        I.W = maxdim >= 2 ? (n[b] + 31) / 32 : 0;
        I.M = maxdim >= 2 ? (n[b] + 63) / 64 : 0;
        I.pt_off = pt_off[b];
        I.pbase = pbase;
        I.slot_base = slots;
        I.cap_off = pairs;
        if (f32) {
            const float t = thr ? ((const float *)thr)[b] : -1.0f;
            I.has_thr = t >= 0.0f;
            I.thr_f = t;
        } else {
            const int64_t t = thr ? ((const int64_t *)thr)[b] : -1;
            I.has_thr = t >= 0;
            I.thr_i = t;
        }
        const int64_t np = (int64_t)n[b] * (n[b] - 1) / 2;
        pbase += n[b];
        slots += (int64_t)n[b] * n[b];
        pairs += n[b] > 0 ? np : 0;
        maxpairs = std::max(maxpairs, np);
        work += (double)np * D[b];
        maxwork = std::max(maxwork, (double)np * D[b]);
        nmax = std::max<int64_t>(nmax, n[b]);
    }
    int lexb = 1, cbits = 0;
    while ((1ll << lexb) < nmax * nmax) lexb++;
    while ((1ll << cbits) < B) cbits++;
    const int cshift = lexb + (f32 ? kVeValueBitsF : kVeValueBitsI);
    if (cshift + cbits > 63 || B > 65535) return PMS_OK;
    hipStream_t s = c->stream;
    const int64_t S = std::max<int64_t>(slots, 1), P = std::max<int64_t>(pairs, 1);
    VeCloud *dcl = (VeCloud *)grow_scratch(c, B_BUILD6, (size_t)B * sizeof(VeCloud));
    uint32_t *ev_s = (uint32_t *)grow_scratch(c, B_BUILD0, P * 4);
    unsigned long long *eval = (unsigned long long *)grow_scratch(c, B_BUILD1, P * 8);
    int32_t *gst_s = (int32_t *)grow_scratch(c, B_BUILD2, P * 4);
    int32_t *gend_s = (int32_t *)grow_scratch(c, B_BUILD3, P * 4);
    int32_t *err = (int32_t *)grow_scratch(c, B_BUILD4, 64);
    Filtration *f = *out;
    pms_status st = filtration_vr_reserve(c, &f, VR_ERANK, S * 4);
    *out = f;
    if (st == PMS_OK) st = filtration_vr_reserve(c, &f, VR_EIDX, S * 4);
    if (st != PMS_OK) return st;
    if (!dcl || !ev_s || !eval || !gst_s || !gend_s || !err) return set_err(c, PMS_ERR_OOM, "builder scratch");
    int32_t *erank = (int32_t *)f->vr[VR_ERANK].p, *eidx = (int32_t *)f->vr[VR_EIDX].p;
    PMS_HIP(hipMemcpyAsync(dcl, h.data(), (size_t)B * sizeof(VeCloud), hipMemcpyHostToDevice, s));
    PMS_HIP(hipMemsetAsync(err, 0, 4, s));
    auto read_clouds = [&]() -> pms_status {
        PMS_HIP(hipMemcpyAsync(h.data(), dcl, (size_t)B * sizeof(VeCloud), hipMemcpyDeviceToHost, s));
        PMS_HIP(hipMemcpyAsync(&herr, err, 4, hipMemcpyDeviceToHost, s));
        PMS_HIP(hipStreamSynchronize(s));
        if (herr == 1) return set_err(c, PMS_ERR_INVALID_ARG, "non-finite FP32 squared distance");
        if (herr == 2) return set_err(c, PMS_ERR_INVALID_ARG, "squared distance >= 2^35 does not fit the order key");
        return PMS_OK;
    };
    // In LDS when every cloud's edges fit (a full cloud of 181 points, a larger
    // truncated one: tried while an eighth of its pairs would fit); the
    // device-wide sort takes the batch when one cloud's do not, or when its
    // distances are too much for the one workgroup it has here.  That takes 0.49 us
    // per 1 000 coordinates of its pairs, the device-wide keys 4.3 us per million of
    // all clouds', and their sort some 100 us more.  Builds to dimension 1 in us,
    // here and device-wide: 181 points of 512 coordinates 4153 and 263; 100 of 64 271
    // and 208, of 32 192 and 204; 60 of 128 200 and 182; 30 of 512 190 and 219; 128
    // clouds of 100 points of 64 435 and 627, of 512 1553 and 1871; 16 of 300 points of
    // 512 10.9 ms and 1.8.
    bool lds = maxpairs <= 8 * kLdsEdges && maxwork <= (double)(1 << 18) + work / 110;
    for (auto &I : h) lds = lds && (I.has_thr || (int64_t)I.n * (I.n - 1) / 2 <= kLdsEdges);
    if (lds) {
        int32_t cap = kVeThreads;  // (a sort has at least one key a thread)
        while (cap < kLdsEdges && cap < maxpairs) cap <<= 1;
        const size_t bytes = (size_t)cap * 8;
        PMS_ALLOW_LDS(f32 ? k_ve_edges<true> : k_ve_edges<false>, kLdsEdges * sizeof(unsigned long long));
        hipEvent_t e0 = nullptr;
        if (c->prof_on) { e0 = prof_event(c); (void)hipEventRecord(e0, s); }
        if (f32) k_ve_edges<true><<<B, kVeThreads, bytes, s>>>(dcl, pts, lexb, cap, ev_s, eval, erank, gst_s, gend_s, err);
        else k_ve_edges<false><<<B, kVeThreads, bytes, s>>>(dcl, pts, lexb, cap, ev_s, eval, erank, gst_s, gend_s, err);
        if (c->prof_on) {
            hipEvent_t e1 = prof_event(c);
            (void)hipEventRecord(e1, s);
            c->pend.push_back({K_VR_EDGES, e0, e1, 8.0 * slots + 20.0 * pairs, 0.0});
        }
        PMS_HIP(hipGetLastError());
        st = read_clouds();
        if (st != PMS_OK) return st;
        for (int b = 0; b < B; b++)
            if (h[(size_t)b].E > cap) lds = false;
    }
    const unsigned gx = (unsigned)std::max<int64_t>(1, std::min<int64_t>((maxpairs + 3) / 4, std::max(16, 16384 / B)));
    if (!lds) {
        unsigned long long *keys = (unsigned long long *)grow_scratch(c, B_BUILD7, P * 8);
        unsigned long long *keys2 = (unsigned long long *)grow_scratch(c, B_BUILD8, P * 8);
        int64_t *first = (int64_t *)grow_scratch(c, B_BUILD9, (size_t)(B + 1) * 8);
        if (!keys || !keys2 || !first) return set_err(c, PMS_ERR_OOM, "builder scratch");
        for (auto &I : h) I.E = 0;
        PMS_HIP(hipMemcpyAsync(dcl, h.data(), (size_t)B * sizeof(VeCloud), hipMemcpyHostToDevice, s));
        if (f32) PMS_LAUNCH(c, K_VR_EDGES, 4.0 * slots + 8.0 * pairs, k_ve_keys<true>, dim3(gx, B), kBlock, dcl, pts, lexb, cshift, keys, erank, err);
        else PMS_LAUNCH(c, K_VR_EDGES, 4.0 * slots + 8.0 * pairs, k_ve_keys<false>, dim3(gx, B), kBlock, dcl, pts, lexb, cshift, keys, erank, err);
        bool in_b = false;
        st = radix_sort<unsigned long long, uint32_t>(c, keys, keys2, nullptr, nullptr, pairs, cshift + cbits, B_AGG, B_AGG2, &in_b);
        if (st == PMS_OK) st = read_clouds();
        if (st != PMS_OK) return st;
        std::vector<int64_t> hf((size_t)B + 1, 0);
        for (int b = 0; b < B; b++) {
            hf[(size_t)b + 1] = hf[(size_t)b] + h[(size_t)b].E;
            h[(size_t)b].gmax = 1;
        }
        PMS_HIP(hipMemcpyAsync(first, hf.data(), hf.size() * 8, hipMemcpyHostToDevice, s));
        PMS_HIP(hipMemcpyAsync(dcl, h.data(), (size_t)B * sizeof(VeCloud), hipMemcpyHostToDevice, s));
        PMS_LAUNCH(c, K_VR_EDGES, 8.0 * pairs + 28.0 * pairs, k_ve_ranks, dim3(gx, B), kBlock, dcl, lexb, cshift,
                   in_b ? keys2 : keys, ev_s, eval, erank, gst_s, gend_s, first);
        PMS_HIP(hipGetLastError());
        st = read_clouds();
        if (st != PMS_OK) return st;
    }
    int64_t E = 0, words = 0, mwords = 0;
    for (int b = 0; b < B; b++) {
        VeCloud &I = h[(size_t)b];
        if (maxdim >= 2 && I.gmax > (maxdim >= 3 ? kVeMaxTies3 : kVeMaxTies)) return PMS_OK;
        if (maxdim < 1) I.E = 0;
        I.eoff = E;
        I.woff = words;
        E += I.E + 1;
        words += (int64_t)I.E * I.W;
        I.moff = mwords;
        mwords += (int64_t)I.E * I.M;
    }
    const int ids[] = {VR_CLOUDS, VR_EV, VR_GST, VR_GEND, VR_TSCAN, VR_APP, VR_APC, VR_REC, VR_MASK, VR_RECD};
    const size_t sz[] = {(size_t)B * sizeof(VeCloud), (size_t)E * 4, (size_t)E * 4, (size_t)E * 4, (size_t)E * 4,
                         (size_t)E * 4, (size_t)E * 4, (size_t)words * 8, (size_t)mwords * 8, maxdim >= 3 ? (size_t)words * 4 : 0};
    for (int k = 0; k < 10; k++)
        if ((st = filtration_vr_reserve(c, &f, ids[k], sz[k])) != PMS_OK) return st;
    f->vr_maxdim = maxdim;
    uint32_t *ev = (uint32_t *)f->vr[VR_EV].p;
    int32_t *gst = (int32_t *)f->vr[VR_GST].p, *gend = (int32_t *)f->vr[VR_GEND].p;
    int32_t *tscan = (int32_t *)f->vr[VR_TSCAN].p, *app = (int32_t *)f->vr[VR_APP].p;
    uint2 *rec = (uint2 *)f->vr[VR_REC].p;
    uint32_t *recd = maxdim >= 3 ? (uint32_t *)f->vr[VR_RECD].p : nullptr;
    VeCloud *cl = (VeCloud *)f->vr[VR_CLOUDS].p;
    PMS_HIP(hipMemcpyAsync(cl, h.data(), (size_t)B * sizeof(VeCloud), hipMemcpyHostToDevice, s));
    int64_t emax = 1, tmax = 1, qmax = 1;
    for (auto &I : h) emax = std::max<int64_t>(emax, I.E);
    // (workgroups per cloud: enough for the largest, about 16 K in all)
    auto grid = [&](int64_t units, int64_t per) {
        return dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>((units + per - 1) / per, std::max(16, 16384 / B))),
                    (unsigned)B);
    };
    uint64_t *mask = (uint64_t *)f->vr[VR_MASK].p;
    int32_t *apc = (int32_t *)f->vr[VR_APC].p;
    if (nmax <= kLdsPoints && E >= kVeManyEdges) {
        const size_t bytes = maxdim >= 2 ? (size_t)nmax * ve_rank_row((int)nmax) * 4 : 0;
        const unsigned parts = (unsigned)std::max<int64_t>(
            1, std::min<int64_t>((emax + kVeMaskThreads - 1) / kVeMaskThreads, std::max(1, 1024 / B)));
        PMS_ALLOW_LDS(k_ve_masks_lds, kLdsPoints * ve_rank_row(kLdsPoints) * 4);
        hipEvent_t e0 = nullptr;
        if (c->prof_on) { e0 = prof_event(c); (void)hipEventRecord(e0, s); }
        k_ve_masks_lds<<<dim3(parts, (unsigned)B), kVeMaskThreads, bytes, s>>>(cl, maxdim, ev_s, gst_s, gend_s, erank, ev,
                                                                              gst, gend, rec, mask, tscan, apc);
        if (c->prof_on) {
            hipEvent_t e1 = prof_event(c);
            (void)hipEventRecord(e1, s);
            c->pend.push_back({K_VR_TRI, e0, e1, 8.0 * words + 28.0 * E, 0.0});
        }
    } else {
        PMS_LAUNCH(c, K_VR_TRI, 8.0 * words + 28.0 * E, k_ve_masks, grid(emax, kWavesPerBlock), kBlock, cl, maxdim, ev_s,
                   gst_s, gend_s, erank, ev, gst, gend, rec, mask, tscan, apc);
    }
    PMS_LAUNCH(c, K_BUILD_SCAN, 8.0 * E, k_ve_scan, (unsigned)B, 1024, cl, tscan);
    PMS_HIP(hipGetLastError());
    PMS_HIP(hipMemcpyAsync(h.data(), cl, (size_t)B * sizeof(VeCloud), hipMemcpyDeviceToHost, s));
    PMS_HIP(hipStreamSynchronize(s));
    int64_t T = 0, Q = 0, words2 = 0;
    for (auto &I : h) {
        I.toff = T;
        T += I.T;
        tmax = std::max(tmax, I.T);
    }
    uint2 *tri = nullptr;
    if (maxdim >= 3) {
        int64_t Wm = 0;
        for (auto &I : h) Wm = std::max<int64_t>(Wm, I.W);
        for (auto &I : h) I.W2 = (int32_t)Wm;
        words2 = T * Wm;
        if ((st = filtration_vr_reserve(c, &f, VR_REC2, (size_t)words2 * 8)) != PMS_OK) return st;
        if ((st = filtration_vr_reserve(c, &f, VR_Q2, (size_t)(T + 1) * 8)) != PMS_OK) return st;
        tri = (uint2 *)grow_scratch(c, B_BUILD10, (size_t)std::max<int64_t>(T, 1) * 8);
        int64_t *tmp = (int64_t *)grow_scratch(c, B_BUILD11, (size_t)((T + kBlock - 1) / kBlock + 2) * 8);
        if (!tri || !tmp) return set_err(c, PMS_ERR_OOM, "builder scratch");
        int64_t *q2 = (int64_t *)f->vr[VR_Q2].p;
        PMS_HIP(hipMemcpyAsync(cl, h.data(), (size_t)B * sizeof(VeCloud), hipMemcpyHostToDevice, s));
        PMS_LAUNCH(c, K_VR_TRI, 8.0 * words2 + 16.0 * T, k_ve_tmasks, grid(tmax, kWavesPerBlock * kTriRun), kBlock,
                   filtration_vr_view(f), (uint2 *)f->vr[VR_REC2].p, tri, q2);
        if ((st = scan_i64(c, q2, T, tmp, &Q)) != PMS_OK) return st;
        PMS_LAUNCH(c, K_FILL, 0, k_ve_qbounds, (unsigned)((B + 255) / 256), 256, cl, B, T, Q, q2);
        PMS_HIP(hipMemcpyAsync(h.data(), cl, (size_t)B * sizeof(VeCloud), hipMemcpyDeviceToHost, s));
        PMS_HIP(hipStreamSynchronize(s));
    }
    int64_t m = 0, nnz = 0;
    f->vr_max_m = 0;
    for (int b = 0; b < B; b++) {
        VeCloud &I = h[(size_t)b];
        I.col_base = m;
        I.nnz_base = nnz;
        if (inst_col_off) inst_col_off[b] = m;
        const int64_t mb = I.n + I.E + I.T + I.Q;
        m += mb;
        nnz += 2LL * I.E + 3 * I.T + 4 * I.Q;
        qmax = std::max(qmax, I.Q);
        f->vr_max_m = std::max(f->vr_max_m, mb);
    }
    if (inst_col_off) inst_col_off[B] = m;
    if (m >= 0x7FFFFFFF) return set_err(c, PMS_ERR_INVALID_ARG, "too many simplices for 32-bit indices");
    st = filtration_reserve(c, &f, m, nnz, f32 ? 1 : 0);
    if (st != PMS_OK) return st;
    if (maxdim >= 3 && (st = filtration_vr_reserve(c, &f, VR_APPT, (size_t)m * 4)) != PMS_OK) return st;
    f->vr_max_n = (int32_t)nmax;
    PMS_HIP(hipMemcpyAsync(cl, h.data(), (size_t)B * sizeof(VeCloud), hipMemcpyHostToDevice, s));
    if (m == 0) {
        const int64_t zero = 0;
        PMS_HIP(hipMemcpyAsync(f->col_ptr, &zero, 8, hipMemcpyHostToDevice, s));
    } else {
        const VeView v = filtration_vr_view(f);
        const VeOut o{m, nnz, f->col_ptr, f->rows, f->dim, f->value, f->crit, f->verts};
        uint2 *rec2 = (uint2 *)f->vr[VR_REC2].p;
        int32_t *appt = maxdim >= 3 ? (int32_t *)f->vr[VR_APPT].p : nullptr;
        const double pb = f32 ? 37.0 : 41.0;
        const int tile = ve_tile(E);
        PMS_LAUNCH(c, K_VR_INDEX, 8.0 * words + 40.0 * E, k_ve_emit, grid(emax, tile), kBlock, v, maxdim, tile, eidx, rec, app, recd);
        if (f32) PMS_LAUNCH(c, K_VR_ROWS, (pb + 8) * E + (pb + 12) * T, k_ve_tris<true>, grid(std::max(emax, nmax), tile), kBlock, v, o, maxdim, tile, eval, appt);
        else PMS_LAUNCH(c, K_VR_ROWS, (pb + 8) * E + (pb + 12) * T, k_ve_tris<false>, grid(std::max(emax, nmax), tile), kBlock, v, o, maxdim, tile, eval, appt);
        if (maxdim >= 3 && T > 0) {
            PMS_LAUNCH(c, K_VR_INDEX, 8.0 * words2, k_ve_tindex, grid(tmax, kBlock), kBlock, v, tri, rec2, appt);
            if (f32) PMS_LAUNCH(c, K_VR_ROWS, (pb + 16) * Q, k_ve_tets<true>, grid(qmax, 2 * kBlock), kBlock, v, o, eval, tri);
            else PMS_LAUNCH(c, K_VR_ROWS, (pb + 16) * Q, k_ve_tets<false>, grid(qmax, 2 * kBlock), kBlock, v, o, eval, tri);
            PMS_LAUNCH(c, K_VR_INDEX, 5.0 * m, k_ve_appt, grid(f->vr_max_m, kBlock), kBlock, v, f->verts, f->dim, appt);
        }
        PMS_HIP(hipGetLastError());
    }
    PMS_HIP(hipStreamSynchronize(s));
    if (c->prof_on) prof_flush(c);
    f->m = m;
    f->nnz = nnz;
    f->value_is_f32 = f32 ? 1 : 0;
    f->vr_count = B;
    f->vr_edges = E;
    *done = 1;
    return PMS_OK;
}

}  // namespace pms
