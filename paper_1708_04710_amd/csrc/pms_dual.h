// A block of the boundary matrix reduced from its rows.
//
// The block of faces of dimension b and cofaces of dimension b + 1 has the
// same pairs as its anti-transpose: the faces' coboundaries as columns, taken
// from the last face to the first, each reduced to its smallest coface (the
// lows of a reduced matrix are unique, Sec. 2.3).  Where cofaces far outnumber
// faces (Vietoris-Rips complexes: 42 triangles per edge on 128 points) this is
// the side to work from: nearly all cofaces are positive, and their columns
// would each be added up to zero (411 M of 481 M additions of 64 full
// 128-point clouds), while most faces are paired at sight (the apparent
// pairs: the first coface of a face, of which the face is the last facet) and
// 15 of 8128 edges of such a cloud are left with 411 additions in all.
//
// The rounds are those of the matrix reduction: every active face adds, in
// one go, the known pivots of its smallest coface, an apparent face or the
// owner settled in an earlier round; where the low has no such pivot it
// claims it (k_dual_claim, after the round, so a round depends only on the
// state before it); of the faces that claim one coface the last one owns it
// and the others, a displaced owner among them, are active again.
//
// One wavefront per face.  The column is a bitmap over the cofaces, with a
// summary of one bit per word: lows only grow, so the next one is found by a
// scan from the last, an addition is one atomic per coface and costs the same
// for any fill-in (36 000 cofaces of 342 000 on a circle), and a column is
// remembered as the list of faces it is the sum of, not as its cofaces.
// Bound by the latency of one addition (two dependent loads, the flips, the
// scan) times the longest chain of them.
#pragma once

#include "pms_common.h"

namespace pms {

constexpr int kDualRounds = 256;  // rounds the counters have room for
constexpr int kDualCounters = 2 * kDualRounds + 3;
// Bits of a bitmap in LDS: with its summary 148 KB of a CU's 160 KB.
constexpr int64_t kDualLdsBits = 1150000;
inline int64_t dual_words(int64_t bits) { return (bits + 31) / 32; }
// LDS bytes of a workgroup: the words (when in LDS) and the summary, padded
// to whole wavefronts of words.
inline int64_t dual_summary_words(int64_t bits) { return ((dual_words(bits) + 31) / 32 + kWave - 1) / kWave * kWave; }

struct DualState {
    int32_t *low_star;         // cofaces: -1 none, >= 0 apparent (the face's column), -2 - key: settled owner
    int2 *list[2];             // active faces (instance, face), by round parity
    // counters, in this order: fail, arena_top, count, head
    int32_t *fail;             // a list outgrew its room: the block is left to the columns' side
    int32_t *arena_top;
    int32_t *count;            // [kDualRounds + 1] active faces of a round
    int32_t *head;             // [kDualRounds] faces taken in a round
    int32_t *vstart, *vlen;    // [key] the faces a column is the sum of, in arena (vlen 0: itself)
    int32_t *klow;             // [key] its smallest coface within the instance, -1: none
    int32_t *arena;            // faces
    int64_t arena_cap;
    int32_t *vtmp;             // [workgroup, vcap] the sum being built
    int32_t vcap;
    uint32_t *words;           // [workgroup, nw0] bitmaps beyond LDS (all zero between faces), or null
    int64_t nw0, nw1;          // words of a bitmap and of its summary
    unsigned long long *adds, *entries;
};

inline void dual_counters(DualState &s, int32_t *p)
{
    s.fail = p;
    s.arena_top = p + 1;
    s.count = p + 2;
    s.head = s.count + kDualRounds + 1;
}

struct DualMap {
    uint32_t *w;   // words (LDS or global)
    uint32_t *s;   // summary (LDS): bit k: word k may be non-zero
    bool lds;
    int64_t nw1;
    uint32_t bits;
    __device__ void toggle(int32_t t) const
    {
        if ((uint32_t)t >= bits) return;  // never (cofaces of one instance); a bound, not a branch
        atomicXor(&w[t >> 5], 1u << (t & 31));
        atomicOr(&s[t >> 10], 1u << ((t >> 5) & 31));
    }
    __device__ uint32_t load(int64_t k) const
    {
        return lds ? w[k] : __hip_atomic_load(&w[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // The smallest set coface >= from, -1 when none; the whole wavefront, all
    // lanes' flips before it done (__syncthreads).
    __device__ int32_t next(int32_t from) const
    {
        const int lane = threadIdx.x & (kWave - 1);
        const int32_t w0 = from >> 5;  // words before it are zero from here on
        for (int64_t b = (w0 >> 5) / kWave * kWave; b < nw1; b += kWave) {
            uint32_t x = s[b + lane];
            if (b + lane < (w0 >> 5)) x = 0;
            else if (b + lane == (w0 >> 5)) x &= ~0u << (w0 & 31);
            uint64_t m = __ballot(x != 0);
            while (m) {
                const int l = __ffsll((long long)m) - 1;
                const uint32_t xs = (uint32_t)__builtin_amdgcn_readlane((int)x, l);
                int32_t k = -1;  // the words of this summary word, one per lane
                if (lane < 32 && ((xs >> lane) & 1u)) k = (int32_t)(((b + l) << 5) + lane);
                uint32_t v = k >= 0 ? load(k) : 0u;
                if (k >= 0 && k == w0) v &= ~0u << (from & 31);
                const uint64_t z = __ballot(v != 0);
                if (z) {
                    const int f = __ffsll((long long)z) - 1;
                    const uint32_t vf = (uint32_t)__builtin_amdgcn_readlane((int)v, f);
                    return (int32_t)((((b + l) << 5) + f) * 32 + __ffs((int)vf) - 1);
                }
                m &= m - 1;
            }
        }
        return -1;
    }
    // Every word back to zero.
    __device__ void clear() const
    {
        const int lane = threadIdx.x & (kWave - 1);
        for (int64_t b = 0; b < nw1; b += kWave) {
            uint32_t x = s[b + lane];
            if (x) s[b + lane] = 0;
            while (x) {
                const int64_t k = ((b + lane) << 5) + __ffs((int)x) - 1;
                x &= x - 1;
                if (lds) w[k] = 0;
                else __hip_atomic_store(&w[k], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
};

// What a lane knows of the smallest coface beyond the last low that it
// flipped in the addition just made: the coface, the face it forms an apparent
// pair with (-1: it is not apparent) and that face's data.  When the next low
// is one of these, the next addition starts without looking it up.
struct DualCand {
    int32_t t, f, d0, d1;
};

// kLds: the bitmap's words are in LDS.  P: the cofaces of a face
//   bind(instance), key(face), face(key); col(t): the column of coface t
//   load(face, d0, d1): the data flip needs
//   int flip(map, face, d0, d1, cur, cand): flips the face's cofaces, returns
//     their number in this lane and fills cand (cofaces beyond cur)
//   int flip_many(map, faces, n): the same for a list, several faces' loads in flight
//   int32_t apparent(t, v): the face of coface t whose low_star is v >= 0 (-1: no such face)
template <class P, bool kLds>
__global__ void __launch_bounds__(kWave) k_dual(P prov, DualState s, int round)
{
    extern __shared__ uint32_t s_map[];
    const int32_t n = s.count[round];
    if ((int32_t)blockIdx.x >= n || *s.fail) return;
    const int lane = threadIdx.x;
    DualMap map;
    map.lds = kLds;
    map.s = s_map;
    map.nw1 = s.nw1;
    map.bits = (uint32_t)(s.nw0 * 32);
    map.w = kLds ? s_map + s.nw1 : s.words + (int64_t)blockIdx.x * s.nw0;
    for (int64_t k = lane; k < s.nw1 + (kLds ? s.nw0 : 0); k += kWave) s_map[k] = 0;
    __syncthreads();
    int32_t *v = s.vtmp + (int64_t)blockIdx.x * s.vcap;
    unsigned long long adds = 0, entries = 0;
    for (;;) {
        int32_t q = 0;
        if (lane == 0) q = atomicAdd(&s.head[round], 1);
        q = bcast_first(q);
        if (q >= n) break;
        const int2 it = s.list[round & 1][q];
        const int32_t face = bcast_first(it.y);
        prov.bind(bcast_first(it.x));
        const int64_t key = prov.key(face);
        const int32_t n0 = s.vlen[key];
        int32_t nv = 1, cur = 0;
        DualCand cand{0x7FFFFFFF, -1, 0, 0};
        if (n0 == 0) {
            int32_t d0, d1;
            if (lane == 0) v[0] = face;
            prov.load(face, d0, d1);
            entries += prov.flip(map, face, d0, d1, -1, cand);
        } else {
            const int32_t *a = s.arena + s.vstart[key];
            cur = s.klow[key];
            nv = n0;
            for (int32_t k = lane; k < n0; k += kWave) v[k] = a[k];
            entries += prov.flip_many(map, a, n0);
        }
        int32_t t;
        bool full = false;
        for (;;) {
            __syncthreads();  // the flips are done
            if (!kLds) __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): also in memory
            t = map.next(cur);
            if (t < 0) break;
            const uint64_t known = __ballot(cand.t == t);
            int32_t f = -1, d0 = 0, d1 = 0;
            if (known) {
                const int l = __ffsll((long long)known) - 1;
                f = __builtin_amdgcn_readlane(cand.f, l);
                d0 = __builtin_amdgcn_readlane(cand.d0, l);
                d1 = __builtin_amdgcn_readlane(cand.d1, l);
            }
            int64_t ko = -1;
            if (f < 0) {
                const int32_t ls = bcast_first(s.low_star[prov.col(t)]);  // (not written during a round)
                if (ls == -1) break;
                if (ls >= 0) {
                    f = bcast_first(prov.apparent(t, ls));
                    if (f < 0) { full = true; break; }
                    prov.load(f, d0, d1);
                } else {
                    ko = -2 - (int64_t)ls;
                    if (ko < key) break;  // an owner further on: it gives way
                }
            }
            cur = t + 1;  // (the addition cancels t)
            cand.t = 0x7FFFFFFF;
            if (ko < 0) {
                if (nv >= s.vcap) { full = true; break; }
                if (lane == 0) v[nv] = f;
                nv++;
                entries += prov.flip(map, f, d0, d1, t, cand);
            } else {
                const int32_t no = s.vlen[ko] > 0 ? s.vlen[ko] : 1;
                if (nv + no > s.vcap) { full = true; break; }
                if (s.vlen[ko] > 0) {
                    const int32_t *a = s.arena + s.vstart[ko];
                    for (int32_t k = lane; k < no; k += kWave) v[nv + k] = a[k];
                    entries += prov.flip_many(map, a, no);
                } else {
                    f = prov.face(ko);
                    if (lane == 0) v[nv] = f;
                    prov.load(f, d0, d1);
                    entries += prov.flip(map, f, d0, d1, t, cand);
                }
                nv += no;
            }
            adds++;
        }
        // remember the sum (itself alone needs no list)
        if (!full && nv > 1 && t >= 0) {
            int32_t at = 0;
            if (lane == 0) at = atomicAdd(s.arena_top, nv);
            at = bcast_first(at);
            if (at < 0 || (int64_t)at + nv > s.arena_cap) full = true;
            else {
                __syncthreads();  // v is written
                for (int32_t k = lane; k < nv; k += kWave) s.arena[at + k] = v[k];
                if (lane == 0) {
                    s.vstart[key] = at;
                    s.vlen[key] = nv;
                }
            }
        }
        if (lane == 0) {
            s.klow[key] = t;
            if (full) *s.fail = 1;
        }
        map.clear();
        __syncthreads();
        if (full) break;
    }
    // entries are counted per lane
    long long e = (long long)entries;
    for (int o = kWave / 2; o > 0; o >>= 1) e += __shfl_xor(e, o, kWave);
    if (lane == 0) {
        if (adds) atomicAdd(s.adds, adds);
        if (e) atomicAdd(s.entries, (unsigned long long)e);
    }
}

// After a round: the claims.  Every face active in it that stopped at a
// coface claims it; the larger key stays, the other one (claimed earlier this
// round, or settled) is active in the next round.
template <class P>
__global__ void __launch_bounds__(kBlock) k_dual_claim(P prov, DualState s, int round)
{
    if (*s.fail) return;
    const int32_t n = s.count[round];
    for (int32_t q = blockIdx.x * kBlock + threadIdx.x; q < n; q += gridDim.x * kBlock) {
        const int2 it = s.list[round & 1][q];
        prov.bind(it.x);
        const int64_t key = prov.key(it.y);
        const int32_t t = s.klow[key];
        if (t < 0) continue;
        const int32_t mine = (int32_t)(-2 - key);
        const int32_t old = atomicMin(&s.low_star[prov.col(t)], mine);
        if (old == -1) continue;
        const int32_t at = atomicAdd(&s.count[round + 1], 1);
        s.list[(round + 1) & 1][at] = make_int2(it.x, old > mine ? prov.face(-2 - (int64_t)old) : it.y);
    }
}

// The counters before the first round (first = 1: no faces listed yet), or
// when the rounds they have room for are used up.
static __global__ void k_dual_counters(DualState s, int first, int32_t n)
{
    for (int k = threadIdx.x; k <= kDualRounds; k += blockDim.x) {
        s.count[k] = k == 0 ? n : 0;
        if (k < kDualRounds) s.head[k] = 0;
    }
    if (first && threadIdx.x == 0) {
        *s.fail = 0;
        *s.arena_top = 0;
    }
}

// k_dual's LDS, allowed and launched.
template <class P>
inline pms_status dual_map_lds(Ctx *c, const P &, const DualState &s)
{
    const int lds = (int)((s.nw1 + (s.words ? 0 : s.nw0)) * 4);
    const void *fn = s.words ? (const void *)k_dual<P, false> : (const void *)k_dual<P, true>;
    PMS_HIP(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    return PMS_OK;
}
template <class P>
inline void dual_launch(Ctx *c, const P &prov, const DualState &s, unsigned blocks, int round)
{
    const size_t lds = (size_t)(s.nw1 + (s.words ? 0 : s.nw0)) * 4;
    if (s.words) k_dual<P, false><<<blocks, kWave, lds, c->stream>>>(prov, s, round);
    else k_dual<P, true><<<blocks, kWave, lds, c->stream>>>(prov, s, round);
}

// Runs the rounds of one block, launch(r) issuing round r's additions.
// count[0] faces are listed.  *rounds grows by the rounds that had active
// faces, *active by their faces; *ok = 0: a list outgrew its room and the
// block is not reduced.
template <class P, class L>
inline pms_status dual_rounds(Ctx *c, const P &prov, const DualState &s, L launch, int kid, int32_t *rounds,
                              int64_t *active, int *ok)
{
    *ok = 1;
    static_assert((kDualRounds + 3) * 4 <= 2048, "the pinned buffer holds the counters");
    const volatile int32_t *h = (const int32_t *)c->host_pinned;  // fail, arena_top, counts
    for (int r = 0;;) {
        // a few rounds per host synchronisation (a round without faces returns at once)
        const int r1 = r + 4 < kDualRounds ? r + 4 : kDualRounds;
        hipEvent_t e0 = nullptr;
        if (c->prof_on) { e0 = prof_event(c); (void)hipEventRecord(e0, c->stream); }
        for (int q = r; q < r1; q++) {
            launch(q);
            k_dual_claim<P><<<32, kBlock, 0, c->stream>>>(prov, s, q);
        }
        if (c->prof_on) {
            hipEvent_t e1 = prof_event(c);
            (void)hipEventRecord(e1, c->stream);
            c->pend.push_back({kid, e0, e1, 0.0, 0.0});
        }
        PMS_HIP(hipGetLastError());
        PMS_HIP(hipMemcpyAsync(c->host_pinned, s.fail, (size_t)(2 + r1 + 1) * 4, hipMemcpyDeviceToHost, c->stream));
        PMS_HIP(hipStreamSynchronize(c->stream));
        for (int q = r; q < r1; q++)
            if (h[2 + q] > 0) {
                (*rounds)++;
                *active += h[2 + q];
            }
        r = r1;
        if (h[0]) {
            *ok = 0;
            return PMS_OK;
        }
        if (h[2 + r] == 0) return PMS_OK;
        if (r == kDualRounds) {  // room for more rounds: their list keeps its parity (kDualRounds is even)
            const int32_t left = h[2 + r];
            k_dual_counters<<<1, kBlock, 0, c->stream>>>(s, 0, left);
            r = 0;
        }
    }
}

}  // namespace pms
