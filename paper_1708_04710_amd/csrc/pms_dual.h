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
// One workgroup per face.  The column is a bitmap over the cofaces in LDS,
// with a summary of one bit per word: lows only grow, so the next one is found
// by a scan from the last, an addition is one LDS atomic per coface and costs
// the same for any fill-in (36 000 cofaces of 342 000 on a circle), and a
// column is remembered as the list of faces it is the sum of, not as its
// cofaces.  Cofaces beyond the bitmap's reach wait in a list until the lows
// get there and the bitmap moves on.  Bound by the latency of one addition
// (dependent loads, the flips, the scan) times the longest chain of them.
#pragma once

#include "pms_common.h"

namespace pms {

constexpr int kDualRounds = 256;  // rounds the counters have room for
constexpr int kDualCounters = 2 * kDualRounds + 3;
// Most bits of a bitmap: with its summary 148 KB of a CU's 160 KB.
constexpr int64_t kDualLdsBits = 1150000;
inline int64_t dual_words(int64_t bits) { return (bits + 31) / 32; }
// Words of its summary, whole wavefronts of them.
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
    int32_t *ovf;              // [workgroup, ovf_cap] cofaces beyond the bitmap, or null (it holds the instance)
    int32_t ovf_cap;
    int64_t nw0, nw1;          // words of a bitmap and of its summary
    unsigned long long *adds, *entries;
    unsigned long long *abytes;  // 8 per entry read (a list word, a bit toggled), or null
};

inline void dual_counters(DualState &s, int32_t *p)
{
    s.fail = p;
    s.arena_top = p + 1;
    s.count = p + 2;
    s.head = s.count + kDualRounds + 1;
}

template <int kT>
struct DualMap {
    uint32_t *w;      // words (LDS)
    uint32_t *s;      // summary (LDS): bit k: word k may be non-zero
    int32_t *ovf;     // cofaces beyond the bitmap
    int32_t *n_ovf;   // (LDS)
    int32_t ovf_cap;
    int32_t base;     // the first coface of the bitmap, a multiple of 1024
    uint32_t bits;
    int32_t nw1;
    __device__ void toggle(int32_t t) const
    {
        const uint32_t k = (uint32_t)(t - base);  // (below base: cancels, nothing below the low is left)
        if (k < bits) {
            atomicXor(&w[k >> 5], 1u << (k & 31));
            atomicOr(&s[k >> 10], 1u << ((k >> 5) & 31));
        } else if (ovf && t >= base) {
            const int32_t at = atomicAdd(n_ovf, 1);
            if (at < ovf_cap) ovf[at] = t;
        }
    }
    // The smallest set coface >= from in the bitmap, -1 when none; every
    // wavefront by itself, all flips before it done.
    __device__ int32_t scan(int32_t from) const
    {
        const int lane = threadIdx.x & (kWave - 1);
        const int32_t f = max(from - base, 0), w0 = f >> 5;  // words before it are zero from here on
        for (int32_t b = (w0 >> 5) / kWave * kWave; b < nw1; b += kWave) {
            uint32_t x = s[b + lane];
            if (b + lane < (w0 >> 5)) x = 0;
            else if (b + lane == (w0 >> 5)) x &= ~0u << (w0 & 31);
            uint64_t m = __ballot(x != 0);
            while (m) {
                const int l = __ffsll((long long)m) - 1;
                const uint32_t xs = (uint32_t)__builtin_amdgcn_readlane((int)x, l);
                int32_t k = -1;  // the words of this summary word, one per lane
                if (lane < 32 && ((xs >> lane) & 1u)) k = ((b + l) << 5) + lane;
                uint32_t v = k >= 0 ? w[k] : 0u;
                if (k == w0) v &= ~0u << (f & 31);
                const uint64_t z = __ballot(v != 0);
                if (z) {
                    const int g = __ffsll((long long)z) - 1;
                    const uint32_t vg = (uint32_t)__builtin_amdgcn_readlane((int)v, g);
                    return base + (((b + l) << 5) + g) * 32 + __ffs((int)vg) - 1;
                }
                m &= m - 1;
            }
        }
        return -1;
    }
    // The smallest set coface >= from, moving the bitmap on when it is used up.
    __device__ int32_t next(int32_t from, int32_t *s_min)
    {
        for (;;) {
            const int32_t t = scan(from);
            __syncthreads();  // scanned by every wavefront before it changes
            if (t >= 0 || !ovf) return t;
            const int32_t n = min(*n_ovf, ovf_cap);
            if (n == 0) return -1;
            clear();
            if (threadIdx.x == 0) *s_min = 0x7FFFFFFF;
            __syncthreads();
            int32_t mn = 0x7FFFFFFF;
            for (int32_t k = threadIdx.x; k < n; k += kT) mn = min(mn, ovf[k]);
            atomicMin(s_min, mn);
            __syncthreads();
            base = *s_min & ~1023;
            __syncthreads();
            if (threadIdx.x == 0) *n_ovf = 0;
            __syncthreads();
            // what stays beyond is moved down, behind the entries read
            for (int32_t k0 = 0; k0 < n; k0 += kT) {
                const int32_t x = k0 + (int32_t)threadIdx.x < n ? ovf[k0 + threadIdx.x] : -1;
                __syncthreads();
                if (x >= 0) toggle(x);
                __syncthreads();
            }
        }
    }
    // Every word back to zero (each thread the words of its summary words).
    __device__ void clear() const
    {
        for (int32_t b = threadIdx.x; b < nw1; b += kT) {
            uint32_t x = s[b];
            if (x) s[b] = 0;
            for (; x; x &= x - 1) w[(b << 5) + __ffs((int)x) - 1] = 0;
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

// P: the cofaces of a face, for workgroups of P::kT threads
//   bind(instance), key(face), face(key); col(t): the column of coface t;
//   floor(face): no coface of it is smaller
//   load(face, d0, d1): the data flip needs
//   int flip(map, face, d0, d1, cur, cand): flips the face's cofaces (the whole
//     workgroup), returns their number in this lane and fills cand (cofaces beyond cur)
//   int flip_many(map, faces, n): the same for a list, several faces' loads in flight
//   int32_t apparent(t, v): the face of coface t whose low_star is v >= 0 (-1: no such face)
template <class P>
__global__ void __launch_bounds__(P::kT) k_dual(P prov, DualState s, int round)
{
    constexpr int kT = P::kT;
    extern __shared__ uint32_t s_map[];
    __shared__ int32_t s_q, s_ovf, s_min, s_at, s_cand[4];
    const int32_t n = s.count[round];
    if ((int32_t)blockIdx.x >= n || *s.fail) return;
    const int tid = threadIdx.x;
    DualMap<kT> map;
    map.s = s_map;
    map.w = s_map + s.nw1;
    map.nw1 = (int32_t)s.nw1;
    map.bits = (uint32_t)(s.nw0 * 32);
    map.ovf = s.ovf ? s.ovf + (int64_t)blockIdx.x * s.ovf_cap : nullptr;
    map.ovf_cap = s.ovf_cap;
    map.n_ovf = &s_ovf;
    for (int64_t k = tid; k < s.nw1 + s.nw0; k += kT) s_map[k] = 0;
    int32_t *v = s.vtmp + (int64_t)blockIdx.x * s.vcap;
    unsigned long long adds = 0, entries = 0;
    for (;;) {
        if (tid == 0) {
            s_q = atomicAdd(&s.head[round], 1);
            s_ovf = 0;
        }
        __syncthreads();
        const int32_t q = bcast_first(s_q);
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
            map.base = prov.floor(face) & ~1023;
            if (tid == 0) v[0] = face;
            prov.load(face, d0, d1);
            entries += prov.flip(map, face, d0, d1, -1, cand);
        } else {
            const int32_t *a = s.arena + s.vstart[key];
            cur = s.klow[key];
            map.base = cur & ~1023;
            nv = n0;
            for (int32_t k = tid; k < n0; k += kT) v[k] = a[k];
            entries += prov.flip_many(map, a, n0);
        }
        int32_t t;
        bool full = false;
        for (;;) {
            __syncthreads();  // the flips are done
            if (s_ovf > s.ovf_cap && s.ovf) { full = true; break; }
            t = map.next(cur, &s_min);
            if (t < 0) break;
            int32_t f = -1, d0 = 0, d1 = 0;
            if (kT == kWave) {
                const uint64_t known = __ballot(cand.t == t);
                if (known) {
                    const int l = __ffsll((long long)known) - 1;
                    f = __builtin_amdgcn_readlane(cand.f, l);
                    d0 = __builtin_amdgcn_readlane(cand.d0, l);
                    d1 = __builtin_amdgcn_readlane(cand.d1, l);
                }
            } else {
                if (tid == 0) s_cand[0] = -1;
                __syncthreads();
                if (cand.t == t) {  // (one lane: a coface is flipped once per addition)
                    s_cand[0] = cand.f;
                    s_cand[1] = cand.d0;
                    s_cand[2] = cand.d1;
                }
                __syncthreads();
                f = bcast_first(s_cand[0]);
                d0 = bcast_first(s_cand[1]);
                d1 = bcast_first(s_cand[2]);
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
                if (tid == 0) v[nv] = f;
                nv++;
                entries += prov.flip(map, f, d0, d1, t, cand);
            } else {
                const int32_t no = s.vlen[ko] > 0 ? s.vlen[ko] : 1;
                if (nv + no > s.vcap) { full = true; break; }
                if (s.vlen[ko] > 0) {
                    const int32_t *a = s.arena + s.vstart[ko];
                    for (int32_t k = tid; k < no; k += kT) v[nv + k] = a[k];
                    entries += prov.flip_many(map, a, no);
                } else {
                    f = prov.face(ko);
                    if (tid == 0) v[nv] = f;
                    prov.load(f, d0, d1);
                    entries += prov.flip(map, f, d0, d1, t, cand);
                }
                nv += no;
            }
            if (tid == 0) adds++;
        }
        // remember the sum (itself alone needs no list)
        __syncthreads();
        if (!full && nv > 1 && t >= 0) {
            if (tid == 0) s_at = atomicAdd(s.arena_top, nv);
            __syncthreads();  // (v is written, too)
            const int32_t at = s_at;
            if (at < 0 || (int64_t)at + nv > s.arena_cap) full = true;
            else {
                for (int32_t k = tid; k < nv; k += kT) s.arena[at + k] = v[k];
                if (tid == 0) {
                    s.vstart[key] = at;
                    s.vlen[key] = nv;
                }
            }
        }
        if (tid == 0) {
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
    if ((tid & (kWave - 1)) == 0) {
        if (adds) atomicAdd(s.adds, adds);
        if (e) atomicAdd(s.entries, (unsigned long long)e);
        if (e && s.abytes) atomicAdd(s.abytes, 8ull * (unsigned long long)e);
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
inline pms_status dual_map_lds(Ctx *c, const P &)
{
    PMS_ALLOW_LDS(k_dual<P>, (dual_words(kDualLdsBits) + dual_summary_words(kDualLdsBits)) * 4);
    return PMS_OK;
}
template <class P>
inline void dual_launch(Ctx *c, const P &prov, const DualState &s, unsigned blocks, int round)
{
    k_dual<P><<<blocks, P::kT, (size_t)(s.nw1 + s.nw0) * 4, c->stream>>>(prov, s, round);
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
    const int most = c->dual.rounds ? c->dual.rounds : kDualRounds;
    for (int r = 0;;) {
        // a few rounds per host synchronisation (a round without faces returns at once)
        const int r1 = r + 4 < most ? r + 4 : most;
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
        if (r == most) {  // room for more rounds: their list keeps its parity (an even number)
            const int32_t left = h[2 + r];
            k_dual_counters<<<1, kBlock, 0, c->stream>>>(s, 0, left);
            r = 0;
        }
    }
}

}  // namespace pms
