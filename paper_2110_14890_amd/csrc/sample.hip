// sample.hip -- query sampling with verified negatives on gfx950.
//
// Positives (smore_sample_positives), one kernel:
//
//  k_positive: PA lanes per query (two for plans that usually accept, up to
//    64 for the others), lane l running attempts l, l + PA, ...;
//    the lowest successful attempt wins.
//    Reverse directional sampling
//    (Sec. 3.1; appendix on reverse directional sampling): attempt t grounds
//    the root among entities with an in-edge, then runs the pre-order walk
//    program compiled from the plan, each projection picking an in-relation
//    of the current entity and an in-neighbour under it.  The first attempt
//    that reaches every anchor, keeps single-projection siblings apart and
//    respects max_fanout wins.  In a whole call (smore_sample) the same
//    lanes then look up the query's forward-cached lists.
//
// Negatives (smore_sample_negatives): bidirectional rejection sampling
// (Sec. 3.2) at the node cut the planner picks for the shape, all on the
// caller's stream with no host synchronisation:
//
//  k_prepare: the forward-cached lists of queries that the call does not
//    sample itself.
//  k_candidates: one wavefront per query draws, verifies and selects until
//    the row is full.  Forward caching turns the anchors into their
//    neighbour lists A_r(a) (sorted CSR groups, staged in LDS when small,
//    used in place when not); a draw without an in-edge, or with in-edges
//    under none of the root's relations, is settled by masks and signatures
//    that fit the caches; the others are verified backward from the
//    candidate; the first occurrences of the non-answers, in draw order, are
//    the negatives, so the output is a function of the draw indices alone.
//    Edge shapes (1p 2i 3i 2u 2in 3in) end here.
//  k_heavy3, k_units3 (3p): the candidates with lists too long for one
//    wavefront to walk.
//  k_finish: the queries that had such candidates (whose lists it decides
//    itself for the other shapes): selection and further draws.
//
// The steps can also be launched apart (smore_sample_negatives_part): the
// preparation, the candidate kernel, the rest.
//
// Shared-candidate minibatches (smore_sample_shared) and verification of
// caller candidates (smore_verify) run the same verification on given
// candidates (k_pairs), each wavefront packing its mask row, then the
// long-list kernels (k_heavy; 3p as above).
#include <hip/hip_runtime.h>

#include <climits>
#include <cstring>
#include <mutex>

#include "philox.h"
#include "rows.h"
#include "smore_internal.h"

namespace smore {
namespace {

constexpr int STAGE = 1024;   // LDS entries per wavefront for staged forward lists

// Draw states.  ST_DEEP exists only inside the candidate kernels: the
// candidate has a backward list, which the deep pass tests.
enum : int32_t { ST_NON = 0, ST_ANS = 1, ST_PEND = 3, ST_DEEP = 4 };

// Accounting of graph reads (bytes, and the 64-byte lines they span).  The
// verification kernel is instantiated with Tally when the caller asks for
// the figures and with NoTally otherwise; NoTally compiles to nothing.
struct NoTally {
    static constexpr bool on = false;
    __device__ __forceinline__ void read(const void*, int32_t) {}
};
struct Tally {
    static constexpr bool on = true;
    uint64_t b = 0, l = 0;
    __device__ __forceinline__ void read(const void* p, int32_t nbytes)
    {
        if (nbytes <= 0) return;
        const uint64_t a = (uint64_t)p;
        b += (uint64_t)nbytes;
        l += ((a + nbytes - 1) >> 6) - (a >> 6) + 1;
    }
};

// Edges [x, y) of v under r when v's node-pointer pair (n0, n1) is known.
// The entries of the last SCAN groups in question (and the next one, for the
// end bound) are loaded at once, so the lookup of an entity with no more
// than that is one dependent step.
constexpr int SCAN = 8;

// One step of an eight-way search of the n > SCAN groups from lo for
// relation r: seven probes at once, after which the group, if the entity
// has it, is among the n left.
template <class T>
__device__ __forceinline__ void group_narrow(const DirView& d, int32_t& lo, int32_t& n, int32_t r, T& tl)
{
    const int32_t q = n >> 3;
    int32_t v[7], c = 0;
#pragma unroll
    for (int k = 0; k < 7; ++k) {
        v[k] = d.grp[lo + q * (k + 1)].x;
        tl.read(&d.grp[lo + q * (k + 1)].x, 4);
    }
#pragma unroll
    for (int k = 0; k < 7; ++k) c += v[k] <= r;
    lo += q * c;
    n = c == 7 ? n - 7 * q : q;
}

template <class T>
__device__ __forceinline__ int2 group_find(const DirView& d, int32_t n0, int32_t n1, int32_t r, T& tl)
{
    int32_t n = n1 - n0;
    while (n > SCAN) group_narrow(d, n0, n, r, tl);
    if (n <= 0) return make_int2(0, 0);
    int2 e[SCAN + 1];
#pragma unroll
    for (int k = 0; k <= SCAN; ++k) e[k] = k <= n ? d.grp[n0 + k] : make_int2(INT_MAX, 0);
    tl.read(d.grp + n0, 8 * (n + 1));
    int2 res = make_int2(0, 0);
#pragma unroll
    for (int k = 0; k < SCAN; ++k)
        if (k < n && e[k].x == r) res = make_int2(e[k].y, e[k + 1].y);
    return res;
}

// group_find of two entities at once (the loads of both in flight together);
// inactive entries return (0, 0).  Entities with more than SCAN groups are
// narrowed eight ways per step first: a wavefront waits for its widest
// lane, and one of 535 groups is three dependent reads and the scan in place
// of ten.
template <class T>
__device__ __forceinline__ void group_find2(const DirView& d, const int32_t* n0, const int32_t* n1,
                                            const bool* act, int32_t r, int2* res, T& tl)
{
    int32_t lo[2], n[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        lo[u] = n0[u];
        n[u] = act[u] ? n1[u] - n0[u] : 0;
    }
    while (n[0] > SCAN || n[1] > SCAN) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
            if (n[u] > SCAN) group_narrow(d, lo[u], n[u], r, tl);
    }
    int2 e[2][SCAN + 1];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
#pragma unroll
        for (int k = 0; k <= SCAN; ++k)
            e[u][k] = (n[u] > 0 && k <= n[u]) ? d.grp[lo[u] + k] : make_int2(INT_MAX, 0);
        if (n[u] > 0) tl.read(d.grp + lo[u], 8 * (n[u] + 1));
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        res[u] = make_int2(0, 0);
#pragma unroll
        for (int k = 0; k < SCAN; ++k)
            if (k < n[u] && e[u][k].x == r) res[u] = make_int2(e[u][k].y, e[u][k + 1].y);
    }
}

// Edges [x, y) of entity v under relation r in one direction ((0, 0) if
// none): the node-pointer pair, then the group lookup.
template <class T>
__device__ __forceinline__ int2 group_range(const DirView& d, int32_t v, int32_t r, T& tl)
{
    const int32_t n0 = d.node[v], n1 = d.node[v + 1];
    tl.read(d.node + v, 8);
    return group_find(d, n0, n1, r, tl);
}

__device__ __forceinline__ int2 group_range(const DirView& d, int32_t v, int32_t r)
{
    NoTally t;
    return group_range(d, v, r, t);
}

// A sorted entity list in memory.
struct FSet {
    const int32_t* p;
    int32_t n;
};

template <class T>
__device__ __forceinline__ bool has(const int32_t* p, int32_t n, int32_t x, bool count, T& tl)
{
    int32_t lo = 0, hi = n;
    while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if (count) tl.read(p + mid, 4);
        if (p[mid] < x) lo = mid + 1; else hi = mid;
    }
    if (lo < n && count) tl.read(p + lo, 4);
    return lo < n && p[lo] == x;
}

// Wave-uniform copy of a value every lane holds (the compiler then keeps
// loops and exits that depend on it converged).
__device__ __forceinline__ int32_t uni(int32_t x) { return __builtin_amdgcn_readfirstlane(x); }

// Lane k's copy of a value (k wave-uniform).
__device__ __forceinline__ int32_t readlane(int32_t x, int k) { return __builtin_amdgcn_readlane(x, k); }

__device__ __forceinline__ uint64_t lanes_below(int lane)
{
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// Four independent membership searches of x[0..3] in the sorted list
// B[0..nb) (nb wave-uniform): branchless, the same number of steps in every
// lane, and the four loads of a step independent of each other, so a lane
// keeps four dependent chains in flight.  A key of -1 never matches.
template <class T>
__device__ __forceinline__ void search4(const int32_t* B, int32_t nb, const int32_t* x, bool* found,
                                        bool count, T& tl)
{
    int32_t base[4] = {0, 0, 0, 0};
    if (nb <= 0) {
        found[0] = found[1] = found[2] = found[3] = false;
        return;
    }
    for (int32_t n = nb; n > 1;) {
        const int32_t half = n >> 1;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (count) tl.read(B + base[k] + half, 4);
            base[k] = B[base[k] + half] <= x[k] ? base[k] + half : base[k];
        }
        n -= half;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (count) tl.read(B + base[k], 4);
        found[k] = B[base[k]] == x[k];
    }
}

// search4 with a target list per key (lists of different lengths; the loop
// runs until every key of the lane is settled), and three probes per step
// where four or more entries remain (a quaternary search: fewer dependent
// reads, more reads in all).
template <class T>
__device__ __forceinline__ void search4q(const int32_t* const* B, const int32_t* nb, const int32_t* x,
                                         const bool* count, bool* found, T& tl)
{
    int32_t base[4] = {0, 0, 0, 0}, n[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) n[k] = nb[k];
    for (;;) {
        bool more = false;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (n[k] >= 4) {
                const int32_t q = n[k] >> 2;
                const int32_t* b = B[k] + base[k];
                if (count[k]) { tl.read(b + q, 4); tl.read(b + 2 * q, 4); tl.read(b + 3 * q, 4); }
                const int32_t v1 = b[q], v2 = b[2 * q], v3 = b[3 * q];
                base[k] += q * ((v1 <= x[k]) + (v2 <= x[k]) + (v3 <= x[k]));
                n[k] -= 3 * q;
            } else if (n[k] > 1) {
                const int32_t half = n[k] >> 1;
                if (count[k]) tl.read(B[k] + base[k] + half, 4);
                base[k] = B[k][base[k] + half] <= x[k] ? base[k] + half : base[k];
                n[k] -= half;
            }
            more |= n[k] > 1;
        }
        if (!more) break;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        found[k] = false;
        if (nb[k] > 0) {
            if (count[k]) tl.read(B[k] + base[k], 4);
            found[k] = B[k][base[k]] == x[k];
        }
    }
}

// Does some element of K[0..nk) occur in L[0..nl)?  Whole wavefront, 256
// keys per step (four per lane).  k_glob / l_glob: whether reads of the
// list count as graph traffic.
template <class T>
__device__ bool wave_any(const int32_t* K, int32_t nk, bool k_glob, const int32_t* L, int32_t nl,
                         bool l_glob, int lane, T& tl)
{
    for (int32_t k0 = 0; k0 < nk; k0 += 256) {
        int32_t x[4];
        bool f[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int32_t i = k0 + 64 * k + lane;
            x[k] = i < nk ? K[i] : -1;
        }
        if (k_glob && lane == 0) tl.read(K + k0, 4 * min(256, nk - k0));
        search4(L, nl, x, f, l_glob, tl);
        if (__ballot(f[0] || f[1] || f[2] || f[3])) return true;
    }
    return false;
}

// Do the sorted lists A and B share an element?  The shorter is the key
// list, searched in the longer.
template <class T>
__device__ bool wave_meet(const int32_t* A, int32_t na, bool a_glob, const int32_t* B, int32_t nb,
                          bool b_glob, int lane, T& tl)
{
    if (na <= nb) return wave_any(A, na, a_glob, B, nb, b_glob, lane, tl);
    return wave_any(B, nb, b_glob, A, na, a_glob, lane, tl);
}

// Does the sorted graph list S share one element with both A and B?  The
// shortest of the three is the key list, searched in the other two.
template <class T>
__device__ bool wave_meet3(const int32_t* S, int32_t ns, FSet A, FSet B, int lane, T& tl)
{
    const int32_t *K = S, *L1 = A.p, *L2 = B.p;
    int32_t nk = ns, n1 = A.n, n2 = B.n;
    bool kg = true, g1 = false, g2 = false;   // lookups inside forward lists are not counted
    if (A.n < nk && A.n <= B.n) {
        K = A.p; nk = A.n; kg = false;
        L1 = S; n1 = ns; g1 = true;
    } else if (B.n < nk) {
        K = B.p; nk = B.n; kg = false;
        L2 = S; n2 = ns; g2 = true;
    }
    for (int32_t k0 = 0; k0 < nk; k0 += 256) {
        int32_t x[4];
        bool f1[4], f2[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int32_t i = k0 + 64 * k + lane;
            x[k] = i < nk ? K[i] : -1;
        }
        if (kg && lane == 0) tl.read(K + k0, 4 * min(256, nk - k0));
        search4(L1, n1, x, f1, g1, tl);
        search4(L2, n2, x, f2, g2, tl);
        const bool hit = (f1[0] && f2[0]) || (f1[1] && f2[1]) || (f1[2] && f2[2]) || (f1[3] && f2[3]);
        if (__ballot(hit)) return true;
    }
    return false;
}

// Does the sorted graph list S share an element with A that is not in B
// (the set difference of an intersection with a complemented operand)?
// The shorter of S and A is the key list, searched in the other and in B.
template <class T>
__device__ bool wave_meet_minus(const int32_t* S, int32_t ns, FSet A, FSet B, int lane, T& tl)
{
    const int32_t *K = S, *L = A.p;
    int32_t nk = ns, nl = A.n;
    bool kg = true, lg = false;   // lookups inside forward lists are not counted
    if (A.n < ns) {
        K = A.p; nk = A.n; kg = false;
        L = S; nl = ns; lg = true;
    }
    for (int32_t k0 = 0; k0 < nk; k0 += 256) {
        int32_t x[4];
        bool f1[4], f2[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int32_t i = k0 + 64 * k + lane;
            x[k] = i < nk ? K[i] : -1;
        }
        if (kg && lane == 0) tl.read(K + k0, 4 * min(256, nk - k0));
        search4(L, nl, x, f1, lg, tl);
        search4(B.p, B.n, x, f2, false, tl);
        const bool hit = (f1[0] && !f2[0]) || (f1[1] && !f2[1]) || (f1[2] && !f2[2]) || (f1[3] && !f2[3]);
        if (__ballot(hit)) return true;
    }
    return false;
}

// ------------------------------------------------------------- positive
__device__ __forceinline__ int32_t sel4(int i, int32_t a, int32_t b, int32_t c, int32_t d)
{
    return i == 0 ? a : i == 1 ? b : i == 2 ? c : d;
}

__device__ __forceinline__ int32_t reg5(int i, const int32_t* e)
{
    return i == 0 ? e[0] : i == 1 ? e[1] : i == 2 ? e[2] : i == 3 ? e[3] : e[4];
}

// Relation grounded for relation slot sl (-1 if no step has it).
__device__ __forceinline__ int32_t slot_rel(const WalkProgram& wp, const int32_t* qr, int sl)
{
    int32_t v = -1;
    for (int k = 0; k < wp.n_steps; ++k)
        if (wp.rel_slot[k] == sl) v = sel4(k, qr[0], qr[1], qr[2], -1);
    return v;
}

// Is t in the complemented operand's set: A_r0(a) for one step, or the
// entities reached from A_r0(a) under r1 for two (some y of A_r0(a) with
// (y, r1, t) an edge)?  At lane level: the shorter of A_r0(a) and t's
// in-list under r1 is walked and each entry searched in the longer.
__device__ bool neg_member(const GraphView& g, int steps, int32_t a, int32_t r0, int32_t r1, int32_t t)
{
    NoTally none;
    const int2 f = group_range(g.fwd, a, r0);
    const int32_t nf = f.y - f.x;
    if (steps == 1) return nf > 0 && has(g.fwd.nbr + f.x, nf, t, false, none);
    const int2 b = group_range(g.rev, t, r1);
    const int32_t nb = b.y - b.x;
    if (nf == 0 || nb == 0) return false;
    const bool fk = nf <= nb;
    const int32_t* K = fk ? g.fwd.nbr + f.x : g.rev.nbr + b.x;
    const int32_t* L = fk ? g.rev.nbr + b.x : g.fwd.nbr + f.x;
    const int32_t nk = fk ? nf : nb, nl = fk ? nb : nf;
    for (int32_t i = 0; i < nk; ++i)
        if (has(L, nl, K[i], false, none)) return true;
    return false;
}

// Attempts of one query run PA at a time, on PA neighbouring lanes (lane l
// of the group takes attempts l, l + PA, ...): the lowest successful
// attempt of a group step is the first successful attempt overall, so the
// result is that of trying them one after the other.  positive_lanes chooses
// PA.

// One attempt t of query q: true and the grounded registers when accepted.
__device__ __forceinline__ bool pos_attempt(const GraphView& g, const WalkProgram& wp,
                                            const SampleParams& p, uint32_t q, int t, int32_t* e,
                                            int32_t* qr)
{
    e[0] = e[1] = e[2] = e[3] = e[4] = -1;
    qr[0] = qr[1] = qr[2] = -1;
    if (g.n_active == 0) return false;
    e[0] = g.active_in[reduce_range(draw64(p.seed, TAG_POS, q, t, 0), (uint32_t)g.n_active)];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        if (k >= wp.n_steps) break;
        const bool sib = wp.neg_steps > 0 && k == wp.neg_first;
        const int after = wp.neg_steps > 0 && k >= wp.neg_first ? 1 : 0;
        if (sib) {
            // sibling entity of the complemented operand: uniform over
            // A_r(x) of step sib_step, a list that holds that step's entity
            const int32_t x = reg5(wp.sib_step + 1, e);
            const int32_t r = sel4(wp.sib_step, qr[0], qr[1], qr[2], -1);
            const int2 fr = group_range(g.fwd, x, r);
            if (fr.y == fr.x) return false;
            const uint64_t u = draw64(p.seed, TAG_POS, q, t, 1 + 2 * k);
            e[WALK_SIB] = g.fwd.nbr[fr.x + (int32_t)reduce_range(u, (uint32_t)(fr.y - fr.x))];
        }
        const int32_t v = reg5(wp.src[k], e);
        const uint64_t u0 = draw64(p.seed, TAG_POS, q, t, 1 + 2 * k + after);
        const uint64_t u1 = draw64(p.seed, TAG_POS, q, t, 2 + 2 * k + after);
        const int32_t s0 = g.rev.node[v], s1 = g.rev.node[v + 1];
        if (s0 == s1) return false;                       // no in-edge: dead end
        const int32_t s = s0 + (int32_t)reduce_range(u0, (uint32_t)(s1 - s0));
        const int2 gr = g.rev.grp[s];
        const int32_t len = g.rev.grp[s + 1].y - gr.y;
        const int32_t x = g.rev.nbr[gr.y + (int32_t)reduce_range(u1, (uint32_t)len)];
        if (p.max_fanout > 0) {
            const int2 fr = group_range(g.fwd, x, gr.x);
            if (fr.y - fr.x > p.max_fanout) return false;
        }
        e[k + 1] = x;
        qr[k] = gr.x;
    }
    for (int pr = 0; pr < wp.n_pairs; ++pr) {
        const int32_t xa = reg5(wp.anchor_reg[wp.pair_anchor[pr][0]], e);
        const int32_t xb = reg5(wp.anchor_reg[wp.pair_anchor[pr][1]], e);
        const int32_t ra = slot_rel(wp, qr, wp.pair_rel[pr][0]);
        const int32_t rb = slot_rel(wp, qr, wp.pair_rel[pr][1]);
        if (xa == xb && ra == rb) return false;           // degenerate sibling branches
    }
    if (wp.neg_steps > 0) {   // the intersection's entity must stay outside the complemented set
        const int32_t a = reg5(wp.anchor_reg[wp.neg_anchor], e);
        const int32_t r0 = slot_rel(wp, qr, wp.neg_rel[0]);
        const int32_t r1 = wp.neg_steps > 1 ? slot_rel(wp, qr, wp.neg_rel[1]) : -1;
        if (neg_member(g, wp.neg_steps, a, r0, r1, reg5(wp.neg_target, e))) return false;
    }
    return true;
}

// --------------------------------------------------------------- negatives
// Lists per shape (anchor slot, relation slot) at the cut the planner picks:
//   1p {a0}, 2p/3p {V1}, 2i/3i/2u/2in/3in {anchors}, ip/up/inp {Y0, Y1},
//   pi/pin {V1, a1}, pni {V1 of the complemented chain, a1}.
// cached = forward caching to the cut (A_r(a) at a cut node one projection
// above the anchor); otherwise the list is the anchor's neighbour list used
// for an edge test at a cut placed on the anchor, which may be decided from
// either end of the edge.  n_anc / n_rel: slots the shape uses.
template <int QT> struct Shape;
#define SHAPE(Q, NF, NA, NR, A0, A1, A2, R0, R1, R2, C0, C1, C2)                                 \
    template <> struct Shape<Q> {                                                              \
        static constexpr int nf = NF, n_anc = NA, n_rel = NR;                                  \
        static constexpr int fa[3] = {A0, A1, A2}, fr[3] = {R0, R1, R2}, cached[3] = {C0, C1, C2}; \
    };
SHAPE(Q1P, 1, 1, 1, 0, 0, 0, 0, 0, 0, 0, 0, 0)
SHAPE(Q2P, 1, 1, 2, 0, 0, 0, 0, 0, 0, 1, 0, 0)
SHAPE(Q3P, 1, 1, 3, 0, 0, 0, 0, 0, 0, 1, 0, 0)
SHAPE(Q2I, 2, 2, 2, 0, 1, 0, 0, 1, 0, 0, 0, 0)
SHAPE(Q3I, 3, 3, 3, 0, 1, 2, 0, 1, 2, 0, 0, 0)
SHAPE(QIP, 2, 2, 3, 0, 1, 0, 0, 1, 0, 1, 1, 0)
SHAPE(QPI, 2, 2, 3, 0, 1, 0, 0, 2, 0, 1, 0, 0)
SHAPE(Q2U, 2, 2, 2, 0, 1, 0, 0, 1, 0, 0, 0, 0)
SHAPE(QUP, 2, 2, 3, 0, 1, 0, 0, 1, 0, 1, 1, 0)
SHAPE(Q2IN, 2, 2, 2, 0, 1, 0, 0, 1, 0, 0, 0, 0)
SHAPE(Q3IN, 3, 3, 3, 0, 1, 2, 0, 1, 2, 0, 0, 0)
SHAPE(QINP, 2, 2, 3, 0, 1, 0, 0, 1, 0, 1, 1, 0)
SHAPE(QPIN, 2, 2, 3, 0, 1, 0, 0, 2, 0, 1, 0, 0)
SHAPE(QPNI, 2, 2, 3, 0, 1, 0, 0, 2, 0, 1, 0, 0)
#undef SHAPE

// Shapes whose last step into the root is the backward step of a two-hop
// chain under relation slot 1 (else slot 2), and shapes whose second list
// is a forward-cached set the deep test needs staged.
template <int QT> constexpr bool chain_r1 = QT == Q2P || QT == QPI || QT == QPIN || QT == QPNI;
template <int QT> constexpr bool two_cached = QT == QIP || QT == QUP || QT == QINP;
// Shapes with a backward step that can meet a long list (the others decide
// every candidate by edge tests).
template <int QT> constexpr bool has_long_lists = QT == Q2P || QT == Q3P || QT == QPI || QT == QPIN ||
                                                  QT == QPNI || two_cached<QT>;

// Lists that test a candidate by one edge into the root: c is an answer
// only if c is in list f for every f of `mask` (any f when `any`).  When
// these lists are staged in LDS they decide the draws without a single
// graph read; otherwise the in-edge mask does.
// Relation slots of the projections that end at the root (bit s: slot s),
// positive operands only: an answer has an in-edge under each of them (any
// one of them for a union).
template <int QT> struct RootRels { static constexpr int mask = 0, any = 0; };
template <> struct RootRels<Q1P> { static constexpr int mask = 1, any = 0; };
template <> struct RootRels<Q2P> { static constexpr int mask = 2, any = 0; };
template <> struct RootRels<Q3P> { static constexpr int mask = 4, any = 0; };
template <> struct RootRels<Q2I> { static constexpr int mask = 3, any = 0; };
template <> struct RootRels<Q3I> { static constexpr int mask = 7, any = 0; };
template <> struct RootRels<QIP> { static constexpr int mask = 4, any = 0; };
template <> struct RootRels<QPI> { static constexpr int mask = 6, any = 0; };
template <> struct RootRels<Q2U> { static constexpr int mask = 3, any = 1; };
template <> struct RootRels<QUP> { static constexpr int mask = 4, any = 0; };
template <> struct RootRels<Q2IN> { static constexpr int mask = 1, any = 0; };
template <> struct RootRels<Q3IN> { static constexpr int mask = 3, any = 0; };
template <> struct RootRels<QINP> { static constexpr int mask = 4, any = 0; };
template <> struct RootRels<QPIN> { static constexpr int mask = 2, any = 0; };
template <> struct RootRels<QPNI> { static constexpr int mask = 4, any = 0; };

template <int QT> struct RootLists { static constexpr int mask = 0, any = 0; };
template <> struct RootLists<Q1P> { static constexpr int mask = 1, any = 0; };
template <> struct RootLists<Q2I> { static constexpr int mask = 3, any = 0; };
template <> struct RootLists<Q3I> { static constexpr int mask = 7, any = 0; };
template <> struct RootLists<QPI> { static constexpr int mask = 2, any = 0; };
template <> struct RootLists<Q2U> { static constexpr int mask = 3, any = 1; };
// with negation, only the positive operands' lists are necessary conditions
template <> struct RootLists<Q2IN> { static constexpr int mask = 1, any = 0; };
template <> struct RootLists<Q3IN> { static constexpr int mask = 3, any = 0; };
template <> struct RootLists<QPNI> { static constexpr int mask = 2, any = 0; };

// The candidate kernel runs one wavefront and one query per workgroup: queries
// differ widely in cost, and the hardware dispatcher hands each freed slot the
// next query, where a fixed share per wavefront leaves the kernel waiting on
// its slowest shares.
constexpr int CWG = 64;
constexpr int HEAVY_WG = 256;    // threads of the heavy-queue workgroups
constexpr int QF = 8;            // int32 per query in the per-query block
constexpr int PERSIST_BLOCKS = 2048;
constexpr int FINISH_WAVES = 4096;    // wavefronts of the finishing kernel: as many as run at once
// 3p long-list work in bounded units: the long-list kernel expands at most
// UNIT_Y entities y of an item and searches at most UNIT_PAIRS pairs of one
// y itself; the rest become units of the unit queue (UNITS_PER_QUERY slots
// per query), which the unit kernel then takes, so one huge item is spread
// over many wavefronts instead of setting the kernel's length alone.
constexpr int UNIT_Y = 256;
constexpr int UNIT_PAIRS = 1024;
constexpr int UNITS_PER_QUERY = 64;

// Workspace carved out of the caller's buffer.
struct Ws {
    int32_t* ctrl;    // [0] queue pushes [2] queries to finish [5] 3p units pushed
    int32_t* qf;      // [B][QF]: list k at [2k, 2k+1) edge range; [6] bit k: list k staged,
                      // [7] the draws of a query to finish, [4] (where no third list
                      // is) how many of them are non-answers and how many pending
    uint8_t* status;  // [B][neg_tries] ST_*
    int32_t* act[2];  // [0] queries to finish [1] by query: negatives selected so far (and from
                      // bit 16 on the finishing workgroups that are done with its first range)
    int2* queue;      // (query, draw) items
    int64_t qcap;
    int4* units;      // 3p long-list units: (item, a, b, kind), counted by ctrl[5]
    int64_t ucap;
};

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Candidate j of query b: draw j of the query's own stream, pick(U(NEG, q,
// 0, j), V) with q = query_offset + b (Sec. 3.2: candidates uniform over the
// entities), or entry j of the caller's list or the shared set, -1 when it
// is not an entity.  Every kernel that needs a candidate takes it from here,
// so the draws are recomputed where they are used instead of being stored
// and read back.
__device__ __forceinline__ int32_t candidate(const SampleParams& p, int32_t V, int32_t b, int32_t j)
{
    if (p.shared_mode != 0) {
        const int32_t c = p.shared[(int64_t)p.cand_stride * b + j];
        return (uint32_t)c >= (uint32_t)V ? -1 : c;
    }
    const uint32_t q = (uint32_t)(p.query_offset + (uint64_t)b);
    return (int32_t)reduce_range(draw64(p.seed, TAG_NEG, q, 0, (uint32_t)j), (uint32_t)V);
}

// Rounds of candidate draws.  A query first takes n_neg draws plus a small
// margin (a query rarely rejects more than a few percent of its draws).  One
// still short of n_neg then takes its own next range: the draws its deficit
// needs at the acceptance rate it has had so far, with a margin
// (next_round_end).  Rounds are a scheduling detail: a query's negatives are
// its first n_neg accepted draws in draw order whatever the rounds were.
constexpr int WIN = 576;   // draws of a window
inline int32_t first_margin(const SampleParams& p)
{
    const int64_t e = (int64_t)p.n_neg + p.n_neg / 32 + 8;
    return (int32_t)(e < p.neg_tries ? e : p.neg_tries);
}

// Entries per query of the long-list queue.
inline int32_t max_round_len(const SampleParams& p)
{
    const int32_t e0 = first_margin(p);
    return e0 > p.neg_tries - e0 ? e0 : p.neg_tries - e0;
}

// A batch under 4,096 queries does not fill the GPU's wavefronts, and its
// time is that of its slowest ones: there the first round fills its last 64
// draws up, and takes 64 more where fewer than 16 would be left to add, so
// that fewer queries need another chain of dependent reads.  Above, the draws
// themselves are the cost.  A round that fits one window stays in it (n_neg
// 537 to 551: with 640 draws the selection table is one of its own, which
// leaves a CU nine wavefronts in place of 16).  The queue has to hold the round.
inline int32_t first_round(const SampleParams& p)
{
    const int32_t e = first_margin(p);
    if (p.batch >= 4096) return e;
    int32_t full = (e + 16 + 63) / 64 * 64;
    if (e <= WIN) full = min(full, WIN);
    return max(e, min(full, min(p.neg_tries, max_round_len(p))));
}

// End of the next range of a query that has `kept` accepted draws among its
// first `end`: the deficit over that acceptance rate, a quarter more, and
// 16 draws; everything up to neg_tries when nothing was accepted yet.
__device__ __forceinline__ int32_t next_round_end(const SampleParams& p, int32_t end, int32_t kept)
{
    if (kept <= 0) return p.neg_tries;
    const int64_t need = (int64_t)(p.n_neg - kept) * end;
    const int64_t more = (need * 5 + 4 * (int64_t)kept - 1) / (4 * (int64_t)kept) + 16;
    return (int32_t)(end + more < p.neg_tries ? end + more : p.neg_tries);
}

// The draws a query leaves to the finishing kernel, kept in its per-query
// block (two 16-bit draw indices).
static_assert(SMORE_MAX_NEG_TRIES < 65536, "draw indices must fit 16 bits");
__host__ __device__ __forceinline__ int32_t pack_range(int32_t a, int32_t b) { return a | (b << 16); }
__host__ __device__ __forceinline__ int32_t range_lo(int32_t r) { return r & 0xFFFF; }
__host__ __device__ __forceinline__ int32_t range_hi(int32_t r) { return (int32_t)((uint32_t)r >> 16); }

// The draw at which a query's row is likely to be full, given the non-answers
// `non`, answers `ans` and pending candidates `pend` of its first `base` draws:
// base when these should do.  Where answers were met, the pending ones are
// taken for answers mostly.  n_neg distinct non-answers of V * a take
// -V ln(1 - n_neg / (V a)) draws.
__device__ __forceinline__ int32_t likely_end(const SampleParams& p, int32_t V, int32_t base, int32_t non,
                                              int32_t ans, int32_t pend)
{
    const float a = ((float)non + (float)pend / (float)(ans + 1)) / (float)base;
    const float x = (float)p.n_neg / ((float)V * a);
    if (!(x < 0.99f)) return p.neg_tries;
    const float d = -(float)V * log1pf(-x);
    if (d <= (float)base) return base;
    return d * 1.1f + 16.0f < (float)p.neg_tries ? (int32_t)(d * 1.1f) + 16 : p.neg_tries;
}

size_t ws_layout(const SampleParams& p, Ws* w, char* base)
{
    const int64_t B = p.batch, T = p.neg_tries > 0 ? p.neg_tries : 1;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char* ptr = base ? base + off : nullptr;
        off += align256(bytes);
        return ptr;
    };
    Ws x;
    x.ctrl = (int32_t*)take(64 * sizeof(int32_t));
    x.qf = (int32_t*)take((size_t)B * QF * sizeof(int32_t));
    x.status = (uint8_t*)take((size_t)B * T);
    x.act[0] = (int32_t*)take((size_t)B * sizeof(int32_t));
    x.act[1] = (int32_t*)take((size_t)B * sizeof(int32_t));
    x.qcap = B * (int64_t)max_round_len(p);
    x.queue = (int2*)take((size_t)x.qcap * sizeof(int2));
    x.ucap = B * (int64_t)UNITS_PER_QUERY;
    x.units = (int4*)take((size_t)x.ucap * sizeof(int4));
    if (w) *w = x;
    return off;
}

// Tally of one lane summed over its wavefront and added to the query's
// counters (the wavefront must be converged).
template <class T>
__device__ __forceinline__ void flush_tally(T& tl, int64_t* stats, int32_t b, int lane, int slot = 0)
{
    if constexpr (T::on) {
        uint64_t x = tl.b, y = tl.l;
        for (int s = 32; s > 0; s >>= 1) {
            x += __shfl_xor(x, s);
            y += __shfl_xor(y, s);
        }
        if (lane == 0 && (x | y)) {
            atomicAdd((unsigned long long*)&stats[4 * (int64_t)b + slot], (unsigned long long)x);
            atomicAdd((unsigned long long*)&stats[4 * (int64_t)b + slot + 1], (unsigned long long)y);
        }
        tl.b = tl.l = 0;
    }
}

// LDS of one wavefront of the candidate kernels.  Staged lists keep their
// order in `stage` and have a hashed bit set each in bits() (split evenly
// between the shape's lists): a value whose bit is clear is not in the list,
// so one LDS read settles nearly every lookup, and only the others bisect
// the list.  The sizes keep it at 10,240 bytes, eight of the 1,280-byte units
// that LDS is given out in: 16 wavefronts per CU, as their registers allow.
constexpr int DPW = WIN / 64;
constexpr int WORDS = WIN / 32;
constexpr int DEEPQ = 192;       // deep items held before a pass over 64 of them: 63 + one step of 128
constexpr int BIT_WORDS = 256;
struct alignas(16) WaveLds {
    int32_t stage[STAGE + BIT_WORDS];   // the lists, their bits after them; or the selection table
    int32_t cand[WIN];      // the window's candidates (complemented: left to the long-list kernels)
    int32_t ds[DEEPQ];      // deep items: start of the backward list
    uint16_t dl[DEEPQ];     //             its length, at most 65,535
    uint16_t dj[DEEPQ];     //             index in the window
    uint16_t sj[WIN];       // survivors of the first test: index in the window
    uint32_t non[WORDS];    // bit i: candidate i is a non-answer
    __device__ __forceinline__ uint32_t* bits() { return (uint32_t*)stage + STAGE; }
    __device__ __forceinline__ const uint32_t* bits() const { return (const uint32_t*)stage + STAGE; }
};

static_assert(sizeof(WaveLds) <= 10240, "LDS of a wavefront");

// A query's forward-cached list: edges [beg, beg + n), and where it is staged.
struct FList {
    int32_t beg, n, off;
    bool lds;
};

// log2 of the bits per list
template <int QT> constexpr int bit_log = Shape<QT>::nf == 1 ? 13 : Shape<QT>::nf == 2 ? 12 : 11;
template <int QT> __device__ __forceinline__ uint32_t bit_slot(int f, int32_t x)
{
    return ((uint32_t)f << bit_log<QT>) | (((uint32_t)x * 0x9E3779B1u) >> (32 - bit_log<QT>));
}
template <int QT> __device__ __forceinline__ bool maybe_in(const WaveLds& L, int f, int32_t x)
{
    const uint32_t h = bit_slot<QT>(f, x);
    return L.bits()[h >> 5] >> (h & 31) & 1u;
}

// Is x in the staged list F?
__device__ __forceinline__ bool in_stage(const WaveLds& L, const FList& F, int32_t x)
{
    int32_t lo = F.off, hi = F.off + F.n;
    while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if (L.stage[mid] < x) lo = mid + 1; else hi = mid;
    }
    return lo < F.off + F.n && L.stage[lo] == x;
}

// Is x in the sorted list p[0..n)?  Seven probes per step where eight or
// more entries remain: a third of the dependent reads of a bisection.
template <class T>
__device__ __forceinline__ bool has8(const int32_t* p, int32_t n, int32_t x, bool count, T& tl)
{
    while (n >= 8) {
        const int32_t q = n >> 3;
        int32_t v[7], c = 0;
#pragma unroll
        for (int k = 0; k < 7; ++k) {
            v[k] = p[q * (k + 1)];
            if (count) tl.read(p + q * (k + 1), 4);
        }
#pragma unroll
        for (int k = 0; k < 7; ++k) c += v[k] <= x;
        p += q * c;
        n = c == 7 ? n - 7 * q : q;
    }
    bool hit = false;
#pragma unroll
    for (int k = 0; k < 7; ++k) {
        if (k < n) {
            if (count) tl.read(p + k, 4);
            hit = hit || p[k] == x;
        }
    }
    return hit;
}

// Membership in list f.  The list is accounted once per query when it is
// cached; lookups in it are not graph traffic of the method, wherever the
// list lives.
template <int QT>
__device__ __forceinline__ bool in_list(const GraphView& g, const WaveLds& L, const FList* F, int f,
                                        int32_t x)
{
    NoTally none;
    if (F[f].lds) return maybe_in<QT>(L, f, x) && in_stage(L, F[f], x);
    return has8(g.fwd.nbr + F[f].beg, F[f].n, x, false, none);
}

// Is (a, r, c) an edge?  From the anchor's list (f) when it is staged,
// otherwise from c's reverse list under r (c's node pair already loaded).
template <int QT, class T>
__device__ __forceinline__ bool edge_test(const GraphView& g, const WaveLds& L, const FList* F, int f,
                                          int32_t a, int32_t r, int32_t c, int32_t n0, int32_t n1, T& tl)
{
    if (F[f].lds) return maybe_in<QT>(L, f, c) && in_stage(L, F[f], c);
    const int2 s = group_find(g.rev, n0, n1, r, tl);
    return s.y > s.x && has8(g.rev.nbr + s.x, s.y - s.x, a, true, tl);
}

// Decision of a shape made of edge tests alone.
template <int QT, class T>
__device__ __forceinline__ int32_t edges_decide(const GraphView& g, const WaveLds& L, const FList* F,
                                                const int32_t* anc, const int32_t* rel, int32_t c,
                                                int32_t n0, int32_t n1, T& tl)
{
    auto edge = [&](int f) { return edge_test<QT>(g, L, F, f, anc[f], rel[f], c, n0, n1, tl); };
    bool ans = edge(0);
    if (QT == Q2I || QT == Q3I || QT == Q3IN) ans = ans && edge(1);
    if (QT == Q2U) ans = ans || edge(1);
    if (QT == Q2IN) ans = ans && !edge(1);
    if (QT == Q3I) ans = ans && edge(2);
    if (QT == Q3IN) ans = ans && !edge(2);
    return ans ? ST_ANS : ST_NON;
}

// First, shallow decision of two candidates c[0], c[1] (act[u]: slot in use)
// at lane level, with the dependent steps of both interleaved: ST_NON or
// ST_ANS when it is settled by the cached lists and c's own groups, else
// ST_DEEP with c's backward list [lst.x, lst.y).
template <int QT, class T>
__device__ __forceinline__ void shallow_test2(const GraphView& g, const WaveLds& L, const FList* F,
                                              const int32_t* anc, const int32_t* rel, const int32_t* c,
                                              const bool* act, int32_t* st, int2* lst, T& tl)
{
    int32_t n0[2], n1[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        n0[u] = n1[u] = 0;
        if (act[u]) {
            n0[u] = g.rev.node[c[u]];
            n1[u] = g.rev.node[c[u] + 1];
            tl.read(g.rev.node + c[u], 8);
        }
    }
    if constexpr (!has_long_lists<QT>) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
            st[u] = act[u] ? edges_decide<QT>(g, L, F, anc, rel, c[u], n0[u], n1[u], tl) : ST_NON;
        return;
    }
    bool live[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        live[u] = act[u];
        if (QT == QPI || QT == QPNI || QT == QPIN) {
            const bool e = act[u] && edge_test<QT>(g, L, F, 1, anc[1], rel[2], c[u], n0[u], n1[u], tl);
            live[u] = act[u] && (QT == QPIN ? !e : e);
        }
    }
    const int32_t rb = chain_r1<QT> ? rel[1] : rel[2];
    int2 sr[2];
    group_find2(g.rev, n0, n1, live, rb, sr, tl);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        st[u] = ST_NON;
        if (!live[u]) continue;
        if (sr[u].y == sr[u].x) {
            if (QT == QPNI) st[u] = ST_ANS;   // nothing reaches c through the complemented chain
        } else {
            lst[u] = sr[u];
            st[u] = ST_DEEP;
        }
    }
}

// Highest lane whose exclusive prefix excl is <= idx (binary lifting over
// the wavefront; every lane must be active).  excl is nondecreasing over
// the lanes and 0 in lane 0.
__device__ __forceinline__ int owner_lane(int32_t idx, int32_t excl)
{
    int lo = 0;
#pragma unroll
    for (int step = 32; step >= 1; step >>= 1) {
        const int cand = lo + step;
        const int32_t ev = __shfl(excl, cand > 63 ? 63 : cand);
        if (cand <= 63 && ev <= idx) lo = cand;
    }
    return lo;
}

__device__ __forceinline__ int32_t excl_prefix(int32_t v, int lane, int32_t* total)
{
    int32_t incl = v;
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t t = __shfl_up(incl, d);
        if (lane >= d) incl += t;
    }
    *total = uni(__shfl(incl, 63));
    return incl - v;
}

// The deep pass over up to 64 candidates, one per lane: lane l's candidate
// has the backward list [start, start + len) (len 0: none).  Returns the
// lanes whose chain meets the cached lists, and in *pend those left to a
// whole wavefront.  All (entry, list) pairs to test are laid out over the
// lanes, with keys from the shorter of the backward list and the cached one
// (for 3p the entries y of all lists 64 at a time, and of each 64 the pairs
// of R_r1(y) and F0), so the dependent reads of the pass are those of its
// deepest candidate, not the sum over a lane's entries (one lane walking its
// own list: 172 + 77 us in two rounds for 512 3p queries x 128 on an
// FB15k-237-shaped graph; laid out: 67 us for all draws).  A candidate with
// over DEEP_LONG pairs, or past DEEP_TOTAL pairs of the pass, is left, and
// so is everything once the query has taken DEEP_STEPS steps (`steps` counts
// them down): a wavefront of its own (or, for 3p, several) shortens the
// longest wavefront of the call.  48 steps: 3p x 1,000 negatives on an
// FB400k-shaped graph 360 us a call, the FB15k-237-shaped step 385; 12: 301
// and 379; 4: 312 and 508.  Two pairs per lane and step pay for the short
// chains of the other shapes (FB400k-shaped 2p 87 -> 69 us with the keys
// from the shorter list), not for 3p (Freebase-shaped step 618 against 604).
constexpr int DEEP_LONG = 512, DEEP_TOTAL = 4096, DEEP_STEPS = 12;
constexpr int DEEP_LEN = 65535;   // lengths are kept in 16 bits; one that long is left

// Drops from np the candidates the pass leaves (all but `cap` pairs of it);
// returns the lanes dropped.
__device__ __forceinline__ uint64_t deep_limit(int32_t& np, int32_t cap, int lane)
{
    bool over = np > DEEP_LONG;
    if (over) np = 0;
    int32_t tot;
    const int32_t ex = excl_prefix(np, lane, &tot);
    if (tot > cap) {
        over = over || (np > 0 && ex + np > cap);
        if (over) np = 0;
    }
    return __ballot(over);
}

// Bits of the owners of the lanes where `hit` holds.
__device__ __forceinline__ uint64_t owners_of(bool hit, int owner)
{
    uint64_t m = __ballot(hit), res = 0;
    while (m) {
        res |= 1ull << readlane(owner, __ffsll((unsigned long long)m) - 1);
        m &= m - 1;
    }
    return res;
}

// Entry off of the list p[0..len), read by one lane of a step whose next
// lanes read the entries after it: accounted once per run of lanes, by the
// lane that holds the list's first entry or starts the step.
template <class T>
__device__ __forceinline__ void tally_run(T& tl, const int32_t* p, int32_t off, int32_t len, int lane)
{
    if (off == 0 || lane == 0) tl.read(p + off, 4 * min(len - off, 64 - lane));
}

// Entry k of list f.
__device__ __forceinline__ int32_t list_entry(const GraphView& g, const WaveLds& L, const FList& F, int32_t k)
{
    return F.lds ? L.stage[F.off + k] : g.fwd.nbr[F.beg + k];
}

// The 3p pass over candidates with at most two entities y each, none of them
// with more than two pairs: each lane takes its own, four lists side by side
// and no layout.  Returns false, and nothing else, for other candidates.
template <int QT>
__device__ __forceinline__ bool short_pass3(const GraphView& g, const WaveLds& L, const FList* F,
                                            const int32_t* rel, int32_t start, int32_t len, uint64_t* ans)
{
    if (__ballot(len > 2)) return false;
    NoTally none;
    const int32_t nf = F[0].n;
    const uint32_t b1 = sig_bit(rel[1]);
    int32_t y[2] = {0, 0}, n0[2] = {0, 0}, n1[2] = {0, 0};
    bool on[2];
    int2 s[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        on[k] = k < len;
        if (on[k]) y[k] = g.rev.nbr[start + k];
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        if (!on[k]) continue;
        n0[k] = g.rev.node[y[k]];
        n1[k] = g.rev.node[y[k] + 1];
        on[k] = (g.sig[y[k]] & b1) != 0;   // else no in-edge under r1
    }
    group_find2(g.rev, n0, n1, on, rel[1], s, none);
    if (__ballot(min(s[0].y - s[0].x, nf) > 2 || min(s[1].y - s[1].x, nf) > 2)) return false;
    bool hit = false;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int32_t n2 = s[k].y - s[k].x;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (i >= min(n2, nf)) continue;
            if (n2 <= nf) hit = hit || in_list<QT>(g, L, F, 0, g.rev.nbr[s[k].x + i]);
            else hit = hit || has8(g.rev.nbr + s[k].x, n2, list_entry(g, L, F[0], i), false, none);
        }
    }
    *ans = __ballot(hit);
    return true;
}

template <int QT, class T>
__device__ __forceinline__ uint64_t deep_pass(const GraphView& g, const WaveLds& L, const FList* F,
                                              const int32_t* rel, int32_t start, int32_t len, int lane,
                                              int32_t cap, int32_t& steps, uint64_t* pend, T& tl)
{
    uint64_t left = 0, ans = 0;
    if constexpr (QT != Q3P) {
        // keys of a list longer than the cached ones: their entries (both
        // for a union of chains)
        const int32_t nf = QT == QUP ? F[0].n + F[1].n : F[0].n;
        int32_t np = len >= DEEP_LEN ? INT_MAX : min(len, nf);
        left = deep_limit(np, cap, lane);
        int32_t total;
        const int32_t ex = excl_prefix(np, lane, &total);
        for (int32_t p0 = 0; p0 < total; p0 += 128) {
            if (--steps < 0) {   // the candidates that reach past pair p0
                left |= __ballot(np > 0 && ex + np > p0);
                break;
            }
            bool on[2], hit[2];
            int it[2];
            int32_t off[2], st[2], ln[2], y[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int32_t pi = p0 + 64 * u + lane;
                on[u] = pi < total;
                it[u] = owner_lane(min(pi, total - 1), ex);
                off[u] = pi - __shfl(ex, it[u]);
                st[u] = __shfl(start, it[u]);
                ln[u] = __shfl(len, it[u]);
                hit[u] = false;
                y[u] = -1;
                if (on[u]) {
                    if (ln[u] <= nf) {
                        y[u] = g.rev.nbr[st[u] + off[u]];
                        tally_run(tl, g.rev.nbr + st[u], off[u], ln[u], lane);
                    } else if (QT == QUP && off[u] >= F[0].n) {
                        y[u] = list_entry(g, L, F[1], off[u] - F[0].n);
                    } else {
                        y[u] = list_entry(g, L, F[0], off[u]);
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (!on[u]) continue;
                if (ln[u] <= nf) {
                    hit[u] = in_list<QT>(g, L, F, 0, y[u]);
                    if (QT == QUP) hit[u] = hit[u] || in_list<QT>(g, L, F, 1, y[u]);
                } else {
                    hit[u] = has8(g.rev.nbr + st[u], ln[u], y[u], true, tl);
                }
                if (QT == QIP) hit[u] = hit[u] && in_list<QT>(g, L, F, 1, y[u]);
                if (QT == QINP) hit[u] = hit[u] && !in_list<QT>(g, L, F, 1, y[u]);
            }
            ans |= owners_of(hit[0], it[0]) | owners_of(hit[1], it[1]);
        }
    } else {
        left = deep_limit(len, cap, lane);
        int32_t total;
        const int32_t ex = excl_prefix(len, lane, &total);
        const uint32_t b1 = sig_bit(rel[1]);
        const int32_t nf = F[0].n;
        for (int32_t y0 = 0; y0 < total; y0 += 64) {
            if (--steps < 0) {
                left |= __ballot(len > 0 && ex + len > y0);
                break;
            }
            const bool on = y0 + lane < total;
            const int it = owner_lane(min(y0 + lane, total - 1), ex);
            const int32_t yat = y0 + lane - __shfl(ex, it), at = __shfl(start, it) + yat;
            const int32_t ylen = __shfl(len, it);
            int2 s2 = make_int2(0, 0);
            if (on && !((ans | left) >> it & 1)) {
                // y without an in-edge under r1's signature class has none under r1
                const int32_t y = g.rev.nbr[at];
                tally_run(tl, g.rev.nbr + at - yat, yat, ylen, lane);
                tl.read(g.sig + y, 1);
                const int32_t a0 = g.rev.node[y], a1 = g.rev.node[y + 1];
                if (g.sig[y] & b1) {
                    tl.read(g.rev.node + y, 8);
                    s2 = group_find(g.rev, a0, a1, rel[1], tl);
                }
            }
            const int32_t n2 = s2.y - s2.x;
            int32_t np = min(n2, nf);
            const uint64_t over = deep_limit(np, cap, lane);
            if (over) left |= owners_of(over >> lane & 1, it);
            int32_t ptotal;
            const int32_t pex = excl_prefix(np, lane, &ptotal);
            for (int32_t p0 = 0; p0 < ptotal; p0 += 64) {
                if (--steps < 0) {
                    left |= owners_of(np > 0 && pex + np > p0, it);
                    break;
                }
                const int32_t pi = p0 + lane;
                const int yl = owner_lane(min(pi, ptotal - 1), pex);
                const int32_t off = pi - __shfl(pex, yl);
                const int32_t lx = __shfl(s2.x, yl), ln = __shfl(n2, yl);
                const int who = __shfl(it, yl);
                bool hit = false;
                if (pi < ptotal && !((ans | left) >> who & 1)) {
                    if (ln <= nf) {
                        tally_run(tl, g.rev.nbr + lx, off, ln, lane);
                        hit = in_list<QT>(g, L, F, 0, g.rev.nbr[lx + off]);
                    } else {
                        hit = has8(g.rev.nbr + lx, ln, list_entry(g, L, F[0], off), true, tl);
                    }
                }
                ans |= owners_of(hit, who);
            }
        }
    }
    *pend = left & ~ans;
    return ans;
}

// Wavefront decision for a queued candidate (the one-hop operand of
// pi / pin / pni has already been tested at lane level).
// s is the candidate's backward list under the last relation (wave-uniform).
template <int QT, class T>
__device__ bool heavy_test(const GraphView& g, const FSet* F, const int32_t* rel, int2 s, int lane,
                           T& tl)
{
    const int32_t* S = g.rev.nbr + s.x;
    const int32_t ns = s.y - s.x;
    if (QT == Q2P || QT == QPI || QT == QPIN) return wave_meet(S, ns, true, F[0].p, F[0].n, false, lane, tl);
    if (QT == QPNI) return !wave_meet(S, ns, true, F[0].p, F[0].n, false, lane, tl);
    if (QT == QIP) return wave_meet3(S, ns, F[0], F[1], lane, tl);
    if (QT == QINP) return wave_meet_minus(S, ns, F[0], F[1], lane, tl);
    if (QT == QUP)
        return wave_meet(S, ns, true, F[0].p, F[0].n, false, lane, tl) ||
               wave_meet(S, ns, true, F[1].p, F[1].n, false, lane, tl);
    return false;
}

__device__ __forceinline__ bool query_ok(const GraphView& g, const smore_sample_out& out, int32_t b,
                                         int n_anc, int n_rel, int32_t R, int32_t* anc, int32_t* rel)
{
    bool ok = !out.positive || out.positive[b] >= 0;   // verification has no positives
    for (int k = 0; k < 3; ++k) {
        rel[k] = out.relations[3 * (int64_t)b + k];
        anc[k] = out.anchors[3 * (int64_t)b + k];
        if (k < n_rel && (rel[k] < 0 || rel[k] >= R)) ok = false;
        if (k < n_anc && (anc[k] < 0 || anc[k] >= g.V)) ok = false;
    }
    return ok;
}

// Counters of a call: queued pairs, queries to finish, units.
__device__ __forceinline__ void reset_counters(const Ws& ws)
{
    ws.ctrl[0] = 0;
    ws.ctrl[2] = 0;
    ws.ctrl[5] = 0;
}

// The preparation of the negatives as part of the positives' kernel: the
// shape's lists (Shape), or nf = -1 for a call that only samples positives.
struct PrepLists {
    int32_t nf;
    int32_t fa[3], fr[3];
};

// Preparation of a query whose lists' edge ranges r are held by its lanes
// l = 0, 1, 2 (lane base + l of the wavefront): ranges, and the staging plan
// in list order.
__device__ __forceinline__ int32_t write_lists(int32_t* q, int2 r, int l, int base, int nf)
{
    if (l < nf) {
        q[2 * l] = r.x;
        q[2 * l + 1] = r.y;
    }
    int32_t used = 0, staged = 0;
    for (int k = 0; k < nf; ++k) {
        const int32_t n = __shfl(r.y - r.x, base + k);
        if (n <= STAGE - used) {
            staged |= 1 << k;
            used += n;
        }
    }
    if (l == 0) q[6] = staged;
    return staged;
}

// With a preparation to do, the lanes of a query share its winning row and
// look its lists up, lane l list l (the plan has at most PA): the chain of
// reads of k_prepare without its launch, which was 5 to 8 us of a call.
template <int PA>
__global__ __launch_bounds__(256) void k_positive(GraphView g, WalkProgram wp, SampleParams p,
                                                  smore_sample_out out, PrepLists lists, Ws ws)
{
    const int32_t gid = blockIdx.x * blockDim.x + threadIdx.x;
    const int32_t b = gid / PA;
    const int l = gid % PA;
    if (b >= p.batch) return;   // whole groups: PA divides the workgroup size
    const bool prepare = lists.nf >= 0;
    if (prepare && gid == 0) reset_counters(ws);
    const uint32_t q = (uint32_t)(p.query_offset + (uint64_t)b);
    const int gbase = (threadIdx.x & 63) & ~(PA - 1);
    int32_t e[5], qr[3];
    int win = -1;
    for (int t0 = 0; t0 < p.pos_tries; t0 += PA) {
        const int t = t0 + l;
        const bool ok = t < p.pos_tries && pos_attempt(g, wp, p, q, t, e, qr);
        const uint64_t m = (__ballot(ok) >> gbase) & (~0ull >> (64 - PA));
        if (m) {
            win = t0 + __ffsll((unsigned long long)m) - 1;
            break;
        }
    }
    int32_t A[3], R[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        A[k] = win >= 0 && k < wp.n_anchor ? reg5(wp.anchor_reg[k], e) : -1;
        R[k] = win >= 0 ? slot_rel(wp, qr, k) : -1;
    }
    if (l == (win < 0 ? 0 : win % PA)) {   // the lane that ran the winning attempt writes the row
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            out.anchors[3 * (int64_t)b + k] = A[k];
            out.relations[3 * (int64_t)b + k] = R[k];
        }
        out.positive[b] = win < 0 ? -1 : e[0];
        out.n_valid[b] = win < 0 ? -1 : 0;
        out.pos_attempts[b] = win < 0 ? p.pos_tries : win + 1;
    }
    if (!prepare) return;
    int32_t* qf = ws.qf + (int64_t)b * QF;
    if (win < 0) {
        if (l == 0) {
            write_undrawn_row(p, out, b, false);
            qf[6] = -1;   // skipped by the candidate kernel
        }
        return;
    }
    const int from = gbase + win % PA;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        A[k] = __shfl(A[k], from);
        R[k] = __shfl(R[k], from);
    }
    int2 r = make_int2(0, 0);
    if (l < lists.nf)
        r = group_range(g.fwd, sel4(lists.fa[l], A[0], A[1], A[2], -1), sel4(lists.fr[l], R[0], R[1], R[2], -1));
    write_lists(qf, r, l, gbase, lists.nf);
}

// Per query: validity, forward-cached lists, staging plan, for queries that
// the same call does not sample.
// Four neighbouring lanes per query: lane f looks up list f, so the
// dependent lookups of a query's lists run side by side; the staging plan
// is made from the sizes of all its lists, in list order.
template <int QT, class T>
__global__ __launch_bounds__(256) void k_prepare(GraphView g, SampleParams p, smore_sample_out out,
                                                 Ws ws, int64_t* stats, int32_t R)
{
    const int32_t gid = blockIdx.x * blockDim.x + threadIdx.x;
    const int32_t b = gid >> 2;
    const int f = gid & 3;
    if (b >= p.batch) return;   // whole groups: 4 divides the workgroup size
    if (gid == 0) reset_counters(ws);
    int32_t anc[3], rel[3];
    int32_t* q = ws.qf + (int64_t)b * QF;
    if (f == 0 && stats)
        for (int k = 0; k < 4; ++k) stats[4 * (int64_t)b + k] = 0;
    if (!query_ok(g, out, b, Shape<QT>::n_anc, Shape<QT>::n_rel, R, anc, rel)) {
        if (f == 0) {
            write_undrawn_row(p, out, b, false);
            q[6] = -1;   // skipped by the rounds
        }
        return;
    }
    T tl;
    int2 r = make_int2(0, 0);
    if (f < Shape<QT>::nf) r = group_range(g.fwd, anc[Shape<QT>::fa[f]], rel[Shape<QT>::fr[f]], tl);
    const int base = (threadIdx.x & 63) & ~3;
    const int32_t staged = write_lists(q, r, f, base, Shape<QT>::nf);
    (void)staged;
    if constexpr (T::on) {
        // forward caching reads the list once; a staged anchor list too
        if (f < Shape<QT>::nf && (Shape<QT>::cached[f] || (staged >> f & 1)))
            tl.read(g.fwd.nbr + r.x, 4 * (r.y - r.x));
        uint64_t x = tl.b, y = tl.l;
        x += __shfl_xor(x, 1);
        y += __shfl_xor(y, 1);
        x += __shfl_xor(x, 2);
        y += __shfl_xor(y, 2);
        if (f == 0) {
            stats[4 * (int64_t)b] = (int64_t)x;
            stats[4 * (int64_t)b + 1] = (int64_t)y;
        }
    }
}

// Calls with n_neg = 0 draw nothing: one thread per query writes its
// n_valid (0, or -1 for a skipped query), and for per-query sampling its
// draw count.  No workspace is read or written.
template <int QT>
__global__ __launch_bounds__(256) void k_no_draws(GraphView g, SampleParams p, smore_sample_out out,
                                                  int64_t* stats, int32_t R)
{
    const int32_t b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= p.batch) return;
    int32_t anc[3], rel[3];
    const bool ok = query_ok(g, out, b, Shape<QT>::n_anc, Shape<QT>::n_rel, R, anc, rel);
    write_undrawn_row(p, out, b, ok);
    if (stats)
        for (int k = 0; k < 4; ++k) stats[4 * (int64_t)b + k] = 0;
}

// The candidate kernels run one wavefront per query.  The query's lists are
// staged once into the wave's LDS slice.  Draws are taken a window of at
// most WIN at a time: every lane computes WIN / 64 draws and reads their
// in-edge bits (all loads in flight together); the draws with an in-edge are
// compacted into the wave's survivor list and then verified one per lane, so
// a window costs one dependent chain per 64 survivors instead of one per
// draw slot.  The window's candidates stay in LDS, its verdicts in one bit
// per draw, and the same wavefront selects the window's negatives.

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// First-occurrence table of the selection: tcap values in LDS, its own
// (own = 1) or over the staged lists and their bits.  At most 13/16 of it is
// filled: a window after the first holds that many draws less the values
// kept before it.
struct Table {
    int32_t tcap, own;
};
constexpr int TABLE_OVER = STAGE + BIT_WORDS;
__host__ __device__ __forceinline__ int32_t table_room(int32_t tcap) { return tcap / 16 * 13; }
__device__ __forceinline__ uint32_t table_slot(int32_t tcap, int32_t c)
{
    return __umulhi((uint32_t)c * 0x9E3779B1u, (uint32_t)tcap);
}
__device__ __forceinline__ uint32_t table_next(int32_t tcap, uint32_t h)
{
    return h + 1 == (uint32_t)tcap ? 0 : h + 1;
}

// Table holding the first acc negatives of a row (all its kept values).
__device__ __forceinline__ void table_fill(int32_t* tab, int32_t tcap, const int32_t* row, int32_t acc,
                                           int lane)
{
    for (int32_t k = 4 * lane; k < tcap; k += 256) *(int4*)(tab + k) = make_int4(-1, -1, -1, -1);
    if (acc > 0) {
        // rows are written by this wave, or by an earlier kernel
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    }
    wave_sync();
    for (int32_t k = lane; k < acc; k += 64) {
        const int32_t c = row[k];
        uint32_t h = table_slot(tcap, c);
        while (atomicCAS(&tab[h], -1, c) != -1) h = table_next(tcap, h);
    }
    wave_sync();
}

// Ordered selection over one window: candidate i < n (draw j0 + i) is kept
// iff it is a non-answer and no earlier draw had its value; the first n_neg
// kept are the row.  Answers never enter the table: a value has the same
// verdict at each of its draws.  A lane's first probes are in flight
// together, and only the values that met another one probe on.  Returns the
// row's length after the window.
__device__ __forceinline__ int32_t select_window(const SampleParams& p, const smore_sample_out& out,
                                                 int32_t b, WaveLds& L, int32_t* tab, int32_t tcap,
                                                 int32_t j0, int32_t n, int32_t acc, int lane)
{
    const uint64_t below = lanes_below(lane);
    int32_t* row = out.negatives + (int64_t)b * p.n_neg;
    uint32_t mine = 0, again = 0, todo = 0;   // bit k: candidate 64 k + lane
    {
        int32_t c[DPW], old[DPW];
#pragma unroll
        for (int k = 0; k < DPW; ++k) {
            c[k] = old[k] = -1;
            if (64 * k >= n) continue;
            const int32_t i = 64 * k + lane;
            if (i < n && (L.non[i >> 5] >> (i & 31) & 1u)) {
                c[k] = L.cand[i];
                const uint32_t h = table_slot(tcap, c[k]);
                old[k] = atomicCAS(&tab[h], -1, c[k]);
                L.sj[i] = (uint16_t)h;   // the survivor list is done with: slots of the values
            }
        }
#pragma unroll
        for (int k = 0; k < DPW; ++k) {
            if (c[k] < 0) continue;
            if (old[k] == -1) mine |= 1u << k;
            else if (old[k] == c[k]) again |= 1u << k;
            else todo |= 1u << k;
        }
    }
    while (todo) {
        const int k = __ffs(todo) - 1, i = 64 * k + lane;
        const int32_t c = L.cand[i];
        uint32_t h = L.sj[i];
        int32_t old;
        do {
            h = table_next(tcap, h);
            old = atomicCAS(&tab[h], -1, c);
        } while (old != -1 && old != c);
        L.sj[i] = (uint16_t)h;
        todo &= todo - 1;
        if (old == -1) mine |= 1u << k;
        else again |= 1u << k;
    }
    if (__ballot(again != 0)) {
        // some value was met again (rare): of the window's draws of a value
        // new to the table the first has it.  Slots of such values hold the
        // least draw of the value for a moment, as -2 - draw under a
        // maximum, which leaves the values of earlier windows alone.
        wave_sync();
        for (uint32_t m = mine; m; m &= m - 1) tab[L.sj[64 * (__ffs(m) - 1) + lane]] = INT_MIN;
        wave_sync();
        const uint32_t all = mine | again;
        for (uint32_t m = all; m; m &= m - 1) {
            const int i = 64 * (__ffs(m) - 1) + lane;
            atomicMax(&tab[L.sj[i]], -2 - i);
        }
        wave_sync();
        mine = 0;
        for (uint32_t m = all; m; m &= m - 1) {
            const int k = __ffs(m) - 1, i = 64 * k + lane;
            if (tab[L.sj[i]] == -2 - i) mine |= 1u << k;
        }
        wave_sync();
        for (uint32_t m = mine; m; m &= m - 1) {
            const int i = 64 * (__ffs(m) - 1) + lane;
            tab[L.sj[i]] = L.cand[i];
        }
        wave_sync();
    }
#pragma unroll
    for (int k = 0; k < DPW; ++k) {
        if (64 * k >= n) break;
        const bool kept = mine >> k & 1;
        const uint64_t keep = __ballot(kept);
        const int32_t rank = acc + __popcll(keep & below);
        if (kept && rank < p.n_neg) {
            row[rank] = L.cand[64 * k + lane];
            if (rank == p.n_neg - 1) out.neg_draws[b] = j0 + 64 * k + lane + 1;
        }
        acc = uni(min(p.n_neg, acc + __popcll(keep)));
    }
    return acc;
}

// Modes of the candidate kernels: the first kernel of a call, which leaves a
// query with long lists to the long-list kernels and the finishing kernel;
// and given candidates (shared or per query), whose verdicts are packed into
// mask rows.
enum : int { DRAW_FIRST = 0, DRAW_GIVEN = 1 };

// One query on one wavefront.
template <int QT, class T, int MODE>
__device__ __forceinline__ void query_draws(const GraphView& g, const SampleParams& p,
                                            const smore_sample_out& out, const Ws& ws, int64_t* stats,
                                            uint32_t* mask, const Table& tb, int32_t* own_tab,
                                            WaveLds& L, int32_t b, int32_t j_first, int lane)
{
    const uint64_t below = lanes_below(lane);
    const int32_t words = (p.n_neg + 31) >> 5;
    int32_t* qb = ws.qf + (int64_t)b * QF;
    const int32_t staged = uni(qb[6]);
    if (staged < 0) {   // query without a valid positive
        if constexpr (MODE == DRAW_GIVEN)
            for (int32_t k = lane; k < words; k += 64) mask[(int64_t)b * words + k] = 0;
        return;
    }
    int32_t anc[3], rel[3];
    for (int k = 0; k < 3; ++k) {
        anc[k] = uni(out.anchors[3 * (int64_t)b + k]);
        rel[k] = uni(out.relations[3 * (int64_t)b + k]);
    }
    T tl;
    FList F[3];
    int32_t used = 0;
#pragma unroll
    for (int f = 0; f < 3; ++f) {
        F[f] = FList{0, 0, 0, false};
        if (f >= Shape<QT>::nf) continue;
        F[f].beg = uni(qb[2 * f]);
        F[f].n = uni(qb[2 * f + 1]) - F[f].beg;
        F[f].lds = staged >> f & 1;
        F[f].off = used;
        if (F[f].lds) used += F[f].n;
    }
    // copy of the staged lists into the wave's LDS slice, with their bits
    auto stage_lists = [&]() {
        for (int k = lane; k < BIT_WORDS; k += 64) L.bits()[k] = 0;
        wave_sync();
#pragma unroll
        for (int f = 0; f < Shape<QT>::nf; ++f) {
            if (!F[f].lds) continue;
            for (int32_t k0 = lane; k0 < F[f].n; k0 += 256) {   // four loads in flight
                int32_t x[4];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    x[u] = k0 + 64 * u < F[f].n ? g.fwd.nbr[F[f].beg + k0 + 64 * u] : -1;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (k0 + 64 * u >= F[f].n) break;
                    const uint32_t h = bit_slot<QT>(f, x[u]);
                    L.stage[F[f].off + k0 + 64 * u] = x[u];
                    atomicOr(&L.bits()[h >> 5], 1u << (h & 31));
                }
            }
        }
        wave_sync();
    };
    uint8_t* sv = ws.status + (int64_t)b * p.neg_tries;
    int32_t* tab = tb.own ? own_tab : L.stage;
    // first test of every draw: the bits of the staged root-edge lists when
    // the shape has them (LDS only; the survivors are then looked up in the
    // lists), else the in-edge mask; in the latter case the lists are copied
    // while the first window's mask words are in flight
    constexpr int RM = RootLists<QT>::mask;
    const bool use_lists = RM != 0 && (RootLists<QT>::any ? (staged & RM) == RM : (staged & RM) != 0);
    // signature bits an answer must carry
    uint32_t need = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k)
        if (RootRels<QT>::mask >> k & 1) need |= sig_bit(rel[k]);
    int32_t acc = 0, base = 0, end = j_first, cnt = 0;
    bool deferred = false;
    int32_t non_left = 0, pend_left = 0;   // states of the draws that are left
    int32_t steps = DEEP_STEPS;
    int32_t jsel = 0;     // draws [0, jsel) are selected
    bool to_stage = used > 0;
    bool table = false;   // the table holds the row so far
    while (base < end) {
        const int32_t n = MODE == DRAW_GIVEN ? min(end - base, WIN)
                                             : min(end - base, min(WIN, table_room(tb.tcap) - acc));
        const int32_t stop = base + n;
        if (use_lists && to_stage) {
            stage_lists();
            to_stage = false;
        }
        // Every answer of every shape is reached by a projection, so a
        // draw without an in-edge is a non-answer, and so is one whose
        // in-relation signature (a byte per entity) lacks the classes of
        // the relations that end at the root.  Which array is read first
        // depends on what fits the L2 (g.first_test): the signatures
        // themselves, or a mask of the entities with an in-edge (one bit
        // per entity, or per four entities), after which only the draws it
        // passes read their signature.
        int32_t c[DPW];
        uint32_t word[DPW];
        const int test = use_lists ? -1 : g.first_test;
#pragma unroll
        for (int k = 0; k < DPW; ++k) {
            const int32_t j = base + k * 64 + lane;
            c[k] = -1;
            word[k] = 0;
            if (j < stop) {
                c[k] = candidate(p, g.V, b, j);   // -1 (given candidates only): never a negative
                if (c[k] >= 0) {
                    if (test == TEST_SIG) word[k] = g.sig[c[k]];
                    if (test == TEST_MASK) word[k] = g.has_in[c[k] >> 5] >> (c[k] & 31) & 1u;
                    if (test == TEST_MASK4) word[k] = g.has_in4[c[k] >> 7] >> (c[k] >> 2 & 31) & 1u;
                }
                L.cand[k * 64 + lane] = c[k];
            }
        }
        if (to_stage) {
            stage_lists();
            to_stage = false;
        }
        if (!use_lists) {
#pragma unroll
            for (int k = 0; k < DPW; ++k) {
                // accounted as one line per draw, whichever array
                if (c[k] >= 0) tl.read(g.has_in + (c[k] >> 5), 4);
                uint32_t sg = word[k];
                if (test != TEST_SIG) sg = word[k] ? (uint32_t)g.sig[c[k]] : 0u;
                word[k] = (RootRels<QT>::any ? (sg & need) != 0 : (sg & need) == need) ? 1u : 0u;
            }
        }
        if (use_lists) {
#pragma unroll
            for (int k = 0; k < DPW; ++k) {
                if (c[k] < 0) continue;   // past the window, or not an entity
                bool hit = !RootLists<QT>::any;
#pragma unroll
                for (int f = 0; f < 3; ++f) {
                    if (!(RM >> f & 1) || !F[f].lds) continue;
                    const bool h = maybe_in<QT>(L, f, c[k]);
                    hit = RootLists<QT>::any ? (hit || h) : (hit && h);
                }
                word[k] = hit ? 1u : 0u;
            }
        }
        int32_t nsurv = 0;
#pragma unroll
        for (int k = 0; k < DPW; ++k) {
            const bool live = c[k] >= 0;
            const bool in = live && word[k];
            const uint64_t ml = __ballot(live), m = __ballot(in);
            if (lane < 2) L.non[2 * k + lane] = (uint32_t)(ml >> (32 * lane));
            if (in) L.sj[nsurv + __popcll(m & below)] = (uint16_t)(k * 64 + lane);
            nsurv += __popcll(m);
        }
        wave_sync();
        bool left = false;   // some candidate of this lane is left to the long-list kernels
        // verdict of candidate i: non-answers keep their bit
        auto settle = [&](int32_t i, int32_t st) {
            if (st == ST_NON) return;
            atomicAnd(&L.non[i >> 5], ~(1u << (i & 31)));
            if (st == ST_PEND) {
                left = true;
                if constexpr (MODE != DRAW_GIVEN) L.cand[i] = ~L.cand[i];
                if constexpr (MODE == DRAW_GIVEN || (MODE == DRAW_FIRST && QT == Q3P)) {
                    const int32_t slot = atomicAdd(&ws.ctrl[0], 1);   // capacity covers a round
                    ws.queue[slot] = make_int2(b, base + i);
                }
            }
        };
        // shallow pass over the survivors, 128 at a time; candidates with a
        // backward list are collected for the deep pass
        int32_t ndeep = 0;
        for (int32_t s0 = 0;; s0 += 128) {
            if (s0 < nsurv) {
                bool act[2];
                int32_t cc[2], ii[2], st[2];
                int2 lst[2] = {make_int2(0, 0), make_int2(0, 0)};
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int32_t at = s0 + 64 * u + lane;
                    act[u] = at < nsurv;
                    ii[u] = act[u] ? L.sj[at] : 0;
                    cc[u] = act[u] ? L.cand[ii[u]] : 0;
                    if (use_lists && act[u]) {
                        bool hit = !RootLists<QT>::any;
#pragma unroll
                        for (int f = 0; f < 3; ++f) {
                            if (!(RM >> f & 1) || !F[f].lds) continue;
                            if (RootLists<QT>::any) hit = hit || in_stage(L, F[f], cc[u]);
                            else hit = hit && in_stage(L, F[f], cc[u]);
                        }
                        act[u] = hit;
                    }
                }
                shallow_test2<QT>(g, L, F, anc, rel, cc, act, st, lst, tl);
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    if (act[u] && st[u] != ST_DEEP) settle(ii[u], st[u]);
                    if constexpr (has_long_lists<QT>) {
                        const bool deep = act[u] && st[u] == ST_DEEP;
                        const uint64_t m = __ballot(deep);
                        if (deep) {
                            const int32_t at = ndeep + __popcll(m & below);
                            L.ds[at] = lst[u].x;
                            L.dl[at] = (uint16_t)min(lst[u].y - lst[u].x, 65535);
                            L.dj[at] = (uint16_t)ii[u];
                        }
                        ndeep += __popcll(m);
                    }
                }
                wave_sync();
            }
            const bool more = s0 + 128 < nsurv;
            if constexpr (has_long_lists<QT>) {
                while (ndeep >= 64 || (!more && ndeep > 0)) {   // the newest 64 (at the end: all)
                    const int32_t d0 = max(0, ndeep - 64), at = d0 + lane;
                    const bool on = at < ndeep;
                    const int32_t ds = on ? L.ds[at] : 0, dl = on ? L.dl[at] : 0;
                    uint64_t over = 0, hit = 0;
                    // 3p, 8,192 queries x 500 candidates on a graph of 1,000 entities:
                    // laid out 175 us, each lane its own 157.  Sampling keeps the layout:
                    // with both forms in its kernel 1,024 x 32 there went from 25.0 to 27.0
                    // us and the Freebase-shaped step from 589 to 594.
                    bool done = false;
                    if constexpr (QT == Q3P && MODE == DRAW_GIVEN) done = short_pass3<QT>(g, L, F, rel, ds, dl, &hit);
                    if (!done) hit = deep_pass<QT>(g, L, F, rel, ds, dl, lane, DEEP_TOTAL, steps, &over, tl);
                    // pni: a meeting chain means c is in the complemented set
                    const bool ans = (hit >> lane & 1) != (QT == QPNI);
                    if (on) settle(L.dj[at], over >> lane & 1 ? ST_PEND : ans ? ST_ANS : ST_NON);
                    ndeep = d0;
                }
                wave_sync();
            }
            if (!more) break;
        }
        const bool any_left = __ballot(left) != 0;
        if constexpr (MODE == DRAW_GIVEN) {
            const int32_t at = (base >> 5) + lane;
            const uint32_t bits = lane < WORDS && 32 * lane < n ? L.non[lane] : 0u;
            if (lane < WORDS && at < words) mask[(int64_t)b * words + at] = bits;
            cnt += __popc(bits);
        } else {
            deferred = deferred || any_left;
            if (deferred) {
                for (int32_t i0 = 0; i0 < n; i0 += 64) {
                    const int32_t i = i0 + lane;
                    const int32_t st = i >= n ? ST_ANS
                                       : L.non[i >> 5] >> (i & 31) & 1u ? ST_NON
                                       : L.cand[i] < 0 ? ST_PEND : ST_ANS;
                    if (i < n) sv[base + i] = (uint8_t)st;
                    non_left += __popcll(__ballot(st == ST_NON));
                    pend_left += __popcll(__ballot(st == ST_PEND));
                }
            } else {
                if (!table) table_fill(tab, tb.tcap, out.negatives + (int64_t)b * p.n_neg, acc, lane);
                table = tb.own;
                to_stage = used > 0 && !tb.own;   // the table lies over the lists
                acc = select_window(p, out, b, L, tab, tb.tcap, base, n, acc, lane);
                jsel = stop;
                if (acc >= p.n_neg) break;
            }
        }
        base = stop;
        if (MODE != DRAW_GIVEN && !deferred && base >= end && base < p.neg_tries)
            end = next_round_end(p, base, acc);
        wave_sync();   // the next window reuses the lists
    }
    if constexpr (MODE == DRAW_GIVEN) {
        for (int32_t k = ((base + 31) >> 5) + lane; k < words; k += 64) mask[(int64_t)b * words + k] = 0;
        for (int s = 32; s > 0; s >>= 1) cnt += __shfl_xor(cnt, s);
        if (lane == 0) out.n_valid[b] = cnt;
    } else if (deferred) {
        if (lane == 0) {
            qb[7] = pack_range(jsel, base);
            if constexpr (Shape<QT>::nf < 3) qb[4] = pack_range(non_left, pend_left);
            ws.act[1][b] = acc;
            ws.act[0][atomicAdd(&ws.ctrl[2], 1)] = b;
        }
    } else {
        int32_t* row = out.negatives + (int64_t)b * p.n_neg;
        for (int32_t k = acc + lane; k < p.n_neg; k += 64) row[k] = -1;
        if (lane == 0) {
            out.n_valid[b] = acc;
            if (acc < p.n_neg) out.neg_draws[b] = p.neg_tries;
        }
    }
    flush_tally(tl, stats, b, lane);
}

// One query per workgroup: queries differ widely in cost, and the hardware
// dispatcher hands each freed slot the next query.
template <int QT, class T>
__global__ __launch_bounds__(CWG, 4) void k_candidates(GraphView g, SampleParams p, smore_sample_out out,
                                                    Ws ws, int64_t* stats, Table tb, int32_t j_first)
{
    __shared__ WaveLds L;
    extern __shared__ __align__(16) int32_t own_tab[];
    query_draws<QT, T, DRAW_FIRST>(g, p, out, ws, stats, nullptr, tb, own_tab, L, blockIdx.x, j_first,
                                   threadIdx.x);
}

// Given candidates (p.shared): mask rows and counts of the pairs.
template <int QT>
__global__ __launch_bounds__(CWG, 4) void k_pairs(GraphView g, SampleParams p, smore_sample_out out, Ws ws,
                                               uint32_t* mask)
{
    __shared__ WaveLds L;
    const int32_t n = p.n_shared ? min(p.n_neg, uni(*p.n_shared)) : p.n_neg;
    query_draws<QT, NoTally, DRAW_GIVEN>(g, p, out, ws, nullptr, mask, Table{0, 0}, nullptr, L,
                                         blockIdx.x, n, threadIdx.x);
}

// Verdict of a queued pair by the long-list kernels: its state, or for given
// candidates (mask not NULL) its bit of the mask row and the row's count.
__device__ __forceinline__ void put_verdict(const SampleParams& p, const smore_sample_out& out,
                                            const Ws& ws, uint32_t* mask, int32_t b, int32_t j, bool ans)
{
    if (!mask) {
        ws.status[(int64_t)b * p.neg_tries + j] = ans ? ST_ANS : ST_NON;
    } else {
        uint32_t* w = mask + (int64_t)b * ((p.n_neg + 31) >> 5) + (j >> 5);
        const uint32_t bit = 1u << (j & 31);
        if (ans) {
            if (atomicAnd(w, ~bit) & bit) atomicSub(&out.n_valid[b], 1);
        } else {
            if (!(atomicOr(w, bit) & bit)) atomicAdd(&out.n_valid[b], 1);
        }
    }
}

// Persistent wavefronts draining the heavy queue of given candidates (a
// sampling call's long lists are the finishing kernel's).  Wavefront w takes items
// w, w + nwaves, ... (no shared counter to contend on).  It looks up its
// next 64 items at once, one per lane: the queue entry, the candidate, the
// query's relations and cached lists, and the candidate's backward list,
// so those dependent reads overlap instead of preceding each test in turn.
template <int QT>
__global__ __launch_bounds__(HEAVY_WG) void k_heavy(GraphView g, SampleParams p, smore_sample_out out,
                                                    Ws ws, uint32_t* mask)
{
    constexpr int NF = Shape<QT>::nf;
    const int lane = threadIdx.x & 63;
    const int32_t total = uni(ws.ctrl[0]);
    const int32_t nwaves = gridDim.x * (HEAVY_WG / 64);
    const int32_t w0 = uni(blockIdx.x * (HEAVY_WG / 64) + (threadIdx.x >> 6));
    NoTally none;
    for (int64_t base = w0; base < total; base += 64 * (int64_t)nwaves) {
        const int64_t mine = base + (int64_t)lane * nwaves;
        int32_t mb = 0, mj = 0;
        int32_t mrel[3] = {0, 0, 0}, mf[2 * NF];
        int2 ms = make_int2(0, 0);
#pragma unroll
        for (int f = 0; f < 2 * NF; ++f) mf[f] = 0;
        if (mine < total) {
            const int2 it = ws.queue[mine];
            mb = it.x;
            mj = it.y;
#pragma unroll
            for (int k = 0; k < 3; ++k) mrel[k] = out.relations[3 * (int64_t)mb + k];
            const int32_t* qb = ws.qf + (int64_t)mb * QF;
#pragma unroll
            for (int f = 0; f < 2 * NF; ++f) mf[f] = qb[f];
            ms = group_range(g.rev, candidate(p, g.V, it.x, it.y), chain_r1<QT> ? mrel[1] : mrel[2]);
        }
        const int32_t n = uni((int32_t)min((int64_t)64, (total - base + nwaves - 1) / nwaves));
        for (int k = 0; k < n; ++k) {
            const int32_t b = readlane(mb, k);
            int32_t rel[3];
#pragma unroll
            for (int q = 0; q < 3; ++q) rel[q] = readlane(mrel[q], k);
            FSet F[3];
#pragma unroll
            for (int f = 0; f < 3; ++f) {
                if (f < NF) {
                    const int32_t beg = readlane(mf[2 * f], k), end = readlane(mf[2 * f + 1], k);
                    F[f] = FSet{g.fwd.nbr + beg, end - beg};
                } else {
                    F[f] = FSet{nullptr, 0};
                }
            }
            const int2 s = make_int2(readlane(ms.x, k), readlane(ms.y, k));
            const bool ans = heavy_test<QT>(g, F, rel, s, lane, none);
            if (lane == 0) put_verdict(p, out, ws, mask, b, readlane(mj, k), ans);
        }
    }
}

// OR of a 64-bit value over the wavefront.
__device__ __forceinline__ uint64_t wave_or(uint64_t x)
{
    for (int s = 32; s > 0; s >>= 1)
        x |= (uint64_t)(uint32_t)__shfl_xor((int32_t)(uint32_t)x, s) |
             ((uint64_t)(uint32_t)__shfl_xor((int32_t)(x >> 32), s) << 32);
    return x;
}

// A slice of one queued 3p item, held by one lane: the item's draw (its
// query b and index j), relation r1, forward list F0 = A_r0(a0)
// (edges [f0b, f0b + f0n)), the candidate's list S = R_r2(c) (edges from
// sx), the range [y0, y1) of S's entities to expand and, for each of them,
// the range [k0, k1) of its (y, key) pairs to search (keys from the shorter
// of R_r1(y) and F0).
struct Slice3 {
    bool valid = false;
    int32_t b = -1, j = 0;
    int32_t r1 = 0, f0b = 0, f0n = 0, sx = 0, y0 = 0, y1 = 0, k0 = 0, k1 = 0;
};

// Reserve n unit slots for a wavefront (all lanes call it with the same n):
// the first slot, or -1 when the queue is full, in which case the slots of
// the failed reservation that lie inside the queue are marked unused.
__device__ __forceinline__ int64_t reserve_units(Ws& ws, int32_t n, int lane)
{
    int32_t base = INT_MAX;
    // once the queue is full the counter is left alone (it cannot grow without bound)
    if (lane == 0 && ws.ctrl[5] < ws.ucap) base = atomicAdd(&ws.ctrl[5], n);
    base = uni(__shfl(base, 0));
    if ((int64_t)base + n <= ws.ucap) return base;
    for (int64_t k = (int64_t)base + lane; k < ws.ucap; k += 64) ws.units[k] = make_int4(-1, 0, 0, 2);
    return -1;
}

// Decide the slices of a wavefront, one per lane: the entities y of all of
// them expanded 64 at a time (signature class, then the group under r1),
// and the (y, key) pairs of all of them searched 256 at a time; a hit makes
// its slice's item an answer, whose remaining y's and pairs are dropped,
// the rest being laid out again after every step.  With PUSH (the
// long-list kernel), y's beyond the first UNIT_Y of a slice and pairs
// beyond the first UNIT_PAIRS of one y go to the unit queue (item index q)
// when it has room, else they are decided here.  Returns the answer bits.
template <bool PUSH, class T>
__device__ uint64_t decide_slices3(const GraphView& g, Ws& ws, Slice3 w, int64_t q, int lane, T& tl)
{
    if constexpr (PUSH) {
        const int32_t ny = w.valid ? w.y1 - w.y0 : 0;
        const int32_t nu = ny > UNIT_Y ? (ny - UNIT_Y + UNIT_Y - 1) / UNIT_Y : 0;
        int32_t tot;
        const int32_t ex = excl_prefix(nu, lane, &tot);
        if (tot > 0) {
            const int64_t at = reserve_units(ws, tot, lane);
            if (at >= 0) {
                for (int32_t k = 0; k < nu; ++k) {
                    const int32_t a = w.y0 + UNIT_Y * (k + 1);
                    ws.units[at + ex + k] = make_int4((int32_t)q, a, min(a + UNIT_Y, w.y1), 0);
                }
                if (nu > 0) w.y1 = w.y0 + UNIT_Y;
            }
        }
    }
    uint64_t ans = 0;     // bit i: the item of lane i is an answer
    int32_t ydone = 0;    // y's of this lane's slice expanded so far
    for (;;) {
        const int32_t yrem = (!w.valid || ((ans >> lane) & 1)) ? 0 : (w.y1 - w.y0) - ydone;
        int32_t ytotal;
        const int32_t yex = excl_prefix(yrem, lane, &ytotal);
        if (ytotal == 0) break;
        const int it = owner_lane(min(lane, ytotal - 1), yex);
        const int32_t ypos = __shfl(w.y0, it) + __shfl(ydone, it) + lane - __shfl(yex, it);
        const int32_t isx = __shfl(w.sx, it), ir1 = __shfl(w.r1, it);
        const int32_t if0b = __shfl(w.f0b, it), if0n = __shfl(w.f0n, it);
        int32_t k0 = __shfl(w.k0, it), k1 = __shfl(w.k1, it);
        int2 s2 = make_int2(0, 0);
        if (lane < ytotal) {
            // y without an in-edge under r1's signature class has none under r1
            const int32_t y = g.rev.nbr[isx + ypos];
            tl.read(g.rev.nbr + isx + ypos, 4);
            tl.read(g.sig + y, 1);
            if (g.sig[y] & sig_bit(ir1)) s2 = group_range(g.rev, y, ir1, tl);
        }
        const int32_t len = s2.y - s2.x;
        const bool kil = len <= if0n;            // search R_r1(y)'s entries in F0
        const int32_t nall = len > 0 ? min(len, if0n) : 0;
        if constexpr (PUSH) {
            // pairs beyond the first UNIT_PAIRS of a y: units of UNIT_PAIRS keys
            const int32_t nu = nall > UNIT_PAIRS ? (nall - 1) / UNIT_PAIRS : 0;
            if (__ballot(nu > 0)) {
                int32_t tot;
                const int32_t ex = excl_prefix(nu, lane, &tot);
                const int64_t at = reserve_units(ws, tot, lane);
                if (at >= 0) {
                    const int32_t iq = __shfl((int32_t)q, it);
                    for (int32_t k = 0; k < nu; ++k)
                        ws.units[at + ex + k] = make_int4(iq, ypos, UNIT_PAIRS * (k + 1), 1);
                    if (nu > 0) k1 = UNIT_PAIRS;
                }
            }
        }
        const int32_t kb = min(k0, nall), ke = min(k1, nall);   // this y's keys [kb, ke)
        int32_t pdone = 0;
        for (;;) {
            const int32_t rem = ((ans >> it) & 1) ? 0 : ke - kb - pdone;
            int32_t ptotal;
            const int32_t pex = excl_prefix(rem, lane, &ptotal);
            if (ptotal == 0) break;
            const int32_t* Bk[4];
            int32_t nbk[4], x[4], who[4];
            bool cnt[4], found[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int32_t pi = 64 * u + lane;
                const int32_t pq = pi < ptotal ? pi : ptotal - 1;
                const int yl = owner_lane(pq, pex);
                const int32_t off = __shfl(kb, yl) + __shfl(pdone, yl) + pq - __shfl(pex, yl);
                const int32_t lx = __shfl(s2.x, yl), ln = __shfl(len, yl);
                const int32_t k_in_l = __shfl((int32_t)kil, yl);
                const int32_t fb = __shfl(if0b, yl), fn = __shfl(if0n, yl);
                who[u] = __shfl(it, yl);
                Bk[u] = g.fwd.nbr + fb;
                nbk[u] = 0;
                x[u] = -1;
                cnt[u] = false;
                if (pi < ptotal) {
                    if (k_in_l) {
                        x[u] = g.rev.nbr[lx + off];
                        tl.read(g.rev.nbr + lx + off, 4);
                        nbk[u] = fn;
                    } else {
                        x[u] = g.fwd.nbr[fb + off];
                        Bk[u] = g.rev.nbr + lx;
                        nbk[u] = ln;
                        cnt[u] = true;
                    }
                }
            }
            search4q(Bk, nbk, x, cnt, found, tl);
            uint64_t m = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (found[u]) m |= 1ull << who[u];
            ans |= wave_or(m);
            pdone += min(rem, max(0, 256 - pex));   // this step took pairs pex .. 255
        }
        ydone += min(yrem, max(0, 64 - yex));       // this chunk took y's yex .. 63
    }
    return ans;
}

// The slice of queued item qi: the whole list S, all keys.
template <class T>
__device__ __forceinline__ Slice3 item_slice3(const GraphView& g, const SampleParams& p,
                                              const smore_sample_out& out, const Ws& ws, int64_t qi, T& tl)
{
    Slice3 w;
    const int2 it = ws.queue[qi];
    w.valid = true;
    w.b = it.x;
    w.j = it.y;
    const int32_t c = candidate(p, g.V, it.x, it.y);
    w.r1 = out.relations[3 * (int64_t)w.b + 1];
    const int32_t r2 = out.relations[3 * (int64_t)w.b + 2];
    const int32_t* qb = ws.qf + (int64_t)w.b * QF;
    w.f0b = qb[0];
    w.f0n = qb[1] - w.f0b;
    const int2 S = group_range(g.rev, c, r2, tl);
    w.sx = S.x;
    w.y0 = 0;
    w.y1 = S.y - S.x;
    w.k0 = 0;
    w.k1 = INT_MAX;
    return w;
}

// The long-list kernel of 3p, batched: wavefront w takes items w,
// w + nwaves, ... like k_heavy, but decides up to 64 of them together, one
// per lane (decide_slices3), so their dependent chains overlap instead of
// running one item after the other; the parts of huge items go to the unit
// queue.  It writes every item's state.  With the read tally, a batch's
// reads are charged to the query of its first item (the sums over all
// queries are exact).
template <class T>
__global__ __launch_bounds__(HEAVY_WG) void k_heavy3(GraphView g, SampleParams p, smore_sample_out out,
                                                     Ws ws, int64_t* stats, uint32_t* mask)
{
    const int lane = threadIdx.x & 63;
    const int32_t total = uni(ws.ctrl[0]);
    const int32_t nwaves = gridDim.x * (HEAVY_WG / 64);
    const int32_t w0 = uni(blockIdx.x * (HEAVY_WG / 64) + (threadIdx.x >> 6));
    T tl;
    for (int64_t base = w0; base < total; base += 64 * (int64_t)nwaves) {
        const int64_t mine = base + (int64_t)lane * nwaves;
        Slice3 w;
        if (mine < total) w = item_slice3(g, p, out, ws, mine, tl);
        const uint64_t ans = decide_slices3<true>(g, ws, w, mine, lane, tl);
        if (mine < total) put_verdict(p, out, ws, mask, w.b, w.j, (ans >> lane) & 1);
        flush_tally(tl, stats, uni(__shfl(w.b, 0)), lane, 2);
    }
}

// Is the queued pair already an answer?  (Every queued pair has had a
// verdict from the long-list kernel before.)
__device__ __forceinline__ bool is_answer(const SampleParams& p, const Ws& ws, const uint32_t* mask,
                                          int32_t b, int32_t j)
{
    if (!mask) return ws.status[(int64_t)b * p.neg_tries + j] == ST_ANS;
    return !(mask[(int64_t)b * ((p.n_neg + 31) >> 5) + (j >> 5)] >> (j & 31) & 1u);
}

// The units the long-list kernel left: wavefront w takes units w,
// w + nwaves, ..., up to 64 at a time, one per lane; a unit of an item
// already decided an answer is skipped, and a hit makes its item an answer
// (units never clear a state, so their order does not matter).
template <class T>
__global__ __launch_bounds__(HEAVY_WG) void k_units3(GraphView g, SampleParams p, smore_sample_out out,
                                                     Ws ws, int64_t* stats, uint32_t* mask)
{
    const int lane = threadIdx.x & 63;
    const int32_t total = uni((int32_t)min((int64_t)ws.ctrl[5], ws.ucap));
    const int32_t nwaves = gridDim.x * (HEAVY_WG / 64);
    const int32_t w0 = uni(blockIdx.x * (HEAVY_WG / 64) + (threadIdx.x >> 6));
    T tl;
    for (int64_t base = w0; base < total; base += 64 * (int64_t)nwaves) {
        const int64_t mine = base + (int64_t)lane * nwaves;
        Slice3 w;
        if (mine < total) {
            const int4 u = ws.units[mine];
            if (u.w != 2) {
                w = item_slice3(g, p, out, ws, u.x, tl);
                if (is_answer(p, ws, mask, w.b, w.j)) {
                    w.valid = false;
                } else if (u.w == 0) {           // entities [a, b) of S, all keys
                    w.y0 = u.y;
                    w.y1 = u.z;
                } else {                         // entity a of S, keys [b, b + UNIT_PAIRS)
                    w.y0 = u.y;
                    w.y1 = u.y + 1;
                    w.k0 = u.z;
                    w.k1 = u.z + UNIT_PAIRS;
                }
            }
        }
        const uint64_t ans = decide_slices3<false>(g, ws, w, -1, lane, tl);
        if (w.valid && ((ans >> lane) & 1)) put_verdict(p, out, ws, mask, w.b, w.j, true);
        flush_tally(tl, stats, uni(__shfl(max(w.b, 0), 0)), lane, 2);
    }
}

// ------------------------------------------------------ finishing kernel
// A query's anchors, relations and forward lists, which are read in place.
struct QueryLists {
    int32_t anc[3], rel[3];
    FList F[3];
};

template <int QT>
__device__ __forceinline__ QueryLists query_lists(const smore_sample_out& out, const Ws& ws, int32_t b)
{
    const int32_t* qb = ws.qf + (int64_t)b * QF;
    QueryLists q;
#pragma unroll
    for (int f = 0; f < 3; ++f) {
        q.anc[f] = uni(out.anchors[3 * (int64_t)b + f]);
        q.rel[f] = uni(out.relations[3 * (int64_t)b + f]);
        q.F[f] = FList{0, 0, 0, false};
        if (f >= Shape<QT>::nf) continue;
        q.F[f].beg = uni(qb[2 * f]);
        q.F[f].n = uni(qb[2 * f + 1]) - q.F[f].beg;
    }
    return q;
}

// A query's states, written and read by several workgroups (shared) or by
// one.  Shared ones go past the L2, which other workgroups have their own of,
// so that no fence has to empty it: with fences the 64 queries x 16 negatives
// of 2p on a dense graph took 160 us, without 60.
struct States {
    uint8_t* p;
    bool shared;
    __device__ __forceinline__ int32_t get(int32_t j) const
    {
        return shared ? __hip_atomic_load(p + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : p[j];
    }
    __device__ __forceinline__ void put(int32_t j, int32_t st) const
    {
        if (shared) __hip_atomic_store(p + j, (uint8_t)st, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else p[j] = (uint8_t)st;
    }
};

// States of the draws [j, j + 64) below j1, one per lane: what the candidate
// kernel does with them, but for 3p every candidate with a backward list is
// left pending.
template <int QT, class T>
__device__ __forceinline__ void finish_draws(const GraphView& g, const SampleParams& p, const WaveLds& L,
                                             const QueryLists& q, int32_t b, int32_t j, int32_t j1,
                                             const States& sv, int lane, T& tl)
{
    j += lane;
    uint32_t need = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k)
        if (RootRels<QT>::mask >> k & 1) need |= sig_bit(q.rel[k]);
    int32_t c[2] = {0, 0}, st[2] = {ST_NON, ST_NON};
    bool act[2] = {false, false};
    int2 lst[2] = {make_int2(0, 0), make_int2(0, 0)};
    if (j < j1) {
        c[0] = candidate(p, g.V, b, j);
        tl.read(g.has_in + (c[0] >> 5), 4);
        bool in = true;
        if (g.first_test == TEST_MASK) in = g.has_in[c[0] >> 5] >> (c[0] & 31) & 1u;
        if (g.first_test == TEST_MASK4) in = g.has_in4[c[0] >> 7] >> (c[0] >> 2 & 31) & 1u;
        const uint32_t sg = in ? (uint32_t)g.sig[c[0]] : 0u;
        act[0] = RootRels<QT>::any ? (sg & need) != 0 : (sg & need) == need;
    }
    shallow_test2<QT>(g, L, q.F, q.anc, q.rel, c, act, st, lst, tl);
    if (!act[0]) st[0] = ST_NON;
    const bool deep = act[0] && st[0] == ST_DEEP;
    if constexpr (QT == Q3P) {
        if (deep) st[0] = ST_PEND;
    } else if (__ballot(deep)) {
        int32_t steps = INT_MAX;
        uint64_t over;
        const uint64_t hit = deep_pass<QT>(g, L, q.F, q.rel, lst[0].x, deep ? lst[0].y - lst[0].x : 0, lane,
                                           INT_MAX, steps, &over, tl);
        if (deep) st[0] = over >> lane & 1 ? ST_PEND : (hit >> lane & 1) != (QT == QPNI) ? ST_ANS : ST_NON;
    }
    if (j < j1) sv.put(j, st[0]);
}

// Verdicts of up to 64 pending draws, one per lane (on: the lane has one).
// Their lists are looked up side by side; for 3p all entities and pairs are
// laid out over the lanes, for the other shapes the pairs of the lists a
// wavefront may walk, and the others are met one after the other.
template <int QT, class T>
__device__ __forceinline__ void finish_pending(const GraphView& g, const SampleParams& p, Ws& ws,
                                               const WaveLds& L, const QueryLists& q, int32_t b, int32_t j,
                                               bool on, const States& sv, int lane, T& tl)
{
    int2 s = make_int2(0, 0);
    if (on) s = group_range(g.rev, candidate(p, g.V, b, j), q.rel[chain_r1<QT> ? 1 : 2], tl);
    uint64_t ans;
    if constexpr (QT == Q3P) {
        Slice3 w;
        w.valid = on;
        w.b = b;
        w.j = j;
        w.r1 = q.rel[1];
        w.f0b = q.F[0].beg;
        w.f0n = q.F[0].n;
        w.sx = s.x;
        w.y1 = s.y - s.x;
        w.k1 = INT_MAX;
        ans = decide_slices3<false>(g, ws, w, -1, lane, tl);
    } else {
        int32_t steps = INT_MAX;
        uint64_t over;
        ans = deep_pass<QT>(g, L, q.F, q.rel, s.x, s.y - s.x, lane, INT_MAX, steps, &over, tl);
        if (QT == QPNI) ans = ~ans & ~over;
        FSet F[3];
#pragma unroll
        for (int f = 0; f < 3; ++f) F[f] = FSet{g.fwd.nbr + q.F[f].beg, q.F[f].n};
        for (; over; over &= over - 1) {
            const int k = __ffsll((unsigned long long)over) - 1;
            if (heavy_test<QT>(g, F, q.rel, make_int2(readlane(s.x, k), readlane(s.y, k)), lane, tl))
                ans |= 1ull << k;
        }
    }
    if (on) sv.put(j, ans >> lane & 1 ? ST_ANS : ST_NON);
}

// The queries that had long lists among their first draws: their verdicts
// (for 3p the long-list kernels have settled them), selection, and whatever
// further draws the queries need, a range at a time.  A workgroup takes a
// query: draws and pending lists are dealt over its wavefronts, selection is
// the first one's.  (A kernel of its own for the long lists was a launch of
// 4 to 16 us for a few queries.)  Where the workgroups outnumber the queries,
// several share a query's first range, and with it the further draws it is
// likely to need; the last one to be done with its share goes on alone.
template <int QT, class T>
__global__ __launch_bounds__(1024) void k_finish(GraphView g, SampleParams p, smore_sample_out out, Ws ws,
                                                 int64_t* stats, Table tb)
{
    __shared__ WaveLds L;
    __shared__ uint16_t items[SMORE_MAX_NEG_TRIES];   // pending draws of the range
    __shared__ int32_t n_items, count, next[2];
    extern __shared__ __align__(16) int32_t own_tab[];
    int32_t* tab = tb.own ? own_tab : L.stage;
    const int tid = threadIdx.x, lane = tid & 63, w = uni(tid >> 6), nw = blockDim.x >> 6;
    const int32_t n = uni(ws.ctrl[2]);
    // workgroups per query: one where the call fills the GPU
    const int32_t per = nw > 4 && n < (int32_t)gridDim.x ? gridDim.x / max(n, 1) : 1;
    for (int32_t task = blockIdx.x; task < n * per; task += gridDim.x) {
        const int32_t b = uni(ws.act[0][task / per]);
        int32_t share = task % per;
        const QueryLists q = query_lists<QT>(out, ws, b);
        const int32_t range = uni(ws.qf[(int64_t)b * QF + 7]);
        int32_t* row = out.negatives + (int64_t)b * p.n_neg;
        int32_t j0 = range_lo(range), mid = range_hi(range), j1 = mid;
        int32_t acc = uni(ws.act[1][b]) & 0xFFFF;
        int32_t shares = 1;
        if (per > 1) {
            // all of a query's workgroups have to come to the same shares, whenever
            // each of them starts: counts that none of them changes.  (The states
            // do change: a workgroup that came late saw fewer pending ones, and
            // with other shares the query was never finished.)
            int32_t non = 0, pend = 0;
            if constexpr (QT == Q3P) {
                // verdicts of earlier kernels: none is pending, none is changed here
                if (tid == 0) count = 0;
                __syncthreads();
                for (int32_t j = j0 + 64 * w; j < j1; j += 64 * nw) {
                    const int32_t st = j + lane < j1 ? ws.status[(int64_t)b * p.neg_tries + j + lane] : ST_ANS;
                    non += __popcll(__ballot(st == ST_NON));
                }
                if (lane == 0) atomicAdd(&count, non);
                __syncthreads();
                non = uni(count);
            } else {
                const int32_t left = uni(ws.qf[(int64_t)b * QF + 4]);
                non = range_lo(left);
                pend = range_hi(left);
            }
            j1 = likely_end(p, g.V, mid, acc + non, mid - j0 - non - pend, pend);
            shares = min(per, max(1, (pend + j1 - mid + nw - 1) / nw));   // a wavefront has work in each
        }
        if (share >= shares) continue;
        const States sv{ws.status + (int64_t)b * p.neg_tries, shares > 1};
        bool first = true;
        T tl;
        for (;;) {
            // states of the draws [mid, j1) and verdicts of the pending ones of
            // [j0, j1): runs of `each` draws, dealt over shares and wavefronts.  A
            // query that is short of a few draws has them taken by all wavefronts, a
            // few each, since a step lasts as long as the longest lists of its draws
            // (256 queries x 200 of 2p on a dense graph: 64 draws a wavefront in
            // ranges of at least 64 per wavefront 285 us, this way 182).
            const int32_t each = shares > 1 ? min(64, max(1, (j1 - j0) / (shares * nw)))
                                            : min(64, max(1, (j1 - j0 + nw - 1) / nw));
            for (int32_t r = share + shares * w; mid < j1 && j0 + r * each < j1; r += shares * nw) {
                const int32_t ja = max(j0 + r * each, mid), jb = min(j0 + (r + 1) * each, j1);
                if (ja < jb) finish_draws<QT>(g, p, L, q, b, ja, jb, sv, lane, tl);
            }
            flush_tally(tl, stats, b, lane);
            if (QT != Q3P || mid < j1) {
                if (tid == 0) n_items = 0;
                __syncthreads();
                for (int32_t k = tid;; k += blockDim.x) {
                    const int32_t r = share + shares * (k / each), j = j0 + r * each + k % each;
                    if (j0 + r * each >= j1) break;
                    if (j < j1 && sv.get(j) == ST_PEND) items[atomicAdd(&n_items, 1)] = (uint16_t)j;
                }
                __syncthreads();
                const int32_t m = uni(n_items), mine = min(64, (m + nw - 1) / nw);
                for (int32_t k = mine * w; k < m; k += mine * nw) {
                    const bool on = lane < mine && k + lane < m;
                    finish_pending<QT>(g, p, ws, L, q, b, on ? items[k + lane] : 0, on, sv, lane, tl);
                }
                flush_tally(tl, stats, b, lane, 2);
            }
            if (shares > 1) {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                __builtin_amdgcn_s_waitcnt(0);   // each wavefront's states are written when its workgroup counts
                __syncthreads();
                if (tid == 0) next[0] = atomicAdd(&ws.act[1][b], 1 << 16) >> 16;
                __syncthreads();
                if (uni(next[0]) + 1 < shares) break;
                share = 0;
                shares = 1;
            }
            __syncthreads();
            if (w == 0) {
                if (first) table_fill(tab, tb.tcap, row, acc, lane);
                first = false;
                while (j0 < j1 && acc < p.n_neg) {
                    const int32_t m = min(j1 - j0, min(WIN, table_room(tb.tcap) - acc));
                    for (int k = 0; 64 * k < m; ++k) {
                        const int32_t i = 64 * k + lane;
                        const bool non = i < m && sv.get(j0 + i) == ST_NON;
                        const uint64_t bits = __ballot(non);
                        if (i < m) L.cand[i] = candidate(p, g.V, b, j0 + i);
                        if (lane < 2) L.non[2 * k + lane] = (uint32_t)(bits >> (32 * lane));
                    }
                    wave_sync();
                    acc = select_window(p, out, b, L, tab, tb.tcap, j0, m, acc, lane);
                    j0 += m;
                    wave_sync();
                }
                if (lane == 0) {
                    next[0] = j0;
                    next[1] = acc < p.n_neg ? next_round_end(p, j0, acc) : j0;
                }
            }
            __syncthreads();
            j0 = mid = uni(next[0]);
            j1 = uni(next[1]);
            if (j0 < j1) continue;
            if (w == 0) {
                for (int32_t k = acc + lane; k < p.n_neg; k += 64) row[k] = -1;
                if (lane == 0) {
                    out.n_valid[b] = acc;
                    if (acc < p.n_neg) out.neg_draws[b] = p.neg_tries;
                }
            }
            break;
        }
        __syncthreads();   // the next query takes the table and the list
    }
}

__device__ __forceinline__ void ht_insert(int32_t* tv, int32_t* tj, uint32_t mask, int shift,
                                          int32_t c, int32_t j)
{
    uint32_t h = ((uint32_t)c * 0x9E3779B1u) >> shift;
    for (;;) {
        const int32_t old = atomicCAS(&tv[h], -1, c);
        if (old == -1 || old == c) {
            atomicMin(&tj[h], j);
            return;
        }
        h = (h + 1) & mask;
    }
}

__device__ __forceinline__ int32_t ht_first(const int32_t* tv, const int32_t* tj, uint32_t mask,
                                            int shift, int32_t c)
{
    uint32_t h = ((uint32_t)c * 0x9E3779B1u) >> shift;
    while (tv[h] != c) h = (h + 1) & mask;
    return tj[h];
}

// first-occurrence table of the shared set: load factor at most 0.6
inline int32_t shared_tcap(int32_t j_end)
{
    int32_t tcap = 64;
    while (tcap * 3 < 5 * j_end) tcap <<= 1;
    return tcap;
}

// Selection table of a call.  A row whose first draws are one window has it
// over the staged lists and their bits (which are copied again if a later
// window is needed), half empty where there is room; a longer row, with
// windows that follow one another, in LDS of its own.  Both hold n_neg
// values and at least 128 more.
inline Table selection_table(const SampleParams& p)
{
    auto blocks = [](int32_t x) { return (x + 255) / 256 * 256; };
    if (first_round(p) <= WIN) return Table{min(blocks(2 * (p.n_neg + 128)), TABLE_OVER), 0};
    return Table{blocks(3 * (p.n_neg + WIN) / 2), 1};
}

inline int check_launch(const char** err)
{
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) { *err = hipGetErrorString(e); return SMORE_E_HIP; }
    return SMORE_OK;
}

// One-shot event pairs of the next negatives call, each independent: around
// the candidate kernel (0), the long-list kernels (1: 3p's two, of the other
// shapes the finishing kernel) and the finishing kernel (2).
struct ProfileArm {
    hipEvent_t start = nullptr, stop = nullptr;
};
thread_local ProfileArm g_prof[3];

// One-shot wait of the next negatives call: its stream waits on this event
// right before the first candidate kernel, after the preparation.
thread_local hipEvent_t g_wait = nullptr;

inline void prof_mark(int which, bool after, hipStream_t st)
{
    ProfileArm& a = g_prof[which];
    if (!a.start || !a.stop) return;
    (void)hipEventRecord(after ? a.stop : a.start, st);
    if (after) a = ProfileArm{};
}

// Wavefronts per query of the finishing kernel: as many as run at once, 4 to
// 16, since a call of few queries would otherwise last as long as one
// wavefront takes for all draws and lists of the worst query (16 queries x
// 1,000 negatives on a graph of 2,000 entities and 300,000 triples, where most
// candidates are answers: one wavefront for the draws 32.1 ms for 3p and 3.7
// for 2p, sixteen, and a query's draws dealt over several workgroups, 0.30 and
// 0.20).  3p leaves it no lists of the first draws: calls that fill the GPU
// run two (Freebase-shaped 3p 387 us with one or two, with four 395; 6,000 x
// 300 on an FB15k-237-shaped graph 575 with one, 397 with two).
template <int QT>
inline int finish_waves(const SampleParams& p)
{
    if (p.batch <= FINISH_WAVES / 16) return 16;
    if (p.batch <= FINISH_WAVES / 8) return 8;
    return QT == Q3P && p.batch >= FINISH_WAVES ? 2 : 4;
}

// The long-list kernels over the queue (mask: see put_verdict).
template <int QT, class T>
int launch_long_lists(const GraphView& gv, const SampleParams& p, const smore_sample_out& out, Ws ws,
                      int64_t* stats, uint32_t* mask, hipStream_t st, const char** err)
{
    int rc;
    if constexpr (QT == Q3P) {
        // a quarter grid: these waves mostly wait on dependent reads, and at
        // four waves per SIMD a full grid would hold the registers that the
        // candidate kernels of shapes sampled beside this one need
        const int grid = mask ? PERSIST_BLOCKS : PERSIST_BLOCKS / 4;
        k_heavy3<T><<<grid, HEAVY_WG, 0, st>>>(gv, p, out, ws, stats, mask);
        if ((rc = check_launch(err))) return rc;
        k_units3<T><<<grid, HEAVY_WG, 0, st>>>(gv, p, out, ws, stats, mask);
    } else {
        k_heavy<QT><<<PERSIST_BLOCKS, HEAVY_WG, 0, st>>>(gv, p, out, ws, mask);
    }
    return check_launch(err);
}

// parts: NEG_PREPARE the per-query preparation, NEG_CANDIDATES the candidate
// kernel, NEG_REST the long-list and finishing kernels.
template <int QT, class T>
int run_negatives(const GraphView& gv, const SampleParams& p, const smore_sample_out& out, Ws ws,
                  int64_t* stats, int32_t R, int parts, hipStream_t st, const char** err)
{
    int rc;
    if (p.n_neg == 0) {   // nothing to draw: no preparation, no workspace
        if (!(parts & NEG_PREPARE)) return SMORE_OK;
        k_no_draws<QT><<<(p.batch + 255) / 256, 256, 0, st>>>(gv, p, out, stats, R);
        return check_launch(err);
    }
    if (parts & NEG_PREPARE) {
        k_prepare<QT, T><<<(p.batch + 63) / 64, 256, 0, st>>>(gv, p, out, ws, stats, R);
        if ((rc = check_launch(err))) return rc;
    }
    const Table tb = selection_table(p);
    const size_t own = tb.own ? (size_t)tb.tcap * sizeof(int32_t) : 0;
    if (parts & NEG_CANDIDATES) {
        if (g_wait) {
            const hipError_t e = hipStreamWaitEvent(st, g_wait, 0);
            g_wait = nullptr;
            if (e != hipSuccess) { *err = hipGetErrorString(e); return SMORE_E_HIP; }
        }
        prof_mark(0, false, st);
        k_candidates<QT, T><<<p.batch, CWG, own, st>>>(gv, p, out, ws, stats, tb, first_round(p));
        if ((rc = check_launch(err))) return rc;
        prof_mark(0, true, st);
    }
    if (!(parts & NEG_REST)) return SMORE_OK;
    // the finishing kernel is the long-list kernel of every shape but 3p
    prof_mark(1, false, st);
    if constexpr (QT == Q3P) {
        if ((rc = launch_long_lists<QT, T>(gv, p, out, ws, stats, nullptr, st, err))) return rc;
        prof_mark(1, true, st);
    }
    prof_mark(2, false, st);
    if constexpr (has_long_lists<QT>) {
        const int nw = finish_waves<QT>(p);
        k_finish<QT, T><<<FINISH_WAVES / nw, 64 * nw, own, st>>>(gv, p, out, ws, stats, tb);
        if ((rc = check_launch(err))) return rc;
    }
    prof_mark(2, true, st);
    prof_mark(1, true, st);
    return SMORE_OK;
}

template <class T>
int dispatch_negatives(QType qt, const GraphView& gv, const SampleParams& p, const smore_sample_out& out,
                       Ws ws, int64_t* stats, int32_t R, int parts, hipStream_t st, const char** err)
{
    switch (qt) {
        case Q1P: return run_negatives<Q1P, T>(gv, p, out, ws, stats, R, parts, st, err);
        case Q2P: return run_negatives<Q2P, T>(gv, p, out, ws, stats, R, parts, st, err);
        case Q3P: return run_negatives<Q3P, T>(gv, p, out, ws, stats, R, parts, st, err);
        case Q2I: return run_negatives<Q2I, T>(gv, p, out, ws, stats, R, parts, st, err);
        case Q3I: return run_negatives<Q3I, T>(gv, p, out, ws, stats, R, parts, st, err);
        case QIP: return run_negatives<QIP, T>(gv, p, out, ws, stats, R, parts, st, err);
        case QPI: return run_negatives<QPI, T>(gv, p, out, ws, stats, R, parts, st, err);
        case Q2U: return run_negatives<Q2U, T>(gv, p, out, ws, stats, R, parts, st, err);
        case QUP: return run_negatives<QUP, T>(gv, p, out, ws, stats, R, parts, st, err);
        case Q2IN: return run_negatives<Q2IN, T>(gv, p, out, ws, stats, R, parts, st, err);
        case Q3IN: return run_negatives<Q3IN, T>(gv, p, out, ws, stats, R, parts, st, err);
        case QINP: return run_negatives<QINP, T>(gv, p, out, ws, stats, R, parts, st, err);
        case QPIN: return run_negatives<QPIN, T>(gv, p, out, ws, stats, R, parts, st, err);
        case QPNI: return run_negatives<QPNI, T>(gv, p, out, ws, stats, R, parts, st, err);
        default: *err = "unknown shape"; return SMORE_E_UNSUPPORTED;
    }
}

// ------------------------------------------------- shared candidate sets
// The minibatch's candidate set: the first n_neg distinct values of the
// draws j < neg_tries of the shared stream, in draw order.  One workgroup
// takes the draws 256 at a time; an LDS table of (value, first draw)
// decides first occurrences (later blocks find the values of earlier ones).
constexpr int SSET_WG = 256;

__global__ __launch_bounds__(SSET_WG) void k_shared_set(SampleParams p, int32_t V, int32_t* shared,
                                                        int32_t* n_shared, int32_t tcap, int tshift)
{
    extern __shared__ int32_t lds[];   // tv[tcap], tj[tcap], wave_cnt[4]: all dynamic
    int32_t* tv = lds;
    int32_t* tj = lds + tcap;
    int32_t* wave_cnt = lds + 2 * tcap;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint32_t tmask = (uint32_t)tcap - 1;
    for (int32_t k = tid; k < tcap; k += SSET_WG) { tv[k] = -1; tj[k] = INT_MAX; }
    __syncthreads();
    int32_t acc = 0;   // the same in every thread: block-wide counts only
    for (int32_t base = 0; base < p.neg_tries && acc < p.n_neg; base += SSET_WG) {
        const int32_t j = base + tid;
        int32_t c = -1;
        if (j < p.neg_tries) {
            c = (int32_t)reduce_range(draw64(p.seed, TAG_SHARED, (uint32_t)p.query_offset, 0, (uint32_t)j),
                                      (uint32_t)V);
            ht_insert(tv, tj, tmask, tshift, c, j);
        }
        __syncthreads();
        const bool first = c >= 0 && ht_first(tv, tj, tmask, tshift, c) == j;
        const uint64_t m = __ballot(first);
        if (lane == 0) wave_cnt[w] = __popcll(m);
        __syncthreads();
        int32_t before = 0, total = 0;
        for (int k = 0; k < SSET_WG / 64; ++k) {
            before += k < w ? wave_cnt[k] : 0;
            total += wave_cnt[k];
        }
        const int32_t rank = acc + before + __popcll(m & lanes_below(lane));
        if (first && rank < p.n_neg) shared[rank] = c;
        acc = min(p.n_neg, acc + total);
        __syncthreads();   // wave_cnt is rewritten by the next block of draws
    }
    for (int32_t k = acc + tid; k < p.n_neg; k += SSET_WG) shared[k] = -1;
    if (tid == 0) *n_shared = acc;
}

// The minibatch's shared candidate set (one workgroup).
int draw_shared_set(const SampleParams& p, int32_t V, int32_t* shared, int32_t* n_shared,
                    hipStream_t st, const char** err)
{
    const int32_t tcap = shared_tcap(p.neg_tries > 0 ? p.neg_tries : 1);
    int tshift = 32;
    for (int32_t x = tcap; x > 1; x >>= 1) --tshift;
    // the table needs up to 64 KiB plus the counts: raise the kernel's LDS
    // limit to the largest request once (the default is 64 KiB in total)
    const size_t lds = ((size_t)2 * tcap + SSET_WG / 64) * sizeof(int32_t);
    static bool attr = false;
    if (!attr) {
        const size_t most = ((size_t)2 * shared_tcap(SMORE_MAX_NEG_TRIES) + SSET_WG / 64) * sizeof(int32_t);
        const hipError_t e = hipFuncSetAttribute((const void*)k_shared_set,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)most);
        if (e != hipSuccess) { *err = hipGetErrorString(e); return SMORE_E_HIP; }
        attr = true;
    }
    k_shared_set<<<1, SSET_WG, lds, st>>>(p, V, shared, n_shared, tcap, tshift);
    return check_launch(err);
}

// Every (query, candidate) pair of p.shared (one set for all queries, or a
// list per query p.cand_stride apart): states, then mask rows and counts.
template <int QT>
int run_pairs(const GraphView& gv, const SampleParams& p, const smore_sample_out& q, Ws ws,
              uint32_t* mask, int32_t R, bool prepared, hipStream_t st, const char** err)
{
    int rc;
    if (p.n_neg == 0) {   // no candidates: n_valid only (0, or -1 for a skipped query)
        k_no_draws<QT><<<(p.batch + 255) / 256, 256, 0, st>>>(gv, p, q, nullptr, R);
        return check_launch(err);
    }
    if (!prepared) {
        k_prepare<QT, NoTally><<<(p.batch + 63) / 64, 256, 0, st>>>(gv, p, q, ws, nullptr, R);
        if ((rc = check_launch(err))) return rc;
    }
    k_pairs<QT><<<p.batch, CWG, 0, st>>>(gv, p, q, ws, mask);
    if ((rc = check_launch(err))) return rc;
    if constexpr (has_long_lists<QT>)
        return launch_long_lists<QT, NoTally>(gv, p, q, ws, nullptr, mask, st, err);
    return SMORE_OK;
}

int dispatch_pairs(QType qt, const GraphView& gv, const SampleParams& p, const smore_sample_out& q,
                   Ws ws, uint32_t* mask, int32_t R, bool prepared, hipStream_t st, const char** err)
{
    switch (qt) {
        case Q1P: return run_pairs<Q1P>(gv, p, q, ws, mask, R, prepared, st, err);
        case Q2P: return run_pairs<Q2P>(gv, p, q, ws, mask, R, prepared, st, err);
        case Q3P: return run_pairs<Q3P>(gv, p, q, ws, mask, R, prepared, st, err);
        case Q2I: return run_pairs<Q2I>(gv, p, q, ws, mask, R, prepared, st, err);
        case Q3I: return run_pairs<Q3I>(gv, p, q, ws, mask, R, prepared, st, err);
        case QIP: return run_pairs<QIP>(gv, p, q, ws, mask, R, prepared, st, err);
        case QPI: return run_pairs<QPI>(gv, p, q, ws, mask, R, prepared, st, err);
        case Q2U: return run_pairs<Q2U>(gv, p, q, ws, mask, R, prepared, st, err);
        case QUP: return run_pairs<QUP>(gv, p, q, ws, mask, R, prepared, st, err);
        case Q2IN: return run_pairs<Q2IN>(gv, p, q, ws, mask, R, prepared, st, err);
        case Q3IN: return run_pairs<Q3IN>(gv, p, q, ws, mask, R, prepared, st, err);
        case QINP: return run_pairs<QINP>(gv, p, q, ws, mask, R, prepared, st, err);
        case QPIN: return run_pairs<QPIN>(gv, p, q, ws, mask, R, prepared, st, err);
        case QPNI: return run_pairs<QPNI>(gv, p, q, ws, mask, R, prepared, st, err);
        default: *err = "unknown shape"; return SMORE_E_UNSUPPORTED;
    }
}

template <int QT> PrepLists lists_of()
{
    PrepLists l{};
    l.nf = Shape<QT>::nf;
    for (int f = 0; f < 3; ++f) {
        l.fa[f] = Shape<QT>::fa[f];
        l.fr[f] = Shape<QT>::fr[f];
    }
    return l;
}

PrepLists prep_lists(QType qt)
{
    switch (qt) {
        case Q1P: return lists_of<Q1P>();
        case Q2P: return lists_of<Q2P>();
        case Q3P: return lists_of<Q3P>();
        case Q2I: return lists_of<Q2I>();
        case Q3I: return lists_of<Q3I>();
        case QIP: return lists_of<QIP>();
        case QPI: return lists_of<QPI>();
        case Q2U: return lists_of<Q2U>();
        case QUP: return lists_of<QUP>();
        case Q2IN: return lists_of<Q2IN>();
        case Q3IN: return lists_of<Q3IN>();
        case QINP: return lists_of<QINP>();
        case QPIN: return lists_of<QPIN>();
        default: return lists_of<QPNI>();
    }
}

GraphView view_of(const smore_graph* g)
{
    GraphView gv;
    gv.fwd = DirView{g->f_node, g->f_grp, g->f_nbr};
    gv.rev = DirView{g->r_node, g->r_grp, g->r_nbr};
    gv.active_in = g->active_in;
    gv.has_in = g->has_in;
    gv.has_in4 = g->has_in4;
    gv.sig = g->sig;
    gv.first_test = g->V <= (1 << 22) ? TEST_SIG : g->V <= (1 << 26) ? TEST_MASK : TEST_MASK4;
    gv.V = g->V;
    gv.n_active = (int32_t)g->n_active;
    return gv;
}

}  // namespace

// Workspace of smore_sample_noalloc: a fixed array in device memory, one
// copy per GPU the library runs on, held until the process ends.  Host code
// never uses the array's name as an address: each device's address comes
// from hipGetSymbolAddress, taken once per device with that device current.
namespace {
static __device__ __align__(256) char scratch[SMORE_NOALLOC_SCRATCH_BYTES];
constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[MAX_DEVICES];
}  // namespace

int scratch_workspace(void** ptr, size_t* bytes, const char** err)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) {
        *err = "no usable current device for the fixed scratch";
        return SMORE_E_HIP;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            *err = e != hipSuccess ? hipGetErrorString(e) : "scratch has no device address";
            return SMORE_E_HIP;
        }
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    *bytes = SMORE_NOALLOC_SCRATCH_BYTES;
    return SMORE_OK;
}

void arm_wait(void* event) { g_wait = (hipEvent_t)event; }

void disarm()
{
    for (ProfileArm& a : g_prof) a = ProfileArm{};
    g_wait = nullptr;
}

void arm_profile(void* start_event, void* stop_event, int which)
{
    ProfileArm& a = g_prof[which];
    a.start = (start_event && stop_event) ? (hipEvent_t)start_event : nullptr;
    a.stop = (start_event && stop_event) ? (hipEvent_t)stop_event : nullptr;
}

size_t negatives_workspace_bytes(const SampleParams& p)
{
    return ws_layout(p, nullptr, nullptr);
}

// Attempt lanes per query (they divide 64).  Attempts past the first
// successful one are wasted reads, so plans that usually succeed at once run
// two.  Plans accept less often per attempt when sibling branches hang off
// the root (two of them must not draw the same in-relation and in-neighbour
// of the root, which seldom has many) or with a complemented operand: four
// lanes, eight with three root siblings; and a maximum expansion C rejects
// every attempt through a wider step: eight lanes.  Such plans get more as
// long as the call stays within one wavefront per SIMD (65,536 lanes), where
// the reads cost nothing and the kernel's time is that of its unluckiest
// query: with 64 lanes in place of 8 and the preparation in the same kernel, a
// 2p call of 1,024 queries at C = 10 (Freebase-shaped, 34 attempts on average)
// went from 137 to 67 us; with 8 in place of 4, 2i x 8,192 from 56 to 49.
inline int positive_lanes(const WalkProgram& wp, const SampleParams& p)
{
    const bool capped = p.max_fanout > 0;
    int pa = (wp.root_pairs >= 3 || capped) ? 8 : (wp.root_pairs > 0 || wp.neg_steps > 0) ? 4 : 2;
    const int most = capped ? 64 : pa > 2 ? 16 : 2;
    while (pa < most && (int64_t)p.batch * pa * 2 <= 65536) pa *= 2;
    return pa;
}

int launch_positive(const smore_graph* g, const WalkProgram& wp, const SampleParams& p,
                    const smore_sample_out& out, int qt, void* workspace, hipStream_t st,
                    const char** err)
{
    Ws ws{};
    PrepLists lists{};
    lists.nf = -1;
    if (workspace) {
        ws_layout(p, &ws, (char*)workspace);
        lists = prep_lists((QType)qt);
    }
    const int pa = positive_lanes(wp, p);
    const unsigned blocks = (unsigned)(((int64_t)p.batch * pa + 255) / 256);
    auto run = [&](auto kernel) { kernel<<<blocks, 256, 0, st>>>(view_of(g), wp, p, out, lists, ws); };
    switch (pa) {
        case 2: run(k_positive<2>); break;
        case 4: run(k_positive<4>); break;
        case 8: run(k_positive<8>); break;
        case 16: run(k_positive<16>); break;
        case 32: run(k_positive<32>); break;
        default: run(k_positive<64>); break;
    }
    return check_launch(err);
}

int launch_negative(const smore_graph* g, QType qt, const SampleParams& p,
                    const smore_sample_out& out, int64_t* stats, void* workspace, size_t ws_bytes,
                    int parts, hipStream_t st, const char** err)
{
    Ws ws;
    const size_t need = ws_layout(p, &ws, (char*)workspace);
    if (p.n_neg > 0 && (!workspace || ws_bytes < need)) {
        *err = "workspace too small (see smore_sample_workspace_bytes)";
        return SMORE_E_INVALID_ARG;
    }
    const GraphView gv = view_of(g);
    return stats ? dispatch_negatives<Tally>(qt, gv, p, out, ws, stats, g->R, parts, st, err)
                 : dispatch_negatives<NoTally>(qt, gv, p, out, ws, nullptr, g->R, parts, st, err);
}

int launch_shared(const smore_graph* g, QType qt, const SampleParams& p0, const smore_sample_out& pos,
                  int32_t* shared, int32_t* n_shared, uint32_t* mask, void* workspace,
                  size_t ws_bytes, hipStream_t st, const char** err)
{
    SampleParams p = p0;
    p.shared_mode = 1;
    p.shared = shared;
    p.n_shared = n_shared;
    p.cand_stride = 0;
    Ws ws;
    const size_t need = ws_layout(p, &ws, (char*)workspace);
    if (p.n_neg > 0 && (!workspace || ws_bytes < need)) {
        *err = "workspace too small (see smore_sample_workspace_bytes)";
        return SMORE_E_INVALID_ARG;
    }
    const GraphView gv = view_of(g);
    const int rc = draw_shared_set(p, gv.V, shared, n_shared, st, err);
    // an empty set leaves nothing to verify: the positives' n_valid (0, or -1
    // without a positive) is the row count, and no mask word exists
    if (rc || p.n_neg == 0) return rc;
    return dispatch_pairs(qt, gv, p, pos, ws, mask, g->R, true, st, err);
}

int launch_verify(const smore_graph* g, QType qt, const SampleParams& p0, const int32_t* anchors,
                  const int32_t* relations, const int32_t* candidates, uint32_t* mask,
                  int32_t* n_valid, void* workspace, size_t ws_bytes, hipStream_t st,
                  const char** err)
{
    SampleParams p = p0;
    p.shared_mode = 2;
    p.shared = candidates;
    p.n_shared = nullptr;
    p.cand_stride = p.n_neg;
    Ws ws;
    const size_t need = ws_layout(p, &ws, (char*)workspace);
    if (p.n_neg > 0 && (!workspace || ws_bytes < need)) {
        *err = "workspace too small (see smore_sample_workspace_bytes)";
        return SMORE_E_INVALID_ARG;
    }
    smore_sample_out q;
    std::memset(&q, 0, sizeof(q));
    q.anchors = (int32_t*)anchors;
    q.relations = (int32_t*)relations;
    q.n_valid = n_valid;
    return dispatch_pairs(qt, view_of(g), p, q, ws, mask, g->R, false, st, err);
}

}  // namespace smore
