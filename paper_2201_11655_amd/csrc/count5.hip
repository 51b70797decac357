// Per-vertex 5-motif counts: the method carried to 5-vertex motifs (Sec. 11 names
// 5-vertex motifs as the next case of the same claims and data structure).
//
// What is counted is what k = 3, 4 count (Sec. 4.1-4.2): every connected 5-set S is
// counted once, its index is read from the induced adjacency matrix (20 bits, first
// entry most significant), mapped to its isomorphism class (9364 weakly connected
// classes) and credited to all five members.
//
// How each set is reached once (Lemma 1 and the BFS shapes of Lemmas 2-4, one level
// further): S is reached from its lowest-rank vertex r only, along its BFS layering
// from r: layer 1 = the members adjacent to r, layer i + 1 = the members adjacent to
// layer i and to no earlier layer.  The layer sizes are the set's shape; five vertices
// have eight: (4) (3,1) (2,2) (2,1,1) (1,3) (1,2,1) (1,1,2) (1,1,1,1), the 4-vertex
// ones of Lemma 2 being the same construction on four.  Members are chosen in the
// order (layer, parent, position in the parent's row), where a member's parent is its
// first neighbour in the previous layer -- a vertex hangs under its lower-index parent,
// the rule of Lemma 3 -- and a candidate under parent x is taken only if it is
// adjacent to no member chosen before x: such a vertex lies in an earlier layer or
// under an earlier parent (the rule of Lemma 4, generalised).  So the layering, the
// parents and the choice order are all fixed by S, and each set is produced once.
//
// Graphs up to kFiveSetsMaxN vertices (k_five_sets).  The first three members T of a set
// fix the candidates C of the fourth: the rest of the third member's layer, then the next
// layer under it.  The last two members are then
//   * two of C: every pair of C once.  Pairs that are not adjacent and whose members have
//     the same arc codes to T share their index, so they are counted as groups, from the
//     number of candidates of each code; an adjacent pair is found from the row of either
//     member and moved to its own index;
//   * one y of C and a neighbour of y that is adjacent to no member of T.
// A workgroup takes a pair {r, a} of first members (from the heaviest roots on) and a wave a
// third member; the arc codes of r, of a and of the third member to all vertices lie in LDS
// as bit planes, so that a pair test is one LDS read.  Credits are summed in an LDS hash of
// (vertex, class), which leaves for the output when it fills: the triples of one pair credit
// the same few thousand cells over and over, and a credit that goes to the output by itself
// is a memory-side atomic.  What bounds it: issue and the latency of the class table's loads
// (2 MiB, in L2).  256 G(n, p) graphs of 20..500 vertices: 34.7 ms a call, 48.2 set by set;
// a fat-tailed graph of 2000 vertices (1.3e9 sets): 30 ms, 244 set by set.
//
// Larger graphs take the same search set by set over the graph in device memory
// (k_five_global): pair tests from the graph's edge hash, rows searched in place.
// Sets are counted per shape (the graph's 8 counters): their sum is the number of
// connected 5-sets.
#include <cmath>
#include <map>

#include <hipcub/hipcub.hpp>

#include "motif_device.h"
#include "vdmc_internal.h"

namespace vdmc {
namespace {

constexpr int64_t kFiveSetsMaxN = 16384;                       // bit planes of 9 members in LDS (36 KiB)
constexpr int64_t kFiveSetsMaxPairs = (int64_t)1 << 24;        // item table of at most 128 MiB
constexpr uint32_t kNone = 0xFFFFFFFFu;
// LDS counter slots per vertex: the 27 classes of 5-sets whose induced subgraph is a tree
// with single arcs (oriented paths, stars and forks without a reciprocal pair), which in a
// sparse digraph hold most of the credits (~84% on G(n, p) graphs of mean degree 10)
constexpr uint32_t kTreeSlots5 = 27;
constexpr int64_t kDenseMaxN = 512;                            // graphs with such counters (55 KiB)
constexpr uint32_t kTreeMark = 0x8000u;                        // these classes in the marked table: mark | slot
constexpr uint32_t kSplitDiv = 32;                             // sub-items of a root: d+ x deg / 32 (best of 2..128)

// bit of the index of a 5-set for the entry (i, j), i != j: rows in order, the diagonal
// skipped, entry (0,1) the most significant of the 20 (Sec. 4.1, Fig. 1)
__host__ __device__ __forceinline__ constexpr uint32_t shift5(uint32_t i, uint32_t j) {
    return 19u - (i * 4u + (j < i ? j : j - 1u));
}
// index bits of the pair (i, t), i < t, from the arc bits b seen from member i
// (bit 0: i -> t, bit 1: t -> i)
__device__ __forceinline__ uint32_t pair_bits(uint32_t i, uint32_t t, uint32_t b) {
    return ((b & 1u) << shift5(i, t)) | ((b >> 1) << shift5(t, i));
}

// A graph in device memory: pair tests and arc bits from the edge hash (one probe
// sequence), rows searched in place.
struct FiveGlobal {
    const uint32_t* off;
    const uint32_t* adj;
    const uint32_t* perm;
    const unsigned long long* eh;
    uint32_t ebits;
    __device__ __forceinline__ bool adjacent(uint32_t u, uint32_t v) const {
        return edge_code(eh, ebits, u, v) != 0u;
    }
    __device__ __forceinline__ uint32_t bits(uint32_t u, uint32_t v) const {
        return edge_code(eh, ebits, u, v);
    }
    __device__ __forceinline__ uint32_t first_above(uint32_t u, uint32_t x) const {
        uint32_t lo = off[u], hi = off[u + 1];
        const uint32_t key = (x + 1u) << 2;
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (adj[mid] < key) lo = mid + 1; else hi = mid;
        }
        return lo;
    }
};

// The members S[0..3] of the set being built (the fifth is the innermost loop's
// candidate).  Named fields rather than an array: a member picked by an index that is not
// a compile-time constant is a select, where an array would be placed in scratch memory.
struct Members {
    uint32_t v0, v1, v2, v3;
    __device__ __forceinline__ uint32_t operator[](uint32_t i) const {
        return i == 0u ? v0 : (i == 1u ? v1 : (i == 2u ? v2 : v3));
    }
};

// y adjacent to none of S[0..lim)
template <class V>
__device__ __forceinline__ bool clear_of(const V& L, const Members& S, uint32_t lim, uint32_t y) {
#pragma unroll
    for (uint32_t m = 0; m < 4; m++)
        if (m < lim && L.adjacent(S[m], y)) return false;
    return true;
}

// Candidates of the next member, given S[0..t): first the rest of S[t-1]'s layer (after
// S[t-1]'s parent and position), then -- phase 1 -- the first member of a new layer under
// the members of S[t-1]'s layer.  pi: S index of the current parent, [pi, pend) the
// parents left in the phase, [j, jend) the rest of the parent's row.
struct Cand {
    uint32_t pi, pend, j, jend, phase, ls, pbits;   // pbits: arc bits of the last candidate with its parent
    template <class V>
    __device__ __forceinline__ void start(const V& L, const Members& S, uint32_t par, uint32_t pos,
                                          uint32_t ls_prev) {
        pi = par;
        pend = ls_prev;
        j = pos + 1u;
        jend = L.off[S[par] + 1u];
        phase = 0u;
        ls = ls_prev;
    }
    // next candidate vertex, or kNone; t = the S index being chosen
    template <class V>
    __device__ __forceinline__ uint32_t next(const V& L, const Members& S, uint32_t t) {
        for (;;) {
            while (j < jend) {
                const uint32_t e = L.adj[j++], y = e >> 2;
                if (clear_of(L, S, pi, y)) {
                    pbits = e & 3u;
                    return y;
                }
            }
            if (++pi < pend) {
                const uint32_t x = S[pi];
                j = L.first_above(x, S[0]);
                jend = L.off[x + 1u];
                continue;
            }
            if (phase == 0u) {   // the layer of S[t-1] is closed: open the next one under it
                phase = 1u;
                pi = ls;
                pend = t;
                const uint32_t x = S[pi];
                j = L.first_above(x, S[0]);
                jend = L.off[x + 1u];
                continue;
            }
            return kNone;
        }
    }
};

// arc bits of (S[m], y) seen from S[m], for the candidate y just returned by c: its
// parent's come with the entry, members before the parent are not adjacent to it (the
// candidate rule), the others are looked up
template <class V>
__device__ __forceinline__ uint32_t arc_of(const V& L, const Members& S, uint32_t m, const Cand& c,
                                           uint32_t y) {
    if (m == c.pi) return c.pbits;
    if (m < c.pi) return 0u;
    return L.bits(S[m], y);
}

// a credit of v sets of class cls to vertex P (original id): one device-scope atomic
struct GlobalSink {
    unsigned long long* out;
    __device__ __forceinline__ void add(uint32_t P, uint32_t cls, uint32_t v) const {
        __hip_atomic_fetch_add(&out[(size_t)P * kClasses5 + cls], (unsigned long long)v, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
};

// v sets of class cls credited to the three members fixed over a depth-2 loop
template <class Sk>
__device__ __forceinline__ void credit3(const Sk& sk, uint32_t P0, uint32_t P1, uint32_t P2, uint32_t cls,
                                        uint32_t v) {
    sk.add(P0, cls, v);
    sk.add(P1, cls, v);
    sk.add(P2, cls, v);
}

// Per-lane cache of the classes credited to S[0], S[1], S[2] over one depth-2 loop (all
// fourth members under one third member): entry = (count << 14) | class, 0 = empty; the
// oldest entry makes room.  A count stays below 2^18: an entry about to pass it takes a
// new slot instead.
struct ClassCache {
    uint32_t e0 = 0, e1 = 0, e2 = 0, e3 = 0, e4 = 0, e5 = 0, e6 = 0, e7 = 0, victim = 0;
    static __device__ __forceinline__ bool take(uint32_t& e, uint32_t cls, uint32_t v) {
        if (e == 0u || (e & 0x3FFFu) != cls || (e >> 14) + v >= (1u << 18)) return false;
        e += v << 14;
        return true;
    }
    template <class Sk>
    __device__ __forceinline__ void add(uint32_t cls, uint32_t v, const Sk& sk, uint32_t P0, uint32_t P1,
                                        uint32_t P2) {
        if (take(e0, cls, v) || take(e1, cls, v) || take(e2, cls, v) || take(e3, cls, v) || take(e4, cls, v) ||
            take(e5, cls, v) || take(e6, cls, v) || take(e7, cls, v))
            return;
        const uint32_t e = (v << 14) | cls;
        uint32_t old;
        switch (victim) {
            case 0: old = e0; e0 = e; break;
            case 1: old = e1; e1 = e; break;
            case 2: old = e2; e2 = e; break;
            case 3: old = e3; e3 = e; break;
            case 4: old = e4; e4 = e; break;
            case 5: old = e5; e5 = e; break;
            case 6: old = e6; e6 = e; break;
            default: old = e7; e7 = e; break;
        }
        victim = (victim + 1u) & 7u;
        if (old) credit3(sk, P0, P1, P2, old & 0x3FFFu, old >> 14);
    }
    template <class Sk>
    __device__ __forceinline__ void flush_all(const Sk& sk, uint32_t P0, uint32_t P1, uint32_t P2) {
        if (e0) credit3(sk, P0, P1, P2, e0 & 0x3FFFu, e0 >> 14);
        if (e1) credit3(sk, P0, P1, P2, e1 & 0x3FFFu, e1 >> 14);
        if (e2) credit3(sk, P0, P1, P2, e2 & 0x3FFFu, e2 >> 14);
        if (e3) credit3(sk, P0, P1, P2, e3 & 0x3FFFu, e3 >> 14);
        if (e4) credit3(sk, P0, P1, P2, e4 & 0x3FFFu, e4 >> 14);
        if (e5) credit3(sk, P0, P1, P2, e5 & 0x3FFFu, e5 >> 14);
        if (e6) credit3(sk, P0, P1, P2, e6 & 0x3FFFu, e6 >> 14);
        if (e7) credit3(sk, P0, P1, P2, e7 & 0x3FFFu, e7 >> 14);
        e0 = e1 = e2 = e3 = e4 = e5 = e6 = e7 = 0u;
        victim = 0u;
    }
};

// v sets of class cls of one context: the fourth member credited now, the three before it
// through the class cache
template <class Sk>
__device__ __forceinline__ void credit_ctx(const Sk& sk, ClassCache& cc, uint32_t P0, uint32_t P1, uint32_t P2,
                                           uint32_t P3, uint32_t cls, uint32_t v) {
    if (v == 0u || cls >= (uint32_t)kClasses5) return;
    sk.add(P3, cls, v);
    cc.add(cls, v, sk, P0, P1, P2);
}

// Per-lane cache of the last member's signatures in one context: entry = (count << 22) |
// (class << 8) | signature, 0 = empty (a signature is never 0: the last member has an
// arc to its parent); the oldest entry makes room.  A count stays below 1023: a signature
// whose entry is full takes a new one.
struct SigCache {
    uint32_t e0 = 0, e1 = 0, e2 = 0, e3 = 0, victim = 0;
    static __device__ __forceinline__ bool take(uint32_t& e, uint32_t sig) {
        if ((e & 255u) != sig || (e >> 22) >= 1023u) return false;
        e += 1u << 22;
        return true;
    }
    static __device__ __forceinline__ uint32_t cls_of(uint32_t e) { return (e >> 8) & 0x3FFFu; }
    // class of a cached signature (its count raised by one), or kNone
    __device__ __forceinline__ uint32_t hit(uint32_t sig) {
        if (take(e0, sig)) return cls_of(e0);
        if (take(e1, sig)) return cls_of(e1);
        if (take(e2, sig)) return cls_of(e2);
        if (take(e3, sig)) return cls_of(e3);
        return kNone;
    }
    template <class Sk>
    __device__ __forceinline__ void insert(uint32_t sig, uint32_t cls, const Sk& sk, ClassCache& cc, uint32_t P0,
                                           uint32_t P1, uint32_t P2, uint32_t P3) {
        const uint32_t e = (1u << 22) | ((cls & 0x3FFFu) << 8) | sig;
        uint32_t old;
        switch (victim) {
            case 0: old = e0; e0 = e; break;
            case 1: old = e1; e1 = e; break;
            case 2: old = e2; e2 = e; break;
            default: old = e3; e3 = e; break;
        }
        victim = (victim + 1u) & 3u;
        credit_ctx(sk, cc, P0, P1, P2, P3, cls_of(old), old >> 22);
    }
    template <class Sk>
    __device__ __forceinline__ void flush_all(const Sk& sk, ClassCache& cc, uint32_t P0, uint32_t P1, uint32_t P2,
                                              uint32_t P3) {
        credit_ctx(sk, cc, P0, P1, P2, P3, cls_of(e0), e0 >> 22);
        credit_ctx(sk, cc, P0, P1, P2, P3, cls_of(e1), e1 >> 22);
        credit_ctx(sk, cc, P0, P1, P2, P3, cls_of(e2), e2 >> 22);
        credit_ctx(sk, cc, P0, P1, P2, P3, cls_of(e3), e3 >> 22);
    }
};

// visited sets of one shape added to the workgroup's shape counters (LDS)
__device__ __forceinline__ void add_shape(unsigned long long* vis, uint32_t s, uint32_t v) {
    if (v) atomicAdd(&vis[s], (unsigned long long)v);
}

// Sub-items per (root, first layer-1 member) of a root with dhi higher neighbours and
// degree deg: the heavy roots' items are cut by the choice of the third member (every
// K-th candidate), so that no single lane carries a hub root's whole subtree.
__device__ __forceinline__ uint32_t item_split(uint32_t dhi, uint32_t deg, uint32_t div) {
    return min(64u, max(1u, (dhi * deg + div - 1u) / div));
}

// Every set of the sub-item k of K of the item (root r, first layer-1 member at entry apos
// of r's row).
template <class V, class Sk>
__device__ void five_item(const V& L, const uint16_t* __restrict__ table, const Sk& sk,
                          uint32_t r, uint32_t apos, uint32_t k, uint32_t K, unsigned long long* vis) {
    Members S{r, L.adj[apos] >> 2, 0u, 0u};
    const uint32_t code1 = pair_bits(0, 1, L.adj[apos] & 3u);
    const uint32_t P0 = L.perm[r], P1 = L.perm[S[1]];
    Cand c2;
    c2.start(L, S, 0u, apos, 1u);   // S[1]'s parent is S[0]; layer 1 starts at index 1
    uint32_t ord2 = 0;
    for (;;) {
        const uint32_t y2 = c2.next(L, S, 2u);
        if (y2 == kNone) break;
        if (ord2++ % K != k) continue;   // another sub-item's third member
        S.v2 = y2;
        const uint32_t par2 = c2.pi, pos2 = c2.j - 1u, ls2 = c2.phase ? 2u : 1u;
        const uint32_t code2 = code1 | pair_bits(0, 2, arc_of(L, S, 0, c2, y2)) | pair_bits(1, 2, arc_of(L, S, 1, c2, y2));
        const uint32_t P2 = L.perm[y2];
        ClassCache cc;
        Cand c3;
        c3.start(L, S, par2, pos2, ls2);
        for (;;) {
            const uint32_t y3 = c3.next(L, S, 3u);
            if (y3 == kNone) break;
            S.v3 = y3;
            const uint32_t par3 = c3.pi, pos3 = c3.j - 1u, ls3 = c3.phase ? 3u : ls2;
            const uint32_t code3 = code2 | pair_bits(0, 3, arc_of(L, S, 0, c3, y3)) |
                                   pair_bits(1, 3, arc_of(L, S, 1, c3, y3)) | pair_bits(2, 3, arc_of(L, S, 2, c3, y3));
            const uint32_t P3 = L.perm[y3];
            Cand c4;
            c4.start(L, S, par3, pos3, ls3);
            uint32_t same = 0, opened = 0;   // sets whose last member continues / opens a layer
            // The last member y4 of a set is credited once per set.  The fixed members are
            // credited per distinct signature of y4 -- its arc bits with S[0..3], which with
            // code3 fix the class -- through a 4-entry cache of (signature, count, class): a
            // context of a sparse graph holds ~8-25 sets with ~4-5 signatures, so this
            // removes most of the fixed members' credits and class reads.  An evicted entry
            // credits S[3], and S[0..2] directly or through the class cache (sink's choice).
            SigCache sc;
            for (;;) {
                const uint32_t y4 = c4.next(L, S, 4u);
                if (y4 == kNone) break;
                const uint32_t b0 = arc_of(L, S, 0, c4, y4), b1 = arc_of(L, S, 1, c4, y4),
                               b2 = arc_of(L, S, 2, c4, y4), b3 = arc_of(L, S, 3, c4, y4);
                const uint32_t sig = b0 | (b1 << 2) | (b2 << 4) | (b3 << 6);
                uint32_t cls = sc.hit(sig);
                if (cls == kNone) {
                    cls = table[code3 | pair_bits(0, 4, b0) | pair_bits(1, 4, b1) | pair_bits(2, 4, b2) |
                                pair_bits(3, 4, b3)];
                    sc.insert(sig, cls, sk, cc, P0, P1, P2, P3);
                }
                if (cls < (uint32_t)kClasses5) sk.add(L.perm[y4], cls, 1u);
                if (c4.phase) opened++; else same++;
            }
            sc.flush_all(sk, cc, P0, P1, P2, P3);
            // shape id: bit 2 = a new layer opens at member 2, bit 1 at member 3, bit 0 at member 4
            const uint32_t base = (ls2 == 2u ? 4u : 0u) | (ls3 == 3u ? 2u : 0u);
            add_shape(vis, base, same);
            add_shape(vis, base | 1u, opened);
        }
        cc.flush_all(sk, P0, P1, P2);
    }
}


// ----------------------------------------------------------------------------- graphs in device memory

struct FiveGlobalArgs {
    FiveGlobal L;
    const uint32_t* split;
    const unsigned long long* hp;   // n + 1: items (sub-items) before each root
    uint32_t n;
    unsigned long long total;
    unsigned long long* out;        // n x 9364, shared by every workgroup
    unsigned long long* stats;
    unsigned long long* cursor;     // item cursor, zeroed before the launch
    const uint16_t* table;
    uint32_t split_div;
};

// items of each root: d+(r) x K(r); cnt[n] = 0 so that an exclusive scan over n + 1 gives the total
__global__ void k_five_counts(const uint32_t* off, const uint32_t* split, uint32_t n, uint32_t div,
                              unsigned long long* cnt) {
    const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r > n) return;
    if (r == n) {
        cnt[n] = 0ull;
        return;
    }
    const uint32_t dhi = off[r + 1] - split[r];
    cnt[r] = (unsigned long long)dhi * item_split(dhi, off[r + 1] - off[r], div);
}

template <int BS>
__global__ __launch_bounds__(BS) void k_five_global(FiveGlobalArgs A) {
    __shared__ unsigned long long s_vis[8];
    const uint32_t tid = threadIdx.x;
    if (tid < 8) s_vis[tid] = 0ull;
    __syncthreads();
    for (;;) {
        const unsigned long long i = atomicAdd(A.cursor, 1ull);
        if (i >= A.total) break;
        uint32_t lo = 0, hi = A.n;   // root: last r with hp[r] <= i
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (A.hp[mid] <= i) lo = mid; else hi = mid;
        }
        const uint32_t r = lo, e = A.L.off[r + 1], sp = A.split[r];
        const uint32_t K = item_split(e - sp, e - A.L.off[r], A.split_div);
        const uint32_t local = (uint32_t)(i - A.hp[r]);
        five_item(A.L, A.table, GlobalSink{A.out}, r, sp + local / K, local % K, K, s_vis);
    }
    __syncthreads();
    if (tid < 8 && s_vis[tid]) atomicAdd(&A.stats[tid], s_vis[tid]);
}

// ----------------------------------------------------------------------------- sets in groups

struct SetsGraph {
    gptr<const uint32_t> off;           // n + 1 (rank space)
    gptr<const uint32_t> adj;           // entries: (nbr_rank << 2) | arc bits
    gptr<const uint32_t> split;         // first entry above the row's vertex
    gptr<const int32_t> perm;           // rank -> original id
    gptr<unsigned long long> out;       // n x 9364, rows by original id
    gptr<unsigned long long> stats;     // 8 shape counters
    uint32_t n;
    uint32_t first;                // items of the graphs before it in the table
};

struct SetsArgs {
    const SetsGraph* graphs;       // device array, or nullptr: the graph `one`
    SetsGraph one;
    const uint2* items;            // per graph from its `first` on: (r, entry of a first layer-1 member in
                                   // r's row); an item covers `step` members from there on, see item_step
    const uint32_t* slots;         // graphs in the order workgroups take them, or nullptr: all `one`
    uint32_t nslots;
    unsigned* cursors;             // slot cursor, then per graph its item cursor and number of items
    const uint16_t* table;         // code -> class id, with LDS counters the marked table
    const uint16_t* slot_cls;      // LDS counter slot -> class (kTreeSlots5 entries)
    uint32_t words;                // words of a bit plane, of the largest graph
    uint32_t dense;                // counters in LDS: the largest graph's vertices, or 0
};

// First layer-1 members of r in one item: about 100 third members, so that an item keeps a
// workgroup busy and a heavy root still spreads over many.
__device__ __forceinline__ uint32_t item_step(uint32_t dhi, uint32_t deg) { return max(1u, 96u / (dhi + deg)); }

// the items of every graph, one workgroup each, in rank order; their number behind the graph's cursor
constexpr int kItemThreads = 1024;
__global__ __launch_bounds__(kItemThreads) void k_five_items(const SetsGraph* graphs, SetsGraph one, uint2* items,
                                                             unsigned* cursors) {
    __shared__ uint32_t part[kItemThreads];
    const SetsGraph G = graphs ? graphs[blockIdx.x] : one;
    const uint32_t tid = threadIdx.x, per = (G.n + kItemThreads - 1) / kItemThreads;
    const uint32_t lo = min(G.n, tid * per), hi = min(G.n, lo + per);
    uint32_t s = 0;
    for (uint32_t r = lo; r < hi; r++) {
        const uint32_t d = G.off[r + 1] - G.split[r], st = d ? item_step(d, G.off[r + 1] - G.off[r]) : 1u;
        s += (d + st - 1u) / st;
    }
    part[tid] = s;
    __syncthreads();
    for (uint32_t o = 1; o < kItemThreads; o <<= 1) {
        const uint32_t v = tid >= o ? part[tid - o] : 0u;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    uint32_t at = G.first + part[tid] - s;
    for (uint32_t r = lo; r < hi; r++) {
        const uint32_t t0 = G.split[r], t1 = G.off[r + 1];
        if (t0 == t1) continue;
        for (uint32_t t = t0, st = item_step(t1 - t0, t1 - G.off[r]); t < t1; t += st) items[at++] = make_uint2(r, t);
    }
    if (tid == kItemThreads - 1) cursors[2u + 2u * blockIdx.x] = part[tid];
}

// outputs, counters and item cursors of every graph to zero (blockIdx.y strides over the
// graphs), the slot cursor too
__global__ __launch_bounds__(256) void k_five_zero(SetsArgs A, uint32_t num) {
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) A.cursors[0] = 0u;
    for (uint32_t g = blockIdx.y; g < num; g += gridDim.y) {
        const SetsGraph& G = A.graphs ? A.graphs[g] : A.one;
        const size_t cells = (size_t)G.n * kClasses5, stride = (size_t)gridDim.x * 256;
        const size_t t0 = (size_t)blockIdx.x * 256 + threadIdx.x;
        if (((uintptr_t)G.out.p & 15u) == 0) {   // 16-byte stores (9364 is even)
            using u64x2 = unsigned long long __attribute__((ext_vector_type(2)));
            const auto o = G.out.as<u64x2>();
            for (size_t i = t0; i < cells / 2; i += stride) o[i] = u64x2{0ull, 0ull};
        } else {
            for (size_t i = t0; i < cells; i += stride) G.out[i] = 0ull;
        }
        if (blockIdx.x == 0 && threadIdx.x < kStatSlots) G.stats[threadIdx.x] = 0ull;
        if (blockIdx.x == 0 && threadIdx.x == 0) A.cursors[1u + 2u * g] = 0u;
    }
}

// State of one wave (a triple of first members at a time).
struct SetsWave {
    uint32_t hist[64];     // candidates by signature (arc codes to r, a, the third member)
    uint32_t lone[48];     // (signature's place, arc code): last members below a candidate (up to 16 signatures)
    uint32_t buf[64];      // candidates in hand: vertex | signature << 14 | phase << 20
    uint32_t lo[64], hi[64];   // their rows
    uint16_t kcls[3 * 64]; // classes of the sets that a neighbour of theirs alone completes, by arc code
    uint16_t cls[256];     // class of two non-adjacent candidates by their signatures (up to 16 of them)
    uint8_t sig[64];       // the signatures that occur
    uint8_t idx[64];       // signature -> its place in sig
};

// a workgroup's credits: counters of the tree classes of every vertex (small graphs), a hash
struct SetsCounters {
    lptr<uint32_t> dense;  // n x kTreeSlots5 (classes marked kTreeMark)
    lptr<uint32_t> key;    // hash: vertex << 14 | class, or kNone
    lptr<uint32_t> val;
    lptr<uint32_t> used;
    uint32_t shift;        // 2^(32 - shift) cells
};

__device__ __forceinline__ uint32_t lds_add(lptr<uint32_t> p, uint32_t v) {
    return __hip_atomic_fetch_add(p.p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// *p = want if it is `expect`; old: what it was
__device__ __forceinline__ bool lds_cas(lptr<uint32_t> p, uint32_t expect, uint32_t want, uint32_t& old) {
    old = expect;
    return __hip_atomic_compare_exchange_strong(p.p, &old, want, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_WORKGROUP);
}

// credit cell (v, cls) += n: the LDS counter of a tree class, else through the hash; a full
// neighbourhood of cells: to the output.  The hash's 32-bit sums carry into the output; a
// dense counter cannot overflow (fewer than 2^32 5-sets hold a vertex of 512).
struct SetsSink {
    const SetsCounters L;
    const SetsGraph G;
    __device__ __forceinline__ gptr<unsigned long long> cell(uint32_t key) const {
        return &G.out[(size_t)G.perm[key >> 14] * kClasses5 + (key & 0x3FFFu)];
    }
    __device__ __forceinline__ uint32_t find(uint32_t key) const {
        const uint32_t mask = ~0u >> L.shift;
        uint32_t h = (key * 2654435761u) >> L.shift;
        for (int i = 0; i < 16; i++, h = (h + 1u) & mask) {
            uint32_t k = L.key[h];
            if (k == kNone) {
                if (lds_cas(&L.key[h], kNone, key, k)) {
                    lds_add(L.used, 1u);
                    return h;
                }
            }
            if (k == key) return h;
        }
        return kNone;
    }
    __device__ __forceinline__ void add(uint32_t v, uint32_t cls, uint32_t n) const {
        if (cls & kTreeMark) {
            lds_add(&L.dense[v * kTreeSlots5 + (cls & 31u)], n);
            return;
        }
        const uint32_t key = (v << 14) | cls, h = find(key);
        if (h == kNone) {
            gadd64(cell(key), n);
            return;
        }
        const uint32_t old = lds_add(&L.val[h], n);
        if (old + n < old) gadd64(cell(key), 1ull << 32);
    }
    __device__ __forceinline__ void sub1(uint32_t v, uint32_t cls) const {
        if (cls & kTreeMark) {
            lds_add(&L.dense[v * kTreeSlots5 + (cls & 31u)], ~0u);
            return;
        }
        const uint32_t key = (v << 14) | cls, h = find(key);
        if (h == kNone) {
            gadd64(cell(key), ~0ull);
            return;
        }
        if (lds_add(&L.val[h], ~0u) == 0u) gadd64(cell(key), 0ull - (1ull << 32));
    }
};

// arc code of a member with vertex z from the member's bit planes (both planes of a word side by side)
__device__ __forceinline__ uint32_t plane_code(const uint2* P, uint32_t z) {
    const uint2 w = P[z >> 5];
    return ((w.x >> (z & 31u)) & 1u) | (((w.y >> (z & 31u)) & 1u) << 1);
}

// index bits of a member t = 3 or 4 with the codes sig to members 0, 1, 2
__device__ __forceinline__ uint32_t sig_bits(uint32_t t, uint32_t sig) {
    return pair_bits(0, t, sig & 3u) | pair_bits(1, t, (sig >> 2) & 3u) | pair_bits(2, t, sig >> 4);
}

// Every set whose first three members are r, a and y2 = the vertex of entry q (of r's row:
// y2 shares a's layer; of a's row: y2 opens the next), by one wave.
__device__ __forceinline__ void five_triple(const SetsGraph& G, const SetsSink& K, SetsWave& S,
                                            const uint16_t* __restrict__ table, const uint2* PR, const uint2* PA,
                                            uint2* PY, uint32_t W, uint32_t r, uint32_t a, uint32_t q, bool same,
                                            unsigned long long* vis) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t y2 = G.adj[q] >> 2;
    const uint32_t ylo = G.off[y2], yhi = G.off[y2 + 1];
    for (uint32_t i = lane; i < W; i += 64) PY[i] = make_uint2(0u, 0u);
    S.hist[lane] = 0u;
    if (lane < 48u) S.lone[lane] = 0u;
    wave_fence();
    for (uint32_t i = ylo + lane; i < yhi; i += 64) {
        const uint32_t e = G.adj[i], z = e >> 2, bit = 1u << (z & 31u);
        if (e & 1u) atomicOr(&PY[z >> 5].x, bit);
        if (e & 2u) atomicOr(&PY[z >> 5].y, bit);
    }
    wave_fence();
    const uint32_t code3 = pair_bits(0, 1, plane_code(PR, a)) | pair_bits(0, 2, plane_code(PR, y2)) |
                           pair_bits(1, 2, plane_code(PA, y2));
    // rows that hold the candidates, one after the other: the rest of the third member's
    // layer (phase 0), then the rows of a (if y2 shares its layer) and of y2 (phase 1)
    const uint32_t l0 = (same ? G.off[r + 1] : G.off[a + 1]) - q - 1u;
    const uint32_t l1 = same ? G.off[a + 1] - G.off[a] : 0u, l2 = yhi - ylo, len = l0 + l1 + l2;
    // candidate i: its vertex, signature and phase as in S.buf, or kNone
    auto candidate = [&](uint32_t i) -> uint32_t {
        if (i >= len) return kNone;
        const uint32_t ph = i >= l0 ? 1u : 0u;
        const uint32_t at = i < l0 ? q + 1u + i : (i < l0 + l1 ? G.off[a] + i - l0 : ylo + i - l0 - l1);
        const uint32_t z = G.adj[at] >> 2;
        if (z <= r) return kNone;
        const uint32_t cr = plane_code(PR, z), ca = plane_code(PA, z), cy = plane_code(PY, z);
        if ((ph || !same) && cr) return kNone;             // adjacent to r: layer 1
        if (i >= l0 + l1 && ca) return kNone;              // adjacent to a: hangs under a, or in y2's layer
        return z | ((cr | (ca << 2) | (cy << 4)) << 14) | (ph << 20);
    };
    uint32_t c0 = 0, c1 = 0;
    for (uint32_t i0 = 0; i0 < len; i0 += 64) {
        const uint32_t c = candidate(i0 + lane);
        if (c != kNone) atomicAdd(&S.hist[(c >> 14) & 63u], 1u);
        c0 += (uint32_t)__popcll(__ballot(c != kNone && !(c >> 20)));
        c1 += (uint32_t)__popcll(__ballot(c != kNone && (c >> 20)));
    }
    if (c0 + c1 == 0u) return;
    wave_fence();
    const bool in = S.hist[lane] != 0u;
    const unsigned long long occ = __ballot(in);
    const uint32_t D = (uint32_t)__popcll(occ);
    if (in) {
        const uint32_t at = (uint32_t)__popcll(occ & ((1ull << lane) - 1ull));
        S.sig[at] = (uint8_t)lane;
        S.idx[lane] = (uint8_t)at;
    }
    wave_fence();
    // ---- pairs of candidates as if not adjacent: the three first members' credits
    const bool small = D <= 16u;
    for (uint32_t i = lane; i < D * D; i += 64) {
        const uint32_t p = i / D, t = i - p * D;
        if (t < p && !small) continue;
        const uint32_t cls = table[code3 | sig_bits(3, S.sig[p]) | sig_bits(4, S.sig[t])];
        if (small) S.cls[i] = (uint16_t)cls;
        if (t < p) continue;
        const uint32_t np = S.hist[S.sig[p]];
        const uint32_t n = p == t ? np * (np - 1u) / 2u : np * S.hist[S.sig[t]];
        if (n) {
            K.add(r, cls, n);
            K.add(a, cls, n);
            K.add(y2, cls, n);
        }
    }
    const uint32_t base = same ? 0u : 4u;
    if (lane == 0) {
        atomicAdd(&vis[base], (unsigned long long)c0 * (c0 - 1u) / 2u);
        atomicAdd(&vis[base + 1u], (unsigned long long)c0 * c1);
        atomicAdd(&vis[base + 2u], (unsigned long long)c1 * (c1 - 1u) / 2u);
    }
    wave_fence();
    auto pair_class = [&](uint32_t s, uint32_t t) -> uint32_t {
        return small ? S.cls[S.idx[s] * D + S.idx[t]] : table[code3 | sig_bits(3, s) | sig_bits(4, t)];
    };
    // ---- the candidates again, 64 in hand at a time
    uint32_t lone0 = 0, lone1 = 0;
    for (uint32_t i0 = 0; i0 < len; i0 += 64) {
        const uint32_t c = candidate(i0 + lane);
        const unsigned long long m = __ballot(c != kNone);
        const uint32_t nb = (uint32_t)__popcll(m);
        if (nb == 0u) continue;
        if (c != kNone) {
            const uint32_t y = c & 0x3FFFu, s = (c >> 14) & 63u, at = (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
            const uint32_t code4 = code3 | sig_bits(3, s);
            S.buf[at] = c;
            S.lo[at] = G.off[y];
            S.hi[at] = G.off[y + 1];
            for (uint32_t k = 0; k < 3; k++) S.kcls[at * 3u + k] = table[code4 | pair_bits(3, 4, k + 1u)];
            // c with every other candidate, by signature, as if not adjacent
            for (uint32_t t = 0; t < D; t++) {
                const uint32_t st = S.sig[t], n = S.hist[st] - (st == s ? 1u : 0u);
                if (n) K.add(y, pair_class(s, st), n);
            }
        }
        wave_fence();
        // 8 lanes per candidate y: y's row above r
        for (uint32_t b0 = 0; b0 < nb; b0 += 8) {
            const uint32_t bi = b0 + (lane >> 3), gl = lane & 7u;
            const bool on = bi < nb;
            const uint32_t e = on ? S.buf[bi] : kNone;
            const uint32_t y = e & 0x3FFFu, s = (e >> 14) & 63u;
            const uint32_t code4 = code3 | sig_bits(3, s);
            uint32_t n1 = 0, n2 = 0, n3 = 0;
            const uint32_t hi = on ? S.hi[bi] : 0u;
            for (uint32_t i = (on ? S.lo[bi] : 0u) + gl; i < hi; i += 8u) {
                const uint32_t ent = G.adj[i], z = ent >> 2, k = ent & 3u;
                if (z <= r) continue;
                const uint32_t cr = plane_code(PR, z), ca = plane_code(PA, z), cy = plane_code(PY, z);
                if (!(cr | ca | cy)) {   // adjacent to none of the first three: the last member
                    n1 += k == 1u;
                    n2 += k == 2u;
                    n3 += k == 3u;
                    K.add(z, S.kcls[bi * 3u + k - 1u], 1u);
                    continue;
                }
                // a candidate too?  It comes after y2 where it shares y2's row of choice.
                const bool in = same ? (cr ? z > y2 : true) : (cr ? false : (ca ? z > y2 : true));
                if (!in || z == a) continue;
                const uint32_t sz = cr | (ca << 2) | (cy << 4);
                const uint32_t was = pair_class(s, sz), is = table[code4 | sig_bits(4, sz) | pair_bits(3, 4, k)];
                K.add(y, is, 1u);
                K.sub1(y, was);
                if (y < z) {
                    K.add(r, is, 1u);
                    K.add(a, is, 1u);
                    K.add(y2, is, 1u);
                    K.sub1(r, was);
                    K.sub1(a, was);
                    K.sub1(y2, was);
                }
            }
            for (int o = 1; o < 8; o <<= 1) {
                n1 += (uint32_t)__shfl_xor((int)n1, o, 64);
                n2 += (uint32_t)__shfl_xor((int)n2, o, 64);
                n3 += (uint32_t)__shfl_xor((int)n3, o, 64);
            }
            if (on && gl < 3u) {
                const uint32_t n = gl == 0u ? n1 : (gl == 1u ? n2 : n3);
                if (n) {
                    K.add(y, S.kcls[bi * 3u + gl], n);
                    if (small) {
                        atomicAdd(&S.lone[S.idx[s] * 3u + gl], n);
                    } else {
                        K.add(r, S.kcls[bi * 3u + gl], n);
                        K.add(a, S.kcls[bi * 3u + gl], n);
                        K.add(y2, S.kcls[bi * 3u + gl], n);
                    }
                    if (e >> 20) lone1 += n;
                    else lone0 += n;
                }
            }
        }
        wave_fence();
    }
    for (uint32_t i = lane; small && i < D * 3u; i += 64) {
        const uint32_t n = S.lone[i];
        if (!n) continue;
        const uint32_t cls = table[code3 | sig_bits(3, S.sig[i / 3u]) | pair_bits(3, 4, i % 3u + 1u)];
        K.add(r, cls, n);
        K.add(a, cls, n);
        K.add(y2, cls, n);
    }
    if (lone0) atomicAdd(&vis[base + 1u], (unsigned long long)lone0);
    if (lone1) atomicAdd(&vis[base + 3u], (unsigned long long)lone1);
    wave_fence();
}

// Per workgroup of BS threads: LDS planes of r, and per wave of a and of the third member;
// the tree counters (A.dense) and the hash of 2^hbits cells.
template <int BS>
__global__ __launch_bounds__(BS) void k_five_sets(SetsArgs A, uint32_t hbits) {
    constexpr uint32_t NWV = BS / 64;
    extern __shared__ uint2 dyn[];
    __shared__ SetsWave wv[NWV];
    __shared__ unsigned long long vis[8];
    __shared__ uint32_t sUsed, sNext, sTask;
    const uint32_t tid = threadIdx.x, wid = tid >> 6, lane = tid & 63u, hn = 1u << hbits;
    uint2* PR = dyn;
    uint2* PA = dyn + (1u + wid) * A.words;
    uint2* PY = dyn + (1u + NWV + wid) * A.words;
    uint32_t* key = (uint32_t*)(dyn + (1u + 2u * NWV) * A.words);
    uint32_t* val = key + hn;
    uint32_t* dense = val + hn;
    const SetsCounters L{dense, key, val, &sUsed, 32u - hbits};
    for (uint32_t i = tid; i < hn; i += BS) {
        key[i] = kNone;
        val[i] = 0u;
    }
    for (uint32_t i = tid; i < A.dense * kTreeSlots5; i += BS) dense[i] = 0u;
    if (tid < 8) vis[tid] = 0ull;
    if (tid == 0) sUsed = 0u;
    for (;;) {   // a slot: a graph's items until none are left
        __syncthreads();
        if (tid == 0) sNext = atomicAdd(&A.cursors[0], 1u);
        __syncthreads();
        const uint32_t slot = sNext;
        if (slot >= A.nslots) break;
        const uint32_t g = A.slots ? A.slots[slot] : 0u;
        const SetsGraph G = A.graphs ? A.graphs[g] : A.one;
        unsigned* cursor = &A.cursors[1u + 2u * g];
        const uint32_t nitems = cursor[1], W = (G.n + 31u) >> 5;
        const SetsSink K{L, G};
        auto empty_hash = [&]() {
            for (uint32_t i = tid; i < hn; i += BS) {
                const uint32_t k = key[i], n = val[i];
                if (k == kNone) continue;
                if (n) gadd64(K.cell(k), n);
                key[i] = kNone;
                val[i] = 0u;
            }
            if (tid == 0) sUsed = 0u;
            __syncthreads();
        };
        __syncthreads();
        if (tid == 0) sNext = atomicAdd(cursor, 1u);
        __syncthreads();
        uint32_t cur_r = kNone, cur_a = kNone;
        bool any = false;
        for (;;) {
            const uint32_t item = sNext;
            const bool full = sUsed > hn / 8u * 5u;
            if (item >= nitems) break;
            any = true;
            const uint2 it = A.items[G.first + item];
            const uint32_t r = it.x, r1 = G.off[r + 1], deg = r1 - G.off[r];
            const uint32_t t1 = min(r1, it.y + item_step(r1 - G.split[r], deg));
            __syncthreads();   // sNext and sUsed are read
            if (full) empty_hash();
            if (r != cur_r)
                for (uint32_t i = tid; i < W; i += BS) PR[i] = make_uint2(0u, 0u);
            if (tid == 0) sTask = 0u;
            __syncthreads();
            if (r != cur_r)
                for (uint32_t i = G.off[r] + tid; i < r1; i += BS) {
                    const uint32_t e = G.adj[i], z = e >> 2, bit = 1u << (z & 31u);
                    if (e & 1u) atomicOr(&PR[z >> 5].x, bit);
                    if (e & 2u) atomicOr(&PR[z >> 5].y, bit);
                }
            cur_r = r;
            if (tid == 0) sNext = atomicAdd(cursor, 1u);
            __syncthreads();
            // tasks: third members, for each a of the item the rest of r's row, then a's row
            uint32_t t = it.y, base = 0, a = G.adj[t] >> 2, a0 = G.off[a], a1 = G.off[a + 1];
            for (;;) {
                uint32_t task = 0;
                if (lane == 0) task = atomicAdd(&sTask, 1u);
                task = (uint32_t)__builtin_amdgcn_readfirstlane((int)task);
                while (t < t1 && task >= base + (r1 - t - 1u) + (a1 - a0)) {
                    base += (r1 - t - 1u) + (a1 - a0);
                    if (++t == t1) break;
                    a = G.adj[t] >> 2;
                    a0 = G.off[a];
                    a1 = G.off[a + 1];
                }
                if (t >= t1) break;
                const uint32_t nx = r1 - t - 1u, i = task - base;
                const bool same = i < nx;
                const uint32_t q = same ? t + 1u + i : a0 + i - nx;
                if (!same) {
                    const uint32_t z = G.adj[q] >> 2;
                    if (z <= r || plane_code(PR, z)) continue;
                }
                if (a != cur_a) {   // this wave's planes of a
                    cur_a = a;
                    for (uint32_t x = lane; x < W; x += 64) PA[x] = make_uint2(0u, 0u);
                    wave_fence();
                    for (uint32_t x = a0 + lane; x < a1; x += 64) {
                        const uint32_t e = G.adj[x], z = e >> 2, bit = 1u << (z & 31u);
                        if (e & 1u) atomicOr(&PA[z >> 5].x, bit);
                        if (e & 2u) atomicOr(&PA[z >> 5].y, bit);
                    }
                    wave_fence();
                }
                five_triple(G, K, wv[wid], A.table, PR, PA, PY, W, r, a, q, same, vis);
            }
            __syncthreads();
        }
        if (!any) continue;   // the graph's items were gone: no counters to give
        // the slot's counters to the graph's output
        __syncthreads();
        empty_hash();
        if (A.dense)
            for (uint32_t i = tid; i < G.n * kTreeSlots5; i += BS) {
                const uint32_t n = dense[i];
                if (!n) continue;
                dense[i] = 0u;
                const uint32_t v = i / kTreeSlots5;
                gadd64(&G.out[(size_t)G.perm[v] * kClasses5 + A.slot_cls[i - v * kTreeSlots5]], n);
            }
        if (tid < 8) {
            if (vis[tid]) gadd64(&G.stats[tid], vis[tid]);
            vis[tid] = 0ull;
        }
    }
}

// code -> class id with the classes of LDS counters replaced by their mark and slot
__global__ __launch_bounds__(256) void k_five_marks(const uint16_t* table, const uint16_t* slot_cls, uint16_t* marked) {
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    const uint16_t c = table[i];
    uint16_t m = c;
    for (uint32_t k = 0; k < kTreeSlots5; k++)
        if (slot_cls[k] == c) m = (uint16_t)(kTreeMark | k);
    marked[i] = m;
}

// Per device: the LDS counter slots, which are the single-arc tree classes found from each
// class's minimal index (four joined pairs, none reciprocal), in ascending class id; the class
// table with them marked (2 MiB).  Built at the first use, kept for the life of the process.
struct FiveSlots {
    uint16_t* marked = nullptr;    // 2^20 entries
    uint16_t* slot_cls = nullptr;  // 32 entries: slot -> class
};
std::mutex g_slots_mu;
std::map<int, FiveSlots> g_slots;
const FiveSlots& five_slots() {
    int dev = 0;
    VDMC_HIP(hipGetDevice(&dev));
    const ClassTable5& t = class_table5();
    std::lock_guard<std::mutex> lock(g_slots_mu);
    auto it = g_slots.find(dev);
    if (it != g_slots.end()) return it->second;
    std::vector<uint16_t> slot_cls(32, 0);
    uint32_t k = 0;
    for (uint32_t c = 0; c < (uint32_t)kClasses5; c++) {
        const uint32_t code = t.codes[c];
        uint32_t joined = 0, recip = 0;
        for (uint32_t i = 0; i < 5; i++)
            for (uint32_t j = i + 1; j < 5; j++) {
                const uint32_t x = (code >> shift5(i, j)) & 1u, y = (code >> shift5(j, i)) & 1u;
                joined += x | y;
                recip += x & y;
            }
        if (joined == 4u && recip == 0u) {
            VDMC_REQUIRE(k < kTreeSlots5, VDMC_ERR_DEVICE, "more single-arc 5-vertex tree classes than slots");
            slot_cls[k++] = (uint16_t)c;
        }
    }
    VDMC_REQUIRE(k == kTreeSlots5, VDMC_ERR_DEVICE,
                 "expected 27 single-arc 5-vertex tree classes, found " + std::to_string(k));
    FiveSlots fs;
    VDMC_HIP(hipMalloc(&fs.slot_cls, 32 * sizeof(uint16_t)));
    const hipError_t e = hipMalloc(&fs.marked, sizeof(uint16_t) << 20);
    if (e != hipSuccess) {
        (void)hipFree(fs.slot_cls);
        VDMC_HIP(e);
    }
    VDMC_HIP(hipMemcpy(fs.slot_cls, slot_cls.data(), 32 * sizeof(uint16_t), hipMemcpyHostToDevice));
    hipLaunchKernelGGL(k_five_marks, dim3((1u << 20) / 256), dim3(256), 0, 0, t.table, fs.slot_cls, fs.marked);
    VDMC_HIP(hipGetLastError());
    VDMC_HIP(hipStreamSynchronize(nullptr));
    return g_slots.emplace(dev, fs).first->second;
}

int g_ncu = -1;
int ncu() {
    if (g_ncu < 0) {
        int dev = 0;
        hipDeviceProp_t prop;
        VDMC_HIP(hipGetDevice(&dev));
        VDMC_HIP(hipGetDeviceProperties(&prop, dev));
        g_ncu = prop.multiProcessorCount;
    }
    return g_ncu;
}

SetsGraph view_of(const vdmc_graph_s* g, uint64_t* out) {
    return SetsGraph{g->off, g->adj, g->split, g->perm, (unsigned long long*)out, g->stats, (uint32_t)g->n, 0u};
}

// LDS of k_five_sets: the largest launch shape that fits.  dense_n: vertices with LDS counters of
// the tree classes.  1024 threads where the bit planes of 16 waves leave room for a hash of 4096
// cells, else 256.  A hash of 8192 cells beside the counters of 512 vertices is why the state of
// a wave is kept this small: 38.3 ms for 256 G(n, p) graphs of 20..500 vertices, 44.4 with 4096.
// (Two triples of 32 lanes a wave, for the 25 or so candidates of a triple there: 51.3 ms.)
struct SetsShape {
    int bs;
    uint32_t hbits;
    size_t lds;
};
SetsShape sets_shape(uint32_t words, uint32_t dense_n) {
    const size_t dense = (size_t)dense_n * kTreeSlots5 * sizeof(uint32_t);
    for (int bs : {1024, 256}) {
        const size_t fixed = sizeof(SetsWave) * (bs / 64) + 256;
        const size_t need = (size_t)(1 + 2 * (bs / 64)) * words * sizeof(uint2) + dense;
        for (uint32_t hb : {13u, 12u}) {
            const size_t lds = need + ((size_t)8 << hb);
            if (fixed + lds <= 163840) return SetsShape{bs, hb, lds};
        }
    }
    throw Error{VDMC_ERR_DEVICE, "bit planes exceed one workgroup's LDS"};
}

// Zeroes the outputs and counters, then counts every graph's items.
void launch_sets(SetsArgs a, uint32_t num, size_t cells, hipStream_t st) {
    const unsigned zx = (unsigned)std::max<size_t>(1, std::min<size_t>((cells / num + 1023) / 1024, 16384 / num + 1));
    hipLaunchKernelGGL(k_five_zero, dim3(zx, std::min<uint32_t>(num, 65535u)), dim3(256), 0, st, a, num);
    VDMC_HIP(hipGetLastError());
    if (a.nslots == 0) return;
    const FiveSlots& fs = five_slots();
    a.table = a.dense ? fs.marked : class_table5().table;
    a.slot_cls = fs.slot_cls;
    const SetsShape sh = sets_shape(a.words, a.dense);
    void (*kern)(SetsArgs, uint32_t) = sh.bs == 1024 ? k_five_sets<1024> : k_five_sets<256>;
    VDMC_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh.lds));
    const unsigned grid = (unsigned)std::min<int64_t>(a.nslots, (int64_t)ncu() * (1024 / sh.bs));
    hipLaunchKernelGGL(kern, dim3(grid), dim3(sh.bs), sh.lds, st, a, sh.hbits);
    VDMC_HIP(hipGetLastError());
}

// cached descriptors of batched 5-vertex launches, by (graphs, outputs): the graph views,
// the item table and its cursor
struct FivePlan {
    std::vector<vdmc_graph_s*> graphs;
    std::vector<uint64_t*> outs;
    SetsGraph* d_graphs = nullptr;
    uint2* d_items = nullptr;
    uint32_t* d_slots = nullptr;
    unsigned* d_cursors = nullptr;
    uint32_t nslots = 0, words = 1, dense = 0;
    size_t cells = 0;
    ~FivePlan() {
        (void)hipFree(d_graphs);
        (void)hipFree(d_items);
        (void)hipFree(d_slots);
        (void)hipFree(d_cursors);
    }
};
std::mutex g_five_mu;
std::vector<FivePlan*> g_five_plans;

// whether k_five_sets takes the graph.  An item costs it some 30 ns (256 workgroups) however few sets
// hang on it, the search set by set the time of its longest item, which grows with the degrees.  So
// graphs of more than kDenseMaxN vertices go set by set if they are paths and cycles, and if no
// degree is above 4 from 20000 pairs on (us set by set and in groups: path of 600 54 and 64, of 5000 114
// and 276; binary tree of 16384 585 and 527; ladder of 16000, 24000 pairs, 461 and 1015; 128 x 128 grid
// 1006 and 1784).
bool takes_sets(const vdmc_graph_s* g) {
    if (g->n > kFiveSetsMaxN || g->pairs > kFiveSetsMaxPairs) return false;
    return g->n <= kDenseMaxN || g->max_deg > 4 || (g->max_deg > 2 && g->pairs < 20000);
}

// 5-vertex counts set by set over the graph in device memory: every workgroup of the grid takes
// sub-items from one cursor and credits the caller's output with device-scope atomics.
// Needs the graph's edge hash and its item prefix (both built at the first such count
// and kept with the graph).
void launch_count5_global(vdmc_graph_s* g, uint64_t* out, hipStream_t st) {
    const ClassTable5& t = class_table5();
    launch_fill_u64((uint64_t*)g->stats, kStatSlots, 0, st);
    if (g->n == 0) return;
    launch_fill_u64(out, (size_t)g->n * kClasses5, 0, st);
    if (g->pairs == 0) return;
    ensure_edge_hash(g, st);
    if (!g->five_hp) {
        const uint32_t n = (uint32_t)g->n;
        unsigned long long* hp = nullptr;
        VDMC_HIP(hipMalloc(&hp, sizeof(unsigned long long) * (n + 2)));   // prefix, then the item cursor
        g->five_hp = hp;   // owned by the graph from here on; five_items 0: not filled yet
        g->five_items = 0;
    }
    if (g->five_items == 0) {
        const uint32_t n = (uint32_t)g->n;
        unsigned long long *cnt = nullptr, *hp = g->five_hp;
        VDMC_HIP(hipMalloc(&cnt, sizeof(unsigned long long) * (n + 1)));
        struct Free {
            void* p;
            ~Free() { (void)hipFree(p); }
        } fcnt{cnt};
        hipLaunchKernelGGL(k_five_counts, dim3((n + 256) / 256), dim3(256), 0, st, g->off, g->split, n, kSplitDiv, cnt);
        VDMC_HIP(hipGetLastError());
        size_t tmp_bytes = 0;
        VDMC_HIP(hipcub::DeviceScan::ExclusiveSum(nullptr, tmp_bytes, cnt, hp, n + 1, st));
        void* tmp = nullptr;
        VDMC_HIP(hipMalloc(&tmp, tmp_bytes ? tmp_bytes : 16));
        Free ftmp{tmp};
        VDMC_HIP(hipcub::DeviceScan::ExclusiveSum(tmp, tmp_bytes, cnt, hp, n + 1, st));
        unsigned long long total = 0;
        VDMC_HIP(hipMemcpyAsync(&total, hp + n, sizeof(total), hipMemcpyDeviceToHost, st));
        VDMC_HIP(hipStreamSynchronize(st));
        g->five_items = total;
    }
    unsigned long long* cursor = g->five_hp + g->n + 1;
    launch_fill_u64((uint64_t*)cursor, 1, 0, st);
    FiveGlobalArgs a{};
    a.L = FiveGlobal{g->off, g->adj, reinterpret_cast<const uint32_t*>(g->perm), g->ehash, g->ehash_bits};
    a.split = g->split;
    a.hp = g->five_hp;
    a.n = (uint32_t)g->n;
    a.total = g->five_items;
    a.out = (unsigned long long*)out;
    a.stats = g->stats;
    a.cursor = cursor;
    a.table = t.table;
    a.split_div = kSplitDiv;
    const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((int64_t)ncu() * 4,
                                                                           (int64_t)((g->five_items + 255) / 256)));
    hipLaunchKernelGGL(k_five_global<256>, dim3(grid), dim3(256), 0, st, a);
    VDMC_HIP(hipGetLastError());
}

}  // namespace

void launch_count5(vdmc_graph_s* g, uint64_t* out, hipStream_t st) {
    g->timed_light = g->timed_hub = false;
    if (!takes_sets(g)) {
        launch_count5_global(g, out, st);
        return;
    }
    SetsArgs a{};
    a.one = view_of(g, out);
    // the item table (8 bytes per pair), then the cursors; kept with the graph
    if (!g->five_tab) {
        void* tab = nullptr;
        VDMC_HIP(hipMalloc(&tab, sizeof(uint2) * (size_t)(g->pairs + 2)));
        g->five_tab = tab;
    }
    uint2* items = (uint2*)g->five_tab;
    a.items = items;
    a.cursors = reinterpret_cast<unsigned*>(items + g->pairs);
    if (!g->five_tab_ready) {
        hipLaunchKernelGGL(k_five_items, dim3(1), dim3(kItemThreads), 0, st, nullptr, a.one, items, a.cursors);
        VDMC_HIP(hipGetLastError());
        g->five_tab_ready = true;
    }
    a.nslots = (uint32_t)std::min<int64_t>((g->pairs + 3) / 4, (int64_t)ncu() * 4);
    a.words = (uint32_t)std::max<int64_t>(1, (g->n + 31) / 32);
    a.dense = g->n <= kDenseMaxN ? (uint32_t)g->n : 0u;
    launch_sets(a, 1, (size_t)g->n * kClasses5, st);
}

void free_five(vdmc_graph_s* g) {
    (void)hipFree(g->five_hp);
    (void)hipFree(g->five_tab);
    g->five_hp = nullptr;
    g->five_tab = nullptr;
    g->five_tab_ready = false;
    g->five_items = 0;
}

// the graphs of one batched launch (all taken by k_five_sets)
static void count5_batch_sets(const std::vector<vdmc_graph_s*>& gs, const std::vector<uint64_t*>& outs,
                              hipStream_t st) {
    if (gs.empty()) return;
    std::lock_guard<std::mutex> lock(g_five_mu);
    FivePlan* plan = nullptr;
    for (FivePlan* p : g_five_plans)
        if (p->graphs == gs && p->outs == outs) {
            plan = p;
            break;
        }
    GraphUse use(gs, st);   // ordered after earlier work on these graphs
    if (!plan) {
        plan = new FivePlan();
        try {
            plan->graphs = gs;
            plan->outs = outs;
            // heaviest graphs first (pairs x squared largest degree as the estimate), so that
            // the last workgroups hold small ones
            std::vector<uint32_t> order(gs.size());
            for (uint32_t i = 0; i < order.size(); i++) order[i] = i;
            const auto work = [&](uint32_t i) { return (double)gs[i]->pairs * gs[i]->max_deg * gs[i]->max_deg; };
            std::stable_sort(order.begin(), order.end(), [&](uint32_t x, uint32_t y) { return work(x) > work(y); });
            // slots: workgroups per graph by its share of the work, about two per compute unit
            double total = 0.0;
            for (uint32_t i : order) total += work(i);
            std::vector<SetsGraph> views;
            std::vector<uint32_t> slots;
            uint32_t nitems = 0;
            int64_t max_n = 1;
            for (uint32_t i : order) {
                const double share = total > 0.0 ? work(i) / total * 2.0 * ncu() : 1.0;
                const uint32_t parts = (uint32_t)std::max(1.0, std::min({std::ceil(share), 64.0, gs[i]->pairs / 16.0}));
                for (uint32_t p = 0; p < parts; p++) slots.push_back((uint32_t)views.size());
                views.push_back(view_of(gs[i], outs[i]));
                views.back().first = nitems;
                nitems += (uint32_t)gs[i]->pairs;
                max_n = std::max(max_n, gs[i]->n);
                plan->cells += (size_t)gs[i]->n * kClasses5;
            }
            plan->nslots = (uint32_t)slots.size();
            plan->words = (uint32_t)((max_n + 31) / 32);
            plan->dense = max_n <= kDenseMaxN ? (uint32_t)max_n : 0u;
            VDMC_HIP(hipMalloc(&plan->d_graphs, sizeof(SetsGraph) * views.size()));
            VDMC_HIP(hipMalloc(&plan->d_items, sizeof(uint2) * std::max<size_t>(nitems, 1)));
            VDMC_HIP(hipMalloc(&plan->d_slots, sizeof(uint32_t) * slots.size()));
            VDMC_HIP(hipMalloc(&plan->d_cursors, sizeof(unsigned) * (2 * views.size() + 2)));
            VDMC_HIP(hipMemcpyAsync(plan->d_graphs, views.data(), sizeof(SetsGraph) * views.size(), hipMemcpyHostToDevice,
                                    st));
            VDMC_HIP(hipMemcpyAsync(plan->d_slots, slots.data(), sizeof(uint32_t) * slots.size(), hipMemcpyHostToDevice,
                                    st));
            hipLaunchKernelGGL(k_five_items, dim3((unsigned)views.size()), dim3(kItemThreads), 0, st, plan->d_graphs,
                               SetsGraph{}, plan->d_items, plan->d_cursors);
            VDMC_HIP(hipGetLastError());
            VDMC_HIP(hipStreamSynchronize(st));   // the host arrays are read by the copies
        } catch (...) {
            delete plan;
            throw;
        }
        g_five_plans.push_back(plan);
        if (g_five_plans.size() > 16) {
            delete g_five_plans.front();
            g_five_plans.erase(g_five_plans.begin());
        }
    }
    for (auto* g : gs) g->timed_light = g->timed_hub = false;
    SetsArgs a{};
    a.graphs = plan->d_graphs;
    a.items = plan->d_items;
    a.slots = plan->d_slots;
    a.nslots = plan->nslots;
    a.cursors = plan->d_cursors;
    a.words = plan->words;
    a.dense = plan->dense;
    launch_sets(a, (uint32_t)gs.size(), plan->cells, st);
}

void count5_batch(const vdmc_graph_s* const* gs_in, int32_t num, uint64_t* const* outs_in, hipStream_t st) {
    // graphs that k_five_sets takes go into batched launches (at most 2 GiB of items each);
    // the others are counted one by one
    for (const bool small : {true, false}) {   // with and without LDS counters
        std::vector<vdmc_graph_s*> gs;
        std::vector<uint64_t*> outs;
        int64_t pairs = 0;
        for (int i = 0; i < num; i++) {
            vdmc_graph_s* g = const_cast<vdmc_graph_s*>(gs_in[i]);
            if (!takes_sets(g) || (g->n <= kDenseMaxN) != small) continue;
            if (pairs + g->pairs > kFiveSetsMaxPairs * 16) {
                count5_batch_sets(gs, outs, st);
                gs.clear();
                outs.clear();
                pairs = 0;
            }
            gs.push_back(g);
            outs.push_back(outs_in[i]);
            pairs += g->pairs;
        }
        count5_batch_sets(gs, outs, st);
    }
    for (int i = 0; i < num; i++) {
        vdmc_graph_s* g = const_cast<vdmc_graph_s*>(gs_in[i]);
        if (takes_sets(g)) continue;
        GraphUse use(g, st);
        launch_count5_global(g, outs_in[i], st);
    }
}

void invalidate_five_plans(vdmc_graph_s* g) {
    std::lock_guard<std::mutex> lock(g_five_mu);
    for (auto it = g_five_plans.begin(); it != g_five_plans.end();) {
        if (std::find((*it)->graphs.begin(), (*it)->graphs.end(), g) != (*it)->graphs.end()) {
            delete *it;
            it = g_five_plans.erase(it);
        } else {
            ++it;
        }
    }
}

}  // namespace vdmc
