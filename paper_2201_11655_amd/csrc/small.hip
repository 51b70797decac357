// Small-graph motif kernel: one workgroup counts a whole graph held in LDS.
//
// For graphs of a few hundred vertices (the batched workload, small served requests)
// a per-root launch leaves most of a workgroup idle: a root of such a graph has a
// handful of higher neighbours.  Here one workgroup takes a whole graph: its rank-space
// CSR (16-bit row entries), a 1-bit adjacency matrix (almost every pair test is one LDS
// read; a set bit is resolved to its arc bits by a search of the LDS row) and per-vertex
// counters live in LDS.
//
// The sets are those of Lemmas 1-4, but most are not visited.  Of the sets of a root r,
// those of three shapes are counted by arc codes as if their members had only the arcs
// that the shape implies, and each set that has another arc is then corrected (its credits
// moved from the tree class to its own):
//   (3,0,0)  triples of N+(r), from the numbers of slots by code;
//   (2,1,0)  a child c of a slot a with a second slot, from the children by code (the rule
//            that c hangs under its lower-rank parent is part of the correction);
//   (1,2,0)  pairs of children of a slot a.
// The fourth, (1,1,1) (a path r - a - c - e), is visited: one credit for e, and for r, a and
// c once per arc code.  Its walk of c's row finds what (2,1,0) and (1,2,0) have to correct
// for c: the entries in N+(r) and those adjacent to a.  An adjacent pair of slots (a
// triangle with r) is queued, and corrects the triples and the children of either.
// In the 4096 graphs of the batched workload (20..500 vertices, mean out-degree 2..8)
// there are 218 k sets a graph, of them 65 k paths, and 14 k corrections: 2.05 ms a call,
// 4.75 with every set visited.  What bounds it: the LDS of the path walk, three reads and an
// atomic per row entry, with one workgroup a CU (128 registers, 16 waves).
//
// k = 3 is the same: pairs of N+(r) and children by code, triangles corrected.
//
// Credits go to LDS counters (k = 3: all 13 classes; k = 4: the 25 tree classes and the 12
// single-arc 4-pair classes, which hold ~99.6% of the credits of sparse graphs); the other
// classes go straight to the graph's output with workgroup-scope atomics (the output block
// of a graph belongs to one workgroup for the whole launch; every such atomic is a
// memory-side operation, so they are kept rare).
// The LDS counters are stored to the output once per graph (their classes never reach
// the output otherwise).  u32 counters cannot overflow: a vertex of a graph with
// n <= kSmallMaxN lies in fewer than 2^32 k-sets, and a correction is arithmetic mod 2^32.
#include "motif_device.h"
#include "vdmc_internal.h"

namespace vdmc {
namespace {

__device__ __forceinline__ uint32_t lane_of() { return threadIdx.x & 63u; }

// LDS counter slots per vertex for k = 4: the 25 tree classes, then the 12 classes whose
// four joined pairs are all single arcs (directed 4-cycles and tailed triangles without a
// reciprocal pair).  In a sparse digraph these are the next most frequent after the trees
// (each further arc or reciprocation costs another factor of p): together they hold ~99.6%
// of the credits of the batch workload, and only the rest goes to the output with
// memory-side atomics.
constexpr uint32_t kSingleArc4 = 12;
constexpr uint32_t kSlots4 = (uint32_t)kCompact4 + kSingleArc4;

// bit of the 4-vertex index for the entry (i, j), i != j: rows in order, the diagonal
// skipped, entry (0,1) the most significant of the 12 (Sec. 4.1)
__device__ __forceinline__ uint32_t bit4(uint32_t code, uint32_t i, uint32_t j) {
    return (code >> (11u - (3u * i + (j < i ? j : j - 1u)))) & 1u;
}

// wg-scope atomic add on a graph's output (the block is owned by this workgroup)
__device__ __forceinline__ void out_add(gptr<unsigned long long> p, unsigned long long v) {
    __hip_atomic_fetch_add(p.p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// exclusive prefix sum of a[0..len) in place (LDS), returns the total; every thread of
// the workgroup must call it.  Each thread sums a contiguous chunk; the chunk sums are
// scanned within each wave by shuffles and across the BS / 64 waves by the first wave.
// part: BS / 64 words of LDS scratch.
template <int BS>
__device__ uint32_t block_exclusive_scan(uint32_t* a, uint32_t len, uint32_t* part) {
    constexpr uint32_t NWV = BS / 64;
    const uint32_t tid = threadIdx.x, lane = lane_of(), wave = tid >> 6;
    const uint32_t per = (len + BS - 1) / BS;
    const uint32_t lo = min(len, tid * per), hi = min(len, lo + per);
    uint32_t s = 0;
    for (uint32_t i = lo; i < hi; i++) s += a[i];
    uint32_t x = s;   // inclusive scan of the chunk sums within the wave
    for (uint32_t o = 1; o < 64; o <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) part[wave] = x;
    __syncthreads();
    if (tid < 64) {   // inclusive scan of the wave totals
        uint32_t w = tid < NWV ? part[tid] : 0u;
        for (uint32_t o = 1; o < NWV; o <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)w, o, 64);
            if (lane >= o) w += y;
        }
        if (tid < NWV) part[tid] = w;
    }
    __syncthreads();
    uint32_t run = (wave ? part[wave - 1] : 0u) + x - s;
    for (uint32_t i = lo; i < hi; i++) {
        const uint32_t v = a[i];
        a[i] = run;
        run += v;
    }
    const uint32_t total = part[NWV - 1];
    __syncthreads();
    return total;
}

// largest i in [0, len) with pre[i] <= q (pre ascending, pre[0] = 0 <= q)
__device__ __forceinline__ uint32_t upper_idx(const uint32_t* pre, uint32_t len, uint32_t q) {
    uint32_t lo = 0, hi = len;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (pre[mid] <= q) lo = mid; else hi = mid;
    }
    return lo;
}

struct SmallLds {
    const uint32_t* off;
    const uint16_t* adj;   // entries (nbr_rank << 2) | arc bits; ranks below 1024 fit 16 bits
    const uint32_t* split;
    const uint32_t* bits;
    const uint32_t* arcs;   // bit (u, v): arc u -> v; nullptr where LDS has no room for it
    uint32_t W;
    __device__ __forceinline__ bool adjacent(uint32_t u, uint32_t v) const {
        return (bits[u * W + (v >> 5)] >> (v & 31u)) & 1u;
    }
    // the bitmap word of row u that holds v's bit, and the bit itself
    __device__ __forceinline__ uint32_t word(uint32_t u, uint32_t v) const { return bits[u * W + (v >> 5)]; }
    static __device__ __forceinline__ bool bit(uint32_t w, uint32_t v) { return (w >> (v & 31u)) & 1u; }
    // arc bits of (u, v) seen from u for a pair whose adjacency bit is already read
    __device__ __forceinline__ uint32_t code_if(bool is_adj, uint32_t u, uint32_t v) const {
        if (!is_adj) return 0u;
        if (arcs)
            return ((arcs[u * W + (v >> 5)] >> (v & 31u)) & 1u) | (((arcs[v * W + (u >> 5)] >> (u & 31u)) & 1u) << 1);
        uint32_t lo = off[u], hi = off[u + 1];
        const uint32_t key = v << 2;
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (adj[mid] < key) lo = mid + 1; else hi = mid;
        }
        return adj[lo] & 3u;
    }
    // arc bits of (u, v) seen from u, 0 if not adjacent
    __device__ __forceinline__ uint32_t code(uint32_t u, uint32_t v) const { return code_if(adjacent(u, v), u, v); }
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

template <int K>
struct SmallCredit {
    static constexpr uint32_t C = K == 3 ? (uint32_t)kClasses3 : (uint32_t)kClasses4;
    uint32_t nc;              // counters of a vertex: the classes, or kSlots4 of them
    uint32_t* cnt;            // n x nc (LDS)
    const uint8_t* comp;      // class -> counter slot or 0xFF (LDS)
    const uint32_t* perm;     // rank -> original id in the low 10 bits (LDS)
    gptr<unsigned long long> out;
    // one set of class cls
    __device__ __forceinline__ void add1(uint32_t v, uint32_t cls) const {
        const uint32_t s = K == 3 ? cls : comp[cls];
        if (K == 3 || s != 0xFFu) atomicAdd(&cnt[v * nc + s], 1u);
        else out_add(&out[(size_t)(perm[v] & 1023u) * C + cls], 1ull);
    }
    // n sets of the class of counter slot s
    __device__ __forceinline__ void add_s(uint32_t v, uint32_t s, uint32_t n) const { atomicAdd(&cnt[v * nc + s], n); }
    // one set: from the counter slot `was` to class `is`
    __device__ __forceinline__ void move(uint32_t v, uint32_t was, uint32_t is) const {
        add_s(v, was, ~0u);
        add1(v, is);
    }
};

// counter slots (k = 4) of tree classes, by two arc codes x, y in 1..3 at [4 x + y], for a
// third code z in the byte z - 1
struct SmallTrees {
    uint32_t path[16];    // r - a - c - e: x = r to a, y = a to c, z = c to e
    uint32_t path2[16];   // c - a - r - b: x = r to a, y = a to c, z = r to b
    uint32_t starr[16];   // r with three slots
    uint32_t stara[16];   // a with r (x: seen from r) and two children (y, z: seen from a)
};
__device__ __forceinline__ uint32_t byte_of(uint32_t w, uint32_t z) { return (w >> (8u * z - 8u)) & 0xFFu; }
__device__ __forceinline__ uint32_t pick3(uint32_t k, uint32_t a, uint32_t b, uint32_t c) {
    return k == 1u ? a : (k == 2u ? b : c);
}
// pairs of two codes k <= l of three, from the numbers by code
__device__ __forceinline__ uint32_t pairs_of(uint32_t k, uint32_t l, uint32_t a, uint32_t b, uint32_t c) {
    const uint32_t x = pick3(k, a, b, c);
    return k == l ? x * (x - 1u) / 2u : x * pick3(l, a, b, c);
}
// i-th pair of codes k <= l
__device__ __forceinline__ void code_pair(uint32_t i, uint32_t& k, uint32_t& l) {
    k = i < 3u ? 1u : (i < 5u ? 2u : 3u);
    l = i < 3u ? i + 1u : (i < 5u ? i - 1u : 3u);
}
// i-th triple of codes, two bits each, ascending
__device__ __forceinline__ uint32_t code_triple(uint32_t i) {
    constexpr unsigned long long t = 0x15ull | 0x25ull << 6 | 0x35ull << 12 | 0x29ull << 18 | 0x39ull << 24 |
                                     0x3Dull << 30 | 0x2Aull << 36 | 0x3Aull << 42 | 0x3Eull << 48 | 0x3Full << 54;
    return (uint32_t)(t >> (6u * i)) & 63u;
}
// the value of a lane of the same 8, by a cross-lane move: the neighbour (0xB1), the other pair of
// four (0x4E), the mirrored lane of eight (0x141)
template <int CTRL>
__device__ __forceinline__ uint32_t lane8(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ unsigned long long lane8(unsigned long long v) {
    return (unsigned long long)lane8<CTRL>((uint32_t)(v >> 32)) << 32 | lane8<CTRL>((uint32_t)v);
}
// sum over aligned groups of 8 lanes, in every lane
template <class T>
__device__ __forceinline__ T sum8(T v) {
    v += lane8<0xB1>(v);
    v += lane8<0x4E>(v);
    v += lane8<0x141>(v);
    return v;
}
// 10-bit fields to 21-bit fields
__device__ __forceinline__ unsigned long long wide3(uint32_t v) {
    return (v & 1023u) | (unsigned long long)((v >> 10) & 1023u) << 21 | (unsigned long long)(v >> 20) << 42;
}

// The sets of r with the adjacent slots a < b, for lane i0 of step: triples (from the first of
// their adjacent pairs) and children of one that are not adjacent to the other.
__device__ __forceinline__ void fix_triangle(const SmallLds& L, const SmallCredit<4>& cr, const SmallTrees& F,
                                             const uint8_t* table, uint32_t r, uint32_t a, uint32_t b, uint32_t i0,
                                             uint32_t step) {
    const uint32_t ra = L.code(r, a), rb = L.code(r, b), ab = L.code(a, b);
    const uint32_t wr = F.starr[ra * 4u + rb];
    for (uint32_t i = L.split[r] + i0; i < L.off[r + 1]; i += step) {
        const uint32_t c = L.adj[i] >> 2, rc = L.adj[i] & 3u;
        const bool xa = L.adjacent(a, c), xb = L.adjacent(b, c);
        if (c == a || c == b || (xa && c < b) || (xb && c < a)) continue;
        const uint32_t is = table[motif_index4(ra, rb, rc, ab, L.code_if(xa, a, c), L.code_if(xb, b, c))];
        const uint32_t was = byte_of(wr, rc);
        cr.move(r, was, is);
        cr.move(a, was, is);
        cr.move(b, was, is);
        cr.move(c, was, is);
    }
    for (uint32_t side = 0; side < 2; side++) {
        const uint32_t p = side ? b : a, q = side ? a : b, rp = side ? rb : ra, rq = side ? ra : rb;
        const uint32_t pq = side ? swap_arc_bits(ab) : ab, lo = L.off[p];
        for (uint32_t i = L.off[p + 1] - i0; (int32_t)i > (int32_t)lo; i -= step) {
            const uint32_t c = L.adj[i - 1u] >> 2, pc = L.adj[i - 1u] & 3u;
            if (c <= r) break;
            if (L.adjacent(r, c) || L.adjacent(q, c)) continue;
            const uint32_t is = table[motif_index4(rp, rq, 0u, pq, pc, 0u)];
            const uint32_t was = byte_of(F.path2[rp * 4u + pc], rq);
            cr.move(r, was, is);
            cr.move(a, was, is);
            cr.move(b, was, is);
            cr.move(c, was, is);
        }
    }
}

template <int BS, int K>
__global__ __launch_bounds__(BS, 4) void k_small(SmallArgs A) {
    extern __shared__ uint32_t dyn[];
    __shared__ uint8_t sTable[K == 3 ? 64 : 4096];
    __shared__ uint8_t sComp[256];
    __shared__ uint8_t sSame[K == 4 ? 256 : 1];        // class -> class
    __shared__ uint8_t sSlotCls[64];
    __shared__ uint32_t sMask[8];   // k = 4: 256-bit mask of the single-arc 4-pair classes
    __shared__ uint32_t sPart[BS / 64];
    __shared__ uint32_t sGraph;
    constexpr uint32_t kTriQueue = K == 4 ? 512 : 1;   // G(n, p) has about deg^3 / 6
    __shared__ uint32_t sTri[kTriQueue];              // triangles (r, a, b), 10 bits each
    __shared__ uint32_t sTriN;
    __shared__ SmallTrees sTreeSlots[2];               // with kSlots4 counters; with one per class
    constexpr uint32_t C = SmallCredit<K>::C;
    const uint32_t tid = threadIdx.x;
    for (uint32_t i = tid; i < (K == 3 ? 64u : 4096u); i += BS) sTable[i] = A.table[i];
    if (K == 4) {
        // counter slots: the tree classes' from the class tables, then the single-arc
        // 4-pair classes in ascending class id (each found from any of its codes)
        for (uint32_t i = tid; i < 256u; i += BS) {
            sComp[i] = A.comp_of[i];
            sSame[i] = (uint8_t)i;
        }
        for (uint32_t i = tid; i < (uint32_t)kCompact4; i += BS) sSlotCls[i] = A.comp_cls[i];
        if (tid < 8) sMask[tid] = 0u;
        __syncthreads();
        for (uint32_t code = tid; code < 4096u; code += BS) {
            uint32_t joined = 0, recip = 0;
            for (uint32_t i = 0; i < 4; i++)
                for (uint32_t j = i + 1; j < 4; j++) {
                    const uint32_t x = bit4(code, i, j), y = bit4(code, j, i);
                    joined += x | y;
                    recip += x & y;
                }
            const uint32_t cls = sTable[code];
            if (joined == 4u && recip == 0u && cls != 0xFFu) atomicOr(&sMask[cls >> 5], 1u << (cls & 31u));
        }
        __syncthreads();
        if (tid == 0) {
            uint32_t k = 0;
            for (uint32_t c = 0; c < 256u; c++)
                if (((sMask[c >> 5] >> (c & 31u)) & 1u) && sComp[c] == 0xFFu && k < kSingleArc4) {
                    sComp[c] = (uint8_t)(kCompact4 + k);
                    sSlotCls[kCompact4 + k] = (uint8_t)c;
                    k++;
                }
        }
        if (tid < 64) {
            const uint32_t x = (tid >> 2) & 3u, y = tid & 3u;
            for (uint32_t f = 0; tid < 16 && f < 2; f++) {
                const uint8_t* of = f ? sSame : sComp;
                uint32_t w[4] = {0, 0, 0, 0};
                for (uint32_t z = 1; x && y && z < 4; z++) {
                    w[0] |= (uint32_t)of[sTable[motif_index4(x, 0u, 0u, y, 0u, z)]] << (8u * z - 8u);
                    w[1] |= (uint32_t)of[sTable[motif_index4(x, z, 0u, 0u, y, 0u)]] << (8u * z - 8u);
                    w[2] |= (uint32_t)of[sTable[motif_index4(x, y, z, 0u, 0u, 0u)]] << (8u * z - 8u);
                    w[3] |= (uint32_t)of[sTable[motif_index4(x, 0u, 0u, y, z, 0u)]] << (8u * z - 8u);
                }
                sTreeSlots[f].path[tid] = w[0];
                sTreeSlots[f].path2[tid] = w[1];
                sTreeSlots[f].starr[tid] = w[2];
                sTreeSlots[f].stara[tid] = w[3];
            }
        }
    }

    for (uint32_t round = 0;; round++) {
        __syncthreads();
        if (tid == 0) sGraph = A.graphs ? atomicAdd(A.cursor, 1u) : round;   // single graph: taken once
        __syncthreads();
        const uint32_t gidx = sGraph;
        if (gidx >= A.num) break;
        const SmallGraph G = A.graphs ? A.graphs[gidx] : A.one;
        const uint32_t n = G.n, E = G.entries, W = (n + 31u) >> 5;
        // LDS layout
        uint32_t* sOff = dyn;                 // n + 1
        uint32_t* sSplit = sOff + n + 1;      // n
        uint32_t* sPreD = sSplit + n;         // n + 1: upper entries before row r
        uint32_t* sPerm = sPreD + n + 1;      // n + 1: rank -> original id | slots of code 1, 2 << 10, 20
        uint32_t* sBits = sPerm + n + 1;      // n * W
        uint32_t* sPre2 = sBits + n * W;      // E / 2 + 1: depth-2 candidates before each upper entry
        uint16_t* sAdj = reinterpret_cast<uint16_t*>(sPre2 + E / 2 + 1);   // E (u16)
        uint16_t* sRootOf = sAdj + E;         // E / 2 (u16): root of each upper entry
        uint32_t* rest = sPre2 + E / 2 + 1 + (E + E / 2 + 1) / 2;
        // With the LDS that is left: the arcs one way, which turn the search for a pair's codes
        // into two reads; more of the triangle queue, whose overflow costs a search per
        // candidate (600 us instead of 55 in the worst of the batched graphs); then counters of
        // every class, which fit up to n = 160 or so, where a graph of 8 arcs a vertex is dense
        // and the classes beyond kSlots4 are frequent.  4096 G(n, p) graphs: 2.70 ms with none of
        // them, 2.05 with all.
        uint32_t room = A.lds_words - (uint32_t)(rest - dyn) - n * (K == 3 ? C : kSlots4);
        uint32_t* sArcs = nullptr;
        if (K == 4 && room >= n * W) {
            sArcs = rest;
            rest += n * W;
            room -= n * W;
        }
        uint32_t* sTri2 = rest;               // more of the queue
        const uint32_t tri2 = K == 4 ? min(room, 1024u) : 0u;
        rest += tri2;
        room -= tri2;
        const bool full = K == 3 || room >= n * (C - kSlots4);
        const uint32_t NC = full ? C : kSlots4;
        uint32_t* sCnt = rest;                // n * NC
        const SmallTrees& sTrees = sTreeSlots[full ? 1 : 0];
        // ---- stage the graph, clear bitmap, counters and the output block
        for (uint32_t i = tid; i <= n; i += BS) sOff[i] = G.off[i];
        for (uint32_t i = tid; i < n; i += BS) sPerm[i] = (uint32_t)G.perm[i];
        for (uint32_t i = tid; i < E; i += BS) sAdj[i] = (uint16_t)G.adj[i];
        for (uint32_t i = tid; i < n * W; i += BS) {
            sBits[i] = 0u;
            if (sArcs) sArcs[i] = 0u;
        }
        for (uint32_t i = tid; i < n * NC; i += BS) sCnt[i] = 0u;
        if (full) {   // every cell is stored at the end
        } else if (((uintptr_t)G.out.p & 15u) == 0) {   // 16-byte stores, then the odd last cell
            const size_t cells = (size_t)n * C;
            using u64x2 = unsigned long long __attribute__((ext_vector_type(2)));
            const auto o = G.out.as<u64x2>();
            for (size_t i = tid; i < cells / 2; i += BS) o[i] = u64x2{0ull, 0ull};
            if ((cells & 1u) && tid == 0) G.out[cells - 1] = 0ull;
        } else {
            for (size_t i = tid; i < (size_t)n * C; i += BS) G.out[i] = 0ull;
        }
        if (tid == 0) sTriN = 0u;
        if (tid < (uint32_t)kShapes) G.stats[tid] = 0ull;   // this launch's visit counters of the graph
        __syncthreads();
        for (uint32_t r = tid; r < n; r += BS) {
            const uint32_t lo = sOff[r], hi = sOff[r + 1];
            uint32_t s = hi, m = sPerm[r];
            for (uint32_t t = lo; t < hi; t++) {
                const uint32_t v = sAdj[t] >> 2, k = sAdj[t] & 3u;
                atomicOr(&sBits[r * W + (v >> 5)], 1u << (v & 31u));
                if (sArcs && (k & 1u)) atomicOr(&sArcs[r * W + (v >> 5)], 1u << (v & 31u));
                if (v > r && s == hi) s = t;
                if (v > r && k != 3u) m += 1u << (10u * k);
            }
            sPerm[r] = m;
            sSplit[r] = s;
            sPreD[r] = hi - s;
        }
        if (tid == 0) sPreD[n] = 0u;
        __syncthreads();
        const SmallLds L{sOff, sAdj, sSplit, sBits, sArcs, W};
        const uint32_t U = block_exclusive_scan<BS>(sPreD, n + 1, sPart);
        for (uint32_t r = tid; r < n; r += BS)
            for (uint32_t t = sPreD[r]; t < sPreD[r] + sOff[r + 1] - sSplit[r]; t++) sRootOf[t] = (uint16_t)r;
        __syncthreads();

        const SmallCredit<K> cr{NC, sCnt, full ? sSame : sComp, sPerm, G.out};
        // visits of this thread: below 2^31 for every shape, as the CSR is in LDS (sum of d < 2^14)
        uint32_t shp[4] = {0, 0, 0, 0};
        const uint32_t gl = tid & 7u;
        uint32_t pk, pl;   // pair of codes of this lane
        code_pair(min(gl, 5u), pk, pl);
        // ---- upper entries (r, a), 8 lanes each: all that is counted by codes
        for (uint32_t u0 = 0; u0 < U; u0 += BS / 8) {
            const uint32_t u = u0 + (tid >> 3);
            const bool on = u < U;
            const uint32_t r = on ? sRootOf[u] : 0u, lo = sSplit[r], d = sOff[r + 1] - lo, m = sPerm[r];
            const uint32_t ent = on ? sAdj[lo + u - sPreD[r]] : 0u, a = ent >> 2, ra = ent & 3u;
            // a's row above r, from its end
            uint32_t h1 = 0, h2 = 0, h3 = 0;   // children by code
            const uint32_t alo = on ? sOff[a] : 0u, ahi = on ? sOff[a + 1] : 0u;
            for (uint32_t q = ahi; q > alo; q -= min(8u, q - alo)) {
                const uint32_t x = q - alo > gl ? sAdj[q - 1u - gl] : 0u, c = x >> 2, k = x & 3u;
                if (c > r) {
                    if (!L.adjacent(r, c)) {
                        h1 += k == 1u;
                        h2 += k == 2u;
                        h3 += k == 3u;
                        if (K == 3) cr.add_s(c, sTable[motif_index3(ra, 0u, k)], 1u);
                    } else if (c > a) {
                        if (K == 3) {
                            const uint32_t rc = L.code(r, c), is = sTable[motif_index3(ra, rc, k)];
                            const uint32_t was = sTable[motif_index3(ra, rc, 0u)];
                            cr.move(r, was, is);
                            cr.move(a, was, is);
                            cr.move(c, was, is);
                        } else {
                            const uint32_t at = atomicAdd(&sTriN, 1u);
                            if (at < kTriQueue) sTri[at] = r | (a << 10) | (c << 20);
                            else if (at < kTriQueue + tri2) sTri2[at - kTriQueue] = r | (a << 10) | (c << 20);
                        }
                    }
                }
                if (q - alo > 8u && (uint32_t)(sAdj[q - 8u] >> 2) <= r) break;
            }
            h1 = sum8(h1);
            h2 = sum8(h2);
            h3 = sum8(h3);
            if (!on) continue;
            const uint32_t m1 = (m >> 10) & 1023u, m2 = m >> 20, h = h1 + h2 + h3;
            // the other slots
            const uint32_t o1 = m1 - (ra == 1u), o2 = m2 - (ra == 2u), o3 = d - m1 - m2 - (ra == 3u);
            if (K == 3) {
                if (gl < 6u) {   // (1,1) of a; (1,2) of a and r
                    const uint32_t k = gl % 3u + 1u, n = gl < 3u ? pick3(k, o1, o2, o3) : pick3(k, h1, h2, h3);
                    const uint32_t cls = sTable[gl < 3u ? motif_index3(ra, k, 0u) : motif_index3(ra, 0u, k)];
                    if (n) {
                        cr.add_s(a, cls, n);
                        if (gl >= 3u) cr.add_s(r, cls, n);
                    }
                }
                if (gl == 0u) shp[1] += h;
                continue;
            }
            {   // (3,0,0) of a; lanes 6 and 7: a part of the next
                const bool star = gl < 6u;
                const uint32_t k = star ? pk : 3u, l = star ? pl : gl - 4u;
                const uint32_t n = star ? pairs_of(pk, pl, o1, o2, o3) : h3 * pick3(l, o1, o2, o3);
                const uint32_t w = (star ? sTrees.starr : sTrees.path2)[ra * 4u + k];
                if (n) {
                    cr.add_s(a, byte_of(w, l), n);
                    if (!star) cr.add_s(r, byte_of(w, l), n);
                }
            }
            if (h) {
                sPre2[u] = h1 | (h2 << 10) | (h3 << 20);
                {   // (2,1,0) of a, the parent, and r; children of codes 1, 2 and the first of code 3
                    const uint32_t k = gl / 3u + 1u, l = gl % 3u + 1u;
                    const uint32_t n = gl < 7u ? pick3(k, h1, h2, h3) * pick3(l, o1, o2, o3) : 0u;
                    const uint32_t slot = byte_of(sTrees.path2[ra * 4u + k], l);
                    if (n) {
                        cr.add_s(a, slot, n);
                        cr.add_s(r, slot, n);
                    }
                }
                if (gl < 6u) {   // (1,2,0) of a and r
                    const uint32_t n = pairs_of(pk, pl, h1, h2, h3), slot = byte_of(sTrees.stara[ra * 4u + pk], pl);
                    if (n) {
                        cr.add_s(a, slot, n);
                        cr.add_s(r, slot, n);
                    }
                }
                if (gl < 3u) {   // (2,1,0), a the second slot: not with its own children, counted below
                    const uint32_t n = pick3(gl + 1u, h1, h2, h3);
                    if (n) cr.add_s(a, byte_of(sTrees.path2[ra * 4u + gl + 1u], ra), 0u - n);
                }
                if (gl == 0u) {
                    shp[1] += h * (d - 1u);
                    shp[2] += h * (h - 1u) / 2u;
                }
                // the children: (2,1,0) and (1,2,0)
                for (uint32_t q = ahi; q > alo; q -= min(8u, q - alo)) {
                    const uint32_t x = q - alo > gl ? sAdj[q - 1u - gl] : 0u, c = x >> 2, k = x & 3u;
                    if (c > r && !L.adjacent(r, c)) {
                        const uint32_t w2 = sTrees.path2[ra * 4u + k], ws = sTrees.stara[ra * 4u + k];
                        const uint32_t n1 = h1 - (k == 1u), n2 = h2 - (k == 2u), n3 = h3 - (k == 3u);
                        if (o1) cr.add_s(c, w2 & 0xFFu, o1);
                        if (o2) cr.add_s(c, (w2 >> 8) & 0xFFu, o2);
                        if (o3) cr.add_s(c, w2 >> 16, o3);
                        if (n1) cr.add_s(c, ws & 0xFFu, n1);
                        if (n2) cr.add_s(c, (ws >> 8) & 0xFFu, n2);
                        if (n3) cr.add_s(c, ws >> 16, n3);
                    }
                    if (q - alo > 8u && (uint32_t)(sAdj[q - 8u] >> 2) <= r) break;
                }
            } else {
                sPre2[u] = 0u;
            }
        }
        __syncthreads();
        // ---- roots, 8 lanes each: r's triples or pairs of slots; (2,1,0) of every slot as the second
        // slot, with all children of r's slots (its own were taken back above)
        for (uint32_t r = tid >> 3; r < n; r += BS / 8) {
            const uint32_t lo = sSplit[r], d = sOff[r + 1] - lo, u0 = sPreD[r];
            if (d == 0u) continue;
            const uint32_t m1 = (sPerm[r] >> 10) & 1023u, m2 = sPerm[r] >> 20, m3 = d - m1 - m2;
            if (K == 3) {
                const uint32_t n = gl < 6u ? pairs_of(pk, pl, m1, m2, m3) : 0u;
                if (n) cr.add_s(r, sTable[motif_index3(pk, pl, 0u)], n);
                if (gl == 0u) shp[0] += d * (d - 1u) / 2u;
                continue;
            }
            for (uint32_t i = gl; i < 10u; i += 8u) {
                const uint32_t t = code_triple(i), k = t & 3u, l = (t >> 2) & 3u, q = t >> 4;
                const uint32_t x = pick3(k, m1, m2, m3), y = pick3(l, m1, m2, m3), z = pick3(q, m1, m2, m3);
                uint32_t n = x * y * z;
                if (k == q) n = x * (x - 1u) / 2u * (x - 2u) / 3u;
                else if (k == l) n = x * (x - 1u) / 2u * z;
                else if (l == q) n = x * (y * (y - 1u) / 2u);
                if (n) cr.add_s(r, byte_of(sTrees.starr[k * 4u + l], q), n);
            }
            if (gl == 0u) shp[0] += d * (d - 1u) / 2u * (d - 2u) / 3u;
            unsigned long long t1 = 0, t2 = 0, t3 = 0;   // children by code (21-bit fields), per code of their slot
            for (uint32_t i = gl; i < d; i += 8u) {
                const unsigned long long h = wide3(sPre2[u0 + i]);
                const uint32_t x = sAdj[lo + i] & 3u;
                t1 += x == 1u ? h : 0ull;
                t2 += x == 2u ? h : 0ull;
                t3 += x == 3u ? h : 0ull;
            }
            t1 = sum8(t1);
            t2 = sum8(t2);
            t3 = sum8(t3);
            for (uint32_t i = gl; i < d; i += 8u) {
                const uint32_t ent = sAdj[lo + i];
                for (uint32_t x = 1; x < 4; x++) {
                    const unsigned long long tx = x == 1u ? t1 : (x == 2u ? t2 : t3);
                    for (uint32_t k = 1; k < 4; k++) {
                        const uint32_t n = (uint32_t)(tx >> (21u * k - 21u)) & 0x1FFFFFu;
                        if (n) cr.add_s(ent >> 2, byte_of(sTrees.path2[x * 4u + k], ent & 3u), n);
                    }
                }
            }
        }
        if constexpr (K == 4) {
            // candidates of each upper entry (r, a): entries of a's row above r
            __syncthreads();
            for (uint32_t u = tid; u < U; u += BS) {
                const uint32_t r = sRootOf[u], a = sAdj[sSplit[r] + u - sPreD[r]] >> 2;
                sPre2[u] = sOff[a + 1] - L.first_above(a, r);
            }
            if (tid == 0) sPre2[U] = 0u;
            __syncthreads();
            const uint32_t N2 = block_exclusive_scan<BS>(sPre2, U + 1, sPart);
            // ---- depth-2 entries (r, a, c), a run of them per thread: the paths and what a row of
            // c holds to correct.  Runs, not strides: the lanes of a wave then rarely share r and a.
            const uint32_t per = (N2 + BS - 1) / BS, q0 = min(N2, tid * per), q1 = min(N2, q0 + per);
            uint32_t u = q0 < q1 ? upper_idx(sPre2, U + 1, q0) : 0u, next = q0, r = 0, a = 0, ra = 0, t = 0;
            for (uint32_t q = q0; q < q1; q++, t++) {
                if (q == next) {   // the entry's first candidate in this run
                    while (sPre2[u + 1] <= q) u++;
                    next = sPre2[u + 1];
                    r = sRootOf[u];
                    const uint32_t ent = sAdj[sSplit[r] + u - sPreD[r]];
                    a = ent >> 2;
                    ra = ent & 3u;
                    t = sOff[a + 1] - (next - q);
                }
                const uint32_t c = sAdj[t] >> 2, ac = sAdj[t] & 3u;
                if (L.adjacent(r, c)) continue;   // c adjacent to r: depth 1, not 2
                const uint32_t w = sTrees.path[ra * 4u + ac], clo = sOff[c];
                uint32_t np = 0;   // paths by arc code 1, 2, 3: 10-bit fields (a row has < 1024 entries)
                uint32_t hi = sOff[c + 1];
                for (bool more = true; more && hi > clo;) {
                    // up to 64 entries of c's row from its end.  Software pipeline: the entry two
                    // ahead and the bitmap words of the next one are read before this entry's
                    // credit (an LDS atomic, which later reads could not otherwise pass)
                    const uint32_t len = min(64u, hi - clo), top = hi - 1u;
                    unsigned long long odd = 0;   // entries with another arc
                    uint32_t e0 = sAdj[top], e1 = sAdj[top - min(1u, len - 1u)];
                    uint32_t wr0 = L.word(r, e0 >> 2), wa0 = L.word(a, e0 >> 2);
                    uint32_t i = 0;
                    for (; i < len; i++) {
                        const uint32_t e2 = sAdj[top - min(i + 2u, len - 1u)];
                        const uint32_t wr1 = L.word(r, e1 >> 2), wa1 = L.word(a, e1 >> 2);
                        const uint32_t e = e0 >> 2, ce = e0 & 3u;
                        if (e <= r) break;
                        const bool x = (((wr0 | wa0) >> (e & 31u)) & 1u) != 0u;
                        e0 = e1;
                        e1 = e2;
                        wr0 = wr1;
                        wa0 = wa1;
                        if (x) {
                            if (e != a) odd |= 1ull << i;
                        } else {
                            cr.add_s(e, byte_of(w, ce), 1u);
                            np += 1u << (10u * ce - 10u);
                        }
                    }
                    more = i == len;
                    for (; odd; odd &= odd - 1ull) {
                        const uint32_t ent = sAdj[top - (uint32_t)(__ffsll((long long)odd) - 1)];
                        const uint32_t e = ent >> 2, ce = ent & 3u;
                        const bool xr = L.adjacent(r, e), xa = L.adjacent(a, e);
                        const uint32_t ae = L.code_if(xa, a, e);
                        if (xr) {   // (2,1,0) with the second slot e: from the lower parent of c
                            const uint32_t re = L.code_if(true, r, e);
                            const uint32_t was = byte_of(sTrees.path2[ra * 4u + ac], re);
                            cr.add_s(r, was, ~0u);
                            cr.add_s(a, was, ~0u);
                            cr.add_s(e, was, ~0u);
                            cr.add_s(c, was, ~0u);
                            if (a < e) {
                                const uint32_t is = sTable[motif_index4(ra, re, 0u, ae, ac, swap_arc_bits(ce))];
                                cr.add1(r, is);
                                cr.add1(a, is);
                                cr.add1(e, is);
                                cr.add1(c, is);
                            } else {
                                shp[1]--;
                            }
                        } else {    // (1,2,0) with the other child e of a: c here, e from its own row
                            const uint32_t was = byte_of(sTrees.stara[ra * 4u + ac], ae);
                            const uint32_t is = sTable[motif_index4(ra, 0u, 0u, ac, ae, ce)];
                            cr.move(c, was, is);
                            if (c < e) {
                                cr.move(r, was, is);
                                cr.move(a, was, is);
                            }
                        }
                    }
                    hi -= len;
                }
                for (uint32_t k = 0; k < 3; k++) {
                    const uint32_t n = (np >> (10u * k)) & 1023u, s = (w >> (8u * k)) & 0xFFu;
                    if (!n) continue;
                    cr.add_s(r, s, n);
                    cr.add_s(a, s, n);
                    cr.add_s(c, s, n);
                    shp[3] += n;
                }
            }
            // ---- triangles, 8 lanes each: those of the queue, or, where it did not hold them all,
            // the candidates again
            __syncthreads();
            const bool all = sTriN <= kTriQueue + tri2;
            const uint32_t ntri = all ? sTriN : N2;
            for (uint32_t i = tid >> 3; i < ntri; i += BS / 8) {
                uint32_t tr, ta, tb;
                if (all) {
                    const uint32_t x = i < kTriQueue ? sTri[i] : sTri2[i - kTriQueue];
                    tr = x & 1023u;
                    ta = (x >> 10) & 1023u;
                    tb = x >> 20;
                } else {
                    const uint32_t v = upper_idx(sPre2, U + 1, i);
                    tr = sRootOf[v];
                    ta = sAdj[sSplit[tr] + v - sPreD[tr]] >> 2;
                    tb = sAdj[sOff[ta + 1] - (sPre2[v + 1] - i)] >> 2;
                    if (tb < ta || !L.adjacent(tr, tb)) continue;
                }
                fix_triangle(L, cr, sTrees, sTable, tr, ta, tb, tid & 7u, 8u);
            }
        }
        __syncthreads();
        // ---- counters -> output.  The block is this workgroup's and was zeroed above; an
        // LDS-counted class never reaches the output otherwise, so its cells are stored.
        for (uint32_t i = tid; i < n * NC; i += BS) {
            const uint32_t x = sCnt[i];
            if (!x && !full) continue;
            const uint32_t v = i / NC, s = i - v * NC;
            const uint32_t cls = full ? s : sSlotCls[s];
            G.out[(size_t)(sPerm[v] & 1023u) * C + cls] = (unsigned long long)x;
        }
        // visited-set counters per shape: k = 3 -> (1,1), (1,2); k = 4 -> the four shapes
        for (int s = 0; s < (K == 3 ? 2 : 4); s++) {
            unsigned long long x = (unsigned long long)(long long)(int32_t)shp[s];
            for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
            if (lane_of() == 0 && x) gadd64(&G.stats[(K == 3 ? 0 : 2) + s], x);
        }
    }
}

}  // namespace

size_t small_lds_bytes(int64_t n, int64_t entries, int k) {
    const int64_t W = (n + 31) / 32;
    const int64_t nc = k == 3 ? kClasses3 : kSlots4;
    // u32 arrays, then the row entries and the roots of the upper entries (u16)
    const int64_t words = (n + 1) * 3 + n + n * W + n * nc + entries / 2 + 1 + (entries + entries / 2 + 1) / 2;
    return (size_t)words * sizeof(uint32_t);
}

bool small_eligible(int64_t n, int64_t entries, int k) {
    return n >= 1 && n <= kSmallMaxN && small_lds_bytes(n, entries, k) <= kSmallLdsBudget;
}

int small_threads(int variant) { return variant <= 0 ? 256 : (variant == 1 ? 512 : 1024); }

void launch_small(SmallArgs a, int k, int variant, unsigned grid, size_t lds, hipStream_t st) {
    void (*kern)(SmallArgs) = nullptr;
    const int bs = small_threads(variant);
    if (k == 3) kern = bs == 256 ? k_small<256, 3> : (bs == 512 ? k_small<512, 3> : k_small<1024, 3>);
    else kern = bs == 256 ? k_small<256, 4> : (bs == 512 ? k_small<512, 4> : k_small<1024, 4>);
    // all the LDS that the workgroups which a CU holds (16 waves by registers) leave each other
    if (k == 4) {
        const size_t fit = std::max<size_t>(1, std::min<size_t>(163840 / (lds + 9216), (size_t)(1024 / bs)));
        lds = std::max(lds, (163840 / fit - 9216) & ~(size_t)15);
    }
    a.lds_words = (uint32_t)(lds / sizeof(uint32_t));
    VDMC_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(kern, dim3(grid), dim3(bs), lds, st, a);
    VDMC_HIP(hipGetLastError());
}

}  // namespace vdmc
