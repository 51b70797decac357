// Hub-root motif kernel: roots with many higher neighbours.
//
// The sets are those of the per-set kernel (count.hip): every connected k-set once,
// from its lowest-rank vertex r (Lemma 1), along the BFS shapes of Lemma 2 under the
// rules of Lemmas 3-4, its motif index from the arc bits (Sec. 4.1), its class from the
// table and one credit for each of its vertices (Sec. 4.2).  What is specific to hub
// roots is that sets are counted in groups: sets that share all members but one, and
// whose last member has the same arc codes, have one index, so a group costs one class
// lookup and one credit per shared member instead of one per set.
//
//   * one workgroup (16 waves) per root; N+(r) (the "slots") is staged in LDS with a
//     hash from rank to slot; each slot's neighbours among the slots become a short
//     list; its entries above r outside N+(r) mark the depth-2 vertices in an index (a
//     bitmap over ranks or a hash) that numbers them, and the parents A(c) = N(c) n N+(r)
//     of each are gathered into one run;
//   * (3,0,0): 2-bit code rows over the slots, 32 slots a word; the group sizes are
//     popcounts of two slots' rows (phase C4);
//   * (2,1,0), (1,2,0) and (1,1,1): per slot a and child c of a, from the counts of the
//     slots by code, of the other parents of c and of the vertices in c's row (phases D, E);
//   * the end vertices of the (1,1,1) paths lie anywhere in the graph: each one that a
//     root reaches is visited once, from its own row, or, where that would read much more
//     than the paths, credited from the rows of the depth-2 vertices (phase G).
// Credits of slots and of r are summed in LDS.  The others go to compact rows (kCmpRow
// counters per vertex) a 64-byte line at a time, because the memory-side atomics (2.4e10
// lines/s whatever the lanes add within a line) are what bounded a kernel that credited
// set by set; k_expand adds the rows to the output.  Measured (one MI355X): Chung-Lu
// n = 1e5, k = 3 and 4, 1.87e10 sets: 145 ms set by set, 37 ms in groups; R-MAT
// n = 2^15, 1.6e10 sets: 212 ms and 25 ms.
#include "motif_device.h"
#include "vdmc_internal.h"

#include <hipcub/hipcub.hpp>

namespace vdmc {
namespace {

constexpr int HT = 1024;                   // threads per hub workgroup
constexpr int NW = HT / 64;                // waves per workgroup
constexpr uint32_t DMAX = kHubMaxDegree;   // largest |N+(r)| (and largest degree) on the hub path
constexpr uint32_t CW = DMAX / 16;         // words of a 2-bit code row over the slots
constexpr uint32_t SHASH = 4096;           // slot hash entries (u16 slot + 1), load <= 1/2
constexpr uint32_t NSTAR = 10;             // star classes
// LARGE: phase G credits end vertices path by path where the rows of a root's depth-2 vertices hold
// less than 1 / kEndsDiv of the graph's entries, else each end once, from its own row, all of which it
// then reads.  G(n, p) of 1e5 vertices of degree 40, every root one way 58 ms, the other 157; R-MAT
// 2^17 314 and 203.  With 4, 8 and 16: R-MAT 2^17 215, 203 and 204 ms, Chung-Lu 1e6 1.80, 1.85 and 1.91 s,
// G(n, p) of degree 120 1.57, 1.56 and 1.80 s.
constexpr unsigned long long kEndsDiv = 8;
constexpr int64_t kHubSmallN = 65536;      // LARGE above it: Chung-Lu 1e5 38.0 -> 34.7 ms, R-MAT 2^15 23.9 -> 25.2
constexpr unsigned long long INV3 = 0xAAAAAAAAAAAAAAABull;      // 3 * INV3 = 1 mod 2^64

struct HubArgs {
    const uint32_t* off;
    const uint32_t* adj;
    const uint32_t* split;
    const int32_t* perm;
    const uint32_t* hubs;        // hub roots, largest work first
    uint32_t nhub;
    unsigned* cursor;            // root cursor
    const uint8_t* t3;
    const uint8_t* t4;
    const uint8_t* maps;         // [0,256) class -> star slot, [256,512) class -> compact counter (0xFF = none)
    const uint8_t* star_cls;     // star slot -> class
    const uint8_t* cmp_cls;      // compact counter -> class
    unsigned long long* out3;
    unsigned long long* out4;
    unsigned long long* stats;
    int k3;
    uint32_t rank_lo, rank_hi;   // only roots with rank in [rank_lo, rank_hi)
    uint32_t* scratch;           // per workgroup: locoff | rows | parents | poff | cids | pcount | index
    size_t wg_words;
    uint32_t s2cap;
    uint32_t n;                  // vertices
    uint32_t hash_below;         // LARGE: roots with fewer entries index their depth-2 vertices by a hash
    void* cmp;                   // compact rows (n x kCmpRow counters, zeroed), or nullptr
    int cmp_wide;                // 64-bit counters instead of 32-bit
    uint32_t split_roots;        // the first split_roots hub roots (the heaviest) ...
    uint32_t shares;             // ... are each taken by this many workgroups (see k_hub)
};

__device__ __forceinline__ uint32_t lane_id() { return threadIdx.x & 63u; }
__device__ __forceinline__ uint32_t wave_id() { return threadIdx.x >> 6; }

__device__ __forceinline__ void gadd(unsigned long long* out, const int32_t* perm, uint32_t C, uint32_t v,
                                     uint32_t cls, unsigned long long cnt) {
    atomicAdd(&out[(size_t)perm[v] * C + cls], cnt);
}

// f(cls, count) once per distinct class among the lanes that reach it with `active`
template <class F>
__device__ __forceinline__ void by_class(uint32_t cls, bool active, F&& f) {
    unsigned long long m = __ballot(active);
    while (m) {
        const uint32_t leader = (uint32_t)(__ffsll((long long)m) - 1);
        const uint32_t k0 = (uint32_t)__shfl((int)cls, (int)leader, 64);
        const unsigned long long same = __ballot(active && cls == k0) & m;
        if (lane_id() == leader) f(k0, (uint32_t)__popcll(same));
        m &= ~same;
    }
}

// sum over the wave, in every lane
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
    int x = (int)v;
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);   // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);   // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);   // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);   // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return (uint32_t)__builtin_amdgcn_readlane(x, 63);
}

// sum over the 16 lanes of a DPP row, in every one of them
__device__ __forceinline__ uint32_t row16_sum(uint32_t v) {
    int x = (int)v;
    x += __builtin_amdgcn_update_dpp(0, x, 0x128, 0xf, 0xf, false);   // row_ror:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x124, 0xf, 0xf, false);   // row_ror:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x122, 0xf, 0xf, false);   // row_ror:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x121, 0xf, 0xf, false);   // row_ror:1
    return (uint32_t)x;
}

// n (signed) sets to counter s of vertex v's compact row, by the 16 lanes of a line (the whole
// wave calls it): one request per line with a non-zero counter
__device__ __forceinline__ void cmp_line(const HubArgs& A, uint32_t v, uint32_t s, uint32_t n) {
    const bool any = ((__ballot(n != 0u) >> (lane_id() & 48u)) & 0xFFFFull) != 0ull;
    if (!any) return;
    const size_t at = (size_t)v * kCmpRow + s;
    if (A.cmp == nullptr) {
        if (n) gadd(A.out4, A.perm, kClasses4, v, A.cmp_cls[s], (unsigned long long)(long long)(int32_t)n);
    } else if (A.cmp_wide) {
        atomicAdd((unsigned long long*)A.cmp + at, (unsigned long long)(long long)(int32_t)n);
    } else {
        atomicAdd((uint32_t*)A.cmp + at, n);
    }
}

// n sets to counter s of vertex v's compact row, by one lane
__device__ __forceinline__ void cmp_add(const HubArgs& A, uint32_t v, uint32_t s, uint32_t n) {
    const size_t at = (size_t)v * kCmpRow + s;
    if (A.cmp == nullptr) gadd(A.out4, A.perm, kClasses4, v, A.cmp_cls[s], n);
    else if (A.cmp_wide) atomicAdd((unsigned long long*)A.cmp + at, (unsigned long long)n);
    else atomicAdd((uint32_t*)A.cmp + at, n);
}

// the count of code s (0..8) in a depth-2 vertex's parents by code
__device__ __forceinline__ uint32_t parents_of(ulonglong2 pc, uint32_t s) {
    return (uint32_t)(s < 5u ? pc.x >> (12u * s) : pc.y >> (12u * (s - 5u))) & 0xFFFu;
}

// The depth-2 vertices of a root, numbered: a bitmap B over ranks and P[w] = how many lie before
// word w (for words that hold one), or, LARGE, a hash of them, in LDS or in the workgroup's scratch.
// The bitmap costs a root n / 32 words whatever it reaches, the hash 3/2 of its entries: 5000 trees of
// 40 x 4 vertices in 2^22 vertices 27.4 ms with the bitmap, 1.2 with the hash.  A find in the hash costs
// more, which phase E, where most of them are, does without.
template <bool LARGE>
struct Index2 {
    static constexpr uint32_t kTag = 0xFFC00000u;   // hash slot: 10 bits of the product, number + 1; 0 = empty
    bool in_lds, hashed;
    lptr<uint32_t> l;
    gptr<uint32_t> g;
    uint32_t w;                  // words of the bitmap, or slots of the hash
    gptr<const uint32_t> ids;    // number -> vertex
    __device__ __forceinline__ Index2(bool lds, bool hash, uint32_t* lp, uint32_t* gp, uint32_t words,
                                      const uint32_t* v)
        : in_lds(!LARGE || lds), hashed(LARGE && hash), l(lp), g(gp), w(words), ids((uint32_t*)v) {}
    // words of the index for a root with `entries` entries above it in its slots' rows
    static __host__ __device__ __forceinline__ uint32_t slots(uint32_t entries) { return entries + entries / 2u + 1u; }
    __device__ __forceinline__ uint32_t word(uint32_t i) const { return in_lds ? l[i] : g[i]; }
    __device__ __forceinline__ uint32_t before(uint32_t i) const { return in_lds ? l[w + i] : g[w + i]; }
    __device__ __forceinline__ void set(uint32_t i, uint32_t x) const {
        if (in_lds) l[i] = x;
        else g[i] = x;
    }
    __device__ __forceinline__ void set_before(uint32_t i, uint32_t j) const { set(w + i, j); }
    __device__ __forceinline__ uint32_t cas(uint32_t i, uint32_t x) const {   // 0 -> x; what it was
        uint32_t old = 0;
        if (in_lds)
            __hip_atomic_compare_exchange_strong((l + i), &old, x, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WORKGROUP);
        else
            __hip_atomic_compare_exchange_strong((g + i), &old, x, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
        return old;
    }
    __device__ __forceinline__ uint32_t next(uint32_t h) const { return h + 1u < w ? h + 1u : 0u; }
    // marks vertex e; a hash holds e + 1 until number() is called
    __device__ __forceinline__ void mark(uint32_t e) const {
        if (hashed) {
            for (uint32_t h = __umulhi(e * 0x9E3779B1u, w);; h = next(h)) {
                uint32_t k = word(h);
                if (k == 0u) k = cas(h, e + 1u);
                if (k == 0u || k == e + 1u) return;
            }
        }
        const uint32_t bit = 1u << (e & 31u);
        if (in_lds) __hip_atomic_fetch_or((l + (e >> 5)), bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        else __hip_atomic_fetch_or((g + (e >> 5)), bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    // a hash of marks numbered in any order (every thread; *ctr = 0 before, their number after)
    __device__ __forceinline__ void number(uint32_t* ctr, uint32_t* cids) const {
        for (uint32_t i0 = wave_id() * 64u; i0 < w; i0 += HT) {
            const uint32_t i = i0 + lane_id();
            uint32_t k = 0;
            if (i < w) k = in_lds ? l[i] : __hip_atomic_load((g + i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const unsigned long long m = __ballot(k != 0u);
            if (m == 0ull) continue;
            uint32_t j = 0;
            if (lane_id() == 0) j = atomicAdd(ctr, (uint32_t)__popcll(m));
            j = (uint32_t)__builtin_amdgcn_readfirstlane((int)j) + (uint32_t)__popcll(m & ((1ull << lane_id()) - 1ull));
            if (k) {
                cids[j] = k - 1u;
                set(i, (((k - 1u) * 0x9E3779B1u) << 22) | (j + 1u));
            }
        }
    }
    __device__ __forceinline__ void clear() const {
        if (in_lds)
            for (uint32_t i = threadIdx.x; i < w; i += HT) l[i] = 0u;
        else
            for (uint32_t i = threadIdx.x; i < w; i += HT) g[i] = 0u;
    }
    // number of vertex e among the depth-2 vertices, or ~0: from the bitmap; from either
    __device__ __forceinline__ uint32_t find_bit(uint32_t e) const {
        const uint32_t b = word(e >> 5), bit = 1u << (e & 31u);
        return (b & bit) ? before(e >> 5) + (uint32_t)__popc(b & (bit - 1u)) : ~0u;
    }
    __device__ __forceinline__ uint32_t find(uint32_t e) const {
        if (hashed) {
            const uint32_t x = e * 0x9E3779B1u;
            for (uint32_t h = __umulhi(x, w);; h = next(h)) {
                const uint32_t s = word(h);
                if (s == 0u) return ~0u;
                if ((s & kTag) == (x << 22) && ids[(s & ~kTag) - 1u] == e) return (s & ~kTag) - 1u;
            }
        }
        return find_bit(e);
    }
    // from the list of the depth-2 vertices, ascending for the bitmap (every thread of the workgroup)
    __device__ __forceinline__ void fill(uint32_t nc) const {
        clear();
        __syncthreads();
        for (uint32_t j = threadIdx.x; j < nc; j += HT) {
            const uint32_t c = ids[j];
            if (hashed) {
                const uint32_t x = c * 0x9E3779B1u;
                uint32_t h = __umulhi(x, w);
                while (cas(h, (x << 22) | (j + 1u))) h = next(h);
                continue;
            }
            mark(c);
            if (j == 0u || (ids[j - 1u] >> 5) != (c >> 5)) set_before(c >> 5, j);
        }
    }
};

// f(cls, sum of val) once per distinct class among the lanes with `active` (the whole wave calls it)
template <class F>
__device__ __forceinline__ void by_class_sum(uint32_t cls, uint32_t val, bool active, F&& f) {
    unsigned long long m = __ballot(active);
    while (m) {
        const uint32_t leader = (uint32_t)(__ffsll((long long)m) - 1);
        const uint32_t k0 = (uint32_t)__builtin_amdgcn_readlane((int)cls, (int)leader);
        const bool mine = active && cls == k0;
        const uint32_t sum = wave_sum(mine ? val : 0u);
        if (lane_id() == leader) f(k0, sum);
        m &= ~__ballot(mine);
    }
}

__device__ __forceinline__ uint32_t code_at(const uint32_t* row, uint32_t i) {
    return (row[i >> 4] >> ((i & 15u) << 1)) & 3u;
}

__device__ __forceinline__ uint32_t shash(uint32_t x) { return (x * 2654435761u) >> 20; }   // 12 bits

// slot of rank x in the LDS slot hash (u16 slot + 1 per entry), or -1
__device__ __forceinline__ int slot_find(const uint16_t* H, const uint32_t* P, uint32_t x) {
    for (uint32_t h = shash(x);; h = (h + 1u) & (SHASH - 1u)) {
        const uint32_t s = H[h];
        if (s == 0u) return -1;
        if ((P[s - 1u] >> 2) == x) return (int)(s - 1u);
    }
}

// insert slot i (rank x) into the slot hash; 16-bit entries updated through their word
__device__ __forceinline__ void slot_insert(uint16_t* H, uint32_t x, uint32_t i) {
    for (uint32_t h = shash(x);; h = (h + 1u) & (SHASH - 1u)) {
        uint32_t* w = (uint32_t*)&H[h & ~1u];
        const uint32_t sh = (h & 1u) << 4;
        uint32_t old = *w;
        while (((old >> sh) & 0xFFFFu) == 0u) {
            const uint32_t got = atomicCAS(w, old, old | ((i + 1u) << sh));
            if (got == old) return;
            old = got;
        }
    }
}

// bit of rank x in a filter of FILTER_BITS bits
constexpr uint32_t FILTER_BITS = 16384;
__device__ __forceinline__ uint32_t filter_bit(uint32_t x) { return (x * 0x9E3779B1u) >> 18; }

// one dynamic task index per wave (LDS counter)
__device__ __forceinline__ uint32_t wave_task(uint32_t* ctr) {
    uint32_t t = 0;
    if (lane_id() == 0) t = atomicAdd(ctr, 1u);
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)t);
}

__device__ __forceinline__ uint32_t first_above(const uint32_t* adj, uint32_t lo, uint32_t hi, uint32_t r) {
    return lower_bound_rank(adj, lo, hi, r + 1u);
}

// exclusive scan of a[0..len) in place (any memory the workgroup sees), returns the total;
// part: HT words of LDS
__device__ uint32_t block_scan(uint32_t* a, uint32_t len, uint32_t* part) {
    const uint32_t tid = threadIdx.x;
    const uint32_t per = (len + HT - 1) / HT;
    const uint32_t lo = min(len, tid * per), hi = min(len, lo + per);
    uint32_t s = 0;
    for (uint32_t i = lo; i < hi; i++) s += a[i];
    part[tid] = s;
    __syncthreads();
    for (uint32_t off = 1; off < HT; off <<= 1) {
        const uint32_t v = tid >= off ? part[tid - off] : 0u;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    uint32_t run = part[tid] - s;
    for (uint32_t i = lo; i < hi; i++) {
        const uint32_t x = a[i];
        a[i] = run;
        run += x;
    }
    const uint32_t total = part[HT - 1];
    __syncthreads();
    return total;
}

// ----------------------------------------------------------------------------- LDS

constexpr uint32_t U_WORDS = 34000;   // the phase-dependent region (133 KiB)

// the fixed part of it in phases E and G
constexpr uint32_t E_GW = 96;   // words per 16-lane group: 3 lines, 9 + 36 pair counts
constexpr uint32_t E_AW = 200;  // words per wave: a's classes
constexpr uint32_t E_FIX = (HT / 16) * E_GW + NW * E_AW + NW * CW + SHASH / 2;
constexpr uint32_t G_EB = 4;    // end vertices per group between two flushes
constexpr uint32_t G_FIX = (HT / 16) * 16 * G_EB + NW * CW + SHASH / 2 + 32;
constexpr uint32_t G_WIN = 4096;   // least words of a window of ranks

// whether an index of iw words fits LDS for every root of up to D slots: in phases B and G (a hash);
// in phase E too (a bitmap)
bool hash_fits(size_t D, size_t iw) {
    return SHASH / 2 + HT + D * kClasses3 + iw <= U_WORDS && G_FIX + iw + G_WIN <= U_WORDS;
}
bool bitmap_fits(size_t D, size_t iw) {
    return hash_fits(D, iw) && D * 5 + 2 + E_FIX + iw + NW * (FILTER_BITS / 32) <= U_WORDS;
}

struct HubLds {
    uint32_t P[DMAX];                  // slots: (rank << 2) | arc bits r -> slot
    uint16_t locn[DMAX];               // local neighbours per slot
    uint16_t ch1[DMAX], ch2[DMAX];     // depth-2 entries per slot with arc code 1, 2
    unsigned long long root3[kClasses3];
    unsigned long long root4[kClasses4];
    uint8_t t4[4096];
    uint8_t t3[64];
    uint8_t maps[512];
    uint32_t ctr[8];
    uint32_t seg[2];                   // first slot with arc code 2, 3 to r
    unsigned long long ends;           // entries in the rows of the depth-2 vertices (LARGE)
    alignas(16) uint32_t U[U_WORDS];
};
static_assert(sizeof(HubLds) + 16 <= 163840, "one workgroup's LDS");

// the per-wave 2-bit code row over the slots from slot x's local list
__device__ __forceinline__ void build_row(uint32_t* row, const uint32_t* locnbr, uint32_t base, uint32_t cnt) {
    const uint32_t lane = lane_id();
    for (uint32_t i = lane; i < CW; i += 64) row[i] = 0u;
    __threadfence_block();
    for (uint32_t i = lane; i < cnt; i += 64) {
        const uint32_t e = locnbr[base + i];
        atomicOr(&row[(e >> 2) >> 4], (e & 3u) << (((e >> 2) & 15u) << 1));
    }
    __threadfence_block();
}

// ----------------------------------------------------------------------------- hub kernel

// K4 = false (k = 3 alone): phases A, B and C3 only.  A kernel of its own (54 registers), as
// the other's spill, which a launch of some 40 us feels: R-MAT 2^10, five ranges, 271 -> 250 us.
// LARGE (graphs whose bitmap of the depth-2 vertices is not in LDS for every root, or of more than
// kHubSmallN vertices): no part of a root's cost grows with n unless its entries do, see Index2 and
// kEndsDiv.  The other index and way of crediting end vertices take 6 registers more to spill.
template <bool K4, bool LARGE>
__global__ __launch_bounds__(HT) void k_hub(HubArgs A) {
    __shared__ HubLds L;
    __shared__ uint32_t sRoot;
    const uint32_t tid = threadIdx.x, lane = lane_id(), wid = wave_id();
    for (uint32_t i = tid; K4 && i < 4096; i += HT) L.t4[i] = A.t4[i];
    for (uint32_t i = tid; i < 64; i += HT) L.t3[i] = A.t3[i];
    for (uint32_t i = tid; K4 && i < 512; i += HT) L.maps[i] = A.maps[i];
    const uint8_t* star_of = L.maps;
    const uint8_t* cmp_of = L.maps + 256;
    uint32_t* S = A.scratch + (size_t)blockIdx.x * A.wg_words;
    uint32_t* locoff = S;                                        // DMAX + 2
    // rows: slot x has the words [locoff[x], locoff[x + 1]): its local entries from the
    // front, its depth-2 entries from the back (rank, then index of the vertex, and code)
    uint32_t* locnbr = locoff + DMAX + 2;                        // s2cap
    uint32_t* parents = locnbr + A.s2cap;                        // s2cap: A(c) of every depth-2 vertex
    uint32_t* poff = parents + A.s2cap;                          // s2cap: first parent of the j-th
    uint32_t* cids = poff + A.s2cap;                             // s2cap: its rank (ascending)
    // s2cap x 16 bytes: first an entry's place among its parents (one word each), then the
    // parents of the j-th by the codes (to r, to c): nine 12-bit counts, five in the first
    // word, four in the second, and above them the mask of the non-zero ones
    ulonglong2* pcount = (ulonglong2*)(S + ((DMAX + 2 + 4 * (size_t)A.s2cap + 3) & ~(size_t)3));
    uint32_t* place = (uint32_t*)pcount;
    uint32_t* gidx = (uint32_t*)(pcount + A.s2cap);              // the index of the depth-2 vertices when
                                                                 // LDS has no room (LARGE)
    const uint32_t nbw = (A.n + 31u) >> 5;
    unsigned long long shp[kShapes] = {0, 0, 0, 0, 0, 0};

    // The heaviest hub roots (the first A.split_roots of the queue) are each taken by
    // A.shares workgroups, so that no single root's workgroup is the critical path.  Each
    // stages the whole root (its lists live in its own scratch) and does the share of every
    // phase's tasks that is its own: slots x with x % G == share and, in phase G, paths over
    // depth-2 vertices c with c % G == share.  Its counters are partial sums (signed: a group
    // and its correction may fall to different shares), flushed with atomics like a whole
    // root's.  Later roots are taken whole (G = 1).
    const uint32_t split_tasks = A.split_roots * A.shares;
    for (;;) {
        __syncthreads();
        if (tid == 0) sRoot = atomicAdd(&A.cursor[0], 1u);
        __syncthreads();
        const uint32_t vi = sRoot;
        const uint32_t G = vi < split_tasks ? A.shares : 1u;
        const uint32_t hi_idx = vi < split_tasks ? vi / G : A.split_roots + (vi - split_tasks);
        const uint32_t share = vi < split_tasks ? vi - hi_idx * G : 0u;
        if (hi_idx >= A.nhub) break;
        const uint32_t r = A.hubs[hi_idx];
        if (r < A.rank_lo || r >= A.rank_hi) continue;   // uniform over the workgroup
        const uint32_t s0 = A.split[r];
        const uint32_t D = A.off[r + 1] - s0;
        // ---- phase A: stage the slots, the lengths of their rows above r, clear counters
        uint16_t* H = (uint16_t*)L.U;   // slot hash (phases A-B)
        // Slots ordered by their arc code to r, by rank within a code.  Any fixed order of
        // N+(r) enumerates each set once ((3,0,0) takes a < b < c, (2,1,0) hangs c under
        // its lowest parent); this one gives the lanes of a step over consecutive slots
        // the same code to r, so that sets without extra pairs share their class.
        if (wid == 0) {
            const unsigned long long below = (1ull << lane) - 1ull;
            uint32_t n1 = 0, n2 = 0;
            for (uint32_t q0 = 0; q0 < D; q0 += 64) {
                const uint32_t k = q0 + lane < D ? (A.adj[s0 + q0 + lane] & 3u) : 0u;
                n1 += (uint32_t)__popcll(__ballot(k == 1u));
                n2 += (uint32_t)__popcll(__ballot(k == 2u));
            }
            uint32_t o[4] = {0u, 0u, n1, n1 + n2};
            if (lane < 2) L.seg[lane] = n1 + (lane ? n2 : 0u);
            for (uint32_t q0 = 0; q0 < D; q0 += 64) {
                const bool in = q0 + lane < D;
                const uint32_t e = in ? A.adj[s0 + q0 + lane] : 0u, k = e & 3u;
                const unsigned long long m1 = __ballot(in && k == 1u), m2 = __ballot(in && k == 2u),
                                         m3 = __ballot(in && k == 3u);
                const unsigned long long mk = k == 1u ? m1 : (k == 2u ? m2 : m3);
                if (in) L.P[o[k] + (uint32_t)__popcll(mk & below)] = e;
                o[1] += (uint32_t)__popcll(m1);
                o[2] += (uint32_t)__popcll(m2);
                o[3] += (uint32_t)__popcll(m3);
            }
        }
        for (uint32_t i = tid; i < SHASH / 2; i += HT) L.U[i] = 0u;
        for (uint32_t i = tid; i < kClasses3; i += HT) L.root3[i] = 0ull;
        for (uint32_t i = tid; K4 && i < kClasses4; i += HT) L.root4[i] = 0ull;
        if (tid < 8) L.ctr[tid] = 0u;
        __syncthreads();
        for (uint32_t i = tid; i < D; i += HT) {
            const uint32_t x = L.P[i] >> 2;
            locoff[i] = A.off[x + 1] - first_above(A.adj, A.off[x], A.off[x + 1], r);
            slot_insert(H, x, i);
        }
        if (tid == 0) locoff[D] = 0u;
        __syncthreads();
        uint32_t* part = L.U + SHASH / 2;   // HT words after the slot hash
        const uint32_t entries = block_scan(locoff, D + 1, part);
        // ---- phase B: rows of the slots: local lists, depth-2 entries, k = 3 (1,2)
        uint32_t* R3 = L.U + SHASH / 2 + HT;   // D x 13 k = 3 counters of the slots
        if (A.k3)
            for (uint32_t i = tid; i < D * kClasses3; i += HT) R3[i] = 0u;
        // the index of the depth-2 vertices, in LDS where it fits
        const uint32_t used = SHASH / 2 + HT + (A.k3 ? D * kClasses3 : 0u);
        const bool hashed = LARGE && entries < A.hash_below;
        const uint32_t iw = hashed ? Index2<LARGE>::slots(entries) : 2u * nbw;   // its words
        const uint32_t isz = hashed ? iw : nbw;
        const bool kept = LARGE && used + iw > U_WORDS;   // in scratch: phases E and G find it there
        const Index2<LARGE> X2(!kept, hashed, L.U + used, gidx, isz, cids);
        if (K4) X2.clear();
        __syncthreads();
        for (;;) {
            const uint32_t x = wave_task(&L.ctr[0]);
            if (x >= D) break;
            const bool own = x % G == share;   // staging for every slot, credits for its own
            const uint32_t vx = L.P[x] >> 2, rx = L.P[x] & 3u;
            const uint32_t hi = A.off[vx + 1];
            const uint32_t base = locoff[x];
            const uint32_t end = locoff[x + 1];
            const uint32_t lo = hi - (end - base);
            uint32_t nloc = 0, nch = 0, nc1 = 0, nc2 = 0;
            for (uint32_t q0 = lo; q0 < hi; q0 += 64) {
                const uint32_t q = q0 + lane;
                const bool in = q < hi;
                uint32_t e = 0, ec = 0;
                int sl = -1;
                if (in) {
                    e = A.adj[q] >> 2;
                    ec = A.adj[q] & 3u;
                    sl = slot_find(H, L.P, e);
                }
                const bool local = in && sl >= 0, d2 = in && sl < 0;
                const unsigned long long ml = __ballot(local);
                if (local)
                    locnbr[base + nloc + (uint32_t)__popcll(ml & ((1ull << lane) - 1ull))] = ((uint32_t)sl << 2) | ec;
                nloc += (uint32_t)__popcll(ml);
                if (A.k3) {   // (1,2): r - x - e
                    const uint32_t cls = L.t3[motif_index3(rx, 0u, ec)];
                    by_class(cls, own && d2, [&](uint32_t k, uint32_t n) {
                        atomicAdd(&L.root3[k], (unsigned long long)n);
                        atomicAdd(&R3[x * kClasses3 + k], n);
                    });
                    if (own && d2) {
                        gadd(A.out3, A.perm, kClasses3, e, cls, 1ull);
                        shp[1]++;
                    }
                }
                if (K4) {   // depth-2 entry (x, e): e marked, the entry behind x's row
                    const unsigned long long md = __ballot(d2);
                    if (d2) {
                        X2.mark(e);
                        locnbr[end - 1u - nch - (uint32_t)__popcll(md & ((1ull << lane) - 1ull))] = (e << 2) | ec;
                    }
                    nch += (uint32_t)__popcll(md);
                    nc1 += (uint32_t)__popcll(__ballot(d2 && ec == 1u));
                    nc2 += (uint32_t)__popcll(__ballot(d2 && ec == 2u));
                }
            }
            if (lane == 0) {
                L.locn[x] = (uint16_t)nloc;
                L.ch1[x] = (uint16_t)nc1;
                L.ch2[x] = (uint16_t)nc2;
            }
        }
        __syncthreads();
        // the depth-2 vertices numbered (cids; by the bitmap in rank order), their parents gathered:
        // A(c_j) = parents[poff[j] .. poff[j + 1])
        uint32_t ngroups = 0;
        if (K4) {
            if (hashed) {
                X2.number(&L.ctr[1], cids);
                __syncthreads();
                ngroups = L.ctr[1];
            } else {
                for (uint32_t i = tid; i < nbw; i += HT) X2.set_before(i, (uint32_t)__popc(X2.word(i)));
                __syncthreads();
                ngroups = kept ? block_scan(gidx + nbw, nbw, part) : block_scan(L.U + used + nbw, nbw, part);
                for (uint32_t i = tid; i < nbw; i += HT) {
                    uint32_t at = X2.before(i);
                    for (uint32_t w = X2.word(i); w; w &= w - 1u) cids[at++] = (i << 5) + (uint32_t)__ffs((int)w) - 1u;
                }
            }
            for (uint32_t j = tid; j <= ngroups; j += HT) poff[j] = 0u;
            __syncthreads();
            for (uint32_t x = wid; x < D; x += NW) {
                const uint32_t end = locoff[x + 1], m = end - locoff[x] - L.locn[x];
                for (uint32_t i = lane; i < m; i += 64) {
                    const uint32_t ent = locnbr[end - 1u - i], j = X2.find(ent >> 2);
                    locnbr[end - 1u - i] = (j << 2) | (ent & 3u);
                    place[end - 1u - i] = atomicAdd(&poff[j], 1u);
                }
            }
            __syncthreads();
            block_scan(poff, ngroups + 1u, part);
            for (uint32_t x = wid; x < D; x += NW) {
                const uint32_t end = locoff[x + 1], m = end - locoff[x] - L.locn[x];
                for (uint32_t i = lane; i < m; i += 64) {
                    const uint32_t ent = locnbr[end - 1u - i];
                    parents[poff[ent >> 2] + place[end - 1u - i]] = (x << 2) | (ent & 3u);
                }
            }
            __syncthreads();
            // the parents of each depth-2 vertex counted by their codes to r and to it
            for (uint32_t j0 = wid * 4u; j0 < ngroups; j0 += NW * 4u) {
                const uint32_t j = j0 + (lane >> 4);
                const uint32_t f0 = j < ngroups ? poff[j] : 0u, f1 = j < ngroups ? poff[j + 1] : 0u;
                unsigned long long lo = 0, hi = 0;
                for (uint32_t i = 0; __ballot(f0 + i < f1); i += 16u) {
                    const uint32_t f = f0 + i + (lane & 15u);
                    const uint32_t pe = f < f1 ? parents[f] : 0u;
                    const uint32_t code = f < f1 ? ((L.P[pe >> 2] & 3u) - 1u) * 3u + (pe & 3u) - 1u : 9u;
#pragma unroll
                    for (uint32_t q = 0; q < 9; q++) {
                        const unsigned long long n = __popcll((__ballot(code == q) >> (lane & 48u)) & 0xFFFFull);
                        if (q < 5) lo += n << (12u * q);
                        else hi += n << (12u * (q - 5u));
                        if (n) hi |= 1ull << (48u + q);
                    }
                }
                if ((lane & 15u) == 0u && j < ngroups) pcount[j] = make_ulonglong2(lo, hi);
            }
            __syncthreads();
        }
        // ---- phase C3: k = 3 (1,1): pairs a < b of slots, lanes over b
        if (A.k3) {
            uint32_t* rows = R3 + DMAX * kClasses3;   // per wave: one code row
            for (;;) {
                const uint32_t a = wave_task(&L.ctr[3]) * G + share;
                if (a + 1 >= D) break;
                uint32_t* BA = rows + wid * CW;
                build_row(BA, locnbr, locoff[a], L.locn[a]);
                const uint32_t ra = L.P[a] & 3u;
                for (uint32_t b0 = a + 1; b0 < D; b0 += 64) {
                    const uint32_t b = b0 + lane;
                    const bool in = b < D;
                    uint32_t cls = 0xFFu;
                    if (in) cls = L.t3[motif_index3(ra, L.P[b] & 3u, code_at(BA, b))];
                    by_class(cls, in, [&](uint32_t k, uint32_t n) {
                        atomicAdd(&L.root3[k], (unsigned long long)n);
                        atomicAdd(&R3[a * kClasses3 + k], n);
                    });
                    if (in) {
                        atomicAdd(&R3[b * kClasses3 + cls], 1u);
                        shp[0]++;
                    }
                }
            }
            __syncthreads();
            for (uint32_t i = tid; i < D * kClasses3; i += HT) {
                const uint32_t x = R3[i];
                if (x) gadd(A.out3, A.perm, kClasses3, L.P[i / kClasses3] >> 2, i % kClasses3, x);
            }
            for (uint32_t i = tid; i < kClasses3; i += HT)
                if (L.root3[i]) gadd(A.out3, A.perm, kClasses3, r, i, L.root3[i]);
        }
        if (!K4) continue;
        const uint32_t seg2 = __builtin_amdgcn_readfirstlane(L.seg[0]), seg3 = __builtin_amdgcn_readfirstlane(L.seg[1]);
        __syncthreads();
        auto seg_at = [&](uint32_t k) -> uint32_t { return k < 2u ? 0u : (k == 2u ? seg2 : (k == 3u ? seg3 : D)); };
        // ---- phase C4: (3,0,0): three slots.  A lane owns the slot a it credits; the pairs
        // {b < c} of other slots come from the 2-bit code rows of b, 32 c's a word: the
        // number of c's of one arc code to r (a run of slots) with codes ac and bc is a
        // popcount of the rows' planes, so a group of sets that share r, a, b and the index
        // costs one lane a few instructions.  Pairs whose b is adjacent to a are counted as
        // if it were not, then moved to their index, one lane per adjacent pair (a, b).
        // Every set is counted from each of its three slots; r takes a third of the sums,
        // exactly, mod 2^64 (also when the tasks are shared by several workgroups).
        {
            const uint32_t W = (D + 31u) >> 5;
            const bool inl = D * (NSTAR + 2u * (W | 1u)) <= U_WORDS;   // star counters in LDS
            uint32_t* R4 = L.U;                                        // D x 10 star counters
            uint2* X = (uint2*)(L.U + (inl ? D * NSTAR : 0u));         // D rows of Wb words, both planes
            const uint32_t smax = (U_WORDS - (inl ? D * NSTAR : 0u)) / (2u * D);
            const uint32_t Wb = (W | 1u) <= smax ? W : ((smax & 1u) ? smax : smax - 1u);
            const uint32_t S1 = Wb | 1u;                               // odd stride: no bank conflicts
            const uint32_t CB = D <= 256u ? 8u : (D <= 512u ? 16u : 32u);   // b's per task
            const uint32_t nag = (D + 63u) >> 6;
            if (inl)
                for (uint32_t i = tid; i < D * NSTAR; i += HT) R4[i] = 0u;
            // n sets of slot a with index code `code`
            auto add_a = [&](uint32_t a, uint32_t cls, uint32_t n) {
                const uint32_t s = star_of[cls];
                if (inl && s < NSTAR) atomicAdd(&R4[a * NSTAR + s], n);
                else gadd(A.out4, A.perm, kClasses4, L.P[a] >> 2, cls, (unsigned long long)(long long)(int32_t)n);
            };
            auto add_r = [&](uint32_t cls, uint32_t n) {
                atomicAdd(&L.root4[cls], (unsigned long long)(long long)(int32_t)n * INV3);
            };
            // s[i][j] (all, bit 0, bit 1, both) -> sets by the codes 0..3 of both pairs
            auto exact = [](uint32_t (&s)[16]) {
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    s[0 + j] += s[12 + j] - s[4 + j] - s[8 + j];
                    s[4 + j] -= s[12 + j];
                    s[8 + j] -= s[12 + j];
                }
#pragma unroll
                for (int i = 0; i < 16; i += 4) {
                    s[i] += s[i + 3] - s[i + 1] - s[i + 2];
                    s[i + 1] -= s[i + 3];
                    s[i + 2] -= s[i + 3];
                }
            };
            // slots of the word w whose arc code to r is k
            auto seg_word = [&](uint32_t k, uint32_t w) {
                const uint32_t lo = seg_at(k), hi = seg_at(k + 1), b0 = w << 5;
                uint32_t m = ~0u;
                if (lo > b0) m &= lo - b0 < 32u ? ~0u << (lo - b0) : 0u;
                if (hi < b0 + 32u) m &= hi > b0 ? ~(~0u << (hi - b0)) : 0u;
                return m;
            };
            for (uint32_t w0 = 0; w0 < W; w0 += Wb) {
                const uint32_t wn = min(Wb, W - w0);
                __syncthreads();
                for (uint32_t i = tid; i < D * S1; i += HT) X[i] = make_uint2(0u, 0u);
                if (tid < 2) L.ctr[4 + tid] = 0u;
                __syncthreads();
                for (uint32_t x = wid; x < D; x += NW) {
                    const uint32_t base = locoff[x], nl = L.locn[x];
                    for (uint32_t i = lane; i < nl; i += 64) {
                        const uint32_t e = locnbr[base + i], w = (e >> 7) - w0, bit = 1u << ((e >> 2) & 31u);
                        if (w < wn) {
                            uint32_t* p = &X[x * S1 + w].x;
                            if (e & 1u) atomicOr(p, bit);
                            if (e & 2u) atomicOr(p + 1, bit);
                        }
                    }
                }
                __syncthreads();
                const uint32_t ntask = nag * ((min(D, (w0 + wn) << 5) + CB - 1u) / CB);
                for (;;) {   // lanes over a, b's in turn
                    const uint32_t t = wave_task(&L.ctr[4]) * G + share;
                    if (t >= ntask) break;
                    const uint32_t ch = t / nag, ag = t - ch * nag;
                    const uint32_t a = ag * 64u + lane;
                    const bool alive = a < D;
                    const uint32_t ra = alive ? L.P[a] & 3u : 0u;
                    for (uint32_t rb = 1; rb < 4; rb++) {
                        const uint32_t blo = max(ch * CB, seg_at(rb)), bhi = min(ch * CB + CB, seg_at(rb + 1));
                        if (blo >= bhi) continue;
                        for (uint32_t rc = rb; rc < 4; rc++) {
                            const uint32_t clo = max(seg_at(rc), blo + 1u), chi = seg_at(rc + 1);
                            if (clo >= chi) continue;
                            const uint32_t wlo = max(clo >> 5, w0), whi = min(((chi - 1u) >> 5) + 1u, w0 + wn);
                            uint32_t s[16] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
                            for (uint32_t w = wlo; w < whi; w++) {
                                const uint32_t sm = seg_word(rc, w);
                                const uint2 aw = alive ? X[a * S1 + w - w0] : make_uint2(0u, 0u);
                                const uint32_t a0 = aw.x, a1 = aw.y, a01 = a0 & a1;
                                const uint32_t ae = alive ? ((a >> 5) == w ? ~(1u << (a & 31u)) : ~0u) : 0u;
                                for (uint32_t b = blo; b < bhi; b++) {
                                    if ((b >> 5) > w) break;
                                    const uint32_t v = (b >> 5) == w ? sm & ~((2u << (b & 31u)) - 1u) : sm;
                                    const uint2 bw = X[b * S1 + w - w0];
                                    const uint32_t b0 = __builtin_amdgcn_readfirstlane(bw.x) & v;
                                    const uint32_t b1 = __builtin_amdgcn_readfirstlane(bw.y) & v;
                                    if (a != b) {
                                        s[0] += __popc(ae & v);
                                        s[4] += __popc(a0 & v);
                                        s[8] += __popc(a1 & v);
                                        s[12] += __popc(a01 & v);
                                        if (b0 | b1) {
                                            const uint32_t b01 = b0 & b1;
                                            s[1] += __popc(ae & b0);
                                            s[5] += __popc(a0 & b0);
                                            s[9] += __popc(a1 & b0);
                                            s[13] += __popc(a01 & b0);
                                            s[2] += __popc(ae & b1);
                                            s[6] += __popc(a0 & b1);
                                            s[10] += __popc(a1 & b1);
                                            s[14] += __popc(a01 & b1);
                                            if (b01) {
                                                s[3] += __popc(ae & b01);
                                                s[7] += __popc(a0 & b01);
                                                s[11] += __popc(a1 & b01);
                                                s[15] += __popc(a01 & b01);
                                            }
                                        }
                                    }
                                }
                            }
                            shp[2] += s[0];
                            exact(s);
#pragma unroll
                            for (uint32_t q = 0; q < 16; q++) {
                                const uint32_t n = s[q];
                                if (!__ballot(n != 0u)) continue;
                                const uint32_t cls = n ? L.t4[motif_index4(ra, rb, rc, 0u, q >> 2, q & 3u)] : 0xFFu;
                                if (n) add_a(a, cls, n);
                                by_class_sum(cls, n, n != 0u, add_r);
                            }
                        }
                    }
                }
                for (;;) {   // adjacent pairs (a, b): a fixed, lanes over b
                    const uint32_t a = wave_task(&L.ctr[5]) * G + share;
                    if (a >= D) break;
                    const uint32_t nl = L.locn[a];
                    if (nl == 0u) continue;
                    const uint32_t base = locoff[a], ra = L.P[a] & 3u;
                    for (uint32_t i0 = 0; i0 < nl; i0 += 64) {
                        const bool on = i0 + lane < nl;
                        const uint32_t ent = on ? locnbr[base + i0 + lane] : 0u;
                        const uint32_t b = ent >> 2, ab = ent & 3u, rb = L.P[b] & 3u;
                        for (uint32_t rc = 1; rc < 4; rc++) {
                            const uint32_t clo = seg_at(rc), chi = seg_at(rc + 1);
                            if (clo >= chi) continue;
                            const uint32_t wlo = max(clo >> 5, w0), whi = min(((chi - 1u) >> 5) + 1u, w0 + wn);
                            uint32_t s[16] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
                            for (uint32_t w = wlo; w < whi; w++) {
                                uint32_t v = seg_word(rc, w);
                                if ((a >> 5) == w) v &= ~(1u << (a & 31u));
                                if (!on || (b >> 5) > w) v = 0u;
                                else if ((b >> 5) == w) v &= ~((2u << (b & 31u)) - 1u);
                                const uint2 aw = X[a * S1 + w - w0], bw = X[b * S1 + w - w0];
                                const uint32_t a0 = __builtin_amdgcn_readfirstlane(aw.x);
                                const uint32_t a1 = __builtin_amdgcn_readfirstlane(aw.y);
                                const uint32_t b0 = bw.x & v, b1 = bw.y & v, b01 = b0 & b1;
                                s[0] += __popc(v);
                                s[1] += __popc(b0);
                                s[2] += __popc(b1);
                                s[3] += __popc(b01);
                                if (a0 | a1) {
                                    const uint32_t a01 = a0 & a1;
                                    s[4] += __popc(a0 & v);
                                    s[5] += __popc(a0 & b0);
                                    s[6] += __popc(a0 & b1);
                                    s[7] += __popc(a0 & b01);
                                    s[8] += __popc(a1 & v);
                                    s[9] += __popc(a1 & b0);
                                    s[10] += __popc(a1 & b1);
                                    s[11] += __popc(a1 & b01);
                                    s[12] += __popc(a01 & v);
                                    s[13] += __popc(a01 & b0);
                                    s[14] += __popc(a01 & b1);
                                    s[15] += __popc(a01 & b01);
                                }
                            }
                            exact(s);
#pragma unroll
                            for (uint32_t q = 0; q < 16; q++) {
                                const uint32_t n = s[q];
                                if (!__ballot(n != 0u)) continue;
                                const uint32_t k0 = n ? L.t4[motif_index4(ra, rb, rc, 0u, q >> 2, q & 3u)] : 0xFFu;
                                const uint32_t k1 = n ? L.t4[motif_index4(ra, rb, rc, ab, q >> 2, q & 3u)] : 0xFFu;
                                by_class_sum(k0, n, n != 0u, [&](uint32_t k, uint32_t m) {
                                    add_a(a, k, 0u - m);
                                    add_r(k, 0u - m);
                                });
                                by_class_sum(k1, n, n != 0u, [&](uint32_t k, uint32_t m) {
                                    add_a(a, k, m);
                                    add_r(k, m);
                                });
                            }
                        }
                    }
                }
            }
            __syncthreads();
            if (inl)
                for (uint32_t i = tid; i < D * NSTAR; i += HT) {
                    const uint32_t x = R4[i];
                    if (x)
                        gadd(A.out4, A.perm, kClasses4, L.P[i / NSTAR] >> 2, A.star_cls[i % NSTAR],
                             (unsigned long long)(long long)(int32_t)x);
                }
        }
        __syncthreads();
        if (!LARGE || ngroups > 0u) {   // LARGE: no depth-2 vertex, no more sets
        // ---- phase D: per slot x, the other slots by their codes to r and to x (NX), and x's
        // (2,1,0) sets as the second slot y: below every other slot x' and its children, by
        // code, as if none were adjacent to y (the children that x and x' share are taken out
        // in phase E).
        const uint32_t nxw = (D * 5u + 1u) & ~1u;
        uint16_t* NX = (uint16_t*)L.U;               // D x 10: [9] slots by codes, children of code 3
        {
            uint32_t* SX = L.U + nxw;                // [9] children of the slots of a code, by code
            uint32_t* CW18 = SX + 16 + wid * 20;     // per wave: 9 counts, 9 sums
            if (tid < 16) SX[tid] = 0u;
            if (tid == 0) L.ctr[4] = 0u;
            __syncthreads();
            for (uint32_t x = tid; x < D; x += HT) {
                const uint32_t n1 = L.ch1[x], n2 = L.ch2[x], q = ((L.P[x] & 3u) - 1u) * 3u;
                const uint32_t n3 = locoff[x + 1] - locoff[x] - L.locn[x] - n1 - n2;
                NX[x * 10 + 9] = (uint16_t)n3;
                if (n1) atomicAdd(&SX[q], n1);
                if (n2) atomicAdd(&SX[q + 1], n2);
                if (n3) atomicAdd(&SX[q + 2], n3);
            }
            __syncthreads();
            auto children = [&](uint32_t x, uint32_t k) -> uint32_t {
                return k == 1u ? L.ch1[x] : (k == 2u ? L.ch2[x] : NX[x * 10 + 9]);
            };
            for (;;) {
                const uint32_t x = wave_task(&L.ctr[4]);
                if (x >= D) break;
                const bool own = x % G == share;
                const uint32_t rx = L.P[x] & 3u, base = locoff[x], nl = L.locn[x];
                auto add_x = [&](uint32_t cls, uint32_t n) { gadd(A.out4, A.perm, kClasses4, L.P[x] >> 2, cls, n); };
                uint32_t c9[9] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u}, l9[9] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
                for (uint32_t i0 = 0; i0 < nl; i0 += 64) {
                    const bool on = i0 + lane < nl;
                    const uint32_t ent = on ? locnbr[base + i0 + lane] : 0u;
                    const uint32_t y = ent >> 2, k = ent & 3u, ry = L.P[y] & 3u;
#pragma unroll
                    for (uint32_t q = 0; q < 9; q++)
                        c9[q] += (uint32_t)__popcll(__ballot(on && ry == q / 3u + 1u && k == q % 3u + 1u));
                    if (own)   // x as the second slot below its local neighbour y
#pragma unroll
                        for (uint32_t xc = 1; xc < 4; xc++) {
                            const uint32_t n = on ? children(y, xc) : 0u;
                            if (!__ballot(n != 0u)) continue;
                            const uint32_t cls = n ? L.t4[motif_index4(ry, rx, 0u, swap_arc_bits(k), xc, 0u)] : 0xFFu;
                            by_class_sum(cls, n, n != 0u, add_x);
#pragma unroll
                            for (uint32_t p = 0; p < 3; p++) l9[p * 3 + xc - 1u] += wave_sum(ry == p + 1u ? n : 0u);
                        }
                }
#pragma unroll
                for (uint32_t q = 0; q < 9; q++)
                    if (lane == q) {
                        NX[x * 10 + q] = (uint16_t)c9[q];
                        CW18[9 + q] = l9[q];
                    }
                __threadfence_block();
                if (own && lane < 9u) {   // parents of code p + 1 that are not adjacent to x, children of code xc
                    const uint32_t p = lane / 3u, xc = lane % 3u + 1u;
                    const uint32_t v = SX[lane] - (p + 1u == rx ? children(x, xc) : 0u) - CW18[9 + lane];
                    if (v) add_x(L.t4[motif_index4(p + 1u, rx, 0u, 0u, xc, 0u)], v);
                }
                __threadfence_block();
            }
        }
        __syncthreads();
        // ---- phase E: the sets below one slot a and one child c of a.  A wave takes a and marks
        // its children in a bitmap over the depth-2 vertices; 16 lanes take a child c:
        //   (2,1,0): a second slot of the group of its codes to r and a (NX), without the other
        //     parents x of c; a pair of parents once, from the lower slot (Lemma 3's rule);
        //   (1,2,0) and (1,1,1): c's row above r is walked, an e outside N(r) is another child
        //     of a (the pair with its arcs) or the end of the path r - a - c - e (the Lemma-4
        //     rule); the children of a that are not adjacent to c are a group by their code.
        // The sets are counted by arc codes.  c's credits leave as whole 64-byte lines of the
        // compact rows (a memory-side atomic costs the same for one counter as for a line of
        // them); a's and r's are summed in LDS.
        const uint32_t gl = lane & 15u;
        {
            constexpr uint32_t GW = E_GW, AW = E_AW, FW = FILTER_BITS / 32, FIX = E_FIX;
            // a's children as a bitmap a plane over the depth-2 vertices (their arc codes), where
            // LDS holds that for every wave beside the index; else as a filter over hashed ranks
            // in front of a search of a's row (hubs with very many depth-2 vertices, and those with
            // few, whose hash is not needed here then)
            const uint32_t jw = (ngroups + 31u) >> 5;
            const bool coded = !hashed && nxw + FIX + iw + 2u * NW * jw <= U_WORDS;
            const uint32_t mw = coded ? 2u * jw : FW;               // words per wave
            const bool in_lds = nxw + FIX + iw + NW * mw <= U_WORDS;
            uint32_t* GC = L.U + nxw + (tid >> 4) * GW;
            uint32_t* AC = L.U + nxw + (HT / 16) * GW + wid * AW;
            uint32_t* BX = L.U + nxw + (HT / 16) * GW + NW * AW + wid * CW;   // per wave: a's code row
            uint16_t* H2 = (uint16_t*)(L.U + nxw + (HT / 16) * GW + NW * AW + NW * CW);
            uint32_t* M0 = L.U + nxw + FIX + wid * mw;              // children with arc bit 0, or the filter
            uint32_t* M1 = M0 + jw;                                 // children with arc bit 1
            const Index2<LARGE> X2(in_lds, false, L.U + nxw + FIX + NW * mw, gidx, isz, cids);
            for (uint32_t i = nxw + tid; i < nxw + FIX; i += HT) L.U[i] = 0u;
            for (uint32_t i = lane; i < mw; i += 64) M0[i] = 0u;
            if (tid == 0) L.ctr[6] = 0u;
            __syncthreads();
            for (uint32_t i = tid; i < D; i += HT) slot_insert(H2, L.P[i] >> 2, i);
            if (!hashed && (!LARGE || in_lds || !kept)) X2.fill(ngroups);
            __syncthreads();
            auto add_r = [&](uint32_t cls, uint32_t n) {
                atomicAdd(&L.root4[cls], (unsigned long long)(long long)(int32_t)n);
            };
            auto add_a = [&](uint32_t cls, uint32_t n) { atomicAdd(&AC[cls], n); };
            for (;;) {
                const uint32_t a = wave_task(&L.ctr[6]) * G + share;
                if (a >= D) break;
                const uint32_t end = locoff[a + 1], nloc = L.locn[a], m = end - locoff[a] - nloc;
                if (m == 0u) continue;
                const uint32_t ra = L.P[a] & 3u;
                const uint32_t m1 = L.ch1[a], m2 = L.ch2[a], m3 = m - m1 - m2;
                if (nloc) build_row(BX, locnbr, locoff[a], nloc);
                if (lane < 6u) {   // (1,2,0) of a and r: pairs of children by code, as if not adjacent
                    const uint32_t k = lane < 3u ? 1u : (lane < 5u ? 2u : 3u);
                    const uint32_t l = lane < 3u ? lane + 1u : (lane < 5u ? lane - 1u : 3u);
                    const uint32_t nk = k == 1u ? m1 : (k == 2u ? m2 : m3), nl = l == 1u ? m1 : (l == 2u ? m2 : m3);
                    const uint32_t n = k == l ? nk * (nk - 1u) / 2u : nk * nl;
                    if (n) {
                        const uint32_t cls = L.t4[motif_index4(ra, 0u, 0u, k, l, 0u)];
                        add_a(cls, n);
                        add_r(cls, n);
                    }
                }
                if (lane == 0u) shp[4] += (unsigned long long)m * (m - 1u) / 2u;
                for (uint32_t i = lane; i < m; i += 64) {   // depth-2 entries of a's row: (j << 2) | code
                    const uint32_t ent = locnbr[end - 1u - i], j = ent >> 2;
                    if (coded) {
                        if (ent & 1u) atomicOr(&M0[j >> 5], 1u << (j & 31u));
                        if (ent & 2u) atomicOr(&M1[j >> 5], 1u << (j & 31u));
                    } else {
                        const uint32_t b = filter_bit(cids[j]);
                        atomicOr(&M0[b >> 5], 1u << (b & 31u));
                    }
                }
                __threadfence_block();
                // The loads of the next children are issued before this one's atomics: entry, then
                // vertex and parents, row, first 16 entries of it, each where the one before has
                // arrived (vector memory operations finish in order, so a load after an atomic
                // waits for it)
                const auto entry = [&](uint32_t i) { return i < m ? locnbr[end - 1u - i] : 0u; };
                uint32_t ent = entry(lane >> 4), ent1 = entry(4u + (lane >> 4));
                uint32_t c = cids[ent >> 2], f0 = poff[ent >> 2], f1 = poff[(ent >> 2) + 1u];
                uint32_t q0 = A.off[c] + gl, q1 = (lane >> 4) < m ? A.off[c + 1] : 0u;
                uint32_t x0 = q0 < q1 ? A.adj[q0] : 0u;
                for (uint32_t i0 = 0; i0 < m; i0 += 4u) {
                    const uint32_t i = i0 + (lane >> 4);
                    const bool on = i < m;
                    const uint32_t ac = ent & 3u, na = f1 - f0;
                    const uint32_t cn = cids[ent1 >> 2], f0n = poff[ent1 >> 2], f1n = poff[(ent1 >> 2) + 1u];
                    const uint32_t ent2 = entry(i + 8u);
                    if (on && na > 1u)   // the other parents of c by codes, those above a in the high half
                        for (uint32_t f = gl; f < na; f += 16u) {
                            const uint32_t pe = parents[f0 + f], x = pe >> 2;
                            if (x == a) continue;
                            const uint32_t ax = nloc ? code_at(BX, x) : 0u;
                            atomicAdd(&GC[57u + (((L.P[x] & 3u) - 1u) * 3u + (pe & 3u) - 1u) * 4u + ax],
                                      x > a ? 0x10001u : 1u);
                        }
                    const uint32_t q0n = A.off[cn] + gl, q1n = i + 4u < m ? A.off[cn + 1] : 0u;
                    uint32_t e12 = 0, e3 = 0;   // e's outside N(r) by arc code (1 | 2 << 16, 3)
                    for (uint32_t q = q0; q < q1; q += 16u) {
                        const uint32_t ee = q == q0 ? x0 : A.adj[q], e = ee >> 2, ce = ee & 3u;
                        if (e <= r || slot_find(H2, L.P, e) >= 0) continue;
                        if (ce == 3u) e3++;
                        else e12 += ce == 1u ? 1u : 1u << 16;
                        uint32_t ae = 0;   // e another child of a: its code
                        if (coded) {
                            const uint32_t j = X2.find_bit(e);
                            if (j == ~0u) continue;
                            ae = ((M0[j >> 5] >> (j & 31u)) & 1u) | (((M1[j >> 5] >> (j & 31u)) & 1u) << 1);
                        } else {
                            const uint32_t b = filter_bit(e);
                            if (!((M0[b >> 5] >> (b & 31u)) & 1u)) continue;
                            uint32_t lo = 0, hi = m;
                            if (!hashed) {   // a's row is in the order of the bitmap's numbers
                                const uint32_t j = X2.find_bit(e);
                                if (j == ~0u) continue;
                                while (lo + 1u < hi) {
                                    const uint32_t mid = (lo + hi) >> 1;
                                    if ((locnbr[end - 1u - mid] >> 2) <= j) lo = mid; else hi = mid;
                                }
                                const uint32_t x = locnbr[end - 1u - lo];
                                ae = (x >> 2) == j ? x & 3u : 0u;
                            } else {
                                while (lo + 1u < hi) {
                                    const uint32_t mid = (lo + hi) >> 1;
                                    if (cids[locnbr[end - 1u - mid] >> 2] <= e) lo = mid; else hi = mid;
                                }
                                const uint32_t x = locnbr[end - 1u - lo];
                                ae = cids[x >> 2] == e ? x & 3u : 0u;
                            }
                        }
                        if (ae) atomicAdd(&GC[48u + (ae - 1u) * 3u + ce - 1u], e > c ? 0x10001u : 1u);
                    }
                    const uint32_t x0n = q0n < q1n ? A.adj[q0n] : 0u;
                    e12 = row16_sum(e12);
                    e3 = row16_sum(e3);
                    __threadfence_block();
                    auto add_c = [&](uint32_t cls, uint32_t n) {
                        const uint32_t s = cmp_of[cls];
                        if (s < kCmpRow) atomicAdd(&GC[s], n);
                        else gadd(A.out4, A.perm, kClasses4, c, cls, (unsigned long long)(long long)(int32_t)n);
                    };
                    if (on && gl < 9u) {   // pairs of adjacent children: ae = gl / 3 + 1, ce = gl % 3 + 1
                        const uint32_t n = GC[48u + gl] & 0xFFFFu, nu = GC[48u + gl] >> 16;
                        const uint32_t ae = gl / 3u + 1u, ce = gl % 3u + 1u;
                        if (n) {
                            const uint32_t cls = L.t4[motif_index4(ra, 0u, 0u, ac, ae, ce)];
                            add_c(cls, n);
                            // c is no end of the paths r - a - e - c (phase G counts it as one)
                            add_c(L.t4[motif_index4(ra, 0u, 0u, ae, 0u, swap_arc_bits(ce))], 0u - n);
                            if (nu) {   // from the child of the lower rank: the pair, for a and r
                                const uint32_t st = L.t4[motif_index4(ra, 0u, 0u, ac, ae, 0u)];
                                add_a(cls, nu);
                                add_r(cls, nu);
                                add_a(st, 0u - nu);
                                add_r(st, 0u - nu);
                            }
                        }
                    } else if (on && gl < 12u) {   // (1,1,1): ends of code k
                        const uint32_t k = gl - 8u;
                        const uint32_t n = (k == 3u ? e3 : (k == 1u ? e12 & 0xFFFFu : e12 >> 16)) -
                                           (GC[47u + k] & 0xFFFFu) - (GC[50u + k] & 0xFFFFu) - (GC[53u + k] & 0xFFFFu);
                        if (n) {
                            const uint32_t cls = L.t4[motif_index4(ra, 0u, 0u, ac, 0u, k)];
                            add_c(cls, n);
                            add_a(cls, n);
                            add_r(cls, n);
                            shp[5] += (unsigned long long)(long long)(int32_t)n;
                        }
                    } else if (on && gl < 15u) {   // (1,2,0) with the children of code k not adjacent to c
                        const uint32_t k = gl - 11u, s = 45u + 3u * k;
                        const uint32_t n = (k == 1u ? m1 : (k == 2u ? m2 : m3)) - (k == ac ? 1u : 0u) -
                                           (GC[s] & 0xFFFFu) - (GC[s + 1u] & 0xFFFFu) - (GC[s + 2u] & 0xFFFFu);
                        if (n) add_c(L.t4[motif_index4(ra, 0u, 0u, ac, k, 0u)], n);
                    }
                    if (on && gl < 12u) {   // (2,1,0) under a: second slots by codes p + 1 to r and k to a
                        const uint32_t p = gl >> 2, k = gl & 3u;
                        uint32_t n;
                        if (k) n = NX[a * 10 + p * 3 + k - 1u];
                        else
                            n = seg_at(p + 2u) - seg_at(p + 1u) - (p + 1u == ra ? 1u : 0u) - NX[a * 10 + p * 3] -
                                NX[a * 10 + p * 3 + 1] - NX[a * 10 + p * 3 + 2];
                        if (na > 1u)
                            for (uint32_t xc = 0; xc < 3; xc++) n -= GC[57u + (p * 3u + xc) * 4u + k] & 0xFFFFu;
                        if (n) {
                            const uint32_t cls = L.t4[motif_index4(ra, p + 1u, 0u, k, ac, 0u)];
                            add_c(cls, n);
                            add_a(cls, n);
                            add_r(cls, n);
                            shp[3] += n;
                        }
                    }
                    if (on && na > 1u)
                        for (uint32_t q = gl; q < 36u; q += 16u) {   // pairs of parents (a, x)
                            const uint32_t w = GC[57u + q], n = w & 0xFFFFu, nu = w >> 16;
                            if (!n) continue;
                            const uint32_t rx = q / 12u + 1u, xc = q % 12u / 4u + 1u, ax = q & 3u;
                            const uint32_t cls = L.t4[motif_index4(ra, rx, 0u, ax, ac, xc)];
                            add_a(cls, n);
                            // a was counted as the second slot below x and c (phase D)
                            add_a(L.t4[motif_index4(rx, ra, 0u, swap_arc_bits(ax), xc, 0u)], 0u - n);
                            if (nu) {
                                add_c(cls, nu);
                                add_r(cls, nu);
                                shp[3] += nu;
                            }
                        }
                    __threadfence_block();
#pragma unroll
                    for (uint32_t ln = 0; ln < kCmpRow; ln += 16u) {   // c's counters, a line at a time
                        const uint32_t n = GC[ln + gl];
                        GC[ln + gl] = 0u;
                        cmp_line(A, c, ln + gl, n);
                    }
                    for (uint32_t q = 48u + gl; q < 93u; q += 16u) GC[q] = 0u;
                    __threadfence_block();
                    ent = ent1;
                    ent1 = ent2;
                    c = cn;
                    f0 = f0n;
                    f1 = f1n;
                    q0 = q0n;
                    q1 = q1n;
                    x0 = x0n;
                }
                if (coded) {
                    for (uint32_t i = lane; i < m; i += 64) {
                        const uint32_t j = locnbr[end - 1u - i] >> 2;
                        M0[j >> 5] = 0u;
                        M1[j >> 5] = 0u;
                    }
                } else {
                    for (uint32_t i = lane; i < FW; i += 64) M0[i] = 0u;
                }
                __threadfence_block();
                for (uint32_t k = lane; k < kClasses4; k += 64) {
                    const uint32_t n = AC[k];
                    AC[k] = 0u;
                    if (n) gadd(A.out4, A.perm, kClasses4, L.P[a] >> 2, k, (unsigned long long)(long long)(int32_t)n);
                }
                __threadfence_block();
            }
        }
        __syncthreads();
        // ---- phase G: the end vertices of the (1,1,1) paths, each once per root and window of
        // ranks: marked in a bitmap from the rows of the depth-2 vertices, then 16 lanes per
        // end e walk e's row: its depth-2 neighbours c and their parents (pcount, by codes) are
        // its paths, parents adjacent to e included (phase E took those out).  Credited path by
        // path instead, the ends alone would take a memory-side atomic per (1,1,1) set.  LARGE, roots
        // with few of them (kEndsDiv): from c's row, an atomic per e and code of c's parents.
        {
            constexpr uint32_t EB = G_EB, GW = 16 * EB, FIX = G_FIX;   // a group: 16 path counters per end vertex
            const bool in_lds = FIX + iw + G_WIN <= U_WORDS;
            uint32_t* GC = L.U + (tid >> 4) * GW;
            uint16_t* LST = (uint16_t*)(L.U + (HT / 16) * GW + wid * CW);   // per wave: 256 marked vertices
            uint16_t* H2 = (uint16_t*)(L.U + (HT / 16) * GW + NW * CW);
            uint32_t* KS = L.U + FIX - 32;   // path counter of the codes ((r -> a, a -> c) - 1) * 3 + (c -> e) - 1
            const Index2<LARGE> X2(in_lds, hashed, L.U + FIX, gidx, isz, cids);
            uint32_t* BM = L.U + FIX + (in_lds ? iw : 0u);
            const uint32_t win = min(nbw, U_WORDS - (uint32_t)(BM - L.U));   // words of a window
            for (uint32_t i = tid; i < FIX - 32; i += HT) L.U[i] = 0u;
            if (tid < 27u)
                KS[tid] = cmp_of[L.t4[motif_index4(tid / 9u + 1u, 0u, 0u, tid % 9u / 3u + 1u, 0u, tid % 3u + 1u)]];
            __syncthreads();
            for (uint32_t i = tid; i < D; i += HT) slot_insert(H2, L.P[i] >> 2, i);
            bool direct = false;
            if (LARGE) {
                unsigned long long sum = 0;
                if (tid == 0) L.ends = 0ull;
                if (tid < 2) L.ctr[6 + tid] = 0u;
                __syncthreads();
                for (uint32_t j = tid; j < ngroups; j += HT) {
                    const uint32_t c = cids[j];
                    if (c % G == share) sum += A.off[c + 1] - A.off[c];
                }
                if (sum) atomicAdd(&L.ends, sum);
                __syncthreads();
                direct = L.ends * kEndsDiv < (unsigned long long)A.off[A.n];
            }
            if (direct) {
                for (;;) {   // 16 lanes per depth-2 vertex c
                    const uint32_t t = wave_task(&L.ctr[6]);
                    if (t * 4u >= ngroups) break;
                    const uint32_t j = t * 4u + (lane >> 4);
                    const uint32_t c = j < ngroups ? cids[j] : 0u;
                    const bool own = j < ngroups && c % G == share;
                    const ulonglong2 pc = own ? pcount[j] : make_ulonglong2(0ull, 0ull);
                    const uint32_t q1 = own ? A.off[c + 1] : 0u;
                    for (uint32_t q = (own ? A.off[c] : 0u) + gl; q < q1; q += 16u) {
                        const uint32_t ee = A.adj[q], e = ee >> 2, ce = (ee & 3u) - 1u;
                        if (e <= r || slot_find(H2, L.P, e) >= 0) continue;
                        for (uint32_t mk = (uint32_t)(pc.y >> 48); mk; mk &= mk - 1u) {
                            const uint32_t s = (uint32_t)__ffs((int)mk) - 1u;
                            cmp_add(A, e, KS[s * 3u + ce], parents_of(pc, s));
                        }
                    }
                }
            } else {
            if (!LARGE || in_lds || !kept) X2.fill(ngroups);
            for (uint32_t w0 = (r + 1u) >> 5; w0 < nbw; w0 += win) {
                const uint32_t wn = min(win, nbw - w0), e0 = w0 << 5;
                __syncthreads();
                for (uint32_t i = tid; i < wn; i += HT) BM[i] = 0u;
                if (tid < 2) L.ctr[6 + tid] = 0u;
                __syncthreads();
                for (;;) {
                    const uint32_t t = wave_task(&L.ctr[6]);
                    if (t * 4u >= ngroups) break;
                    const uint32_t j = t * 4u + (lane >> 4);
                    const uint32_t c = j < ngroups ? cids[j] : 0u;
                    const bool own = j < ngroups && c % G == share;
                    const uint32_t q1 = own ? A.off[c + 1] : 0u;
                    for (uint32_t q = (own ? A.off[c] : 0u) + gl; q < q1; q += 16u) {
                        const uint32_t e = A.adj[q] >> 2, i = e - e0;
                        if (e > r && i < (wn << 5) && slot_find(H2, L.P, e) < 0) atomicOr(&BM[i >> 5], 1u << (i & 31u));
                    }
                }
                __syncthreads();
                for (;;) {   // 256 ranks a wave
                    const uint32_t b0 = wave_task(&L.ctr[7]) * 8u;
                    if (b0 >= wn) break;
                    uint32_t word = lane < 8u && b0 + lane < wn ? BM[b0 + lane] : 0u;
                    uint32_t pos = 0, total = 0;
                    for (uint32_t i = 0; i < 8; i++) {
                        const uint32_t m = (uint32_t)__popc((uint32_t)__builtin_amdgcn_readlane((int)word, (int)i));
                        pos += i < lane ? m : 0u;
                        total += m;
                    }
                    for (; word; word &= word - 1u)
                        LST[pos++] = (uint16_t)(lane * 32u + (uint32_t)__ffs((int)word) - 1u);
                    __threadfence_block();
                    // EB vertices a group, then their credits: vector memory operations finish in
                    // order, so a load after an atomic waits for the atomic
                    // (and the first loads of the next vertex come before this one's parents)
                    const uint32_t eg = e0 + (b0 << 5);
                    const auto end_at = [&](uint32_t i) { return eg + (i < total ? LST[i] : 0u); };
                    uint32_t q0 = A.off[end_at(lane >> 4)] + gl;
                    uint32_t q1 = (lane >> 4) < total ? A.off[end_at(lane >> 4) + 1u] : 0u;
                    uint32_t x0 = q0 < q1 ? A.adj[q0] : 0u;
                    for (uint32_t i0 = 0; i0 < total; i0 += 4u * EB) {
                        for (uint32_t eb = 0; eb < EB; eb++) {
                            const uint32_t in = i0 + (eb + 1u) * 4u + (lane >> 4), en = end_at(in);
                            const uint32_t q0n = A.off[en] + gl, q1n = in < total ? A.off[en + 1u] : 0u;
                            for (uint32_t q = q0; q < q1; q += 16u) {
                                const uint32_t ee = q == q0 ? x0 : A.adj[q], c = ee >> 2;
                                const uint32_t ce = swap_arc_bits(ee & 3u) - 1u;
                                if (c <= r || (G > 1u && c % G != share)) continue;
                                const uint32_t j = X2.find(c);
                                if (j == ~0u) continue;
                                const ulonglong2 pc = pcount[j];
                                for (uint32_t mk = (uint32_t)(pc.y >> 48); mk; mk &= mk - 1u) {
                                    const uint32_t s = (uint32_t)__ffs((int)mk) - 1u;
                                    atomicAdd(&GC[eb * 16u + KS[s * 3u + ce]], parents_of(pc, s));
                                }
                            }
                            q0 = q0n;
                            q1 = q1n;
                            x0 = q0 < q1 ? A.adj[q0] : 0u;
                        }
                        __threadfence_block();
#pragma unroll
                        for (uint32_t eb = 0; eb < EB; eb++) {
                            const uint32_t i = i0 + eb * 4u + (lane >> 4);
                            const uint32_t n = GC[eb * 16u + gl];
                            GC[eb * 16u + gl] = 0u;
                            cmp_line(A, e0 + (b0 << 5) + (i < total ? LST[i] : 0u), gl, n);
                        }
                        __threadfence_block();
                    }
                }
            }
            }
        }
        }
        __syncthreads();
        for (uint32_t i = tid; i < kClasses4; i += HT)
            if (L.root4[i]) gadd(A.out4, A.perm, kClasses4, r, i, L.root4[i]);
    }
    for (int s = 0; s < kShapes; s++) {
        unsigned long long x = shp[s];
        if (s == 2) x *= INV3;   // (3,0,0) sets were seen from each of their three slots
        for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
        if (lane == 0 && x) atomicAdd(&A.stats[s], x);
    }
}

// the compact rows of the hub path added to the output (48 lanes per vertex), atomically: two
// graphs' accumulated ranges may add to one output from two streams
__global__ __launch_bounds__(192) void k_expand(const void* cmp, int wide, int64_t n, const int32_t* __restrict__ perm,
                                                const uint8_t* __restrict__ cmp_cls, unsigned long long* out4) {
    const uint32_t s = threadIdx.x % kCmpRow, cls = cmp_cls[s];
    for (int64_t v = blockIdx.x * 4ll + threadIdx.x / kCmpRow; v < n; v += gridDim.x * 4ll) {
        const size_t at = (size_t)v * kCmpRow + s;
        const unsigned long long x = wide ? ((const unsigned long long*)cmp)[at] : ((const uint32_t*)cmp)[at];
        if (x) gadd64(&out4[(size_t)perm[v] * kClasses4 + cls], x);
    }
}

// ----------------------------------------------------------------------------- binning

constexpr int BT = 256;
constexpr double kShareWork3 = 1e6;   // in the unit of the hub queue's key

// every pair {u < v} into the edge hash, one thread per row (entries from split[u] on)
__global__ void k_edge_hash(const uint32_t* __restrict__ off, const uint32_t* __restrict__ split,
                            const uint32_t* __restrict__ adj, int64_t n, unsigned long long* table, uint32_t bits) {
    const uint32_t mask = (1u << bits) - 1u;
    for (int64_t u = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; u < n; u += (int64_t)gridDim.x * blockDim.x) {
        for (uint32_t t = split[u]; t < off[u + 1]; t++) {
            const uint32_t e = adj[t];
            const unsigned long long key = ((unsigned long long)u << 32) | ((unsigned long long)(e >> 2) << 2);
            for (uint32_t h = edge_slot(key, bits);; h = (h + 1u) & mask)
                if (atomicCAS(&table[h], 0ull, key | (e & 3u)) == 0ull) break;
        }
    }
}

// part of the ranks that holds rank r
__host__ __device__ inline uint32_t rank_part(uint32_t r, uint32_t n) {
    return (uint32_t)((unsigned long long)r * kRankParts / n);
}

// Per root, 16 lanes: the entries s2 of its slots' rows above it, its bin and sort key.  Hub
// roots come first, largest estimated work first, then the light tiers.  tot: [0] largest s2
// of a hub root, [1] largest |N+(r)| of all roots, [2..6] roots per bin (hubs, tiers 0..3); by_rank:
// s2 + 1 of the hub roots by kRankParts equal parts of the ranks, the sums, then the largest.
static_assert(kRankParts == 256, "a thread of k_root_work per part of the ranks");
__global__ __launch_bounds__(256) void k_root_work(const uint32_t* __restrict__ off, const uint32_t* __restrict__ adj,
                                                   const uint32_t* __restrict__ split,
                                                   const uint32_t* __restrict__ roots, int64_t nroots,
                                                   uint32_t hub_min, uint32_t hub_ok, uint32_t light_ok,
                                                   unsigned long long* __restrict__ wkey,
                                                   unsigned long long* __restrict__ tot,
                                                   unsigned long long* __restrict__ by_rank, uint32_t n) {
    __shared__ unsigned long long sh[8];
    __shared__ unsigned long long part[kRankParts], most[kRankParts];
    if (threadIdx.x < 8) sh[threadIdx.x] = 0ull;
    part[threadIdx.x] = most[threadIdx.x] = 0ull;
    __syncthreads();
    const uint32_t gl = threadIdx.x & 15u;
    for (int64_t i = blockIdx.x * 16ll + threadIdx.x / 16; i < nroots; i += gridDim.x * 16ll) {
        const uint32_t r = roots[i];
        const uint32_t s = split[r], e = off[r + 1], d = e - s;
        unsigned long long s2 = 0;
        for (uint32_t t = s + gl; t < e; t += 16u) {
            const uint32_t a = adj[t] >> 2;
            s2 += off[a + 1] - lower_bound_rank(adj, off[a], off[a + 1], r + 1);
        }
        for (int o = 8; o > 0; o >>= 1) s2 += __shfl_xor(s2, o, 64);
        if (gl != 0u) continue;
        int tier = light_ok ? light_tier(d, s2) : 3;
        // hub path: from hub_min higher neighbours on, and roots too large for the light kernel
        const bool hub = hub_ok && d <= DMAX && (d >= hub_min || (tier == 3 && d <= 32u));
        // work of a hub root, for the queue's order and for sharing: its triples of slots against its
        // entries (these weighed 50 and 500: R-MAT 2^15 24.9 and 23.6 ms, Chung-Lu 1e5 36.8 and 36.5, now
        // 24.8 and 36.6; the triples ten times as much: R-MAT 2^13 5.1 and 4.5 ms, Chung-Lu 1e5 38.8)
        const unsigned long long dd = d;
        wkey[i] = hub ? ~(dd * (dd - 1) * (dd - 2) / 100 + 150 * s2 + 4) : ~0ull - 3ull + (unsigned long long)tier;
        atomicMax(&sh[1], dd);
        if (hub) {
            atomicMax(&sh[0], s2);
            atomicAdd(&part[rank_part(r, n)], s2 + 1ull);
            atomicMax(&most[rank_part(r, n)], s2 + 1ull);
        }
        atomicAdd(&sh[hub ? 2 : 3 + tier], 1ull);
    }
    __syncthreads();
    if (part[threadIdx.x]) {
        atomicAdd(&by_rank[threadIdx.x], part[threadIdx.x]);
        atomicMax(&by_rank[kRankParts + threadIdx.x], most[threadIdx.x]);
    }
    if (threadIdx.x < 2) atomicMax(&tot[threadIdx.x], sh[threadIdx.x]);
    else if (threadIdx.x < 7 && sh[threadIdx.x]) atomicAdd(&tot[threadIdx.x], sh[threadIdx.x]);
}

__global__ void k_zero_u32(unsigned* p, int n) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0;
}

int g_num_cu = -1;

int hub_workgroups() {
    if (g_num_cu < 0) {
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess)
            g_num_cu = prop.multiProcessorCount;
        else
            g_num_cu = 256;
    }
    return g_num_cu;
}

}  // namespace

void free_hub_scratch(vdmc_graph_s* g) {
    if (!g->hub_scratch) return;
    wait_graph(g);
    (void)hipFree(g->hub_scratch);
    g->hub_scratch = nullptr;
}

void free_hub(vdmc_graph_s* g) {
    wait_graph(g);
    free_hub_scratch(g);
    (void)hipFree(g->hub_queue);   // and hubs
    g->light = g->hubs = nullptr;
    g->hub_queue = nullptr;
    g->hub_scratch_need = 0;
    g->nhub = g->nlight = 0;
    g->bins_hub_min = -1;
}

size_t hub_scratch_need(const vdmc_graph_s* g) { return g->nhub > 0 ? g->hub_scratch_need : 0; }

void ensure_hub_scratch(vdmc_graph_s* g) {
    if (g->nhub == 0 || g->hub_scratch) return;
    VDMC_HIP(hipMalloc(&g->hub_scratch, g->hub_scratch_need));
}

void ensure_edge_hash(vdmc_graph_s* g, hipStream_t st) {
    if (g->ehash) return;
    uint32_t eb = 10;   // load <= 1/4
    while (((size_t)1 << eb) < 4 * (size_t)std::max<int64_t>(g->pairs, 1)) eb++;
    const size_t eh_bytes = ((size_t)1 << eb) * sizeof(unsigned long long);
    struct Table {   // the graph's once it is filled
        unsigned long long* p = nullptr;
        ~Table() { (void)hipFree(p); }
    } t;
    VDMC_HIP(hipMalloc(&t.p, eh_bytes));
    VDMC_HIP(hipMemsetAsync(t.p, 0, eh_bytes, st));
    const unsigned blocks = (unsigned)std::min<int64_t>((g->n + BT - 1) / BT, 65536);
    if (blocks > 0)
        hipLaunchKernelGGL(k_edge_hash, dim3(blocks), dim3(BT), 0, st, g->off, g->split, g->adj, g->n, t.p, eb);
    VDMC_HIP(hipGetLastError());
    VDMC_HIP(hipStreamSynchronize(st));
    std::swap(g->ehash, t.p);
    g->ehash_bits = eb;
}

void ensure_bins(vdmc_graph_s* g, hipStream_t st) {
    const int hub_min = g->hub_min;
    if (g->bins_hub_min == hub_min) return;
    free_hub(g);   // waits for running work on the old bins
    HubPlan& hub = g->hub = HubPlan();
    const int64_t nr = g->nroots;
    DeviceTemps tmp((size_t)nr * 40 + (1u << 20));
    // The hub path needs every degree <= DMAX (slot arrays; parents of a depth-2 vertex counted in
    // 12 bits, pairs below a slot in 16; numbers of depth-2 vertices in 22) and ranks below 2^26 (its
    // bitmap of them, at most 16 MiB a workgroup)
    const uint32_t hub_ok = (g->max_deg <= (int32_t)DMAX && g->n < ((int64_t)1 << 26)) ? 1u : 0u;
    const uint32_t light_ok = g->max_deg < kLightMaxDegree ? 1u : 0u;
    unsigned long long* wkey = tmp.alloc<unsigned long long>(nr + 1);
    unsigned long long* wkey_s = tmp.alloc<unsigned long long>(nr + 1);
    unsigned long long* d_tot = tmp.alloc<unsigned long long>(8 + 2 * kRankParts);
    unsigned long long tot[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    int64_t nhub = 0;
    std::vector<unsigned long long> hub_keys;   // sorted work keys of the hub roots (~work)
    VDMC_HIP(hipMalloc(&g->hub_queue, 64 + (nr + 1) * sizeof(uint32_t)));   // the cursors, then the binned roots
    g->hubs = (uint32_t*)g->hub_queue + 16;
    if (nr > 0) {
        launch_fill_u64((uint64_t*)d_tot, 8 + 2 * kRankParts, 0, st);
        const unsigned blocks = (unsigned)std::min<int64_t>((nr + 15) / 16, 16384);
        hipLaunchKernelGGL(k_root_work, dim3(blocks), dim3(256), 0, st, g->off, g->adj, g->split, g->roots, nr,
                           (uint32_t)hub_min, hub_ok, light_ok, wkey, d_tot, d_tot + 8, (uint32_t)g->n);
        VDMC_HIP(hipGetLastError());
        // hub roots by work, then the tiers, each in rank order
        size_t sb = 0;
        int ni = (int)nr;
        VDMC_HIP(hipcub::DeviceRadixSort::SortPairs(nullptr, sb, wkey, wkey_s, g->roots, g->hubs, ni, 0, 64, st));
        void* t2 = tmp.alloc<uint8_t>(sb);
        VDMC_HIP(hipcub::DeviceRadixSort::SortPairs(t2, sb, wkey, wkey_s, g->roots, g->hubs, ni, 0, 64, st));
        VDMC_HIP(hipMemcpyAsync(tot, d_tot, sizeof(tot), hipMemcpyDeviceToHost, st));
        VDMC_HIP(hipStreamSynchronize(st));
        nhub = (int64_t)tot[2];
        if (nhub > 0) {
            hub_keys.resize((size_t)nhub);
            VDMC_HIP(hipMemcpyAsync(hub_keys.data(), wkey_s, nhub * sizeof(unsigned long long), hipMemcpyDeviceToHost,
                                    st));
            VDMC_HIP(hipMemcpyAsync(g->hub.parts, d_tot + 8, sizeof(g->hub.parts), hipMemcpyDeviceToHost, st));
            VDMC_HIP(hipStreamSynchronize(st));
        }
        // Hub roots whose estimated work exceeds a fair share of the device (the total over
        // twice the workgroups) would each be the critical path on one workgroup: the
        // leading ones of the queue (largest first) are shared by G workgroups, G from the
        // heaviest root's excess, at most 8.
        if (nhub > 0) {
            double total = 0.0;
            for (unsigned long long k : hub_keys) total += (double)(~k);
            const double fair = total / (2.0 * hub_workgroups());
            size_t h = 0;
            while (h < hub_keys.size() && h < 4096 && (double)(~hub_keys[h]) > fair) h++;
            const double top = (double)(~hub_keys[0]);
            const uint32_t shares = fair > 0.0 ? (uint32_t)std::min(8.0, std::ceil(top / fair)) : 1u;
            hub.split_roots = shares >= 2 ? (uint32_t)h : 0u;
            hub.shares = std::max(1u, shares);
            // k = 3 alone: staging is most of a root's work and sharing repeats it, so only roots
            // above kShareWork3 (some 400 slots) as well are shared.  R-MAT 2^12, three ranges:
            // 291 us, 347 with the line of k = 4, 364 without sharing.
            h = 0;
            while (h < hub_keys.size() && h < 4096 && (double)(~hub_keys[h]) > std::max(fair, kShareWork3)) h++;
            hub.split_roots3 = shares >= 2 ? (uint32_t)h : 0u;
        }
    }
    const unsigned long long max_s2 = tot[0];
    const int32_t maxhi = (int32_t)tot[1];
    g->nhub = nhub;
    g->light = g->hubs + nhub;
    g->nlight = nr - nhub;
    for (int t = 0; t < 4; t++) g->ntier[t] = (int64_t)tot[3 + t];
    // light roots: fewer than hub_min higher neighbours (every root when the hub path is off)
    g->light_max_d = hub_ok ? std::min<int32_t>(maxhi, hub_min - 1) : maxhi;
    if (nhub > 0) {
        const int wgs = hub_workgroups();
        const size_t s2cap = (size_t)max_s2 + 64;
        const size_t nbw = ((size_t)g->n + 31) / 32, base = (DMAX + 2) + 8 * s2cap + 4;
        // The index of the depth-2 vertices (see Index2): a bitmap for roots with nbw / 2 entries or more
        // (R-MAT 2^19 0.88 s, from nbw on 0.91), none if no root has nbw: bitmaps in scratch leave
        // workgroups out where nbw is large against the roots' rows (G(n, p) of 1e6 vertices of degree
        // 40, a bitmap from nbw / 16 on, 24 workgroups: 2.5 s, 0.71 without).
        const bool fits = bitmap_fits((size_t)maxhi, 2 * nbw);
        const bool large = !fits || g->n > kHubSmallN;
        const size_t hash_below = max_s2 < nbw ? (size_t)0xFFFFFFFFu : nbw / 2;
        const size_t most = std::min<size_t>(max_s2, hash_below);   // entries of a root with a hash
        size_t index = 0;                                           // scratch for it, where LDS may not hold it
        if (!fits && max_s2 >= nbw) index = 2 * nbw;
        if (large && !hash_fits((size_t)maxhi, Index2<true>::slots((uint32_t)most)))
            index = std::max<size_t>(index, Index2<true>::slots((uint32_t)most));
        const size_t wg_words = (base + index + 63) & ~(size_t)63;
        hub.large = large;
        hub.hash_below = (uint32_t)hash_below;
        hub.wg_words = wg_words;
        hub.s2cap = (uint32_t)s2cap;
        // Workgroups: one per compute unit, no more than there are roots and shares of roots.
        // Compact rows: a class of a vertex has at most 2 max_deg^3 paths or stars in a call, which
        // 32 bits hold up to degree 1290.  Together they stay within the scratch of one workgroup
        // per compute unit with its index in LDS; graphs whose rows would take more than half of that
        // go without.
        const size_t wg_bytes = wg_words * sizeof(uint32_t);
        const size_t room = ((base + 60 + 63) & ~(size_t)63) * sizeof(uint32_t) * (size_t)wgs;
        const double dm = (double)g->max_deg;
        const int wide = 2.0 * dm * dm * dm >= 4294967296.0 ? 1 : 0;
        const size_t rows = (((size_t)g->n * kCmpRow * (wide ? 8 : 4)) + 255) & ~(size_t)255;
        const bool use_rows = rows <= room / 2;
        const size_t parts = (size_t)nhub + (size_t)hub.split_roots * (hub.shares - 1u);
        size_t nwg = std::min<size_t>((size_t)wgs, parts);
        nwg = std::max<size_t>(1, std::min(nwg, (use_rows ? room - rows : room) / wg_bytes));
        hub.wgs = (uint32_t)nwg;
        hub.row_bytes = use_rows ? rows : 0;
        hub.row_wide = wide != 0;
        g->hub_scratch_need = hub.row_bytes + wg_bytes * nwg;
    }
    g->bins_hub_min = hub_min;
}

bool launch_hub(vdmc_graph_s* g, int k3, int k4, uint64_t* out3, uint64_t* out4, hipStream_t st,
                uint32_t rank_lo, uint32_t rank_hi, const hipEvent_t* around) {
    if (g->nhub == 0) return false;
    // s2 + 1 of the hub roots in the range, those of its first and last part by their share of its ranks
    double work = 0.0;
    unsigned long long most = 0;   // the largest of a root there
    const uint32_t n = (uint32_t)g->n;
    rank_hi = std::min(rank_hi, n);
    for (uint64_t lo = rank_lo, hi; lo < rank_hi; lo = hi) {
        const uint64_t p = rank_part((uint32_t)lo, n);
        const uint64_t p0 = (p * n + kRankParts - 1) / kRankParts, p1 = ((p + 1) * n + kRankParts - 1) / kRankParts;
        hi = std::min<uint64_t>(rank_hi, p1);
        work += (double)g->hub.parts[p] * (double)(hi - lo) / (double)(p1 - p0);
        most = std::max(most, g->hub.parts[kRankParts + p]);
    }
    if (work == 0.0) return false;
    ensure_hub_scratch(g);
    const ClassTables& t = class_tables();
    HubArgs a;
    a.off = g->off;
    a.adj = g->adj;
    a.split = g->split;
    a.perm = g->perm;
    a.hubs = g->hubs;
    a.nhub = (uint32_t)g->nhub;
    a.cursor = g->hub_queue;
    a.t3 = t.t3;
    a.t4 = t.t4;
    a.maps = t.maps4;
    a.star_cls = t.star_cls;
    a.cmp_cls = t.cmp_cls;
    a.out3 = (unsigned long long*)out3;
    a.out4 = (unsigned long long*)out4;
    a.stats = g->stats;
    a.k3 = k3;
    a.rank_lo = rank_lo;
    a.rank_hi = rank_hi;
    // the compact rows come first, then the workgroups' scratch
    a.n = n;
    a.hash_below = g->hub.hash_below;
    // rows are cleared and read for every vertex: not for a few small roots (Chung-Lu 1e6, 100 roots from
    // rank 10000 on, 0.4 n entries: 1.71 ms with rows, 1.65 without; 500 roots, 2 n entries: 3.79 and
    // 4.19; the root of rank 0 alone, 0.45 n entries: 515 and 532)
    const bool rows = 2.0 * work >= (double)n || 16ull * most >= n;
    a.cmp = k4 && g->hub.row_bytes && rows ? g->hub_scratch : nullptr;
    a.cmp_wide = g->hub.row_wide;
    a.scratch = (uint32_t*)((char*)g->hub_scratch + g->hub.row_bytes);
    a.wg_words = g->hub.wg_words;
    a.s2cap = g->hub.s2cap;
    const unsigned wgs = g->hub.wgs;
    // the heaviest hub roots, shared (set at binning)
    a.split_roots = k4 ? g->hub.split_roots : g->hub.split_roots3;
    a.shares = g->hub.shares;
    hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, st, g->hub_queue, 16);
    if (a.cmp) launch_fill_u64((uint64_t*)a.cmp, g->hub.row_bytes / 8, 0, st);
    // around[0] and around[1] bracket the hub path, around[2] marks the end of k_hub
    if (around) VDMC_HIP(hipEventRecord(around[0], st));
    if (!k4) hipLaunchKernelGGL((k_hub<false, false>), dim3(wgs), dim3(HT), 0, st, a);
    else if (g->hub.large) hipLaunchKernelGGL((k_hub<true, true>), dim3(wgs), dim3(HT), 0, st, a);
    else hipLaunchKernelGGL((k_hub<true, false>), dim3(wgs), dim3(HT), 0, st, a);
    VDMC_HIP(hipGetLastError());
    if (around) VDMC_HIP(hipEventRecord(around[2], st));
    if (a.cmp) {
        const unsigned blocks = (unsigned)std::min<int64_t>((g->n + 3) / 4, 65536);
        hipLaunchKernelGGL(k_expand, dim3(blocks), dim3(4 * kCmpRow), 0, st, a.cmp, a.cmp_wide, g->n, g->perm,
                           a.cmp_cls,
                           a.out4);
        VDMC_HIP(hipGetLastError());
    }
    if (around) VDMC_HIP(hipEventRecord(around[1], st));
    return true;
}

}  // namespace vdmc
