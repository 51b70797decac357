// Per-edge motif counts (Sec. 11: "count per edge" as a minimal change of the method:
// the edges of each set are credited instead of its vertices).
//
// Output rows are the vertex pairs {lo < hi} joined in G_U, in ascending (lo, hi) order
// of original ids (vdmc_edge_list).  The edge index maps every pair's slot in the
// graph's edge hash to its row, and every CSR entry to the row of its pair.
//
// k_edge_sets counts a root r's sets by its upper entries (r, a), a wave each, as small.hip
// does for vertices: by arc codes as if the members had only the arcs that the shape implies,
// and then each set that has another arc is corrected.  The pair (r, a) takes the part of
// the slot a there, (a, c) that of the child c, (c, e) that of the end vertex of a path; a
// further pair gets only the corrected sets.  The arcs of r and of a are in LDS, as bit planes or
// a hash (see Arcs), so that testing an entry of c's row costs two LDS reads.
// What bounds it: the memory-side atomics on the pairs (a, c) and (c, e) (2.4e10 a second);
// the pair (r, a) is summed in LDS.  Power-law graph of 3001 vertices, 20 k pairs, 25 M sets,
// k = 4: 0.55 ms a call, 16.1 with the per-set kernel (count.hip, EdgeSink), which remains for
// graphs of more vertices (kEdgeSetsMaxN: what the planes' LDS and the cells' 16 bits hold) and for
// k = 3 in graphs of small rows.
#include <hipcub/hipcub.hpp>

#include <algorithm>

#include "motif_device.h"
#include "vdmc_internal.h"

namespace vdmc {
namespace {

constexpr int ET = 256;
constexpr int64_t kPlanesN = 8192;   // up to here the planes leave room for the 16 waves that registers allow

unsigned blocks_of(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + ET - 1) / ET, 65536)); }

// entries above the diagonal (the pair's lower-rank row), per row
__global__ void k_upper_counts(const uint32_t* __restrict__ off, const uint32_t* __restrict__ split, int64_t n,
                               uint32_t* __restrict__ cnt) {
    for (int64_t u = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; u < n; u += (int64_t)gridDim.x * blockDim.x)
        cnt[u] = off[u + 1] - split[u];
}

// one key per pair: (lo << 32) | hi in original ids; value = its index in rank order
__global__ void k_pair_keys(const uint32_t* __restrict__ off, const uint32_t* __restrict__ split,
                            const uint32_t* __restrict__ adj, const int32_t* __restrict__ perm, int64_t n,
                            const uint32_t* __restrict__ uoff, unsigned long long* __restrict__ keys,
                            uint32_t* __restrict__ vals) {
    for (int64_t u = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; u < n; u += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t s = split[u], base = uoff[u];
        for (uint32_t t = s; t < off[u + 1]; t++) {
            const uint32_t a = (uint32_t)perm[u], b = (uint32_t)perm[adj[t] >> 2];
            const uint32_t i = base + (t - s);
            keys[i] = ((unsigned long long)min(a, b) << 32) | max(a, b);
            vals[i] = i;
        }
    }
}

__global__ void k_rows(const unsigned long long* __restrict__ keys_s, const uint32_t* __restrict__ vals_s,
                       int64_t P, uint32_t* __restrict__ row_of, int32_t* __restrict__ elo,
                       int32_t* __restrict__ ehi) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < P; i += (int64_t)gridDim.x * blockDim.x) {
        row_of[vals_s[i]] = (uint32_t)i;
        elo[i] = (int32_t)(keys_s[i] >> 32);
        ehi[i] = (int32_t)(keys_s[i] & 0xFFFFFFFFu);
    }
}

// every pair's edge-hash slot -> its output row
__global__ void k_slot_rows(const uint32_t* __restrict__ off, const uint32_t* __restrict__ split,
                            const uint32_t* __restrict__ adj, int64_t n, const uint32_t* __restrict__ uoff,
                            const uint32_t* __restrict__ row_of, const unsigned long long* __restrict__ table,
                            uint32_t bits, uint32_t* __restrict__ epid) {
    for (int64_t u = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; u < n; u += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t s = split[u], base = uoff[u];
        for (uint32_t t = s; t < off[u + 1]; t++) {
            const uint32_t h = edge_find(table, bits, (uint32_t)u, adj[t] >> 2);
            if (h != 0xFFFFFFFFu) epid[h] = row_of[base + (t - s)];
        }
    }
}

// every CSR entry -> the output row of its pair, every upper entry -> its root; a wave per row
__global__ __launch_bounds__(ET) void k_entry_rows(gptr<const uint32_t> off, gptr<const uint32_t> split,
                                                   gptr<const uint32_t> adj, int64_t n, gptr<const uint32_t> uoff,
                                                   gptr<const unsigned long long> table, uint32_t bits,
                                                   gptr<const uint32_t> epid, gptr<uint32_t> eid,
                                                   gptr<uint32_t> root_of) {
    const uint32_t lane = threadIdx.x & 63u;
    for (int64_t u = blockIdx.x * (int64_t)(ET / 64) + (threadIdx.x >> 6); u < n; u += (int64_t)gridDim.x * (ET / 64)) {
        const uint32_t s = split[u];
        for (uint32_t t = off[u] + lane; t < off[u + 1]; t += 64) {
            const uint32_t h = edge_find(table, bits, (uint32_t)u, adj[t] >> 2);
            eid[t] = h != 0xFFFFFFFFu ? epid[h] : 0u;
            if (t >= s) root_of[uoff[u] + (t - s)] = (uint32_t)u;
        }
    }
}

constexpr uint32_t kRootRow = 12;   // per root: children of its slots by both codes (9), its slots by code (3)

struct EdgeArgs {
    gptr<const uint32_t> off, adj, split;
    gptr<const uint32_t> eid;      // CSR entry -> output row
    gptr<const uint32_t> root_of;  // upper entry -> r
    gptr<const uint32_t> uoff;     // r -> its first upper entry
    gptr<uint32_t> kids;           // upper entry (r, a) -> children of a by code
    gptr<uint32_t> rows;           // r -> kRootRow
    gptr<const unsigned long long> table;
    gptr<const uint32_t> epid;
    uint32_t bits, words, n, pairs;
    const uint8_t* tab;            // code -> class
    gptr<unsigned long long> out;
    gptr<unsigned long long> stats;
};

__device__ __forceinline__ uint32_t esum8(uint32_t v) {
    v += (uint32_t)__shfl_xor((int)v, 1, 64);
    v += (uint32_t)__shfl_xor((int)v, 2, 64);
    v += (uint32_t)__shfl_xor((int)v, 4, 64);
    return v;
}

// children of a by code for every upper entry (r, a), 8 lanes each: entries of a's row above r
// that are not adjacent to r
__global__ __launch_bounds__(ET) void k_edge_kids(EdgeArgs A) {
    const uint32_t gl = threadIdx.x & 7u;
    const uint32_t step = gridDim.x * (ET / 8);
    for (uint32_t u0 = blockIdx.x * (ET / 8); u0 < A.pairs; u0 += step) {
        const uint32_t u = u0 + (threadIdx.x >> 3);
        const bool on = u < A.pairs;
        uint32_t h1 = 0, h2 = 0, h3 = 0;
        if (on) {
            const uint32_t r = A.root_of[u], a = A.adj[A.split[r] + (u - A.uoff[r])] >> 2, alo = A.off[a];
            for (uint32_t q = A.off[a + 1]; q > alo; q -= min(8u, q - alo)) {
                const uint32_t x = q - alo > gl ? A.adj[q - 1u - gl] : 0u, c = x >> 2, k = x & 3u;
                if (c > r && edge_find(A.table, A.bits, r, c) == 0xFFFFFFFFu) {
                    h1 += k == 1u;
                    h2 += k == 2u;
                    h3 += k == 3u;
                }
                if (q - alo > 8u && (A.adj[q - 8u] >> 2) <= r) break;
            }
        }
        h1 = esum8(h1);
        h2 = esum8(h2);
        h3 = esum8(h3);
        if (on && gl < 3u) A.kids[(size_t)3 * u + gl] = gl == 0u ? h1 : (gl == 1u ? h2 : h3);
    }
}

// per root, a wave: children of all slots by both codes, slots by code; the visits of the shapes
// that these fix
template <bool K4>
__global__ __launch_bounds__(ET) void k_edge_roots(EdgeArgs A) {
    const uint32_t lane = threadIdx.x & 63u;
    unsigned long long v0 = 0, v1 = 0;
    for (uint32_t r = blockIdx.x * (ET / 64) + (threadIdx.x >> 6); r < A.n; r += gridDim.x * (ET / 64)) {
        const uint32_t lo = A.split[r], d = A.off[r + 1] - lo, u = A.uoff[r];
        if (d == 0u) continue;
        uint32_t t[kRootRow] = {0};
        for (uint32_t i = lane; i < d; i += 64) {
            const uint32_t x = A.adj[lo + i] & 3u;
            for (uint32_t c = 1; c < 4; c++)
                for (uint32_t k = 0; k < 3; k++) t[(c - 1) * 3 + k] += x == c ? A.kids[(size_t)3 * (u + i) + k] : 0u;
            for (uint32_t c = 1; c < 4; c++) t[8 + c] += x == c;
        }
        uint32_t all = 0;
        for (uint32_t k = 0; k < kRootRow; k++) {
            for (int o = 1; o < 64; o <<= 1) t[k] += (uint32_t)__shfl_xor((int)t[k], o, 64);
            if (k < 9) all += t[k];
            if (lane == 0) A.rows[(size_t)r * kRootRow + k] = t[k];
        }
        const unsigned long long dd = d;
        v0 += K4 ? (dd * (dd - 1) / 2 * (dd - 2)) / 3 : dd * (dd - 1) / 2;
        v1 += K4 ? all * (dd - 1) : (unsigned long long)all;
    }
    if (lane == 0 && v0) gadd64(&A.stats[K4 ? 2 : 0], v0);
    if (lane == 0 && v1) gadd64(&A.stats[K4 ? 3 : 1], v1);
}

__device__ __forceinline__ uint32_t epick(uint32_t k, const uint32_t (&v)[3]) {
    return k == 1u ? v[0] : (k == 2u ? v[1] : v[2]);
}
__device__ __forceinline__ unsigned long long epairs(uint32_t k, uint32_t l, const uint32_t (&v)[3]) {
    const unsigned long long x = epick(k, v);
    return k == l ? x * (x - 1u) / 2u : x * epick(l, v);
}
__device__ __forceinline__ void epair(uint32_t i, uint32_t& k, uint32_t& l) {
    k = i < 3u ? 1u : (i < 5u ? 2u : 3u);
    l = i < 3u ? i + 1u : (i < 5u ? i - 1u : 3u);
}
// The arcs of a pair's member to other vertices: two bit planes of n bits, or, HASH, cells of the
// entries (epoch of the pair << 18 | vertex << 2 | code; a cell of another epoch is empty).  Planes are
// one read a test, but at n = 65536 they leave a CU one workgroup, which is too few for rows of some
// entries: G(n, p) of degree 2, k = 4, 769 us with planes, 664 with the hash; of degree 6 2007 and 1447;
// Chung-Lu 3e4 16.1 and 15.3 ms.  (Epochs: a wave takes a pair in 8192 x 4, and rows that the hash
// takes have fewer than 3072 entries, so at most 3073 of 16384.)
template <bool HASH>
struct Arcs {
    uint2* planes;
    uint32_t* cells;
    uint32_t mask, epoch;
    __device__ __forceinline__ uint32_t bits(uint32_t v) const {
        if (HASH) {
            for (uint32_t h = v * 2654435761u >> 15;; h++) {
                const uint32_t x = cells[h & mask];
                if ((x >> 18) != epoch) return 0u;
                if (((x >> 2) & 0xFFFFu) == v) return x & 3u;
            }
        }
        const uint2 w = planes[v >> 5];
        return ((w.x >> (v & 31u)) & 1u) | (((w.y >> (v & 31u)) & 1u) << 1);
    }
    __device__ __forceinline__ void set(uint32_t ent) const {
        const uint32_t v = ent >> 2;
        if (HASH) {
            for (uint32_t h = v * 2654435761u >> 15;; h++) {
                uint32_t x = cells[h & mask];
                while ((x >> 18) != epoch) {
                    const uint32_t got = atomicCAS(&cells[h & mask], x, (epoch << 18) | ent);
                    if (got == x) return;
                    x = got;
                }
            }
        }
        const uint32_t bit = 1u << (v & 31u);
        if (ent & 1u) atomicOr(&planes[v >> 5].x, bit);
        if (ent & 2u) atomicOr(&planes[v >> 5].y, bit);
    }
};
// A wave per upper entry (r, a), from the roots of the largest degrees on.
template <bool K4, bool HASH>
__global__ __launch_bounds__(ET) void k_edge_sets(EdgeArgs A) {
    constexpr uint32_t C = K4 ? (uint32_t)kClasses4 : (uint32_t)kClasses3;
    constexpr uint32_t NWV = ET / 64;
    constexpr unsigned long long kLess = ~0ull;   // one set less
    extern __shared__ uint2 dyn[];
    __shared__ unsigned long long rows[NWV][K4 ? 3 : 1][C];   // classes of (r, a); of a triangle's (r, b), (a, b)
    __shared__ uint8_t tab[K4 ? 4096 : 64];
    const uint32_t tid = threadIdx.x, wid = tid >> 6, lane = tid & 63u, gl = tid & 7u;
    // per wave: arcs of r to its slots; k = 4: arcs of a to the vertices above r
    constexpr uint32_t NT = K4 ? 2u : 1u;
    uint2* const my = dyn + wid * NT * A.words;
    Arcs<HASH> PR{my, (uint32_t*)my, 2u * A.words - 1u, 0u}, PA{my + A.words, (uint32_t*)(my + A.words), 2u * A.words - 1u, 0u};
    unsigned long long(&RA)[C] = rows[wid][0];
    for (uint32_t i = tid; i < (K4 ? 4096u : 64u); i += ET) tab[i] = A.tab[i];
    // the planes are zero between two pairs: cleared here, then where a pair has set them
    for (uint32_t i = lane; i < NT * A.words; i += 64) my[i] = make_uint2(0u, 0u);
    for (uint32_t i = lane; i < C * (K4 ? 3u : 1u); i += 64) RA[i] = 0ull;
    __syncthreads();
    auto add = [&](uint32_t row, uint32_t cls, unsigned long long n) { gadd64(&A.out[(size_t)row * C + cls], n); };
    auto move = [&](uint32_t row, uint32_t was, uint32_t is) {
        add(row, was, kLess);
        add(row, is, 1ull);
    };
    auto lmove = [&](unsigned long long* row, uint32_t was, uint32_t is) {
        atomicAdd(&row[was], kLess);
        atomicAdd(&row[is], 1ull);
    };
    auto row_of = [&](uint32_t x, uint32_t y) { return A.epid[edge_find(A.table, A.bits, x, y)]; };
    auto idx4 = [&](uint32_t p01, uint32_t p02, uint32_t p03, uint32_t p12, uint32_t p13, uint32_t p23) -> uint32_t {
        return tab[motif_index4(p01, p02, p03, p12, p13, p23)];
    };
    unsigned long long v1 = 0, v2 = 0, v3 = 0;   // (2,1,0) less, (1,2,0), (1,1,1)
    for (uint32_t u = blockIdx.x * NWV + wid; u < A.pairs; u += gridDim.x * NWV) {
        const uint32_t r = A.root_of[u], lo = A.split[r], rend = A.off[r + 1], t = lo + (u - A.uoff[r]);
        const uint32_t ent = A.adj[t], a = ent >> 2, ra = ent & 3u, alo = A.off[a], aend = A.off[a + 1];
        if (HASH) PA.epoch = ++PR.epoch;
        wave_fence();
        for (uint32_t i = lo + lane; i < rend; i += 64) PR.set(A.adj[i]);
        uint32_t abeg = aend;   // a's first entry above r
        for (bool more = true; more && abeg > alo;) {
            const uint32_t x = lane < abeg - alo ? A.adj[abeg - 1u - lane] : 0u;
            const bool in = (x >> 2) > r;
            if (K4 && in) PA.set(x);
            const uint32_t cnt = (uint32_t)__popcll(__ballot(in));
            abeg -= cnt;
            more = cnt == 64u;
        }
        wave_fence();
        // ---- (r, a): sets by code
        const gptr<const uint32_t> T = &A.rows[(size_t)r * kRootRow];
        const uint32_t h[3] = {A.kids[(size_t)3 * u], A.kids[(size_t)3 * u + 1u], A.kids[(size_t)3 * u + 2u]};
        const uint32_t o[3] = {T[9] - (ra == 1u), T[10] - (ra == 2u), T[11] - (ra == 3u)};
        if (lane < (K4 ? 30u : 6u)) {
            unsigned long long n;
            uint32_t cls, k, l;
            if (!K4) {
                k = lane % 3u + 1u;
                n = lane < 3u ? epick(k, o) : epick(k, h);
                cls = tab[lane < 3u ? motif_index3(ra, k, 0u) : motif_index3(ra, 0u, k)];
            } else if (lane < 9u) {    // (2,1,0), a the parent
                k = lane / 3u + 1u;
                l = lane % 3u + 1u;
                n = (unsigned long long)epick(k, h) * epick(l, o);
                cls = idx4(ra, l, 0u, 0u, k, 0u);
            } else if (lane < 15u) {   // (3,0,0)
                epair(lane - 9u, k, l);
                n = epairs(k, l, o);
                cls = idx4(ra, k, l, 0u, 0u, 0u);
            } else if (lane < 21u) {   // (1,2,0)
                epair(lane - 15u, k, l);
                n = epairs(k, l, h);
                cls = idx4(ra, 0u, 0u, k, l, 0u);
            } else {                   // (2,1,0), a the second slot
                k = (lane - 21u) / 3u + 1u;
                l = (lane - 21u) % 3u + 1u;
                n = T[lane - 21u] - (k == ra ? epick(l, h) : 0u);
                cls = idx4(k, ra, 0u, 0u, l, 0u);
            }
            if (n) atomicAdd(&RA[cls], n);
        }
        if (K4 && lane == 0) {
            const unsigned long long x = (unsigned long long)h[0] + h[1] + h[2];
            v2 += x * (x - 1u) / 2u;
        }
        // ---- a's row above r: children c, 8 lanes each; for k = 3 a lane per entry
        if (!K4) {
            for (uint32_t i = abeg + lane; i < aend; i += 64) {
                const uint32_t x = A.adj[i], c = x >> 2, ac = x & 3u, rc = PR.bits(c);
                if (!rc) {
                    add(A.eid[i], tab[motif_index3(ra, 0u, ac)], 1ull);
                } else if (c > a) {
                    const uint32_t was = tab[motif_index3(ra, rc, 0u)], is = tab[motif_index3(ra, rc, ac)];
                    lmove(RA, was, is);
                    move(row_of(r, c), was, is);
                    add(A.eid[i], is, 1ull);
                }
            }
        } else {
            for (uint32_t i0 = abeg; i0 < aend; i0 += 8) {
                const uint32_t i = i0 + (lane >> 3);
                const uint32_t x = i < aend ? A.adj[i] : 0u, c = x >> 2, ac = x & 3u;
                const bool on = i < aend && !PR.bits(c);
                const uint32_t eac = on ? A.eid[i] : 0u, clo = on ? A.off[c] : 0u;
                uint32_t e1 = 0, e2 = 0, e3 = 0;   // paths by their last arc
                for (uint32_t q = on ? A.off[c + 1] : 0u; q > clo; q -= min(8u, q - clo)) {
                    const bool in = gl < q - clo;
                    const uint32_t y = in ? A.adj[q - 1u - gl] : 0u, ece = in ? A.eid[q - 1u - gl] : 0u;
                    const uint32_t e = y >> 2, ce = y & 3u;
                    if (e > r && e != a) {
                        const uint32_t re = PR.bits(e), ae = PA.bits(e);
                        if (re) {          // (2,1,0) with the second slot e: from the lower parent of c
                            const uint32_t was = idx4(ra, re, 0u, 0u, ac, 0u), ere = row_of(r, e);
                            atomicAdd(&RA[was], kLess);
                            add(ere, was, kLess);
                            add(eac, was, kLess);
                            if (a < e) {
                                const uint32_t is = idx4(ra, re, 0u, ae, ac, swap_arc_bits(ce));
                                atomicAdd(&RA[is], 1ull);
                                add(ere, is, 1ull);
                                add(eac, is, 1ull);
                                add(ece, is, 1ull);
                                if (ae) add(row_of(a, e), is, 1ull);
                            } else {
                                v1--;
                            }
                        } else if (ae) {   // (1,2,0) with the other child e
                            const uint32_t was = idx4(ra, 0u, 0u, ac, ae, 0u), is = idx4(ra, 0u, 0u, ac, ae, ce);
                            move(eac, was, is);
                            if (c < e) {
                                lmove(RA, was, is);
                                add(ece, is, 1ull);
                            }
                        } else {           // path
                            add(ece, idx4(ra, 0u, 0u, ac, 0u, ce), 1ull);
                            e1 += ce == 1u;
                            e2 += ce == 2u;
                            e3 += ce == 3u;
                        }
                    }
                    if (q - clo > 8u && (A.adj[q - 8u] >> 2) <= r) break;
                }
                const uint32_t ne[3] = {esum8(e1), esum8(e2), esum8(e3)};
                if (!on) continue;
                // (a, c): 3 classes each of (2,1,0), (1,2,0) and (1,1,1)
                for (uint32_t j = gl; j < 9u; j += 8u) {
                    const uint32_t k = j % 3u + 1u;
                    const uint32_t n = j < 3u ? epick(k, o) : (j < 6u ? epick(k, h) - (k == ac) : epick(k, ne));
                    const uint32_t cls = j < 3u ? idx4(ra, k, 0u, 0u, ac, 0u)
                                                : (j < 6u ? idx4(ra, 0u, 0u, ac, k, 0u) : idx4(ra, 0u, 0u, ac, 0u, k));
                    if (n) {
                        add(eac, cls, n);
                        if (j >= 6u) {
                            atomicAdd(&RA[cls], (unsigned long long)n);
                            v3 += n;
                        }
                    }
                }
            }
            // ---- triangles (r, a, b), a < b: triples of slots from the first of their adjacent pairs,
            // and children of one of a, b that are not adjacent to the other
            unsigned long long* RB = rows[wid][K4 ? 1 : 0];
            unsigned long long* AB = rows[wid][K4 ? 2 : 0];
            for (uint32_t i0 = abeg; i0 < aend; i0 += 64) {
                const uint32_t x = i0 + lane < aend ? A.adj[i0 + lane] : 0u;
                unsigned long long todo = __ballot((x >> 2) > a && PR.bits(x >> 2));
                for (; todo; todo &= todo - 1ull) {
                    const int src = __ffsll((long long)todo) - 1;
                    const uint32_t y = (uint32_t)__shfl((int)x, src, 64), b = y >> 2, ab = y & 3u;
                    const uint32_t rb = PR.bits(b);
                    wave_fence();
                    for (uint32_t j = lo + lane; j < rend; j += 64) {
                        const uint32_t z = A.adj[j], c = z >> 2, rc = z & 3u;
                        if (c == a || c == b) continue;
                        const uint32_t xa = PA.bits(c);
                        if (xa && c < b) continue;
                        const uint32_t xb = edge_code(A.table, A.bits, b, c);
                        if (xb && c < a) continue;
                        const uint32_t was = idx4(ra, rb, rc, 0u, 0u, 0u), is = idx4(ra, rb, rc, ab, xa, xb);
                        lmove(RA, was, is);
                        lmove(RB, was, is);
                        move(A.eid[j], was, is);
                        atomicAdd(&AB[is], 1ull);
                        if (xa) add(row_of(a, c), is, 1ull);
                        if (xb) add(row_of(b, c), is, 1ull);
                    }
                    for (uint32_t j = abeg + lane; j < aend; j += 64) {
                        const uint32_t z = A.adj[j], c = z >> 2, ac = z & 3u;
                        if (PR.bits(c) || edge_code(A.table, A.bits, b, c)) continue;
                        const uint32_t was = idx4(ra, rb, 0u, 0u, ac, 0u), is = idx4(ra, rb, 0u, ab, ac, 0u);
                        lmove(RA, was, is);
                        lmove(RB, was, is);
                        move(A.eid[j], was, is);
                        atomicAdd(&AB[is], 1ull);
                    }
                    const uint32_t blo = A.off[b];
                    for (uint32_t j = A.off[b + 1]; j > blo; j -= min(64u, j - blo)) {
                        const uint32_t z = j - blo > lane ? A.adj[j - 1u - lane] : 0u, c = z >> 2, bc = z & 3u;
                        if (c > r && !PR.bits(c) && !PA.bits(c)) {
                            const uint32_t was = idx4(rb, ra, 0u, 0u, bc, 0u);
                            const uint32_t is = idx4(rb, ra, 0u, swap_arc_bits(ab), bc, 0u);
                            lmove(RA, was, is);
                            lmove(RB, was, is);
                            move(A.eid[j - 1u - lane], was, is);
                            atomicAdd(&AB[is], 1ull);
                        }
                        if (j - blo > 64u && (A.adj[j - 64u] >> 2) <= r) break;
                    }
                    wave_fence();
                    const uint32_t erb = row_of(r, b), eab = A.eid[i0 + (uint32_t)src];
                    for (uint32_t k = lane; k < C; k += 64) {
                        if (RB[k]) add(erb, k, RB[k]);
                        if (AB[k]) add(eab, k, AB[k]);
                        RB[k] = AB[k] = 0ull;
                    }
                    wave_fence();
                }
            }
        }
        wave_fence();
        const uint32_t era = A.eid[t];
        for (uint32_t k = lane; k < C; k += 64) {
            if (!RA[k]) continue;
            add(era, k, RA[k]);
            RA[k] = 0ull;
        }
        if (!HASH) {
            for (uint32_t i = lo + lane; i < rend; i += 64) PR.planes[A.adj[i] >> 7] = make_uint2(0u, 0u);
            if (K4)
                for (uint32_t i = abeg + lane; i < aend; i += 64) PA.planes[A.adj[i] >> 7] = make_uint2(0u, 0u);
        }
        wave_fence();
    }
    if (!K4) return;
    for (int o = 1; o < 64; o <<= 1) {
        v1 += __shfl_xor(v1, o, 64);
        v2 += __shfl_xor(v2, o, 64);
        v3 += __shfl_xor(v3, o, 64);
    }
    if (lane < 3u) {
        const unsigned long long n = lane == 0u ? v1 : (lane == 1u ? v2 : v3);
        if (n) gadd64(&A.stats[3u + lane], n);
    }
}

}  // namespace

// The index is the graph's only once it is complete: a failure on the way leaves the graph
// without one, and the next call builds it.
void ensure_edge_index(vdmc_graph_s* g, hipStream_t st) {
    if (g->epid) return;
    ensure_edge_hash(g, st);
    const int64_t n = g->n, P = g->pairs;
    struct Owner {
        std::vector<void*> v;
        void* alloc(size_t bytes) {
            void* p = nullptr;
            VDMC_HIP(hipMalloc(&p, bytes ? bytes : 16));
            v.push_back(p);
            return p;
        }
        ~Owner() {
            for (void* p : v) (void)hipFree(p);
        }
    } tmp, kept;
    auto* epid = (uint32_t*)kept.alloc(((size_t)1 << g->ehash_bits) * sizeof(uint32_t));
    auto* elo = (int32_t*)kept.alloc(P * sizeof(int32_t));
    auto* ehi = (int32_t*)kept.alloc(P * sizeof(int32_t));
    uint32_t* work = nullptr;
    if (n > 0 && P > 0) {
        uint32_t* cnt = (uint32_t*)tmp.alloc((n + 1) * sizeof(uint32_t));
        uint32_t* uoff = (uint32_t*)tmp.alloc((n + 1) * sizeof(uint32_t));
        auto* keys = (unsigned long long*)tmp.alloc(P * sizeof(unsigned long long));
        auto* keys_s = (unsigned long long*)tmp.alloc(P * sizeof(unsigned long long));
        uint32_t* vals = (uint32_t*)tmp.alloc(P * sizeof(uint32_t));
        uint32_t* vals_s = (uint32_t*)tmp.alloc(P * sizeof(uint32_t));
        uint32_t* row_of = (uint32_t*)tmp.alloc(P * sizeof(uint32_t));
        size_t tb = 0, sb = 0;
        VDMC_HIP(hipcub::DeviceScan::ExclusiveSum(nullptr, tb, cnt, uoff, (int)n, st));
        VDMC_HIP(hipcub::DeviceRadixSort::SortPairs(nullptr, sb, keys, keys_s, vals, vals_s, (int)P, 0, 64, st));
        void* t1 = tmp.alloc(std::max(tb, sb));   // the sort follows the scan on the stream
        // CSR entry -> row, upper entry -> root, and the scratch of k_edge_sets, where there is memory
        // beside what the index needs (the per-set kernel does without)
        const size_t words = (size_t)6 * P + (1 + kRootRow) * (n + 1);
        if (n <= kEdgeSetsMaxN) {
            if (hipMalloc(&work, words * sizeof(uint32_t)) == hipSuccess) {
                kept.v.push_back(work);
            } else {
                (void)hipGetLastError();
                work = nullptr;
            }
        }
        hipLaunchKernelGGL(k_upper_counts, dim3(blocks_of(n)), dim3(ET), 0, st, g->off, g->split, n, cnt);
        VDMC_HIP(hipcub::DeviceScan::ExclusiveSum(t1, tb, cnt, uoff, (int)n, st));
        hipLaunchKernelGGL(k_pair_keys, dim3(blocks_of(n)), dim3(ET), 0, st, g->off, g->split, g->adj, g->perm, n,
                           uoff, keys, vals);
        VDMC_HIP(hipcub::DeviceRadixSort::SortPairs(t1, sb, keys, keys_s, vals, vals_s, (int)P, 0, 64, st));
        hipLaunchKernelGGL(k_rows, dim3(blocks_of(P)), dim3(ET), 0, st, keys_s, vals_s, P, row_of, elo, ehi);
        hipLaunchKernelGGL(k_slot_rows, dim3(blocks_of(n)), dim3(ET), 0, st, g->off, g->split, g->adj, n, uoff, row_of,
                           g->ehash, g->ehash_bits, epid);
        if (work) {
            VDMC_HIP(hipMemcpyAsync(work + 6 * P, uoff, n * sizeof(uint32_t), hipMemcpyDeviceToDevice, st));
            hipLaunchKernelGGL(k_entry_rows, dim3(blocks_of(n * 64)), dim3(ET), 0, st, g->off, g->split, g->adj, n, uoff,
                               g->ehash, g->ehash_bits, epid, work, work + 2 * P);
        }
        VDMC_HIP(hipGetLastError());
        VDMC_HIP(hipStreamSynchronize(st));
    }
    kept.v.clear();   // the graph's from here on
    g->epid = epid;
    g->elo = elo;
    g->ehi = ehi;
    g->ework = work;
}

void launch_edge_sets(vdmc_graph_s* g, int k, uint64_t* out, hipStream_t st) {
    const ClassTables& t = class_tables();
    const int64_t n = g->n, P = g->pairs;
    EdgeArgs a;
    a.off = g->off;
    a.adj = g->adj;
    a.split = g->split;
    a.eid = g->ework;
    a.root_of = g->ework + 2 * P;
    a.kids = g->ework + 3 * P;
    a.uoff = g->ework + 6 * P;
    a.rows = g->ework + 6 * P + n + 1;
    a.table = g->ehash;
    a.epid = g->epid;
    a.bits = g->ehash_bits;
    a.words = (uint32_t)((n + 31) / 32);
    a.n = (uint32_t)n;
    a.pairs = (uint32_t)P;
    a.tab = k == 3 ? t.t3 : t.t4;
    a.out = (unsigned long long*)out;
    a.stats = g->stats;
    // cells for the longest row, three quarters full at most: two in the place of a plane's two words
    uint32_t pairs_of_cells = 32;
    while (3 * pairs_of_cells < 2 * (uint32_t)g->max_deg) pairs_of_cells <<= 1;
    const bool hash = pairs_of_cells < a.words && n > kPlanesN;
    if (hash) a.words = pairs_of_cells;
    const size_t lds = (size_t)(ET / 64) * (k == 3 ? 1 : 2) * a.words * sizeof(uint2);
    const unsigned blocks = (unsigned)std::min<int64_t>((P + ET / 64 - 1) / (ET / 64), 8192);
    hipLaunchKernelGGL(k_edge_kids, dim3(blocks_of(P * 8)), dim3(ET), 0, st, a);
    void (*kern)(EdgeArgs) = k == 3 ? (hash ? k_edge_sets<false, true> : k_edge_sets<false, false>)
                                    : (hash ? k_edge_sets<true, true> : k_edge_sets<true, false>);
    VDMC_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    if (k == 3) hipLaunchKernelGGL((k_edge_roots<false>), dim3(blocks_of(n * 64)), dim3(ET), 0, st, a);
    else hipLaunchKernelGGL((k_edge_roots<true>), dim3(blocks_of(n * 64)), dim3(ET), 0, st, a);
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(ET), lds, st, a);
    VDMC_HIP(hipGetLastError());
}

}  // namespace vdmc

extern "C" {

vdmc_status vdmc_count_edges(vdmc_graph g, int32_t k, uint64_t* out, void* stream) {
    return vdmc::guarded([&] {
        VDMC_REQUIRE(g != nullptr, VDMC_ERR_INVALID_ARG, "graph is NULL");
        VDMC_REQUIRE(k == 3 || k == 4, k == 5 ? VDMC_ERR_UNSUPPORTED : VDMC_ERR_INVALID_ARG, "k must be 3 or 4");
        VDMC_REQUIRE(out != nullptr || g->pairs == 0, VDMC_ERR_INVALID_ARG, "out is NULL");
        VDMC_HIP(hipSetDevice(g->device));
        vdmc::GraphUse use(g, vdmc::as_stream(stream));
        vdmc::launch_count_edges(g, k, out, vdmc::as_stream(stream));
    });
}

vdmc_status vdmc_edge_list(vdmc_graph g, int32_t* lo, int32_t* hi) {
    return vdmc::guarded([&] {
        VDMC_REQUIRE(g != nullptr, VDMC_ERR_INVALID_ARG, "graph is NULL");
        VDMC_REQUIRE((lo && hi) || g->pairs == 0, VDMC_ERR_INVALID_ARG, "lo/hi is NULL");
        VDMC_HIP(hipSetDevice(g->device));
        std::lock_guard<std::mutex> lock(g->mu);
        vdmc::ensure_edge_index(g, nullptr);
        if (g->pairs == 0) return;
        VDMC_HIP(hipMemcpy(lo, g->elo, g->pairs * sizeof(int32_t), hipMemcpyDeviceToHost));
        VDMC_HIP(hipMemcpy(hi, g->ehi, g->pairs * sizeof(int32_t), hipMemcpyDeviceToHost));
    });
}

}  // extern "C"
