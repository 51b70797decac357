// Light-root motif kernel: roots with at most 32 higher neighbours.
//
// The sets are those of the per-set kernel (count.hip), from the same lowest-rank vertex
// r (Lemma 1), along the same shapes (Lemma 2) under the rules of Lemmas 3-4.  That kernel
// reads the CSR in place: every pair test is a chain of dependent loads, which is all the
// time of a small graph.  Here the whole neighbourhood of a root is staged in LDS first:
//   * the slots (N+(r)) and the depth-2 vertices in one hash by rank; a depth-2 vertex
//     carries its arc codes to the slots as two 32-bit masks, a slot its codes to the
//     other slots, so that a pair test is a bit test and a set below one (slot, child) is
//     an iteration over mask bits;
//   * rows are read from the end (the entries above r are a row's suffix), 16 lanes a row;
//   * the slots' and r's credits are summed in LDS; a depth-2 vertex takes one memory-side
//     atomic per class and parent, an end vertex of (1,1,1) one per set.
// What bounds it: the latency of the few dependent loads per root at small sizes, the
// memory-side atomics (2.4e10/s) at large ones.  G(1000, 0.005), k = 3 and 4: 126 us a call,
// 665 with the per-set kernel; G(150, 0.027), k = 4: 45 us, 258.
//
// A root's depth-2 entries must fit the hash; three sizes are built (light_tier), chosen by
// the number of slots and of entries in their rows above r.  Larger roots take the hub path
// or, in graphs that path does not take, the per-set kernel.
#include "motif_device.h"
#include "vdmc_internal.h"

namespace vdmc {
namespace {

constexpr uint32_t kSlotMark = 0x80000000u;

template <uint32_t DM, uint32_t CAP, bool K4>
struct LightLds {
    uint32_t P[DM];                 // slots: (rank << 2) | arc bits r -> slot
    uint32_t PP[DM];                // their original ids
    uint32_t X0[DM], X1[DM];        // arc bits of a slot to the slots, a plane each
    uint32_t CH[DM][3];             // depth-2 entries of a slot by code
    uint32_t SC[K4 ? DM : 1][kCmpRow];   // compact counters of a slot (k = 4)
    uint32_t S3[DM][kClasses3];     // k = 3 counters of a slot
    uint32_t R4[kClasses4];
    uint32_t R3[kClasses3];
    uint32_t K[CAP];                // hash: rank + 1, marked for a slot; 0 = empty
    uint32_t A0[CAP], A1[CAP];      // slot: its index; depth-2 vertex: arc bits slot -> vertex, a plane each
    uint32_t CL[CAP - CAP / 4];     // depth-2 entries: (hash index << 7) | (slot << 2) | code
    uint32_t n2;                    // number of depth-2 entries
};

__device__ __forceinline__ uint32_t lhash(uint32_t x, uint32_t cap) { return (x * 2654435761u >> 16) & (cap - 1u); }

// n sets of class cls to the vertex of original id v.  Ids are read before the atomics of a phase:
// vector memory operations finish in order, so a load after an atomic waits for it.
__device__ __forceinline__ void ladd(gptr<unsigned long long> out, uint32_t C, uint32_t v, uint32_t cls,
                                     unsigned long long n) {
    gadd64(&out[(size_t)v * C + cls], n);
}

// all threads of a root's group have arrived and see each other's LDS writes
template <int BS>
__device__ __forceinline__ void group_sync() {
    if (BS > 64) {
        __syncthreads();
    } else {
        wave_fence();
    }
}

// sum over aligned groups of 8 lanes, in every lane
__device__ __forceinline__ uint32_t sum8(uint32_t v) {
    v += (uint32_t)__shfl_xor((int)v, 1, 64);
    v += (uint32_t)__shfl_xor((int)v, 2, 64);
    v += (uint32_t)__shfl_xor((int)v, 4, 64);
    return v;
}

template <int BS, uint32_t DM, uint32_t CAP, bool K3, bool K4>
__device__ void light_root(const GraphView& gv, const uint8_t* t3, const uint8_t* t4, const uint8_t* cmp_of,
                           const uint8_t* cmp_cls, uint32_t r, LightLds<DM, CAP, K4>& S, unsigned long long* shp) {
    const uint32_t tid = threadIdx.x % BS;
    const uint32_t s = gv.split[r], d = min(gv.off[r + 1] - s, DM);
    const uint32_t pr = gv.perm[r];
    for (uint32_t i = tid; i < d; i += BS) {
        S.P[i] = gv.adj[s + i];
        S.PP[i] = gv.perm[S.P[i] >> 2];
        S.X0[i] = S.X1[i] = 0u;
        for (int k = 0; k < 3; k++) S.CH[i][k] = 0u;
    }
    for (uint32_t i = tid; i < CAP; i += BS) {
        S.K[i] = 0u;
        S.A0[i] = S.A1[i] = 0u;
    }
    if (K4) {
        for (uint32_t i = tid; i < d * kCmpRow; i += BS) (&S.SC[0][0])[i] = 0u;
        for (uint32_t i = tid; i < (uint32_t)kClasses4; i += BS) S.R4[i] = 0u;
    }
    if (K3) {
        for (uint32_t i = tid; i < d * kClasses3; i += BS) (&S.S3[0][0])[i] = 0u;
        for (uint32_t i = tid; i < (uint32_t)kClasses3; i += BS) S.R3[i] = 0u;
    }
    if (tid == 0) S.n2 = 0u;
    group_sync<BS>();
    for (uint32_t i = tid; i < d; i += BS)
        for (uint32_t key = (S.P[i] >> 2) + 1u, h = lhash(key, CAP);; h = (h + 1u) & (CAP - 1u))
            if (atomicCAS(&S.K[h], 0u, key | kSlotMark) == 0u) {
                S.A0[h] = i;
                break;
            }
    group_sync<BS>();
    // ---- rows of the slots, from the end: arcs among the slots, depth-2 entries
    for (uint32_t a = tid >> 4; a < d; a += BS / 16) {
        const uint32_t va = S.P[a] >> 2, ra = S.P[a] & 3u, lo = gv.off[va];
        uint32_t hi = gv.off[va + 1], next = (tid & 15u) < hi - lo ? gv.adj[hi - 1u - (tid & 15u)] : 0u;
        for (; hi > lo; hi -= min(16u, hi - lo)) {
            const bool in = (tid & 15u) < hi - lo;
            const uint32_t ent = next, e = ent >> 2, c = ent & 3u;
            const uint32_t pe = K3 && e > r ? gv.perm[e] : 0u;
            const bool more = hi - lo > 16u;
            next = (tid & 15u) + 16u < hi - lo ? gv.adj[hi - 17u - (tid & 15u)] : 0u;
            const uint32_t first = more ? gv.adj[hi - 16u] >> 2 : 0u;
            if (in && e > r) {
                uint32_t h = lhash(e + 1u, CAP);
                bool slot = false;
                for (;; h = (h + 1u) & (CAP - 1u)) {
                    uint32_t k = S.K[h];
                    if (k == 0u) {
                        if (!K4) break;
                        k = atomicCAS(&S.K[h], 0u, e + 1u);
                        if (k == 0u) break;
                    }
                    if ((k & ~kSlotMark) == e + 1u) {
                        slot = (k & kSlotMark) != 0u;
                        break;
                    }
                }
                if (slot) {
                    const uint32_t x = S.A0[h];
                    if (c & 1u) atomicOr(&S.X0[a], 1u << x);
                    if (c & 2u) atomicOr(&S.X1[a], 1u << x);
                } else {
                    if (K4) {
                        if (c & 1u) atomicOr(&S.A0[h], 1u << a);
                        if (c & 2u) atomicOr(&S.A1[h], 1u << a);
                        atomicAdd(&S.CH[a][c - 1u], 1u);
                        S.CL[atomicAdd(&S.n2, 1u)] = (h << 7) | (a << 2) | c;
                    }
                    if (K3) {   // (1,2): r - a - e
                        const uint32_t cls = t3[motif_index3(ra, 0u, c)];
                        atomicAdd(&S.R3[cls], 1u);
                        atomicAdd(&S.S3[a][cls], 1u);
                        ladd(gv.out3, kClasses3, pe, cls, 1ull);
                        shp[1]++;
                    }
                }
            }
            if (first <= r) break;   // the rest of the row is not above r
        }
    }
    group_sync<BS>();
    auto code = [](uint32_t m0, uint32_t m1, uint32_t x) { return ((m0 >> x) & 1u) | (((m1 >> x) & 1u) << 1); };
    // n sets of class cls to slot a / to r
    auto add_a = [&](uint32_t a, uint32_t cls, uint32_t n) {
        const uint32_t c = cmp_of[cls];
        if (c < kCmpRow) atomicAdd(&S.SC[a][c], n);
        else ladd(gv.out4, kClasses4, S.PP[a], cls, (unsigned long long)(long long)(int32_t)n);
    };
    auto add_r = [&](uint32_t cls, uint32_t n) { atomicAdd(&S.R4[cls], n); };
    // ---- pairs a < b of slots: (1,1), (3,0,0)
    for (uint32_t q = tid; q < d * (d - 1u) / 2u; q += BS) {
        uint32_t b = (uint32_t)((1.0f + sqrtf(1.0f + 8.0f * (float)q)) * 0.5f);
        while (b * (b - 1u) / 2u > q) b--;
        while ((b + 1u) * b / 2u <= q) b++;
        const uint32_t a = q - b * (b - 1u) / 2u;
        const uint32_t ra = S.P[a] & 3u, rb = S.P[b] & 3u;
        const uint32_t a0 = S.X0[a], a1 = S.X1[a], b0 = S.X0[b], b1 = S.X1[b], ab = code(a0, a1, b);
        if (K3) {
            const uint32_t cls = t3[motif_index3(ra, rb, ab)];
            atomicAdd(&S.R3[cls], 1u);
            atomicAdd(&S.S3[a][cls], 1u);
            atomicAdd(&S.S3[b][cls], 1u);
            shp[0]++;
        }
        if (K4) {
            uint32_t run = 0xFFu, n = 0;   // consecutive sets of one class
            for (uint32_t c = b + 1u; c < d; c++) {
                const uint32_t cls = t4[motif_index4(ra, rb, S.P[c] & 3u, ab, code(a0, a1, c), code(b0, b1, c))];
                add_a(c, cls, 1u);
                if (cls != run) {
                    if (n) {
                        add_a(a, run, n);
                        add_a(b, run, n);
                        add_r(run, n);
                    }
                    run = cls;
                    n = 0;
                }
                n++;
            }
            if (n) {
                add_a(a, run, n);
                add_a(b, run, n);
                add_r(run, n);
            }
            shp[2] += d - 1u - b;
        }
    }
    if (K4) {
        const uint32_t n2 = S.n2;
        // ---- (2,1,0) of every depth-2 entry (a, c): a second slot b, not below the lower parent
        for (uint32_t i = tid; i < n2; i += BS) {
            const uint32_t ent = S.CL[i], h = ent >> 7, a = (ent >> 2) & 31u, ac = ent & 3u;
            const uint32_t c = S.K[h] - 1u, c0 = S.A0[h], c1 = S.A1[h], ra = S.P[a] & 3u;
            const uint32_t a0 = S.X0[a], a1 = S.X1[a];
            const uint32_t all = d < 32u ? (1u << d) - 1u : ~0u;
            uint32_t run = 0xFFu, n = 0;
            gptr<unsigned long long> row = &gv.out4[(size_t)gv.perm[c] * kClasses4];
            for (uint32_t m = all & ~(1u << a) & ~((c0 | c1) & ((1u << a) - 1u)); m; m &= m - 1u) {
                const uint32_t b = (uint32_t)__ffs((int)m) - 1u;
                const uint32_t cls = t4[motif_index4(ra, S.P[b] & 3u, 0u, code(a0, a1, b), ac, code(c0, c1, b))];
                add_a(b, cls, 1u);
                shp[3]++;
                if (cls != run) {
                    if (n) {
                        add_a(a, run, n);
                        add_r(run, n);
                        gadd64(&row[run], n);
                    }
                    run = cls;
                    n = 0;
                }
                n++;
            }
            if (n) {
                add_a(a, run, n);
                add_r(run, n);
                gadd64(&row[run], n);
            }
        }
        // ---- (1,2,0) of a and r: pairs of a's children by code, as if not adjacent
        for (uint32_t i = tid; i < d * 6u; i += BS) {
            const uint32_t a = i / 6u, p = i % 6u;
            const uint32_t k = p < 3u ? 0u : (p < 5u ? 1u : 2u), l = p < 3u ? p : (p < 5u ? p - 2u : 2u);
            const uint32_t nk = S.CH[a][k], nl = S.CH[a][l], n = k == l ? nk * (nk - 1u) / 2u : nk * nl;
            if (n) {
                const uint32_t cls = t4[motif_index4(S.P[a] & 3u, 0u, 0u, k + 1u, l + 1u, 0u)];
                add_a(a, cls, n);
                add_r(cls, n);
                shp[4] += n;
            }
        }
        // ---- (1,2,0) and (1,1,1) of every depth-2 entry (a, c), 8 lanes each: c's row above r
        // (the next entry's row is loaded before this one's credits)
        const uint32_t gl = tid & 7u;
        const auto child = [&](uint32_t i) { return i < n2 ? S.K[S.CL[i] >> 7] - 1u : 0u; };
        uint32_t c = child(tid >> 3), lo = gv.off[c], hi0 = (tid >> 3) < n2 ? gv.off[c + 1] : 0u, pc = gv.perm[c];
        uint32_t x0 = hi0 > lo + gl ? gv.adj[hi0 - 1u - gl] : 0u;
        for (uint32_t i0 = 0; i0 < n2; i0 += BS / 8) {
            const uint32_t i = i0 + (tid >> 3);
            const bool on = i < n2;
            const uint32_t ent = on ? S.CL[i] : 0u, a = (ent >> 2) & 31u, ac = ent & 3u, ra = S.P[a] & 3u;
            const uint32_t cn = child(i + BS / 8), lon = gv.off[cn], hin = i + BS / 8 < n2 ? gv.off[cn + 1] : 0u;
            const uint32_t pcn = gv.perm[cn];
            uint32_t x0n = 0;
            uint32_t e1 = 0, e2 = 0, e3 = 0;   // ends of paths by arc code
            uint32_t j1 = 0, j2 = 0, j3 = 0;   // children of a adjacent to c, by their code
            for (uint32_t hi = hi0; hi > lo; hi -= min(8u, hi - lo)) {
                const bool in = gl < hi - lo;
                const uint32_t ee = hi == hi0 ? x0 : (in ? gv.adj[hi - 1u - gl] : 0u), e = ee >> 2, ce = ee & 3u;
                const uint32_t pe = e > r ? gv.perm[e] : 0u;
                const uint32_t first = hi - lo > 8u ? gv.adj[hi - 8u] >> 2 : 0u;
                if (hi == hi0) x0n = hin > lon + gl ? gv.adj[hin - 1u - gl] : 0u;
                if (in && e > r) {
                    uint32_t h = lhash(e + 1u, CAP), k;
                    for (;; h = (h + 1u) & (CAP - 1u)) {
                        k = S.K[h];
                        if (k == 0u || (k & ~kSlotMark) == e + 1u) break;
                    }
                    if (!(k & kSlotMark)) {
                        const uint32_t ae = k ? code(S.A0[h], S.A1[h], a) : 0u;
                        if (ae) {   // e is another child of a
                            const uint32_t cls = t4[motif_index4(ra, 0u, 0u, ac, ae, ce)];
                            ladd(gv.out4, kClasses4, pc, cls, 1ull);
                            j1 += ae == 1u;
                            j2 += ae == 2u;
                            j3 += ae == 3u;
                            if (e > c) {
                                const uint32_t st = t4[motif_index4(ra, 0u, 0u, ac, ae, 0u)];
                                add_a(a, cls, 1u);
                                add_r(cls, 1u);
                                add_a(a, st, ~0u);
                                add_r(st, ~0u);
                            }
                        } else {    // path r - a - c - e
                            ladd(gv.out4, kClasses4, pe, t4[motif_index4(ra, 0u, 0u, ac, 0u, ce)], 1ull);
                            e1 += ce == 1u;
                            e2 += ce == 2u;
                            e3 += ce == 3u;
                        }
                    }
                }
                if (first <= r) break;
            }
            e1 = sum8(e1);
            e2 = sum8(e2);
            e3 = sum8(e3);
            j1 = sum8(j1);
            j2 = sum8(j2);
            j3 = sum8(j3);
            if (on && gl < 6u) {
                const uint32_t k = gl % 3u;
                if (gl < 3u) {
                    const uint32_t n = k == 2u ? e3 : (k == 0u ? e1 : e2);
                    if (n) {
                        const uint32_t cls = t4[motif_index4(ra, 0u, 0u, ac, 0u, k + 1u)];
                        add_a(a, cls, n);
                        add_r(cls, n);
                        ladd(gv.out4, kClasses4, pc, cls, n);
                        shp[5] += n;
                    }
                } else {   // the children of a that are not adjacent to c, by code
                    const uint32_t n = S.CH[a][k] - (k + 1u == ac ? 1u : 0u) -
                                       (k == 2u ? j3 : (k == 0u ? j1 : j2));
                    if (n) ladd(gv.out4, kClasses4, pc, t4[motif_index4(ra, 0u, 0u, ac, k + 1u, 0u)], n);
                }
            }
            c = cn;
            lo = lon;
            hi0 = hin;
            pc = pcn;
            x0 = x0n;
        }
    }
    group_sync<BS>();
    if (K4) {
        for (uint32_t i = tid; i < d * kCmpRow; i += BS) {
            const uint32_t n = (&S.SC[0][0])[i];
            if (n) ladd(gv.out4, kClasses4, S.PP[i / kCmpRow], cmp_cls[i % kCmpRow], n);
        }
        for (uint32_t i = tid; i < (uint32_t)kClasses4; i += BS)
            if (S.R4[i]) ladd(gv.out4, kClasses4, pr, i, S.R4[i]);
    }
    if (K3) {
        for (uint32_t i = tid; i < d * kClasses3; i += BS) {
            const uint32_t n = (&S.S3[0][0])[i];
            if (n) ladd(gv.out3, kClasses3, S.PP[i / kClasses3], i % kClasses3, n);
        }
        for (uint32_t i = tid; i < (uint32_t)kClasses3; i += BS)
            if (S.R3[i]) ladd(gv.out3, kClasses3, pr, i, S.R3[i]);
    }
    group_sync<BS>();
}

// visited sets of the calling workgroup to a graph's shape counters, one atomic per wave and shape
__device__ __forceinline__ void add_shapes(gptr<unsigned long long> stats, unsigned long long* shp) {
    for (int s = 0; s < kShapes; s++) {
        unsigned long long x = shp[s];
        for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
        if ((threadIdx.x & 63u) == 0u && x) gadd64(&stats[s], x);
        shp[s] = 0;
    }
}

// WPB groups of BS threads per workgroup, each with a root of its own
template <int BS, int WPB, uint32_t DM, uint32_t CAP, bool K3, bool K4>
__global__ __launch_bounds__(BS* WPB) void k_light(LightArgs A) {
    static_assert(BS == 64 || WPB == 1, "a group is a wave or the whole workgroup");
    __shared__ LightLds<DM, CAP, K4> lds[WPB];
    __shared__ uint32_t t4w[K4 ? 1024 : 1];
    __shared__ uint8_t t3[64];
    __shared__ uint8_t cmp_of[256];
    __shared__ uint8_t cmp_cls[kCmpRow];
    __shared__ unsigned long long next;
    const uint8_t* t4 = (const uint8_t*)t4w;
    if (K4)
        for (uint32_t i = threadIdx.x; i < 1024u; i += BS * WPB) t4w[i] = ((const uint32_t*)A.t4)[i];
    for (uint32_t i = threadIdx.x; i < 64u; i += BS * WPB) t3[i] = A.t3[i];
    for (uint32_t i = threadIdx.x; i < 256u; i += BS * WPB) cmp_of[i] = A.cmp_of[i];
    if (threadIdx.x < kCmpRow) cmp_cls[threadIdx.x] = A.cmp_cls[threadIdx.x];
    __syncthreads();
    const uint32_t group = threadIdx.x / BS;
    LightLds<DM, CAP, K4>& S = lds[group];
    unsigned long long shp[kShapes] = {0, 0, 0, 0, 0, 0};
    if (A.roots) {   // one graph: roots in turn
        for (int64_t i = (int64_t)blockIdx.x * WPB + group; i < A.nroots; i += (int64_t)gridDim.x * WPB) {
            const uint32_t r = A.roots[K4 ? i : A.nroots - 1 - i];   // all tiers at once: the largest first
            if (r < A.rank_lo || r >= A.rank_hi) continue;   // uniform over the group
            light_root<BS, DM, CAP, K3, K4>(A.gv, t3, t4, cmp_of, cmp_cls, r, S, shp);
        }
        add_shapes(A.gv.stats, shp);
        return;
    }
    int cur = -1;    // many graphs: (graph, root) pairs from a cursor
    for (;;) {
        unsigned long long e0 = 0;
        if (BS > 64) {
            __syncthreads();
            if (threadIdx.x == 0) next = atomicAdd(A.cursor, (unsigned long long)A.tile);
            __syncthreads();
            e0 = next;
        } else {
            if ((threadIdx.x & 63u) == 0u) e0 = atomicAdd(A.cursor, (unsigned long long)A.tile);
            e0 = __shfl(e0, 0, 64);
        }
        if (e0 >= (unsigned long long)A.nroots) break;
        const unsigned long long e1 = min(e0 + A.tile, (unsigned long long)A.nroots);
        for (unsigned long long e = e0; e < e1; e++) {
            const uint2 ent = A.table[K4 ? e : A.nroots - 1 - e];   // x = graph, y = root
            if ((int)ent.x != cur) {
                if (cur >= 0) add_shapes(A.graphs[cur].stats, shp);
                cur = (int)ent.x;
            }
            light_root<BS, DM, CAP, K3, K4>(A.graphs[ent.x], t3, t4, cmp_of, cmp_cls, ent.y, S, shp);
        }
    }
    if (cur >= 0) add_shapes(A.graphs[cur].stats, shp);
}

template <int BS, int WPB, uint32_t DM, uint32_t CAP>
void launch_one(const LightArgs& a, int k3, unsigned grid, hipStream_t st) {
    const dim3 block(BS * WPB);
    if (k3) hipLaunchKernelGGL((k_light<BS, WPB, DM, CAP, true, true>), dim3(grid), block, 0, st, a);
    else hipLaunchKernelGGL((k_light<BS, WPB, DM, CAP, false, true>), dim3(grid), block, 0, st, a);
    VDMC_HIP(hipGetLastError());
}

int light_cus() {
    static int ncu = -1;
    if (ncu < 0) {
        int dev = 0;
        hipDeviceProp_t prop;
        VDMC_HIP(hipGetDevice(&dev));
        VDMC_HIP(hipGetDeviceProperties(&prop, dev));
        ncu = prop.multiProcessorCount;
    }
    return ncu;
}

}  // namespace

void launch_light(LightArgs a, int tier, int k3, int k4, hipStream_t st) {
    if (a.nroots <= 0) return;
    const ClassTables& t = class_tables();
    a.t3 = t.t3;
    a.t4 = t.t4;
    a.cmp_of = t.cmp_of;
    a.cmp_cls = t.cmp_cls;
    const int64_t cus = light_cus();
    // few roots (a workgroup each in one go): four waves each, latency is what counts; many: a wave each
    // (G(n, p) of 600 vertices of degree 10: 81 us, 145 with the line at one workgroup per compute unit; of
    // 2000 vertices of degree 4: 90, 97 with the line at sixteen)
    const bool few = a.roots && a.nroots <= 4 * cus;
    // as many workgroups as registers and LDS hold at once (8-slot kernel, 112 registers: four a compute
    // unit; path of 2^20 vertices 1.78 ms with six, whose last two run alone, 1.43 with four)
    const auto grid = [&](int64_t roots_per_wg, int64_t wgs_per_cu) {
        return (unsigned)std::min<int64_t>((a.nroots + roots_per_wg - 1) / roots_per_wg, cus * wgs_per_cu);
    };
    if (!k4) {   // k = 3 alone hashes the slots only: one kernel and launch for all tiers (537 us with
                 // the sizes of k = 4, 479 so, for R-MAT 2^14 in five ranges)
        if (few) hipLaunchKernelGGL((k_light<256, 1, 32, 64, true, false>), dim3(grid(1, 4)), dim3(256), 0, st, a);
        else hipLaunchKernelGGL((k_light<64, 4, 32, 64, true, false>), dim3(grid(4, 7)), dim3(256), 0, st, a);
        VDMC_HIP(hipGetLastError());
    } else if (tier == 2) launch_one<256, 1, 32, 4096>(a, k3, grid(1, 2), st);
    else if (few) launch_one<256, 1, 32, 512>(a, k3, grid(1, 4), st);
    else if (tier == 1) launch_one<64, 4, 32, 512>(a, k3, grid(4, 2), st);
    else launch_one<64, 4, 8, 128>(a, k3, grid(4, 4), st);
}

}  // namespace vdmc
