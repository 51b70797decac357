"""Workloads of the motif counter: what a program that uses this library has it do.

A case is a dict of plain values.  ``listed()`` gives the standing cases, ``draw(rng)`` one
more of the same ranges, ``prepare(case, seed)`` what a program holds before the call
(arc lists, resident graphs, output buffers, a server), ``run(state)`` one pass through
the public entry points, ``work(case)`` the bytes and operations a pass cannot do without
and ``exact(case, seed)`` the counts by plain numpy, where that is quick.

Graph families (``family``), all seeded and synthetic:
  er       directed G(n, p) with mean out-degree ``deg``, as a raw arc list: a few
           self-loops and repeats are left in, which the library drops
  chunglu  power-law in/out weights (gamma 2.1) clipped at ``clip``, 20% of the arcs
           reciprocated, undirected degrees kept near 2 x clip
  rmat     R-MAT (0.57, 0.19, 0.19, 0.05), n = 2^scale, hubs thinned to ``clip`` x 2

What a pass does (``do``):
  count      count / count34 (k = 34) of one resident graph
  range      the same count as ``parts`` consecutive root-rank ranges, accumulated (the
             unit for spreading one graph over devices)
  fresh      device graph build and count of an arc list that is in device memory (or on
             the host: ``host``), the graph freed afterwards
  undirected count_undirected of one resident graph
  edges      count_edges of one resident graph
  batch      count_batch over ``num`` resident G(n, p) graphs
  serve      ``num`` requests, k = 3 and 4 mixed, through a running server and back
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2201_11655_amd as v


# ---------------------------------------------------------------------------- the cases

def listed():
    return [
        # one small request alone (the smallest graphs of the batch and of the request pool
        # are of this size): launches and latency are all there is
        {"name": "one_small_k4", "do": "count", "family": "er", "n": 150, "deg": 4.0, "k": 4},
        # the G(1000, 0.005) reference graph, both k in one call, resident
        {"name": "er1000_k34", "do": "count", "family": "er", "n": 1000, "deg": 4.95, "k": 34},
        # the same for a graph seen once: arcs in host memory, build, count, free
        {"name": "fresh_er1000_k34", "do": "fresh", "family": "er", "n": 1000, "deg": 4.95, "k": 34, "host": True},
        # the headline batch: 4096 uneven G(n, p) graphs, k = 4, one call
        {"name": "batch4096_k4", "do": "batch", "num": 4096, "n_lo": 20, "n_hi": 500, "deg_lo": 2.0, "deg_hi": 8.0,
         "k": 4},
        # a batch for k = 3 with some graphs that are larger than a whole-graph workgroup takes
        {"name": "batch_mixed_k3", "do": "batch", "num": 700, "n_lo": 20, "n_hi": 1500, "deg_lo": 2.0, "deg_hi": 8.0,
         "k": 3},
        # 5-vertex motifs of a batch
        {"name": "batch256_k5", "do": "batch", "num": 256, "n_lo": 20, "n_hi": 500, "deg_lo": 2.0, "deg_hi": 8.0,
         "k": 5},
        # 5-vertex motifs of one fat-tailed graph that LDS does not hold
        {"name": "chunglu2000_k5", "do": "count", "family": "chunglu", "n": 2000, "deg": 8.4, "clip": 45, "k": 5},
        # a fat-tailed graph of about a million arcs: build and count both k, as in the
        # large runs (arcs already in device memory)
        {"name": "chunglu100k_k34", "do": "fresh", "family": "chunglu", "n": 100_000, "deg": 8.4, "clip": 316, "k": 34,
         "host": False},
        # R-MAT with the heaviest hubs the hub path takes, counted in root ranges: the largest
        {"name": "rmat15_k4_ranges", "do": "range", "family": "rmat", "n": 1 << 15, "deg": 8.0, "clip": 750, "k": 4,
         "parts": 4},
        # undirected motifs of a fat-tailed graph
        {"name": "undirected30k_k4", "do": "undirected", "family": "chunglu", "n": 30_000, "deg": 8.4, "clip": 173,
         "k": 4},
        # per-edge counts of a fat-tailed graph
        {"name": "edges3001_k4", "do": "edges", "family": "chunglu", "n": 3001, "deg": 8.4, "clip": 55, "k": 4},
        # a burst of requests of very uneven size over a pool of resident graphs
        {"name": "serve96", "do": "serve", "num": 96, "pool": 48, "log_lo": 2.0, "log_hi": 4.2, "clip": 1000},
    ]


def _log(rng, lo, hi):
    """An odd-or-even whole number spread evenly over the logarithm of [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _clip(n):
    return max(8, int(round(1000.0 * math.sqrt(n / 1e6))))   # hubs shrink with sqrt(n)


def draw(rng):
    do = rng.choice(["count", "count", "count5", "fresh", "fresh", "range", "undirected", "edges", "batch", "batch",
                     "batch5", "serve"])
    deg = round(rng.uniform(2.0, 10.0), 2)
    if do == "count5":
        if rng.random() < 0.5:   # held in LDS
            return {"do": "count", "family": "er", "n": _log(rng, 40, 500), "deg": min(deg, 6.0), "k": 5}
        n = _log(rng, 520, 2000)
        return {"do": "count", "family": "chunglu", "n": n, "deg": min(deg, 8.4), "clip": _clip(n), "k": 5}
    if do in ("batch", "batch5"):
        lo = rng.randint(5, 40)
        hi = rng.randint(100, 500) if do == "batch5" else rng.choice([rng.randint(60, 500), rng.randint(500, 1400)])
        num = _log(rng, 16, 160) if do == "batch5" else _log(rng, 32, 2500 if hi <= 500 else 500)
        d0 = round(rng.uniform(1.0, 4.0), 2)
        return {"do": "batch", "num": num, "n_lo": lo, "n_hi": hi, "deg_lo": d0,
                "deg_hi": round(d0 + rng.uniform(0.5, 4.0), 2), "k": 5 if do == "batch5" else rng.choice([3, 4, 4])}
    if do == "serve":
        pool = rng.randint(8, 48)
        return {"do": "serve", "num": pool * 2, "pool": pool, "log_lo": 1.5, "log_hi": round(rng.uniform(2.5, 4.0), 2),
                "clip": rng.randint(200, 1000)}
    c = {"do": do}
    if do == "edges":
        c.update(family="chunglu", n=_log(rng, 300, 3001), deg=min(deg, 8.4), k=rng.choice([3, 4]))
    elif do == "undirected":
        c.update(family=rng.choice(["er", "chunglu"]), n=_log(rng, 300, 30_000), deg=min(deg, 8.4), k=rng.choice([3, 4]))
    elif do == "range":
        c.update(family="rmat", n=1 << rng.randint(10, 14), deg=deg, k=rng.choice([3, 4]), parts=rng.randint(2, 5))
        c["clip"] = min(750, c["n"] // 8)
        return c
    else:
        c.update(family=rng.choice(["er", "chunglu"]), n=_log(rng, 60, 80_000), deg=min(deg, 8.4),
                 k=rng.choice([3, 4, 34]))
        if do == "fresh":
            c["host"] = rng.random() < 0.5
    if c["family"] == "chunglu":
        c["clip"] = _clip(c["n"])
    return c


# ---------------------------------------------------------------------------- inputs

def _er(rng, n, deg):
    m = max(1, int(rng.poisson(n * deg)))
    return rng.integers(0, n, m), rng.integers(0, n, m)


def _thin(rng, n, src, dst, cap):
    """Drops arcs of vertices above ``cap`` incident arcs, each with the vertex's excess share."""
    d = np.bincount(src, minlength=n) + np.bincount(dst, minlength=n)
    keep = np.minimum(1.0, cap / np.maximum(d, 1))
    ok = rng.random(src.shape[0]) < keep[src] * keep[dst]
    return src[ok], dst[ok]


def _chunglu(rng, n, deg, clip):
    m = max(1, int(n * deg))
    w = (np.arange(n) + 1.0) ** (-1.0 / 1.1)
    w = np.minimum(w * (m / w.sum()), clip)
    ends = []
    for _ in range(2):
        c = np.cumsum(w[rng.permutation(n)])
        ends.append(np.minimum(np.searchsorted(c, rng.random(m) * c[-1], side="right"), n - 1))
    src, dst = ends
    back = rng.random(m) < 0.2
    return _thin(rng, n, np.concatenate([src, dst[back]]), np.concatenate([dst, src[back]]), 2.2 * clip)


def _rmat(rng, n, deg, clip):
    m = int(n * deg)
    src, dst = np.zeros(m, np.int64), np.zeros(m, np.int64)
    for _ in range(n.bit_length() - 1):
        u = rng.random(m)
        src = (src << 1) | (u >= 0.76)
        dst = (dst << 1) | (((u >= 0.57) & (u < 0.76)) | (u >= 0.95))
    return _thin(rng, n, src, dst, 2 * clip)


def _trim(rng, n, src, dst, pairs):
    """The arcs of exactly ``pairs`` joined vertex pairs: those given, thinned, or filled up
    with uniform ones."""
    extra = rng.integers(0, n, (2, 3 * pairs))
    s, d = np.concatenate([src, extra[0]]), np.concatenate([dst, extra[1]])
    ok = s != d
    s, d = s[ok], d[ok]
    _, first, of = np.unique(np.minimum(s, d) * n + np.maximum(s, d), return_index=True, return_inverse=True)
    given = first < np.count_nonzero(src != dst)
    order = np.argsort(rng.random(len(first)) + ~given, kind="stable")   # the given pairs come first
    keep = np.zeros(len(first), bool)
    keep[order[:pairs]] = True
    keep = keep[of]
    return s[keep], d[keep]


def _arcs(case, rng):
    """(n, src, dst) of a single-graph case, int32."""
    n = case["n"]
    if case["family"] == "er":
        s, d = _er(rng, n, case["deg"])
    elif case["family"] == "chunglu":
        s, d = _chunglu(rng, n, case["deg"], case["clip"])
    else:
        s, d = _rmat(rng, n, case["deg"], case["clip"])
    if case["do"] == "edges":   # one output row per pair: their number belongs to the case
        s, d = _trim(rng, n, s, d, int(0.8 * n * case["deg"]))
    return n, s.astype(np.int32), d.astype(np.int32)


def _many(case, rng):
    """The arc lists of a batch or of a pool; the vertex counts belong to the case."""
    out = []
    if case["do"] == "batch":
        sizes = np.random.default_rng([case["num"], case["n_lo"], case["n_hi"]])
        for n in sizes.integers(case["n_lo"], case["n_hi"] + 1, case["num"]).tolist():
            s, d = _er(rng, n, rng.uniform(case["deg_lo"], case["deg_hi"]))
            out.append((n, s.astype(np.int32), d.astype(np.int32)))
        return out
    sizes = np.random.default_rng([case["pool"], case["clip"]])
    logs = sizes.uniform(case["log_lo"], case["log_hi"], case["pool"])
    for i, n in enumerate(np.rint(10 ** logs).astype(int).tolist()):   # even slots G(n, p), odd slots fat-tailed
        deg = rng.uniform(2.0, 10.0)
        s, d = _er(rng, n, deg) if i % 2 == 0 else _chunglu(rng, n, deg / 1.2, case["clip"])
        out.append((n, s.astype(np.int32), d.astype(np.int32)))
    return out


def _rows(ns, C):
    """One buffer for many outputs and its parts (each starts on a 64-value boundary)."""
    starts, at = [], 0
    for n in ns:
        starts.append(at)
        at += (n * C + 63) // 64 * 64
    flat = torch.zeros(at, dtype=torch.int64, device="cuda")
    return flat, [flat[a:a + n * C].view(n, C) for a, n in zip(starts, ns)]


def _requests(case, rng):
    """(slot of the pool, k) of every request: each graph twice, k = 3 and 4 half and half."""
    reqs = [(i % case["pool"], 3 + (i // case["pool"]) % 2) for i in range(case["num"])]
    return [reqs[i] for i in rng.permutation(len(reqs))]


def prepare(case, seed):
    rng = np.random.default_rng([int(seed), 7])
    do = case["do"]
    st = {"case": case}
    if do == "batch":
        gs = _many(case, rng)
        st["graphs"] = [v.Graph(n, s, d) for n, s, d in gs]
        st["flat"], st["outs"] = _rows([n for n, _, _ in gs], v.num_classes(case["k"]))
        return st
    if do == "serve":
        gs = _many(case, rng)
        st["graphs"] = [v.Graph(n, s, d) for n, s, d in gs]
        st["reqs"] = _requests(case, rng)
        C = {3: v.num_classes(3), 4: v.num_classes(4)}
        st["flats"], parts = {}, {}
        for k in (3, 4):
            st["flats"][k], parts[k] = _rows([gs[i][0] for i, q in st["reqs"] if q == k], C[k])
        st["outs"] = [parts[k].pop(0) for _, k in st["reqs"]]
        st["server"] = v.Server(16 << 30, 32)
        torch.cuda.synchronize()
        return st
    n, src, dst = _arcs(case, rng)
    if do == "fresh":
        if case["host"]:
            st["arcs"] = (n, src, dst)
        else:
            st["arcs"] = (n, torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda())
        return st
    st["graph"] = v.Graph(n, src, dst, undirected=do == "undirected")
    st["n"] = n
    return st


# ---------------------------------------------------------------------------- one pass

def run(st):
    case = st["case"]
    do = case["do"]
    if do == "batch":
        v.count_batch(st["graphs"], case["k"], outs=st["outs"])
        return st["flat"]
    if do == "serve":
        srv = st["server"]
        ids = [srv.submit(st["graphs"][i], k, o) for (i, k), o in zip(st["reqs"], st["outs"])]
        for rid in ids:
            srv.wait(rid)
        return [st["flats"][3], st["flats"][4]]
    if do == "edges":
        return v.count_edges(st["graph"], case["k"])
    if do == "undirected":
        return v.count_undirected(st["graph"], case["k"])
    if do == "range":
        g, parts = st["graph"], case["parts"]
        out = torch.empty((g.n, v.num_classes(case["k"])), dtype=torch.int64, device="cuda")
        # ranges of about equal weight: the heavy roots come first in rank order
        cuts = [0] + [g.n >> (parts - i) for i in range(1, parts)] + [g.n]
        for i in range(parts):
            v.count_range(g, case["k"], out, cuts[i], cuts[i + 1], accumulate=i > 0)
        return out
    g = v.Graph(*st["arcs"]) if do == "fresh" else st["graph"]
    if case["k"] == 34:
        return list(v.count34(g))
    return v.count(g, case["k"])


# ---------------------------------------------------------------------------- what it takes

_CLASSES = {3: 13, 4: 199, 5: 9364}


def work(case):
    """Bytes: each arc read once (8 bytes), each count written once (8 bytes).  Operations:
    the k credits of every connected k-set, the sets estimated as those of a sparse random
    graph (n k^(k-2) / k! x degree^(k-1)), for the fat-tailed families from one seeded
    graph's degrees (trees with k - 1 pairs)."""
    ks = [3, 4] if case["do"] == "serve" or case.get("k") == 34 else [case["k"]]
    if case["do"] in ("batch", "serve"):
        graphs = _many(case, np.random.default_rng([1, 7]))
    else:
        graphs = [_arcs(case, np.random.default_rng([1, 7]))]
    nbytes, ops = 0.0, 0.0
    for n, s, d in graphs:
        deg = np.bincount(s, minlength=n) + np.bincount(d, minlength=n).astype(np.float64)
        for k in ks:
            if k == 3:
                sets = float((deg * (deg - 1) / 2).sum())
            elif k == 4:
                sets = float(((deg[s] - 1) * (deg[d] - 1)).sum() + (deg * (deg - 1) * (deg - 2) / 6).sum())
            else:
                sets = float((deg ** 4).sum() * 125 / 120)
            ops += k * sets
            C = _CLASSES[k] if case["do"] != "undirected" else {3: 2, 4: 6}[k]
            rows = n if case["do"] != "edges" else s.shape[0]
            nbytes += 8.0 * rows * C + (4.0 if len(ks) == 2 else 8.0) * s.shape[0]
    return {"bytes": nbytes, "flops": ops}


# ---------------------------------------------------------------------------- plain numpy counts

def _class_of(k):
    """class id of every motif index (-1: not connected): the rank of its smallest relabelling
    among the connected ones; indices are the adjacency matrix row by row, no diagonal."""
    from itertools import permutations
    pairs = [(i, j) for i in range(k) for j in range(k) if i != j]
    nb = len(pairs)
    codes = np.arange(1 << nb)
    best, arc = codes.copy(), np.zeros((k, k, 1 << nb), bool)
    for b, (i, j) in enumerate(pairs):
        arc[i, j] = (codes >> (nb - 1 - b)) & 1
    for p in permutations(range(k)):
        c = np.zeros_like(codes)
        for b, (i, j) in enumerate(pairs):
            c |= arc[p[i], p[j]].astype(np.int64) << (nb - 1 - b)
        best = np.minimum(best, c)
    reach = arc | arc.transpose(1, 0, 2) | np.eye(k, dtype=bool)[:, :, None]
    for _ in range(2):
        reach = np.any(reach[:, :, None] & reach[None], axis=1)
    conn = reach.all(axis=(0, 1))
    ids = np.full(1 << nb, -1)
    ids[conn] = np.searchsorted(np.unique(best[conn]), best[conn])
    return ids


def _simple(n, src, dst, undirected):
    """Arc keys u * n + v, ascending, without loops and repeats, and the CSR of G_U."""
    s, d = src.astype(np.int64), dst.astype(np.int64)
    if undirected:
        s, d = np.concatenate([s, d]), np.concatenate([d, s])
    arcs = np.unique((s * n + d)[s != d])
    both = np.unique(np.concatenate([arcs, (arcs % n) * n + arcs // n]))
    off = np.searchsorted(both, np.arange(n + 1) * n)
    return arcs, off, both % n


def _sets(n, off, nbr, k):
    """Every connected k-set as ascending columns, grown one neighbour at a time."""
    deg = np.diff(off)
    sets = np.arange(n)[:, None]
    for size in range(2, k + 1):
        grown = []
        for c in range(size - 1):
            rep = deg[sets[:, c]]
            base = np.repeat(np.cumsum(rep) - rep, rep)
            new = nbr[np.repeat(off[sets[:, c]], rep) + np.arange(rep.sum()) - base]
            old = np.repeat(sets, rep, axis=0)
            fresh = (old != new[:, None]).all(axis=1)
            grown.append(np.sort(np.concatenate([old[fresh], new[fresh, None]], axis=1), axis=1))
        grown = np.concatenate(grown)
        key = np.zeros(len(grown), np.int64)
        for c in range(size):
            key = key * n + grown[:, c]
        sets = grown[np.unique(key, return_index=True)[1]]
    return sets


def _counts(n, src, dst, k, edges=False, undirected=False):
    """The counts of one graph: n x classes, or pairs x classes for ``edges``."""
    arcs, off, nbr = _simple(n, src, dst, undirected)
    ids = _class_of(k)
    C = int(ids.max()) + 1
    if undirected:   # keep the classes whose pairs are all joined both ways
        pairs = [(i, j) for i in range(k) for j in range(i + 1, k)]
        order = [(i, j) for i in range(k) for j in range(k) if i != j]
        cols = sorted({int(ids[sum(1 << (len(order) - 1 - order.index(e)) for b, (i, j) in enumerate(pairs)
                                   if m >> b & 1 for e in ((i, j), (j, i)))]) for m in range(1 << len(pairs))} - {-1})
    if len(arcs) == 0:
        return np.zeros((n, len(cols) if undirected else C), np.int64)
    sets = _sets(n, off, nbr, k)
    code = np.zeros(len(sets), np.int64)

    def has(u, w):
        key = u * n + w
        at = np.minimum(np.searchsorted(arcs, key), len(arcs) - 1)
        return arcs[at] == key

    for i in range(k):
        for j in range(k):
            if i != j:
                code = (code << 1) | has(sets[:, i], sets[:, j])
    cls = ids[code]
    if edges:
        rows_of = np.unique(np.minimum(arcs // n, arcs % n) * n + np.maximum(arcs // n, arcs % n))
        out = np.zeros(len(rows_of) * C, np.int64)
        for i in range(k):
            for j in range(i + 1, k):
                key = sets[:, i] * n + sets[:, j]
                at = np.minimum(np.searchsorted(rows_of, key), len(rows_of) - 1)
                ok = rows_of[at] == key
                out += np.bincount(at[ok] * C + cls[ok], minlength=out.size)
        return out.reshape(-1, C)
    out = np.zeros(n * C, np.int64)
    for i in range(k):
        out += np.bincount(sets[:, i] * C + cls, minlength=n * C)
    out = out.reshape(n, C)
    return out[:, cols] if undirected else out


def exact(case, seed):
    """The counts of run(), by enumeration of vertex sets in numpy; None where there are too
    many sets for that (and for k = 5)."""
    if case.get("k") == 5 or case["do"] == "serve" or work(case)["flops"] > 1.2e7:
        return None
    rng = np.random.default_rng([int(seed), 7])
    if case["do"] == "batch":
        k, C, parts = case["k"], _CLASSES[case["k"]], []
        for n, s, d in _many(case, rng):
            flat = np.zeros((n * C + 63) // 64 * 64, np.int64)
            flat[:n * C] = _counts(n, s, d, k).reshape(-1)
            parts.append(flat)
        return np.concatenate(parts)
    n, s, d = _arcs(case, rng)
    if case["k"] == 34:
        return [_counts(n, s, d, 3), _counts(n, s, d, 4)]
    return _counts(n, s, d, case["k"], edges=case["do"] == "edges", undirected=case["do"] == "undirected")
