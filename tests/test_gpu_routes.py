"""GPU parity at the edges of each kernel's range: sizes at which a root, a graph or a launch
takes another kernel or another layout of one, against the CPU oracle, every count equal."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def v():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2201_11655_amd as v
    v.load()
    return v


def _np(t):
    import torch
    torch.cuda.synchronize()
    return t.cpu().numpy().view(np.uint64)


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _er(n, deg, seed):
    rng = np.random.default_rng(seed)
    m = int(n * deg)
    return n, rng.integers(0, n, m).astype(np.int32), rng.integers(0, n, m).astype(np.int32)


def _join(parts):
    """Disjoint union of (n, src, dst)."""
    base, src, dst = 0, [], []
    for n, s, d in parts:
        src.append(s + base)
        dst.append(d + base)
        base += n
    return base, np.concatenate(src).astype(np.int32), np.concatenate(dst).astype(np.int32)


def _arcs(edges, rng):
    """Each pair as one arc either way or, one in five, as both."""
    e = np.asarray(edges, np.int64)
    way = rng.integers(0, 5, len(e))
    fwd, back = e[way != 1], e[(way == 1) | (way == 4)][:, ::-1]
    a = np.concatenate([fwd, back])
    return a[:, 0].astype(np.int32), a[:, 1].astype(np.int32)


def _root(d, entries, seed):
    """A graph with a root of d higher neighbours whose rows above it have `entries` entries:
    the root hangs below a clique of larger degrees, each neighbour has children of its own and
    some of them are joined in pairs."""
    rng = np.random.default_rng(seed)
    per = -(-entries // d)
    h = max(per + 3 - d, 1)                       # lower-ranked neighbours of the root
    edges = [(i, j) for i in range(h) for j in range(i)]
    nxt = h + 1
    edges += [(i, h) for i in range(h)]
    for i in range(h):                            # pendants that keep the clique above the root
        for _ in range(d + 4):
            edges.append((i, nxt))
            nxt += 1
    slots = list(range(nxt, nxt + d))
    nxt += d
    edges += [(h, s) for s in slots]
    kids = []
    for q in range(entries):
        edges.append((slots[q % d], nxt))
        kids.append(nxt)
        nxt += 1
    for i in range(0, len(kids) - 1, 3):          # adjacent children, of one slot or two
        j = (i * 7 + 1) % len(kids)
        edges.append((kids[i], kids[j if j != i else i + 1]))
    s, t = _arcs(edges, rng)
    return nxt, s, t


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("threshold", [32, 1 << 20])
def test_light_roots(v, threshold, batch):
    """Sizes of k_light (8 and 32 slots; 96, 384 and 3072 slots and entries) and their neighbours."""
    parts = [_root(d, total - d, 100 * d + total)
             for d, total in ((1, 3), (8, 96), (8, 97), (9, 60), (31, 384), (31, 385), (31, 3072), (31, 3073),
                              (32, 384), (32, 3072), (33, 400))]
    n, src, dst = _join(parts)
    G = v.Graph(n, src, dst)
    assert v.load().vdmc_set_hub_threshold(G.handle, threshold) == 0
    for k in (3, 4):
        _say(f"light k={k} n={n} m={len(src)} threshold={threshold} batch={batch}")
        want, tot = oracle.count(n, src, dst, k)
        if batch:
            got = v.count_batch([G, v.Graph(*_er(1500, 3, 5))], k)[0]
        else:
            got = v.count(G, k)
        assert (_np(got) == want).all(), (k, threshold)
        sc = list(v.shape_counts(G).values())
        assert sum(sc[:2] if k == 3 else sc[2:]) == int(tot.sum())


def _hub(slots, kids, seed, extra=0):
    """A hub with `slots` neighbours, each with `kids` children; one child in four has a second
    parent or an end vertex, `extra` of them are joined to 20 slots."""
    rng = np.random.default_rng(seed)
    edges = [(0, 1 + i) for i in range(slots)]
    edges += [(1 + int(a), 1 + int(b)) for a, b in rng.integers(0, slots, (slots, 2)) if a != b]
    nxt = 1 + slots
    for i in range(slots):
        for q in range(kids):
            edges.append((1 + i, nxt))
            if q % 8 == 0:
                edges.append((nxt, 1 + int(rng.integers(0, slots))))
            elif q % 8 == 4:
                edges.append((nxt, nxt - 1))
            nxt += 1
    for x in range(extra):
        for i in rng.permutation(slots)[:20]:
            edges.append((nxt, 1 + int(i)))
        nxt += 1
    edges = sorted({(min(a, b), max(a, b)) for a, b in edges if a != b})
    s, t = _arcs(edges, rng)
    return nxt, s, t


@pytest.mark.parametrize("slots,kids,extra,pad", [
    (40, 3, 12, "none"),         # compact rows, bitmaps of a slot's children, index in LDS
    (40, 3, 12, "isolated"),     # no room for compact rows; the index in scratch memory
    (40, 3, 12, "pairs"),        # end vertices in a second window of ranks
    (175, 130, 3, "none"),       # 22750 depth-2 vertices: filter and search instead of bitmaps
    (1300, 0, 2, "none"),        # 64-bit compact rows
])
def test_hub_layouts(v, slots, kids, extra, pad):
    import torch
    n, src, dst = _hub(slots, kids, slots + kids, extra)
    # padding changes no count: vertices of degree 0, or pairs that rank before the leaves
    add = {"none": 0, "isolated": 600_000, "pairs": 900_000}[pad]
    s, d = src, dst
    if pad == "pairs":
        a = np.arange(0, add, 2, dtype=np.int32)
        s, d = np.concatenate([src + add, a]), np.concatenate([dst + add, a + 1])
    first = add if pad == "pairs" else 0
    _say(f"hub slots={slots} kids={kids} extra={extra} pad={pad} n={n + add}")
    G = v.Graph(n + add, s, d)
    for k in (3, 4):
        want, tot = oracle.count(n, src, dst, k)
        out = v.count(G, k)
        assert (_np(out[first:first + n]) == want).all(), k
        assert int(out.sum()) == int(out[first:first + n].sum())
        sc = list(v.shape_counts(G).values())
        assert sum(sc[:2] if k == 3 else sc[2:]) == int(tot.sum())
        del out
    torch.cuda.empty_cache()


def test_whole_graphs(v):
    """k_small: counters of every class or of some, arc bits or none, a triangle queue that
    overflows or not, the largest n, one vertex."""
    cases = [_er(20, 8, 1), _er(60, 30, 2), _er(158, 8, 3), _er(170, 12, 4), _er(230, 20, 5), _er(420, 7, 6),
             _er(500, 8, 7), _er(500, 7.9, 8), _er(620, 1.5, 9), _er(1, 0, 10), _er(3, 4, 11),
             _join([_root(1, 3, 12), _root(2, 4, 13)]), _hub(120, 1, 14, 5)]
    for k in (3, 4):
        _say(f"whole graphs k={k}")
        Gs = [v.Graph(*c) for c in cases]
        for c, G, o in zip(cases, Gs, v.count_batch(Gs, k)):
            want, tot = oracle.count(*c, k)
            assert (_np(o) == want).all(), (k, c[0], len(c[1]))
            sc = list(v.shape_counts(G).values())
            assert sum(sc[:2] if k == 3 else sc[2:]) == int(tot.sum()), (k, c[0])


@pytest.mark.parametrize("case", ["dense40", "er300", "hub", "roots", "planes_full", "too_many_vertices"])
def test_edge_sets(v, case):
    """Per-edge counts: dense, a hub with many parents below it, the largest n of the bit planes
    and one more (per-set kernel)."""
    n, src, dst = {"dense40": lambda: _er(40, 15, 1), "er300": lambda: _er(300, 6, 2),
                   "hub": lambda: _hub(90, 4, 3, 9),
                   "roots": lambda: _join([_root(1, 3, 4), _root(9, 60, 5), _root(33, 300, 6)]),
                   "planes_full": lambda: _hub(70, 2, 7, 4),
                   "too_many_vertices": lambda: _hub(70, 2, 7, 4)}[case]()
    full = {"planes_full": 65536, "too_many_vertices": 65537}.get(case)
    if full:   # the graph's ids at the end, isolated vertices before
        src, dst, n = src + (full - n), dst + (full - n), full
    G = v.Graph(n, src, dst)
    lo, hi = v.edge_list(G)
    for k in (3, 4):
        _say(f"edges {case} k={k} n={n}")
        olo, ohi, want = oracle.count_edges(n, src, dst, k)
        assert (lo == olo).all() and (hi == ohi).all()
        assert (_np(v.count_edges(G, k)) == want).all(), (case, k)
        sc = list(v.shape_counts(G).values())
        tot = oracle.count(n, src, dst, k)[1] if not full else None
        if tot is not None:
            assert sum(sc[:2] if k == 3 else sc[2:]) == int(tot.sum())


@pytest.mark.parametrize("n,pad", [(70, 0), (512, 0), (513, 0), (900, 11000), (900, 16384 - 900), (900, 16385 - 900)])
def test_five_layouts(v, n, pad):
    """k = 5: LDS counters up to 512 vertices, a hash that many classes fill, workgroups of 256
    threads where the bit planes are long, and graphs past them."""
    import torch
    n, src, dst = _er(n, 12 if n == 70 else 1.4, n)
    want, tot = oracle.count(n, src, dst, 5)
    _say(f"five n={n} pad={pad}")
    G = v.Graph(n + pad, src + pad, dst + pad)
    out = v.count(G, 5)
    assert (_np(out[pad:]) == want).all()
    assert int(out[:pad].sum()) == 0
    assert sum(v.shape_counts5(G).values()) == int(tot.sum())
    del out
    torch.cuda.empty_cache()
