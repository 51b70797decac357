"""Calls that share an output or a device with others: every count equal to the count alone."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def v():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2201_11655_amd as v
    v.load()
    return v


def _fat(n, deg, cap, seed):
    """A fat-tailed graph: arcs between vertices drawn by power-law weights clipped at cap."""
    rng = np.random.default_rng(seed)
    m = int(n * deg)
    w = (np.arange(n) + 1.0) ** -0.9
    c = np.cumsum(np.minimum(w * (m / w.sum()), cap))
    src, dst = (np.minimum(np.searchsorted(c, rng.random(m) * c[-1]), n - 1) for _ in range(2))
    return n, src.astype(np.int32), dst.astype(np.int32)


def test_two_handles_accumulate_into_one_output(v):
    """Two handles of one graph add disjoint rank ranges to one buffer, from two streams at once."""
    import torch
    n, src, dst = _fat(30_000, 6, 200, 3)
    A, B = v.Graph(n, src, dst), v.Graph(n, src, dst)
    cut = 40
    want = v.count(A, 4)
    out = torch.zeros_like(want)
    for g, lo, hi in ((A, 0, cut), (B, cut, n)):   # both have their bins and scratch
        v.count_range(g, 4, out, lo, hi, accumulate=True)
    torch.cuda.synchronize()
    assert torch.equal(out, want)
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    for rep in range(20):
        print(f"two handles, pass {rep}", flush=True)
        out.zero_()
        torch.cuda.synchronize()
        for i in range(4):
            v.count_range(A, 4, out, i * cut // 4, (i + 1) * cut // 4, accumulate=True, stream=sa)
        v.count_range(B, 4, out, cut, n, accumulate=True, stream=sb)
        torch.cuda.synchronize()
        assert torch.equal(out, want), rep


@pytest.mark.parametrize("n,deg,cap", [(8192, 1.5, 400), (8193, 1.5, 400), (8193, 1, 3), (20_000, 2, 40), (65_536, 1, 900),
                                       (65_536, 1, 1500), (65_536, 0.6, 4)])
def test_edge_layouts(v, n, deg, cap):
    """Per-edge counts around the number of vertices from which a pair's arcs are held in a hash, with
    rows that the hash or only the planes hold, and k = 3 around the row from which pairs are counted
    in groups, against the oracle and the counts of the same graph."""
    import oracle
    _, src, dst = _fat(n, deg, cap, n + cap)
    rng = np.random.default_rng(cap)
    if cap <= 4:
        src, dst = (rng.integers(0, n, int(n * deg)).astype(np.int32) for _ in range(2))
    keep = rng.random(len(src)) < (0.15 if cap >= 900 else 1.0)    # the oracle's time
    src, dst = src[keep], dst[keep]
    G = v.Graph(n, src, dst)
    lo, hi = v.edge_list(G)
    for k in (3, 4):
        print(f"edges n={n} deg={deg} cap={cap} k={k} max_deg={G.max_deg}", flush=True)
        olo, ohi, want = oracle.count_edges(n, src, dst, k)
        assert (lo == olo).all() and (hi == ohi).all()
        import torch
        got = v.count_edges(G, k)
        torch.cuda.synchronize()
        assert (got.cpu().numpy().view(np.uint64) == want).all(), k


def test_edge_planes_of_the_largest_graph(v):
    """A star of 1600 leaves in 65536 vertices: rows too long for the hash, bit planes of every vertex."""
    import torch
    n, d = 65_536, 1600
    ids = np.random.default_rng(1).permutation(n)[:d + 1].astype(np.int32)
    G = v.Graph(n, np.full(d, ids[0], np.int32), ids[1:])
    for k, sets in ((3, d - 1), (4, (d - 1) * (d - 2) // 2)):
        out = v.count_edges(G, k)
        torch.cuda.synchronize()
        rows = out.cpu().numpy()
        col = np.flatnonzero(rows.any(axis=0))
        assert len(col) == 1 and (rows[:, col[0]] == sets).all(), k


@pytest.mark.parametrize("n,width,legs", [(512, 1, 0), (513, 1, 0), (5000, 1, 0), (13_000, 2, 0), (14_000, 2, 0),
                                          (10_000, 100, 0), (10_200, 100, 0), (6000, 1, 1)])
def test_five_low_degrees(v, n, width, legs):
    """5-vertex counts of paths, ladders, grids and combs on both sides of the number of pairs from which
    they are counted set by set, alone and beside another graph in a batch, against the oracle."""
    import torch
    import oracle
    rng = np.random.default_rng(n)
    i = np.arange(n - n % (width * (1 + legs)))
    if legs:      # a comb: a path with a leg at every vertex
        path, leg = i[i % 2 == 0], i[i % 2 == 1]
        e = np.concatenate([np.stack([path[:-1], path[1:]], 1), np.stack([path, leg], 1)])
    else:         # rows of `width` vertices
        down = i[:-width]
        e = np.stack([down, down + width], 1)
        if width > 1:
            right = i[i % width < width - 1]
            e = np.concatenate([e, np.stack([right, right + 1], 1)])
    flip = rng.random(len(e)) < 0.5
    e[flip] = e[flip][:, ::-1]
    e = np.concatenate([e, e[rng.random(len(e)) < 0.2][:, ::-1]]).astype(np.int32)
    src, dst = e[:, 0].copy(), e[:, 1].copy()
    want, tot = oracle.count(n, src, dst, 5)
    G = v.Graph(n, src, dst)
    H = v.Graph(60, rng.integers(0, 60, 200), rng.integers(0, 60, 200))
    hb = v.count(H, 5).clone()
    print(f"five low degrees n={n} width={width} legs={legs} pairs={G.pairs} max_deg={G.max_deg}", flush=True)
    for outs in ([v.count(G, 5), hb], v.count_batch([G, H], 5)):
        torch.cuda.synchronize()
        assert (outs[0].cpu().numpy().view(np.uint64) == want).all()
        assert sum(v.shape_counts5(G).values()) == int(tot.sum())
        assert torch.equal(outs[1], hb)


def test_threads_with_graphs_of_different_sizes(v):
    """Kernels whose LDS is sized for the graph, launched from several threads for different graphs at
    once: every call succeeds and every count is that of the call alone."""
    import threading
    import torch
    rng = np.random.default_rng(11)
    jobs = []
    for n, deg in ((300, 3.0), (7000, 1.5), (60, 4.0), (450, 6.0), (2500, 2.0), (700, 0.8)):
        G = v.Graph(n, rng.integers(0, n, int(n * deg)), rng.integers(0, n, int(n * deg)))
        jobs.append((G, lambda G, s: v.count_edges(G, 4, stream=s)))
        jobs.append((G, lambda G, s: v.count_edges(G, 3, stream=s)))
        if n <= 700:
            jobs.append((G, lambda G, s: v.count_batch([G], 4, stream=s)[0]))
            jobs.append((G, lambda G, s: v.count(G, 5, stream=s)))
    want = []
    for G, f in jobs:
        want.append(f(G, None).clone())
    torch.cuda.synchronize()
    bad = []

    def work(t):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for rep in range(60):
                i = (t * 5 + rep * (2 * t + 1)) % len(jobs)
                try:
                    got = f_run(i, s)
                    s.synchronize()
                    if not torch.equal(got, want[i]):
                        bad.append((t, i, "counts differ"))
                except v.VdmcError as e:
                    bad.append((t, i, str(e)))

    def f_run(i, s):
        G, f = jobs[i]
        return f(G, s)

    ts = [threading.Thread(target=work, args=(t,)) for t in range(6)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad, bad[:5]


def test_first_batches_beside_other_calls(v):
    """A batch's first call captures its launches; calls on other streams for graphs whose last call was
    on the batch's stream go on meanwhile."""
    import threading
    import torch
    rng = np.random.default_rng(12)
    G = v.Graph(200, rng.integers(0, 200, 600), rng.integers(0, 200, 600))
    Hs = [v.Graph(300, rng.integers(0, 300, 900), rng.integers(0, 300, 900)) for _ in range(16)]
    want_g, want_h = v.count(G, 4).clone(), [v.count(H, 3).clone() for H in Hs]
    outs = [torch.empty_like(want_g) for _ in range(300)]
    first = [torch.empty_like(w) for w in want_h]
    torch.cuda.synchronize()
    bad, done = [], threading.Event()

    def batches():
        s = torch.cuda.Stream()
        try:
            for o in outs:   # another output: another batch to capture
                for H, f in zip(Hs, first):
                    v.count(H, 3, f, stream=s)
                v.count_batch([G], 4, outs=[o], stream=s)
        except v.VdmcError as e:
            bad.append(str(e))
        done.set()

    def others(part):
        s = torch.cuda.Stream()
        got = [torch.empty_like(w) for w in want_h]
        torch.cuda.synchronize()
        try:
            while not done.is_set():
                for i in list(part) * 8:
                    v.count(Hs[i], 3, got[i], stream=s)
                s.synchronize()
            for i in part:
                if not torch.equal(got[i], want_h[i]):
                    bad.append(f"counts of graph {i} differ")
        except v.VdmcError as e:
            bad.append(str(e))

    ts = [threading.Thread(target=batches)] + [threading.Thread(target=others, args=(range(k, 16, 3),)) for k in range(3)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    torch.cuda.synchronize()
    assert not bad, bad[:3]
    for o in outs:
        assert torch.equal(o, want_g)


def test_tuner_leaves_what_no_launch_uses(v):
    """Threads per root and workgroups per CU are the per-set kernel's: a batch without roots of its
    keeps their defaults, and is counted as before tuning; one with such roots is tuned over all."""
    import torch
    rng = np.random.default_rng(13)
    Gs = [v.Graph(n, rng.integers(0, n, 3 * n), rng.integers(0, n, 3 * n)) for n in (60, 1500, 1800)]
    want = [o.clone() for o in v.count_batch(Gs, 3)]
    before = v.tuned_choice(Gs, 3)
    v.tune(Gs, 3)
    after = v.tuned_choice(Gs, 3)
    print(f"tuned {before} -> {after}", flush=True)
    assert after["tuned"] and not before["tuned"]
    for key in ("threads_per_root", "workgroups_per_cu"):
        assert after[key] == before[key], key
    star = v.Graph(1500, np.zeros(60, np.int32), np.arange(1, 61, dtype=np.int32))
    v.set_hub_threshold(star, 1 << 30)      # 60 higher neighbours: neither the hub nor the light-root kernel's
    with_star = Gs + [star]
    want.append(v.count(star, 3).clone())
    v.tune(with_star, 3)
    for batch in (Gs, with_star):
        got = v.count_batch(batch, 3)
        torch.cuda.synchronize()
        for a, b in zip(got, want):
            assert torch.equal(a, b)


@pytest.mark.parametrize("threshold", [32, 1 << 20])
def test_every_graph_of_a_mixed_batch(v, threshold):
    """Batches whose root tables hold roots of every size from several graphs: the counts and the shape
    counters of each, also where a workgroup goes from one graph to the next and back, against the
    oracle."""
    import oracle
    import torch
    import test_gpu_routes as routes
    roots = [routes._root(d, total - d, 7 * d + total) for d, total in
             ((1, 3), (8, 96), (9, 60), (31, 384), (31, 385), (32, 3072), (33, 400))]
    graphs = [_fat(1500, 3, 60, 1), routes._join(roots), routes._er(1100, 4, 2), routes._join(roots[::-1]),
              _fat(2300, 2, 40, 3), routes._er(90, 3, 4)]
    Gs = [v.Graph(*g) for g in graphs]
    for G in Gs:
        v.set_hub_threshold(G, threshold)
    for k in (3, 4):
        print(f"mixed batch k={k} threshold={threshold}", flush=True)
        for rep in range(2):   # captured, then replayed
            outs = v.count_batch(Gs, k) if rep == 0 else v.count_batch(Gs, k, outs=outs)
            torch.cuda.synchronize()
            for i, (g, G, o) in enumerate(zip(graphs, Gs, outs)):
                want, tot = oracle.count(*g, k)
                assert (o.cpu().numpy().view(np.uint64) == want).all(), (k, rep, i)
                sc = list(v.shape_counts(G).values())
                assert sum(sc[:2] if k == 3 else sc[2:]) == int(tot.sum()), (k, rep, i)
