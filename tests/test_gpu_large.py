"""Hub roots in graphs with many vertices: every layout of the depth-2 vertices' index and both ways of
crediting end vertices against the CPU oracle, and a cost and scratch that do not grow with n."""
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


def _hub(slots, kids, leaves, seed):
    """A hub with `slots` neighbours, some joined, each with `kids` children, each with `leaves` leaves;
    one child in eight has a second parent, one in eight is joined to the child before it, and one
    leaf in five has a second child as its neighbour."""
    rng = np.random.default_rng(seed)
    parts = [np.stack([np.zeros(slots, np.int64), 1 + np.arange(slots)], 1)]
    parts.append(1 + rng.integers(0, slots, (slots, 2)))
    c0, nc = 1 + slots, slots * kids
    c = np.arange(nc)
    parts.append(np.stack([1 + c // max(kids, 1), c0 + c], 1))
    q = c[c % 8 == 0]
    parts.append(np.stack([1 + rng.integers(0, slots, len(q)), c0 + q], 1))
    q = c[(c % 8 == 4)]
    parts.append(np.stack([c0 + q, c0 + q - 1], 1))
    l0, nl = c0 + nc, nc * leaves
    x = np.arange(nl)
    parts.append(np.stack([c0 + x // max(leaves, 1), l0 + x], 1))
    q = x[x % 5 == 0]
    if nl:
        parts.append(np.stack([c0 + rng.integers(0, nc, len(q)), l0 + q], 1))
    e = np.concatenate(parts)
    e = np.unique(np.sort(e[e[:, 0] != e[:, 1]], axis=1), axis=0)
    way = rng.integers(0, 5, len(e))
    fwd, back = e[way != 1], e[(way == 1) | (way == 4)][:, ::-1]
    a = np.concatenate([fwd, back])
    return l0 + nl, a[:, 0].astype(np.int32), a[:, 1].astype(np.int32)


@pytest.mark.parametrize("slots,kids,leaves,pad,lone", [
    (40, 3, 1, 0, 66_000),          # bitmap in LDS; end vertices path by path
    (40, 3, 0, 0, 300_000),         # hash in LDS, no end vertices
    (40, 0, 0, 0, 300_000),         # no depth-2 vertices
    (100, 100, 1, 0, 1_200_000),    # hash in LDS, too long for bitmaps of a slot's children
    (175, 130, 1, 0, 1_500_000),    # hash in scratch
    (175, 130, 8, 900_000, 0),      # hash in scratch; end vertices once each, in two windows of ranks
    (175, 130, 1, 0, 400_000),      # bitmap in scratch
    (175, 130, 8, 0, 380_000),      # bitmap in scratch; end vertices once each
    (1300, 5, 1, 0, 700_000),       # many slots: little LDS left in phases B and E
])
def test_large_layouts(v, slots, kids, leaves, pad, lone):
    """pad: vertices joined in pairs, which rank before the leaves; lone: vertices of degree 0."""
    import torch
    n, src, dst = _hub(slots, kids, leaves, slots + kids)
    a = np.arange(0, pad, 2, dtype=np.int32)
    s, d = np.concatenate([src + pad, a]), np.concatenate([dst + pad, a + 1])
    print(f"large slots={slots} kids={kids} leaves={leaves} pad={pad} lone={lone} n={n + pad + lone}", flush=True)
    G = v.Graph(n + pad + lone, s, d)
    want, tot = oracle.count(n, src, dst, 4)
    for out3, out4 in ((None, v.count(G, 4)), v.count34(G)):
        assert (_np(out4[pad:pad + n]) == want).all()
        assert int(out4.sum()) == int(out4[pad:pad + n].sum())
        assert sum(list(v.shape_counts(G).values())[2:]) == int(tot.sum())
        del out4, out3
        torch.cuda.empty_cache()


def test_hub_cost_does_not_grow_with_n(v):
    """500 hubs with trees below them: vertices of degree 0 change nothing but the rows to write."""
    n, src, dst = 500 * 201, [], []
    r = np.repeat(np.arange(500), 40)
    c = 500 + np.arange(500 * 40)
    g, e = np.repeat(c, 4), 500 + 500 * 40 + np.arange(500 * 160)
    src, dst = np.concatenate([r, g]).astype(np.int32), np.concatenate([c, e]).astype(np.int32)
    ms = []
    for m in (n, 2_000_000):
        G = v.Graph(m, src, dst)
        out = v.count(G, 4)
        times = []
        for _ in range(5):
            v.count(G, 4, out)
            times.append(float(v.kernel_times(G)[2]))
        ms.append(min(times))
        del out, G
    print("hub kernel ms", ms, flush=True)
    assert ms[1] < 4 * ms[0] + 0.2


def test_hub_scratch_does_not_grow_with_n(v):
    """A request's scratch is what its hub roots' neighbourhoods take, so that a small budget does."""
    import torch
    src = np.repeat(np.arange(300), 40).astype(np.int32)
    dst = (300 + np.arange(300 * 40)).astype(np.int32)
    n = 4_000_000
    G = v.Graph(n, src, dst)
    out = torch.empty((n, 13), dtype=torch.int64, device="cuda")
    srv = v.Server(32 << 20, 2)
    srv.wait(srv.submit(G, 3, out))
    srv.wait(srv.submit(G, 3, out))     # its bins are known: checked at submission
    want = oracle.count(300 * 41, src, dst, 3)[0]
    assert (_np(out[:300 * 41]) == want).all()
    srv.close()


def test_ranges_without_hub_roots(v):
    """A range of ranks that holds no hub root launches no hub path (vdmc_kernel_times: -1), and ranges
    of a few roots, a part of the ranks or none add up to the whole count."""
    import torch
    n, src, dst = _hub(100, 20, 1, 5)
    for lone in (0, 100_000):
        G = v.Graph(n + lone, src, dst)
        want = v.count(G, 4)
        off, adj, _ = G.export()
        deg = np.diff(off)
        hubs = [r for r in np.nonzero(deg >= 32)[0] if np.count_nonzero(adj[off[r]:off[r + 1]] >> 2 > r) >= 32]
        assert hubs and want[:n].any()
        out = torch.zeros_like(want)
        first = 600                                  # past every hub root and its part of the ranks
        assert max(hubs) < first - (n + lone) // 256
        cuts = sorted([0, hubs[0] + 1, hubs[0] + 2, hubs[-1] + 1, first, first, n // 2, n + lone])
        for lo, hi in zip(cuts[:-1], cuts[1:]):
            v.count_range(G, 4, out, lo, hi, accumulate=True)
            torch.cuda.synchronize()
            ran = v.kernel_times(G)[1] >= 0
            print(f"range {lo}..{hi} hub path {ran}", flush=True)
            if lo >= first:
                assert not ran, (lo, hi)
            if any(lo <= h < hi for h in hubs):
                assert ran, (lo, hi)
        assert torch.equal(out, want), lone
