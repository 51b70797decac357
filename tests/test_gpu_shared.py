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
