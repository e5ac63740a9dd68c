"""Exact edge sampling where its draws change over: half a wave per draw (an odd
number of draws), the tile sums of a chunk four a lane (one tile, a last chunk
of a few), rows of 8 | 9 coordinates, not a
multiple of 4, and the fused (d <= 64) and the sorted draws (d > 64).  A draw's
target, from the documented uniform, has to lie in the interval that the fp64
row gives its pick, within the fp32 rounding of the tile sums (1e-5 of the row);
unaligned rows give the same draws bit for bit."""
import numpy as np
import pytest

from tests.gpu_util import announce, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def stag():
    import torch
    assert torch.cuda.is_available()
    import paper_2407_07096_amd as s
    s.load()
    return s


@pytest.mark.parametrize("n,d,s", [(2, 3, 1), (31, 8, 3), (33, 9, 1), (129, 16, 5), (1000, 30, 3), (4095, 64, 1),
                                   (4129, 65, 3), (301, 130, 3), (8200, 12, 1), (200, 300, 1)])
def test_draws_follow_the_rows(stag, n, d, s):
    import torch
    rng = np.random.default_rng(n + d)
    X = rng.normal(size=(n, d)).astype(np.float32)
    a = 0.3 / d
    announce(f"draws n={n} d={d} s={s}")
    src, dst, w, deg = stag.simgraph_sample(to_dev(X), a, samples_per_node=s, seed=77, mode="exact")
    got = [t.cpu().numpy() for t in (src, dst, w, deg)]
    buf = torch.empty(X.size + 1, dtype=torch.float32, device="cuda")
    buf[1:] = torch.from_numpy(X.reshape(-1)).cuda()
    again = stag.simgraph_sample(buf[1:].view(X.shape), a, samples_per_node=s, seed=77, mode="exact")
    for u, v in zip(got, again):
        assert np.array_equal(u, v.cpu().numpy())
    src, dst, w, deg = got
    assert np.array_equal(src, np.repeat(np.arange(n), s)) and np.all(dst != src)
    assert dst.min() >= 0 and dst.max() < n
    K = np.exp(-a * ((X[:200].astype(np.float64)[:, None] - X.astype(np.float64)[None]) ** 2).sum(-1)) \
        if n * d < 200000 else None
    if K is not None:
        rows = np.arange(len(K))
        K[rows, rows] = 0.0
        cum = np.cumsum(K, axis=1)
        # the uniform of a draw is the documented stream's; its target has to lie
        # in the picked row's interval, up to the tile sums' fp32 rounding
        e = np.arange(len(K) * s)
        u = np.array([oracle_uniform(77, int(i // s), int(i % s)) for i in e])
        target = u * cum[src[e], -1]
        hi = cum[src[e], dst[e]]
        lo = hi - K[src[e], dst[e]]
        slack = 1e-5 * cum[src[e], -1]
        assert np.all(target >= lo - slack) and np.all(target <= hi + slack)


def _mix(z):
    m = (1 << 64) - 1
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & m
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & m
    return z ^ (z >> 31)


def oracle_uniform(seed, i, r):
    m = (1 << 64) - 1
    ds = _mix(_mix(_mix(seed ^ 0x44524157) ^ i))
    return (_mix((ds + (r + 1) * 0x9E3779B97F4A7C15) & m) >> 11) * 2.0 ** -53
