"""The CKNS bucket join where its kernel changes over: row widths around the
padded 16, 32, 64 and 128 (aligned rows and padded copies), buckets of one to a
few hundred queries and members (pairs formed directly, one or two query
tiles, several member ranges), chunks where few and where nearly all pairs
survive, and more than 8 tables.  Candidate and accept counts equal the
oracle's, estimates are within the 1e-9 of test_gpu_lsh; a query's estimate is
bit for bit the same alone, in a batch and from an unaligned row."""
import numpy as np
import pytest

from tests.gpu_util import announce
from tests.test_gpu_lsh import _compare, _randomness, stag  # noqa: F401

pytestmark = pytest.mark.gpu


def _points(n, m, d, rng):
    """Tight groups of 1, 5, 40 and the rest (every pair of a group is near),
    and queries in them and apart."""
    c = rng.normal(size=(4, d)) * 4.0
    g = np.repeat(np.arange(4), [1, 5, 40, n - 46])
    X = c[g] + rng.normal(size=(n, d)) * np.array([0.01, 0.05, 0.05, 0.4])[g][:, None]
    h = rng.integers(0, 4, m)
    Q = c[h] + rng.normal(size=(m, d)) * 0.3
    Q[: min(m, n) // 3] = X[rng.permutation(n)[: min(m, n) // 3]]
    return X.astype(np.float32), Q.astype(np.float32)


@pytest.mark.parametrize("n,m,d,k2", [
    (300, 1, 1, 4), (300, 33, 3, 4), (400, 65, 12, 6), (700, 130, 15, 4), (700, 130, 16, 9), (500, 64, 17, 4),
    (500, 31, 32, 20), (500, 97, 33, 4), (900, 200, 64, 4), (400, 40, 65, 9), (400, 70, 100, 4), (300, 66, 128, 4)])
def test_join_shapes(stag, orc, n, m, d, k2):  # noqa: F811
    import torch
    rng = np.random.default_rng(n + m + d)
    X, Q = _points(n, m, d, rng)
    a = 0.5 / d
    announce(f"lsh join n={n} m={m} d={d} k2={k2}")
    kw = dict(k1=2, k2_constant=k2, p_offset=1)
    _compare(stag, orc, X, Q, a, seed=n + d, check_segments=False, **kw)
    sh, G0, B = _randomness(orc, n, d, a, n + d, **kw)
    from tests.gpu_util import to_dev
    idx = stag.LshIndex(to_dev(X), a, G0=to_dev(G0), b=to_dev(B), seed=n + d, **kw)
    S = idx.query(to_dev(Q)).cpu().numpy()
    part = np.concatenate([idx.query(to_dev(Q[:1])).cpu().numpy(), idx.query(to_dev(Q[1:])).cpu().numpy()]) \
        if m > 1 else S
    assert np.array_equal(S, part)
    buf = torch.empty(Q.size + 1, dtype=torch.float32, device="cuda")
    buf[1:] = torch.from_numpy(Q.reshape(-1)).cuda()
    assert np.array_equal(S, idx.query(buf[1:].view(Q.shape)).cpu().numpy())
    idx.close()


@pytest.mark.parametrize("n,d,s", [(300, 4, 3), (400, 8, 2), (400, 9, 3), (500, 30, 5), (600, 64, 64), (500, 100, 3),
                                   (500, 129, 4), (400, 200, 3), (300, 258, 2)])
def test_draws_from_join_and_walk(stag, orc, n, d, s):  # noqa: F811
    """Edge draws after the join (d <= 128: the levels it flags) and after the
    walk, with rows read one lane each (d <= 8) and by quads, against the
    oracle as in test_gpu_simgraph."""
    from tests.gpu_util import to_dev
    rng = np.random.default_rng(7 * n + d)
    X, _ = _points(n, 1, d, rng)
    a = 0.5 / d
    kw = dict(eps=0.5, k1=2, k2_constant=4)
    announce(f"lsh draws n={n} d={d} s={s}")
    sh, G0, B = _randomness(orc, n, d, a, 31, **kw)
    got = stag.simgraph_sample(to_dev(X), a, samples_per_node=s, mode="lsh", seed=77, G0=to_dev(G0), b=to_dev(B),
                               lsh_seed=0, **kw)
    src, dst, w, deg = (t.cpu().numpy() for t in got)
    osrc, odst, ow, odeg, mg = orc.simgraph_lsh(X, a, s, 77, G0, B, lsh_seed=0, **kw)
    assert np.array_equal(src, osrc)
    assert np.allclose(deg, odeg, rtol=1e-9)
    same = dst == odst
    assert np.all(same[mg > 1e-9])
    ok = same & (dst >= 0)
    assert np.allclose(w[ok], ow[ok], rtol=1e-9)
