"""Exact edge sampling on both sides of the line between the fused and the
sorted draws (d > 64: 7 MiB of data), and over several chunks on each: the target
of a draw has to lie in the interval that the fp64 row gives its pick, within
the fp32 rounding of the tile sums (1e-5 of the row)."""
import numpy as np
import pytest

from tests.gpu_util import announce, to_dev
from tests.test_gpu_draw_rows import oracle_uniform, stag  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,s", [(4129, 65, 3), (7168, 256, 1), (7169, 256, 1), (32300, 65, 1), (9000, 250, 2),
                                   (8129, 260, 3)])
def test_draws_follow_the_rows(stag, n, d, s):  # noqa: F811
    rng = np.random.default_rng(n + d)
    X = rng.normal(size=(n, d)).astype(np.float32)
    a = 0.3 / d
    announce(f"draw paths n={n} d={d} s={s}")
    src, dst, w, deg = (t.cpu().numpy() for t in stag.simgraph_sample(to_dev(X), a, samples_per_node=s, seed=77,
                                                                      mode="exact"))
    assert np.array_equal(src, np.repeat(np.arange(n), s)) and np.all(dst != src)
    rows = np.concatenate([np.arange(60), np.arange(n // 2, n // 2 + 60), np.arange(n - 60, n)])
    Xd = X.astype(np.float64)
    for i in rows:
        K = np.exp(-a * ((Xd - Xd[i]) ** 2).sum(1))
        K[i] = 0.0
        cum = np.cumsum(K)
        for r in range(s):
            j, target = dst[i * s + r], oracle_uniform(77, int(i), r) * cum[-1]
            slack = 1e-5 * cum[-1]
            assert cum[j] - K[j] - slack <= target <= cum[j] + slack, (i, r)
