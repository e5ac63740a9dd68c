"""k-means where its kernels change over: point blocks of 1024 +- 1, the
register paddings of the assignment (1, 2, 4, 8, 16, 24, 32, 48, 64, none), 256
and 257 clusters (listed and accumulated block sums), and more than 1024 blocks
(the seeding scans its block sums in pieces).  Bit-exact against the oracle,
whose order of operations is documented, so there is no tolerance.  The graph
build is checked at runs of empty rows."""
import numpy as np
import pytest

import oracle
from oracle import spectral as ospec
from tests.gpu_util import announce, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def stag():
    import torch
    assert torch.cuda.is_available()
    import paper_2407_07096_amd as s
    s.load()
    return s


@pytest.mark.parametrize("n,dim,k", [(1, 1, 1), (1023, 1, 5), (1024, 2, 64), (1025, 4, 9), (2047, 5, 256),
                                     (2049, 3, 257), (1500, 8, 300), (900, 9, 100), (1200, 17, 30), (1200, 24, 25),
                                     (700, 25, 40), (600, 33, 20), (600, 48, 10), (500, 49, 11), (500, 64, 64),
                                     (500, 65, 7), (300, 1000, 4), (1300, 1, 1200)])
def test_kmeans_edges_bit_exact(stag, n, dim, k):
    rng = np.random.default_rng(n + dim + k)
    P = rng.normal(size=(n, dim)) + 4.0 * rng.integers(0, 3, size=(n, 1))
    announce(f"kmeans n={n} dim={dim} k={k}")
    lab, C, it, seeds = stag.kmeans(to_dev(P), k, seed=k, max_iter=4)
    lo, Co, ito, so = oracle.kmeans(P, k, k, max_iter=4)
    assert np.array_equal(seeds.cpu().numpy(), so) and it == ito
    assert np.array_equal(lab.cpu().numpy(), lo) and np.array_equal(C.cpu().numpy(), Co)


def test_kmeans_more_than_1024_blocks(stag):
    n = 1024 * 1030 + 5
    P = np.random.default_rng(3).normal(size=(n, 1))
    announce(f"kmeans n={n}")
    lab, C, it, seeds = stag.kmeans(to_dev(P), 4, seed=8, max_iter=2)
    lo, Co, ito, so = oracle.kmeans(P, 4, 8, max_iter=2)
    assert np.array_equal(seeds.cpu().numpy(), so) and it == ito
    assert np.array_equal(lab.cpu().numpy(), lo) and np.array_equal(C.cpu().numpy(), Co)


def test_graph_with_runs_of_empty_rows(stag):
    # two cycles of 6 inside 700 vertices, the others isolated (eigenvalue 1):
    # the two zero eigenvalues, then the cycles' 1 - cos(2 pi / 6)
    n = 700
    c = np.arange(6)
    src = np.concatenate([260 + c, 600 + c])
    dst = np.concatenate([260 + (c + 1) % 6, 600 + (c + 1) % 6])
    announce("spectral runs of empty rows")
    lam, U, _ = stag.spectral_embedding(n, to_dev(src.astype(np.int64)), to_dev(dst.astype(np.int64)),
                                        to_dev(np.ones(12)), 6)
    lo, _ = ospec.spectral_embedding(n, src, dst, np.ones(12), 7)
    np.testing.assert_allclose(lam.cpu().numpy(), lo[:6], atol=1e-9)


def test_embedding_when_the_cholesky_factor_breaks_down(stag):
    # nine disjoint edges with self-loops of weight 1e-13: eigenvalues 0 and
    # 2 - 4e-13, nine of each; the block of 16 holds some of the upper ones, so
    # the filter's interval has length 4e-13 and its images differ by 1e25 in
    # size: the block's Gram matrix is singular to rounding
    n = 18
    e = np.arange(0, n, 2)
    src = np.concatenate([e, np.arange(n)])
    dst = np.concatenate([e + 1, np.arange(n)])
    w = np.concatenate([np.ones(len(e)), np.full(n, 1e-13)])
    announce("spectral cholesky breakdown")
    lam, U, it = stag.spectral_embedding(n, to_dev(src.astype(np.int64)), to_dev(dst.astype(np.int64)), to_dev(w), 8)
    U = U.cpu().numpy()
    assert it >= 1
    np.testing.assert_allclose(lam.cpu().numpy(), 0.0, atol=1e-9)
    np.testing.assert_allclose(U.T @ U, np.eye(8), atol=1e-9)
    np.testing.assert_allclose(np.abs(U[0::2]), np.abs(U[1::2]), atol=1e-7)
