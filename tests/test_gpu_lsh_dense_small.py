"""GPU: walked CKNS indexes with dense levels: segments of few members, and
query batches of few rows, against the oracle and bit for bit against a batch
of whole tiles."""
import numpy as np
import pytest
import torch

import oracle as orc
import paper_2407_07096_amd as stag
import synth
from tests.gpu_util import announce, to_dev

pytestmark = pytest.mark.gpu


# segments from none or one member to past the sampled 64 and 256; one copy and
# several; tables (L = 5 and 36) that do not fill a group
@pytest.mark.parametrize("n,d,kw", [
    (2, 256, dict(k1=1, k2_constant=5, p_offset=0)),
    (65, 131, dict(k1=2, k2_constant=5, p_offset=1)),
    (300, 256, dict(k1=3, k2_constant=9, p_offset=0)),
    (300, 20, dict(k1=2, k2_constant=40, p_offset=1)),
    (900, 784, dict(k1=1, k2_constant=8, p_offset=0)),
])
def test_small_batches_and_segments(n, d, kw):
    X = synth.sparse_uniform(n, d, 60 + n) if d > 128 else synth.sample(synth.mixture(d, 1, 60 + n, sigma=0.3), n, 61)
    a = 0.02 if d <= 128 else 1e-3
    sh = orc.lsh_derive(n, a, eps=0.5, **kw)
    G0, B = synth.e2lsh_randomness(sh["K1"] * sh["J"] * sh["L"] * sh["K"], d, 62)
    m = 150
    Q = np.resize(np.concatenate([X, X[:1] + np.float32(0.01)]), (m, d)).astype(np.float32)
    announce(f"lsh dense small n={n} d={d} {kw}")
    idx = stag.LshIndex(to_dev(X), a, G0=to_dev(G0), b=to_dev(B), seed=3, eps=0.5, **kw)
    S, st = idx.query(to_dev(Q), stats=True)
    for k in (1, 16, 17, 64, 65, 128):
        part, ps = idx.query(to_dev(Q[:k]), stats=True)
        torch.cuda.synchronize()
        assert torch.equal(part.view(torch.int64), S[:k].view(torch.int64)), k
        assert torch.equal(ps["n_cand"], st["n_cand"][:k]) and torch.equal(ps["n_acc"], st["n_acc"][:k]), k
    R, sr = orc.lsh_kde(X, Q, a, G0, B, seed=3, return_stats=True, eps=0.5, **kw)
    assert np.array_equal(st["n_cand"].cpu().numpy(), sr["n_cand"])
    assert np.array_equal(st["n_acc"].cpu().numpy(), sr["n_acc"])
    np.testing.assert_allclose(S.cpu().numpy(), R, rtol=1e-9, atol=0)


# 16, 64 and 128 queries per workgroup, by the number of queries; rows on and
# off 16-byte boundaries
@pytest.mark.parametrize("n,d", [(1500, 132), (1100, 259)])
def test_batches_of_every_tile_height(n, d):
    kw = dict(k1=2, k2_constant=6, p_offset=0)
    X, a = synth.sparse_uniform(n, d, 70 + n), 1e-3
    sh = orc.lsh_derive(n, a, eps=0.5, **kw)
    G0, B = synth.e2lsh_randomness(sh["K1"] * sh["J"] * sh["L"] * sh["K"], d, 71)
    Q = np.concatenate([X[:20], synth.sparse_uniform(25, d, 72)])
    announce(f"lsh dense tile heights n={n} d={d}")
    idx = stag.LshIndex(to_dev(X), a, G0=to_dev(G0), b=to_dev(B), seed=3, eps=0.5, **kw)
    R, sr = orc.lsh_kde(X, Q, a, G0, B, seed=3, return_stats=True, eps=0.5, **kw)
    first = None
    for m in (45, 400, 700, 1000, 1400, 2000, 2800, 4000, 5600, 9000, 20000):
        S, st = idx.query(to_dev(np.resize(Q, (m, d))), stats=True)
        torch.cuda.synchronize()
        S, nc, na = (v.cpu().numpy() for v in (S, st["n_cand"], st["n_acc"]))
        first = S[:45] if first is None else first
        np.testing.assert_allclose(first, R, rtol=1e-9, atol=0)
        rows = np.arange(m) % 45
        assert np.array_equal(S, first[rows]), m
        assert np.array_equal(nc, sr["n_cand"][rows]) and np.array_equal(na, sr["n_acc"][rows]), m
