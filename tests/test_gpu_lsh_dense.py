"""GPU: walked CKNS indexes whose levels are dense (pairs formed tile by tile)
against the oracle: candidate and accept counts equal, values within 1e-9 (only
the order of fp64 sums differs), draws as the oracle's."""
import numpy as np
import pytest
import torch

import oracle as orc
import paper_2407_07096_amd as stag
import synth
from tests.gpu_util import announce, to_dev

pytestmark = pytest.mark.gpu


def _setup(n, d, seed, **kw):
    # sparse rows are nearly equidistant: one level takes every pair
    X = synth.sparse_uniform(n, d, seed) if d > 128 else synth.sample(synth.mixture(d, 1, seed, sigma=0.3), n, seed)
    a = 0.02 if d <= 128 else 1e-3
    sh = orc.lsh_derive(n, a, **kw)
    G0, B = synth.e2lsh_randomness(sh["K1"] * sh["J"] * sh["L"] * sh["K"], d, seed + 1)
    return X, a, G0, B


# members around a 128-row tile, one query and one past a tile, rows that start
# off 16 bytes (d = 131), tables past one batch of 8 (L = 9), the walked path of
# narrow rows (L > 32), several copies
@pytest.mark.parametrize("n,d,m,kw", [
    (520, 256, 1, dict(k1=1, k2_constant=8, p_offset=0)),
    (1100, 131, 129, dict(k1=2, k2_constant=9, p_offset=1)),
    (3001, 785, 130, dict(k1=1, k2_constant=8, p_offset=1)),
    (600, 20, 140, dict(k1=2, k2_constant=40, p_offset=0)),
])
def test_dense_levels_match_oracle(n, d, m, kw):
    X, a, G0, B = _setup(n, d, 500 + n, eps=0.5, **kw)
    Q = np.concatenate([X[:1], synth.sparse_uniform(m, d, 9) if d > 128 else X[-m:] + 0.01])[:m].astype(np.float32)
    announce(f"lsh dense n={n} d={d} m={m} {kw}")
    idx = stag.LshIndex(to_dev(X), a, G0=to_dev(G0), b=to_dev(B), seed=3, eps=0.5, **kw)
    S, st = idx.query(to_dev(Q), stats=True)
    one = idx.query(to_dev(Q[-1:]))
    torch.cuda.synchronize()
    R, sr = orc.lsh_kde(X, Q, a, G0, B, seed=3, return_stats=True, eps=0.5, **kw)
    assert np.array_equal(st["n_cand"].cpu().numpy(), sr["n_cand"])
    assert np.array_equal(st["n_acc"].cpu().numpy(), sr["n_acc"])
    np.testing.assert_allclose(S.cpu().numpy(), R, rtol=1e-9, atol=0)
    np.testing.assert_allclose(st["S_copies"].cpu().numpy(), sr["S_copies"], rtol=1e-9, atol=1e-300)
    assert torch.equal(one, S[-1:])  # whatever the batch


@pytest.mark.parametrize("n,d,s,kw", [
    (1030, 300, 7, dict(k1=2, k2_constant=8, p_offset=1)),
    (700, 24, 17, dict(k1=1, k2_constant=36, p_offset=0)),
])
def test_dense_draws_match_oracle(n, d, s, kw):
    X, a, G0, B = _setup(n, d, 900 + n, eps=0.5, **kw)
    announce(f"simgraph lsh dense n={n} d={d} {kw}")
    src, dst, w, deg = stag.simgraph_sample(to_dev(X), a, s, mode="lsh", seed=41, eps=0.5, G0=to_dev(G0), b=to_dev(B),
                                            lsh_seed=2, **kw)
    torch.cuda.synchronize()
    osrc, odst, ow, odeg, mg = orc.simgraph_lsh(X, a, s, 41, G0, B, lsh_seed=2, eps=0.5, **kw)
    assert np.array_equal(src.cpu().numpy(), osrc)
    np.testing.assert_allclose(deg.cpu().numpy(), odeg, rtol=1e-9)
    same = dst.cpu().numpy() == odst
    assert np.all(same[mg > 1e-9]) and same.mean() > 0.99
    np.testing.assert_allclose(w.cpu().numpy()[same], ow[same], rtol=1e-9)


# enough queries that their keys are hashed a block of tables at a time; rows on
# and off 16-byte boundaries, a ragged last block of rows and of tables
@pytest.mark.parametrize("n,d,m,kw", [(900, 132, 13400, dict(k1=1, k2_constant=8, p_offset=0)),
                                      (300, 131, 26001, dict(k1=2, k2_constant=3, p_offset=0))])
def test_hashing_of_many_wide_queries(n, d, m, kw):
    X, a, G0, B = _setup(n, d, 1500 + n, eps=0.5, **kw)
    Q = np.resize(synth.sparse_uniform(700, d, 19), (m, d)).astype(np.float32)
    announce(f"lsh wide hashing n={n} d={d} m={m} {kw}")
    idx = stag.LshIndex(to_dev(X), a, G0=to_dev(G0), b=to_dev(B), seed=3, eps=0.5, **kw)
    S, st = idx.query(to_dev(Q), stats=True)
    R, sr = orc.lsh_kde(X, Q[:700], a, G0, B, seed=3, return_stats=True, eps=0.5, **kw)
    S, nc = S.cpu().numpy(), st["n_cand"].cpu().numpy()
    for k in range(0, m, 700):
        c = min(700, m - k)
        assert np.array_equal(nc[k:k + c], sr["n_cand"][:c])
        np.testing.assert_allclose(S[k:k + c], R[:c], rtol=1e-9, atol=0)
