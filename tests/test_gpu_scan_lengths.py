"""Offsets of near-neighbour lists at the lengths where the prefix sum under
them changes over: one block of 1024 and its neighbours, many blocks, and past
the 4096 blocks whose totals a block still adds itself.  The lists are those of
a few queries over and over, so the offsets have to be the running sums of
their counts, exactly."""
import numpy as np
import pytest

import synth
from tests.gpu_util import announce, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def stag():
    import torch
    assert torch.cuda.is_available()
    import paper_2407_07096_amd as s
    s.load()
    return s


@pytest.mark.parametrize("m", [1, 2, 1023, 1024, 1025, 2048, 100003, 4096 * 1024, 4096 * 1024 + 1])
def test_offsets_are_running_sums(stag, m):
    import torch
    rng = np.random.default_rng(5)
    X = rng.normal(size=(40, 2)).astype(np.float32)
    Q = (rng.normal(size=(37, 2)) * 2.0).astype(np.float32)
    G, b = synth.e2lsh_randomness(3, 2, 9)
    announce(f"scan m={m}")
    t = stag.E2LSHTable(to_dev(X), to_dev(G), to_dev(b), 3, 1)
    off, _ = t.near_neighbours(to_dev(Q))
    counts = np.diff(off.cpu().numpy())
    many = to_dev(Q).repeat((m + 36) // 37, 1)[:m].contiguous()
    got, idx = t.near_neighbours(many)
    want = np.concatenate([[0], np.cumsum(np.tile(counts, (m + 36) // 37)[:m])])
    assert counts.sum() > 0
    assert np.array_equal(got.cpu().numpy(), want) and idx.numel() == want[-1]
    torch.cuda.synchronize()
    t.close()
