"""The KDE-tree sampler where its row reading changes: d = 8 | 9 (a lane per row,
a quad per rows), multiples of 4 and not, around pieces of 16 and 32
coordinates, at every row alignment of a float, and with 8, 16 and 32 lanes per
child (draws that do not fill the last wave).  Against the oracle under the
margin of test_gpu_tree; the alignments among each other bit for bit."""
import numpy as np
import pytest

from tests.gpu_util import announce
from tests.test_gpu_tree import _compare, _gpu, _valid, stag  # noqa: F401


@pytest.mark.gpu
@pytest.mark.parametrize("n,d,s,t,t_deg", [
    (131, 1, 3, 8, 40), (200, 4, 5, 9, 63), (200, 7, 5, 16, 64), (333, 8, 3, 17, 65), (333, 9, 3, 32, 130),
    (100, 12, 1, 8, 128), (101, 16, 1, 16, 30), (203, 17, 3, 32, 200), (150, 20, 7, 8, 64), (150, 31, 1, 8, 64),
    (150, 32, 3, 15, 64), (150, 33, 5, 16, 64), (97, 47, 2, 32, 64), (97, 48, 2, 3, 64), (97, 63, 2, 24, 64),
    (97, 64, 64, 8, 64), (65, 65, 3, 16, 64), (70, 130, 1, 32, 64)])
def test_rows_and_lanes(stag, orc, n, d, s, t, t_deg):  # noqa: F811
    import torch
    X = (np.random.default_rng(n * d).normal(size=(n, d))).astype(np.float32)
    a = 0.4 / d
    announce(f"tree rows n={n} d={d} s={s} t={t} t_deg={t_deg}")
    got = _gpu(stag, X, a, s, t, t_deg, 5 + d)
    _valid(got[0], got[1], n)
    _compare(got, orc.simgraph_tree(X, a, s, t, t_deg, 5 + d))
    buf = torch.empty(X.size + 4, dtype=torch.float32, device="cuda")
    for off in (1, 2, 3):
        buf[off:off + X.size] = torch.from_numpy(X.reshape(-1)).cuda()
        Xd = buf[off:off + X.size].view(X.shape)
        assert Xd.data_ptr() % 16 == 4 * off
        for u, v in zip(got, _gpu(stag, X, a, s, t, t_deg, 5 + d, Xd=Xd)):
            assert np.array_equal(u, v)


def test_draw_quotients():
    # the multiply and shift that replaces e / s, over the whole accepted range
    rng = np.random.default_rng(1)
    for s in list(range(1, 65)) + [65, 100, 1000, 4097, (1 << 20) - 1]:
        l = max(0, (s - 1).bit_length())
        shift = 31 + l
        m = ((1 << shift) + s - 1) // s
        assert m < 1 << 32
        e = np.unique(np.concatenate([rng.integers(0, 2**31 - 1, 2000), np.arange(200), 2**31 - 2 - np.arange(200),
                                      s * rng.integers(0, (2**31 - 2) // s + 1, 500)])).astype(np.uint64)
        e = e[e < 2**31 - 1]
        assert all((int(x) * m) >> shift == int(x) // s for x in e)
