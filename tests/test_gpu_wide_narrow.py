"""Wide rows (d > 256) in launches of few query tiles that do not share chunks
(the exponential kernel, the no-allocation call, the rescue's passes): they take
32 queries a workgroup instead of 128.  Every value has the bits that the same
query has in a large launch, and lies within its bound of the 64-bit sum."""
import ctypes as C

import numpy as np
import pytest

from tests.gpu_util import announce, to_dev

pytestmark = pytest.mark.gpu


def _data(n, m, d, rng):
    X = rng.random((n, d)) * (rng.random((n, d)) < 0.3)
    Q = rng.random((m, d)) * (rng.random((m, d)) < 0.3)
    Q[5:m:7] = X[rng.integers(0, n, len(Q[5:m:7]))]  # some queries are points, some near them
    Q[6:m:7] = X[rng.integers(0, n, len(Q[6:m:7]))] * 1.001
    return X.astype(np.float32), Q.astype(np.float32)


def _check(orc, X, Q, a, kernel, S, B, rows):
    ref = orc.kde_kernel(X, Q[:rows], a, kernel)
    ok = ref > 1e-280
    assert ok.any() and np.all(np.abs(S[:rows][ok] - ref[ok]) <= B[:rows][ok] * ref[ok])


# rows around a tile, a step (256), a sub-chunk (512) and a chunk (4096)
@pytest.mark.parametrize("n,d", [(31, 257), (300, 300), (520, 784), (4100, 320), (9001, 513), (5000, 1024)])
@pytest.mark.parametrize("form", ["fp32", "fp16_split", "bf16_split"])
def test_exponential_bits_of_a_large_launch(orc, n, d, form):
    import torch
    assert torch.cuda.is_available()
    import paper_2407_07096_amd as stag
    rng = np.random.default_rng(n + d)
    chunks = -(-n // 4096)
    big = 128 * (200 // chunks + 1)  # more than 192 pairs: 128 queries a workgroup
    X, Q = _data(n, big, d, rng)
    a = 3.0 / np.sqrt(d)
    Xd, Qd = to_dev(X), to_dev(Q)
    announce(f"wide narrow exponential n={n} d={d} form={form} m={big} and 1..129")
    S, B = (v.cpu().numpy() for v in stag.kde_exact(Xd, Qd, a, form=form, kernel="exponential", return_bound=True))
    for m in (1, 8, 31, 33, 64, 97, 129):
        s, b = stag.kde_exact(Xd, Qd[:m].contiguous(), a, form=form, kernel="exponential", return_bound=True)
        assert np.array_equal(s.cpu().numpy(), S[:m]) and np.array_equal(b.cpu().numpy(), B[:m]), m
    _check(orc, X, Q, a, "exponential", S, B, 129)


@pytest.mark.parametrize("kernel,a", [("exponential", 60.0), ("gaussian", 3.0), ("logistic", 60.0)])
@pytest.mark.parametrize("form", ["fp32", "fp16_split"])
def test_rescued_sums(orc, kernel, a, form):
    # every sum underflows: the maximum and shifted passes on few tiles
    import torch
    assert torch.cuda.is_available()
    import paper_2407_07096_amd as stag
    rng = np.random.default_rng(7)
    n, d, big = 4500, 300, 13000
    X, Q = _data(n, big, d, rng)
    Xd, Qd = to_dev(X), to_dev(Q)
    announce(f"wide narrow rescue {kernel} form={form} m={big} and 1..129")
    S, B = (v.cpu().numpy() for v in stag.kde_exact(Xd, Qd, a, form=form, kernel=kernel, return_bound=True))
    for m in (1, 33, 129):
        s, b = stag.kde_exact(Xd, Qd[:m].contiguous(), a, form=form, kernel=kernel, return_bound=True)
        assert np.array_equal(s.cpu().numpy(), S[:m]) and np.array_equal(b.cpu().numpy(), B[:m]), m
    _check(orc, X, Q, a, kernel, S, B, 129)


@pytest.mark.parametrize("form", ["fp32", "fp16_split", "bf16_split"])
@pytest.mark.parametrize("n,m", [(100, 1), (4097, 32), (9000, 130)])
def test_no_allocation_call(orc, n, m, form):
    import torch
    assert torch.cuda.is_available()
    from paper_2407_07096_amd import _lib as L
    import paper_2407_07096_amd as stag
    lib = stag.load()
    rng = np.random.default_rng(n)
    X, Q = _data(n, m, 400, rng)
    Xd, Qd = to_dev(X), to_dev(Q)
    want, bound = stag.kde_exact(Xd, Qd, 0.05, form=form, return_bound=True)  # shares the chunks
    S, B = torch.empty_like(want), torch.empty_like(bound)
    st = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    announce(f"wide narrow noalloc n={n} m={m} form={form}")
    assert lib.stag_kde_exact_noalloc(Xd.data_ptr(), n, Qd.data_ptr(), m, 400, 0.05, L.FORMS[form], 0, S.data_ptr(),
                                      B.data_ptr(), st) == 0
    assert torch.equal(S, want) and torch.equal(B, bound)
    _check(orc, X, Q, 0.05, "gaussian", S.cpu().numpy(), B.cpu().numpy(), m)
