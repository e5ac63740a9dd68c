"""The CKNS bucket join with more tasks than it takes at once: every pair of
1e5 points shares its buckets (about 1e7 tasks), so the batch is done in
slices.  Estimates and counts are bit for bit those of small batches."""
import ctypes as C

import numpy as np
import pytest

from tests.gpu_util import announce, to_dev

pytestmark = pytest.mark.gpu


def test_sliced_batch_matches_small_batches():
    import torch
    assert torch.cuda.is_available()  # (its HIP runtime is loaded first)
    import paper_2407_07096_amd as stag
    lib = stag.load()
    rng = np.random.default_rng(11)
    n = 100000
    X = to_dev((rng.normal(size=(n, 3)) * 1e-3).astype(np.float32))
    ix = stag.LshIndex(X, 0.5, eps=0.5, k1=1, k2_constant=8.0)
    announce("join slices n=m=100000 d=3, one bucket a table")
    lib.stag_timing_enable(1)
    try:
        S, st = ix.query(X, stats=True)
        buf = C.create_string_buffer(1 << 16)
        lib.stag_timing_report(buf, len(buf))
    finally:
        lib.stag_timing_enable(0)
    counts = {k: int(c) for k, c, _ in (line.split() for line in buf.value.decode().splitlines())}
    assert counts["lsh_join"] >= 2
    for lo, hi in ((0, 64), (n // 2, n // 2 + 3000), (n - 1000, n)):
        S2, st2 = ix.query(X[lo:hi].contiguous(), stats=True)
        assert np.array_equal(S2.cpu().numpy(), S[lo:hi].cpu().numpy())
        for k in st:
            assert np.array_equal(st2[k].cpu().numpy(), st[k][lo:hi].cpu().numpy()), k
