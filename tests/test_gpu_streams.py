"""Calls on several streams and from several threads at once: the workspaces
that they share through the block cache must not mix their results."""
import threading

import numpy as np
import pytest

import synth
from tests.gpu_util import announce, to_dev

pytestmark = pytest.mark.gpu

SIZES = [(4000, 500, 32), (20000, 1000, 64), (9001, 300, 300)]


def _calls():
    import paper_2407_07096_amd as stag
    out = []
    for k, (n, m, d) in enumerate(SIZES):
        rng = np.random.default_rng(100 + k)
        X = to_dev(rng.normal(size=(n, d)).astype(np.float32))
        Q = to_dev(rng.normal(size=(m, d)).astype(np.float32))
        out.append(lambda X=X, Q=Q, d=d: stag.kde_exact(X, Q, 0.5 / d, form="fp16_split"))
    ix = stag.LshIndex(to_dev(synth.config_points(2, n=5000, m=1)[0]), 0.01, eps=0.5, k1=2, k2_constant=8.0)
    Q = to_dev(synth.config_points(2, n=5000, m=700)[1])
    out.append(lambda: ix.query(Q))
    return out


def test_four_streams_and_threads_match_one():
    import torch
    calls = _calls()
    want = [f().cpu().numpy() for f in calls]
    streams = [torch.cuda.Stream() for _ in calls]
    torch.cuda.synchronize()
    announce("four calls on four streams, 12 rounds")
    got = []
    for r in range(12):
        for k, f in enumerate(calls):
            with torch.cuda.stream(streams[(k + r) % len(streams)]):
                got.append((k, f()))
    torch.cuda.synchronize()
    for k, v in got:
        assert np.array_equal(v.cpu().numpy(), want[k])

    announce("four calls from four threads, 12 rounds each")
    bad = []

    def work(k):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            vals = [calls[k]() for _ in range(12)]
        s.synchronize()
        bad.extend(k for v in vals if not np.array_equal(v.cpu().numpy(), want[k]))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(calls))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
