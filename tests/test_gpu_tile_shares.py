"""GPU: launches whose chunks are shared by several workgroups, and the wide
tile, against the oracle and bit for bit against unshared launches."""
import numpy as np
import pytest
import torch

import oracle as orc
import paper_2407_07096_amd as stag
import synth
from tests.gpu_util import announce, to_dev

pytestmark = pytest.mark.gpu


def _data(n, m, d, seed):
    if d > 256:
        X = synth.sparse_uniform(n, d, seed)
        Q = synth.sparse_uniform(m, d, seed + 1)
        return X, Q, 0.02
    mix = synth.mixture(d, 4, seed, sigma=(0.5, 1.0))
    return synth.sample(mix, n, seed + 1), synth.sample(mix, m, seed + 2), 0.64 / d


# Rows around tile, sub-chunk and chunk edges: 31 (one ragged tile), 513 (one row
# past a 512-row sub-chunk), 4097 (one past a chunk), 8191 (one short of two)
CASES = [
    ("fp32", "gaussian", 31, 1, 3), ("fp32", "gaussian", 4097, 129, 40), ("fp32", "logistic", 513, 130, 17),
    ("fp16_split", "gaussian", 8191, 37, 64), ("bf16_split", "logistic", 4097, 5, 96),
    ("bf16_split3", "gaussian", 513, 129, 200), ("fp16_centred", "gaussian", 8191, 130, 128),
    ("fp16_centred", "gaussian", 4097, 40, 250), ("fp16_adaptive", "gaussian", 8191, 60, 70),
    ("fp32", "gaussian", 4097, 129, 257), ("fp16_split", "gaussian", 513, 130, 270),
    ("bf16_split", "gaussian", 8191, 3, 1000), ("fp16_split", "exponential", 257, 129, 300),
    ("fp32", "logistic", 31, 1, 1024), ("fp16_split", "logistic", 4097, 129, 784),
    # rows and queries grouped by one workgroup (up to 8,192) and by three launches
    ("fp32", "gaussian", 8192, 60, 20), ("fp32", "gaussian", 8193, 60, 131), ("fp16_adaptive", "gaussian", 1025, 8193, 24),
]


@pytest.mark.parametrize("form,kernel,n,m,d", CASES)
def test_small_launches_meet_their_bound(form, kernel, n, m, d):
    X, Q, a = _data(n, m, d, 7000 + n + d)
    if kernel != "gaussian":
        a = float(np.sqrt(a))
    announce(f"shared launch form={form} kernel={kernel} n={n} m={m} d={d}")
    S, B = stag.kde_exact(to_dev(X), to_dev(Q), a, form=form, kernel=kernel, return_bound=True)
    torch.cuda.synchronize()
    ref = orc.kde_exact(X, Q, a) if kernel == "gaussian" else orc.kde_kernel(X, Q, a, kernel)
    err = np.abs(S.cpu().numpy() - ref) / ref
    assert np.all(err <= B.cpu().numpy())


# The large call has a workgroup per (query tile, chunk) or fewer shares of a
# chunk; the small ones share it among up to eight.  m = 12,000 (135,000 wide)
# keeps the large call above the sharing rule at two chunks.
@pytest.mark.parametrize("form,kernel,d,m", [
    ("fp32", "gaussian", 16, 12000), ("fp32", "logistic", 33, 12000), ("fp16_split", "gaussian", 64, 12000),
    ("bf16_split", "logistic", 100, 12000), ("bf16_split3", "gaussian", 40, 12000),
    ("fp16_centred", "gaussian", 128, 12000), ("fp16_centred", "gaussian", 160, 12000),
    ("fp32", "gaussian", 300, 135000), ("fp16_split", "logistic", 257, 135000), ("fp16_split", "exponential", 260, 9000)])
def test_results_do_not_depend_on_the_sharing(form, kernel, d, m):
    n = 8191
    X, Q, a = _data(n, 300, d, 8100 + d)
    if kernel != "gaussian":
        a = float(np.sqrt(a))
    Xd = to_dev(X)
    Qd = to_dev(Q)
    big = Qd.repeat((m + 299) // 300, 1)[:m].contiguous()
    announce(f"sharing form={form} kernel={kernel} d={d} m={m}")
    full, fb = stag.kde_exact(Xd, big, a, form=form, kernel=kernel, return_bound=True)
    for k in (1, 129, 300):
        S, B = stag.kde_exact(Xd, Qd[:k].contiguous(), a, form=form, kernel=kernel, return_bound=True)
        assert torch.equal(S, full[:k]) and torch.equal(B, fb[:k]), k


def test_shared_graph_pass_draws_as_the_oracle():
    # 2,500 rows: one chunk shared by eight workgroups per query tile, tile sums stored by each
    n, d, a, s = 2500, 24, 0.05, 6
    X = synth.sample(synth.mixture(d, 4, 91, sigma=(0.5, 1.0)), n, 92)
    announce(f"shared graph pass n={n} d={d}")
    src, dst, w, deg = stag.simgraph_sample(to_dev(X), a, s, mode="exact", form="fp32", seed=5)
    torch.cuda.synchronize()
    ref = orc.kde_exact(X, X, a)
    tol = 1e-4  # the sampler's fp32 tiles expand distances around the origin
    np.testing.assert_allclose(deg.cpu().numpy(), ref, rtol=tol)
    o_src, o_dst, o_w, o_deg, o_mg = orc.simgraph_exact(X, a, s, 5, return_margin=True)
    same = dst.cpu().numpy() == o_dst
    # a draw differs only where its target lies within that error of a boundary
    assert np.all(same | (o_mg < tol))


@pytest.mark.parametrize("form,d", [("fp32", 64), ("fp16_split", 128), ("bf16_split3", 32), ("fp16_adaptive", 96),
                                    ("fp16_centred", 20), ("fp32", 320), ("bf16_split", 260)])
def test_rows_off_16_bytes(form, d):
    # the same rows at a 4-byte offset: read element by element, bit for bit the same operands
    n, m = 1500, 70
    X, Q, a = _data(n, m, d, 9300 + d)
    Xd, Qd = to_dev(X), to_dev(Q)

    def shifted(t):
        buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
        buf[1:] = t.reshape(-1)
        return buf[1:].view(t.shape)
    announce(f"unaligned rows form={form} d={d}")
    S, B = stag.kde_exact(Xd, Qd, a, form=form, return_bound=True)
    S2, B2 = stag.kde_exact(shifted(Xd), shifted(Qd), a, form=form, return_bound=True)
    assert torch.equal(S, S2) and torch.equal(B, B2)
