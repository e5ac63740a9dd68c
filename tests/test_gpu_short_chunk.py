"""GPU: data of one chunk, shared by several workgroups or not by their number
of 32-row tiles: the same bits as an unshared launch on each side of the line,
and sums within the bounds of the oracle."""
import numpy as np
import pytest
import torch

import oracle as orc
import paper_2407_07096_amd as stag
import synth
from tests.gpu_util import announce, to_dev

pytestmark = pytest.mark.gpu

# Tiles on both sides of each line: 16 | 17; 24 | 25 and 48 | 49 (wide rows,
# split and fp32); 32 | 33 (Gaussian, at most 32 coordinates); 63 | 64 (centred
# fp16 above 128).  The large call has 128 query tiles (2,048 for wide rows),
# where no launch shares a chunk.
CASES = [
    ("fp32", "logistic", 40, 16400, (1, 512, 513, 544)), ("bf16_split", "gaussian", 64, 16400, (512, 513, 1100)),
    ("fp16_split", "gaussian", 32, 16400, (1024, 1025)), ("fp16_split", "logistic", 16, 16400, (512, 513)),
    ("fp32", "gaussian", 60, 16400, (512, 513)), ("fp16_centred", "gaussian", 100, 16400, (512, 513)),
    ("fp16_centred", "gaussian", 130, 16400, (2016, 2017)), ("fp32", "gaussian", 257, 262200, (1536, 1537)),
    ("fp16_split", "gaussian", 300, 262200, (768, 769)),
]


@pytest.mark.parametrize("form,kernel,d,m,ns", CASES)
def test_one_chunk_on_both_sides_of_the_line(form, kernel, d, m, ns):
    for n in ns:
        if d > 256:
            X, Q, a = synth.sparse_uniform(n, d, 9), synth.sparse_uniform(260, d, 10), 0.02
        else:
            mix = synth.mixture(d, 4, 9, sigma=(0.5, 1.0))
            X, Q, a = synth.sample(mix, n, 10), synth.sample(mix, 260, 11), 0.64 / d
        if kernel != "gaussian":
            a = float(np.sqrt(a))
        announce(f"one chunk form={form} kernel={kernel} n={n} m={m} d={d}")
        Xd, Qd = to_dev(X), to_dev(Q)
        big = Qd.repeat((m + 259) // 260, 1)[:m].contiguous()
        full, fb = stag.kde_exact(Xd, big, a, form=form, kernel=kernel, return_bound=True)
        for k in (3, 260):
            S, B = stag.kde_exact(Xd, Qd[:k].contiguous(), a, form=form, kernel=kernel, return_bound=True)
            torch.cuda.synchronize()
            assert torch.equal(S.view(torch.int64), full[:k].view(torch.int64)), (n, k)
            assert torch.equal(B.view(torch.int64), fb[:k].view(torch.int64)), (n, k)
        ref = orc.kde_exact(X, Q, a) if kernel == "gaussian" else orc.kde_kernel(X, Q, a, kernel)
        assert np.all(np.abs(S.cpu().numpy() - ref) <= B.cpu().numpy() * ref), n
