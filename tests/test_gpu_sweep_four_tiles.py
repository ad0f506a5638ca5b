"""The batched interval sweep in its four-tile form, with and without gradients,
against the FP64 oracle on sampled signals and intervals: ragged in both, the
first and last interval of a work-group and of the sweep, signals at the edges
of a tile, and (amp = 8) sums that are redone against their own reference."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import assert_close
from paper_2501_04194_amd import stl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,B,N,amp", [(6, 65, 256 * 13108 - 3, 8.0), (20, 4083, 256 * 257 - 3, 0.5),
                                       (17, 4096, 256 * 256 - 1, 8.0)])
@pytest.mark.parametrize("op", ["always", "eventually"])
@pytest.mark.parametrize("grads", [True, False])
def test_against_oracle(T, B, N, amp, op, grads):
    rng = np.random.default_rng(T * B)
    x = rng.uniform(-amp, amp, size=(B, T, 1)).astype(np.float32)
    a = rng.uniform(-2.0, T, size=N).astype(np.float32)
    b = (a + rng.uniform(0.5, T, size=N)).astype(np.float32)
    kw = dict(c=0.0, op=op, beta=10.0, mask_c=2.0, mask_eps=1e-6)
    t = lambda v: torch.from_numpy(v).cuda()
    got = stl.interval_sweep(t(x), t(a), t(b), [1.0], grads=grads, **kw)
    rows = sorted({0, 1, 15, 16, B // 2, B - 2, B - 1})
    cols = np.unique(np.concatenate([[0, 3, 15, 16, 63, 64, 255, 256, N // 2, N - 4, N - 2, N - 1],
                                     rng.integers(0, N, size=40)]))
    ref = oracle.interval_sweep(x[rows], a[cols].astype(np.float64), b[cols].astype(np.float64), [1.0], **kw)
    ri, ci = torch.tensor(rows, device="cuda"), torch.from_numpy(cols).cuda()
    for g, r, scale, what in zip(got if grads else [got], ref, (max(1.0, amp), 2.0 / 40, 2.0 / 40),
                                 ("rho", "d/da", "d/db")):
        assert_close(g[ri][:, ci].cpu().numpy(), r, scale=scale, what="%s T=%d B=%d" % (what, T, B))
