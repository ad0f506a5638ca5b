"""The batched interval sweep on signals with an infinite sample: an interval
that holds it has the infinite value it implies (the other samples' terms vanish
against it), an interval whose support misses it does not see it."""
import numpy as np
import pytest
import torch

from paper_2501_04194_amd import stl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("op", ["always", "eventually"])
@pytest.mark.parametrize("T", [20, 32, 64])
@pytest.mark.parametrize("grads", [True, False])
def test_infinite_sample(T, op, grads):
    rng = np.random.default_rng(T)
    B, N, at = 19, 300, 9
    c, eps = 2.0, 1e-6
    x = rng.uniform(-0.5, 0.5, size=(B, T, 1)).astype(np.float32)
    a = rng.uniform(-4.0, T, size=N)
    b = a + rng.uniform(1.0, T, size=N)
    # the support reaches ln(1/eps) / c = 6.9 steps past the bounds at most, and holds what lies between them
    holds, misses = (a <= at - 1) & (b >= at + 1), (a > at + 9) | (b < at - 9)
    assert holds.sum() > 20 and misses.sum() > 5
    kw = dict(op=op, beta=10.0, mask_c=c, mask_eps=eps, grads=grads)
    bad = x.copy()
    bad[:, at] = np.inf if op == "eventually" else -np.inf
    t = lambda v: torch.from_numpy(np.asarray(v, np.float32)).cuda()
    first = lambda r: (r[0] if grads else r).cpu().numpy().astype(np.float64)
    rho = first(stl.interval_sweep(t(bad), t(a), t(b), [1.0], **kw))
    ref = first(stl.interval_sweep(t(x), t(a), t(b), [1.0], **kw))
    assert (rho[:, holds] == bad[0, at, 0]).all(), rho[:, holds]
    # both meet the oracle's 1e-5 of the value and of the scale 1
    assert (np.abs(rho - ref)[:, misses] <= 2e-5 * (1.0 + np.abs(ref[:, misses]))).all()
