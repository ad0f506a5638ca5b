"""Smooth Until near the end of its FP64 exponent range: a trajectory whose
terms span almost 2^1000, an unbounded interval in which thousands of outputs
share their dominant position, and upstream gradients of 2^24.  The exponents
beta log2(e) u of about 1000 carry half a unit in the last place of float32,
2^-15, once for the product and once for beta log2(e): each term is off by up
to 2 ln(2) 2^-15 = 4.3e-5, a ratio of two of them by 8.5e-5; the bound is 2e-4."""
import numpy as np
import pytest

import oracle
from gpu_util import Gpu, assert_close
from paper_2501_04194_amd import stl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,slots", [(700, 0), (4096, 0), (4096, 1)])
@pytest.mark.parametrize("b", [None, 900])
def test_large_gradients_at_the_range_limit(L, slots, b):
    beta = 8.0
    unit = 1.0 / (beta * np.log2(np.e))
    lin = lambda w: {"op": "linear", "w": w, "c": 0.0}
    spec = {"op": "until", "a": 0, "b": b, "smooth": True, "beta": beta, "left": lin([1.0, 0.0]), "right": lin([0.0, 1.0])}
    x = np.empty((2, L, 2), np.float32)
    x[:, :, 0] = 998.5 * unit           # phi: terms 2^-998.5 of the largest
    x[:, :, 1] = 940.0 * unit
    x[:, 0, 1] = 0.0                    # the largest term
    x[:, L - 1, 1] = 997.0 * unit       # the position that decides the outputs before it
    x[1, L // 2, 1] = 996.0 * unit
    G = np.full((2, L), 2.0 ** 24, np.float32)
    G[1, ::3] *= -0.5
    g = Gpu(spec, 2, launch=stl.Launch(0, 0, slots, 0))
    dx, _ = g.bwd(x, G)
    ref, _ = oracle.backward(spec, x, G)
    mag, _ = oracle.backward(spec, x, np.abs(G))
    assert np.isfinite(dx).all(), "%d of %d values not finite" % ((~np.isfinite(dx)).sum(), dx.size)
    assert_close(dx, ref, rel=2e-4, scale=np.abs(ref).max(), elem_scale=mag, what="dx L=%d" % L)
    assert_close(g.fwd(x), oracle.forward(spec, x), what="root L=%d" % L)
