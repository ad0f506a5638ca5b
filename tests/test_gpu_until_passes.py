"""Smooth Until where the number of outputs per lane changes (an eighth beyond
one and two work-groups' lanes), so that one pass is full and the next has the
fewest or the most outputs it may have.  Same bounds as the other parity tests."""
import numpy as np
import pytest

from gpu_util import check_formula
from paper_2501_04194_amd import stl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("threads,slots", [(64, 0), (256, 0), (64, 1)])
@pytest.mark.parametrize("a,b", [(0, 2), (5, 67), (0, None)])
def test_until_pass_edges(threads, slots, a, b):
    lin = lambda w: {"op": "linear", "w": w, "c": 0.0}
    spec = {"op": "until", "a": a, "b": b, "smooth": True, "beta": 8.0, "left": lin([1.0, 0.0]), "right": lin([0.2, 1.0])}
    rng = np.random.default_rng(threads)
    one = threads + threads // 8
    for L in (threads + 1, one, one + 1, 2 * threads + 1, 2 * one, 2 * one + 1, 4 * threads + 1):
        x = (0.2 + np.cumsum(0.1 * rng.normal(size=(2, L, 2)), axis=1)).astype(np.float32)
        check_formula(spec, x, launch=stl.Launch(threads, 0, slots, 0), what="L=%d nt=%d" % (L, threads))
