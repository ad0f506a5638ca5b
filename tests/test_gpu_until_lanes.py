"""Smooth Until at the edges of its lane layout (1, 2 or 4 outputs per lane,
chosen by length and work-group size): lengths around the lanes' and the
waves' ends, intervals that begin before a lane's last output, intervals
narrower than a lane's outputs, checkpoint blocks (16 steps) and export buffers
(64 lane steps) that end inside or at the interval, sparse adjoints, slots in
LDS and in the workspace.  Same bounds as the other parity tests (gpu_util)."""
import numpy as np
import pytest

from gpu_util import check_formula
from paper_2501_04194_amd import stl

pytestmark = pytest.mark.gpu


def spec(a, b):
    lin = lambda w: {"op": "linear", "w": w, "c": 0.0}
    return {"op": "until", "a": a, "b": b, "smooth": True, "beta": 8.0, "left": lin([1.0, 0.0]), "right": lin([0.2, 1.0])}


def signal(rng, B, L):
    return (0.2 + np.cumsum(0.1 * rng.normal(size=(B, L, 2)), axis=1)).astype(np.float32)


@pytest.mark.parametrize("threads,slots", [(64, 0), (128, 0), (256, 0), (64, 1)])
def test_until_edges(threads, slots):
    rng = np.random.default_rng(threads + slots)
    for L in [1, 2, 3, 5, 63, 64, 65, 127, 129, 131, 255, 257, 300, 515]:
        x = signal(rng, 2, L)
        for a, b in [(0, 0), (0, 1), (0, 2), (1, 2), (2, 2), (3, 5), (0, 15), (1, 16), (4, 63), (5, 67), (20, 200),
                     (0, None), (2, None), (30, None)]:
            check_formula(spec(a, b), x, launch=stl.Launch(threads, 0, slots, 0),
                          what="L=%d [%s,%s] nt=%d" % (L, a, b, threads))


def test_until_sparse_adjoint():
    """Outputs without an adjoint inside a lane, a wave and a whole work-group pass."""
    rng = np.random.default_rng(3)
    x = signal(rng, 2, 1100)
    for hit in ([0], [1, 2, 5], [63, 64, 255, 256], [1023, 1024, 1099]):
        G = np.zeros((2, 1100), np.float32)
        G[:, hit] = rng.normal(size=(2, len(hit)))
        for a, b in [(0, 3), (20, 200), (0, None)]:
            check_formula(spec(a, b), x, G=G, what="G at %s [%s,%s]" % (hit, a, b))
