"""Scan edges of the generic executor: lengths around the wave, the row of 16
lanes, the work-group and odd chunk sizes, blocks of one step up to longer than
the trajectory, every work-group size, with the slots in LDS and in the
workspace.  Same bounds as the other parity tests (gpu_util)."""
import numpy as np
import pytest

from gpu_util import check_formula
from paper_2501_04194_amd import stl

pytestmark = pytest.mark.gpu

LENGTHS = [1, 2, 15, 16, 17, 63, 64, 65, 127, 129, 255, 257, 511, 513, 1025]


def spec(a, b, smooth):
    lin = lambda w, c: {"op": "linear", "w": w, "c": c}
    s = {"smooth": smooth, "beta": 10.0}
    return dict(op="and", children=[
        dict(op="always", a=a, b=b, child=dict(op="or", children=[lin([1.0, 0.5, 0.0], 0.1),
                                                                  lin([0.0, 1.0, -1.0], -0.2)], **s), **s),
        dict(op="eventually", a=0, b=None, child=lin([0.0, 0.0, 1.0], 0.0), **s)], **s)


@pytest.mark.parametrize("threads,slots", [(64, 0), (128, 0), (256, 0), (512, 0), (256, 1)])
@pytest.mark.parametrize("smooth", [False, True])
def test_scan_edges(threads, slots, smooth):
    rng = np.random.default_rng(7)
    for L in LENGTHS:
        x = np.cumsum(0.1 * rng.normal(size=(2, L, 3)), axis=1).astype(np.float32)
        for a, b in [(0, 0), (0, 6), (2, 20), (1, 64), (3, 300), (0, 2000)]:
            check_formula(spec(a, b, smooth), x, launch=stl.Launch(threads, 0, slots, 0),
                          what="L=%d [%d,%d] nt=%d" % (L, a, b, threads), exact_sentinels=False)


@pytest.mark.parametrize("D", [1, 2, 3, 4, 5, 16])
def test_predicate_rows(D):
    """Rows of every width, and x that is not aligned to the row size."""
    import torch
    rng = np.random.default_rng(D)
    A = rng.normal(size=(min(D, 3), D)).tolist()
    f = {"op": "and", "smooth": True, "beta": 5.0, "children": [
        {"op": "linear", "w": rng.normal(size=D).tolist(), "c": 0.3},
        {"op": "norm", "A": A, "p": rng.normal(size=len(A)).tolist(), "r": 0.5, "sign": 1.0},
        {"op": "linear", "w": rng.normal(size=D).tolist(), "c": -0.1}]}
    x = rng.normal(size=(3, 301, D)).astype(np.float32)
    G = rng.normal(size=(3, 301)).astype(np.float32)
    g = check_formula(f, x, G=G, what="D=%d" % D)
    buf = torch.zeros(x.size + 1, device="cuda")
    xu = buf[1:].view(x.shape)
    xu.copy_(torch.from_numpy(x))
    Gd = torch.from_numpy(G).cuda()
    root, dx = g.plan.forward(xu, g.pv), g.plan.backward(xu, Gd, g.pv)[0]
    assert np.array_equal(root.cpu().numpy(), g.fwd(x))
    assert np.array_equal(dx.cpu().numpy(), g.bwd(x, G)[0])
