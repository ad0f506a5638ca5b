"""Formulas of many predicates through stl_forward_static, whose workspace is
fixed: where all their traces at once would not fit on chip, a predicate's trace
takes a slot only until its parent has read it."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2501_04194_amd import stl

E_WORKSPACE = -5


def tree(n, smooth=False):
    s = {"smooth": True, "beta": 8.0} if smooth else {}
    level = [{"op": "linear", "w": [np.cos(k), np.sin(k)], "c": 0.1 * k / n} for k in range(n)]
    op = "and"
    while len(level) > 1:
        level = [dict(op=op, children=level[i:i + 4], **s) for i in range(0, len(level), 4)]
        op = "or" if op == "and" else "and"
    return level[0]


# (formula, B, T, slots in the workspace): 25 floats a timestep and trajectory fit, 33 do not
CASES = [(tree(32), 60, 2700, 0), (tree(32, True), 60, 2700, 0), (tree(32), 1000, 160, 1)]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_accepted(case):
    """The workspace is checked before the missing output: with it too small the status would say so."""
    spec, B, T, slots = CASES[case]
    plan = stl.Plan(spec, 2)
    bt = stl.Batch()
    bt.x, bt.B, bt.T, bt.D = 256, B, T, 2            # (never read: no output, so nothing is launched)
    pv = ctypes.c_void_p(256)
    launch = stl.Launch(0, 0, slots, 0)
    st = stl.lib().stl_forward_static(plan.handle, ctypes.byref(bt), pv, None, None, ctypes.byref(launch), None)
    msg = stl.lib().stl_last_error().decode()
    assert st < 0 and "workspace" not in msg, (st, msg)


@pytest.mark.gpu
@pytest.mark.parametrize("n,smooth,B,T", [(32, False, 300, 1300), (32, True, 300, 1300), (32, False, 60, 2700),
                                          (20, True, 17, 2500), (32, True, 3, 6001)])
def test_values(n, smooth, B, T):
    from gpu_util import check_formula
    spec = tree(n, smooth)
    x = np.cumsum(0.05 * np.random.default_rng(T).normal(size=(B, T, 2)), axis=1).astype(np.float32)
    g = check_formula(spec, x, grads=B <= 17, what="%d predicates T=%d" % (n, T))
    xd = torch.from_numpy(x).cuda()
    ref, nodes = g.plan.forward(xd, g.pv, node_traces=True)
    assert torch.equal(ref, g.plan.forward(xd, g.pv))
    assert torch.equal(ref, g.plan.forward_static(xd, g.pv))


@pytest.mark.gpu
@pytest.mark.parametrize("D,n", [(1, 32), (2, 32), (3, 32), (4, 32), (5, 26)])
@pytest.mark.parametrize("T", [1, 70, 700])
def test_predicates_in_their_place(D, n, T):
    """Every state width's predicate code, slots in the workspace, dense and ragged, norm predicates among
    them where the coefficients allow it."""
    from gpu_util import check_formula
    rng = np.random.default_rng(D * T)

    def pred(k):
        if D <= 2 and k % 4 == 3:
            return {"op": "norm", "A": [[1.0] * D], "p": [0.1], "r": 0.2 + 0.01 * k, "sign": 1.0 if k % 8 == 3 else -1.0}
        return {"op": "linear", "w": [float(v) for v in rng.normal(size=D)], "c": 0.1 * k / n}

    level, op = [pred(k) for k in range(n)], "or"
    while len(level) > 1:
        level = [dict(op=op, children=level[i:i + 4], smooth=True, beta=8.0) for i in range(0, len(level), 4)]
        op = "and" if op == "or" else "or"
    launch = stl.Launch(0, 0, 1, 0)
    x = np.cumsum(0.1 * rng.normal(size=(3, T, D)), axis=1).astype(np.float32)
    check_formula(level[0], x, launch=launch, what="D=%d T=%d" % (D, T))
    off = np.array([0, T, T, T + (T + 1) // 2], dtype=np.int64)
    check_formula(level[0], x.reshape(-1, D)[:off[-1]].copy(), launch=launch, offsets=off, T=T, what="ragged D=%d" % D)
