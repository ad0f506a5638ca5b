"""The one-launch descent at the edges of its layout (lanes per signal, values
per lane, more signals than threads) against the descent composed of one
interval-sweep launch per step.  Both round each step's gradient to float32:
over 60 steps of size 1e-2 the bounds stay within 2e-4 of each other, the
tolerance of the existing comparison over 300 steps."""
import pytest
import torch

from paper_2501_04194_amd import mining

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T", [(1, 1), (1, 20), (2, 1024), (7, 65), (12, 1000), (16, 64), (33, 372), (64, 20), (65, 21),
                                 (500, 24), (511, 24), (512, 20), (513, 20), (1023, 12), (1024, 12), (1025, 11),
                                 (12288, 1)])
def test_descent_layouts(B, T):
    x = torch.from_numpy(mining.make_dataset(B, T=T, seed=B + T)).cuda()
    kw = dict(steps=60, lr=1e-2, gamma=0.1, init=(0.15, 0.8))
    a1, b1, _ = mining.mine(x, **kw)
    a2, b2, _ = mining.mine_stepwise(x, **kw)
    assert abs(a1 - a2) < 2e-4 and abs(b1 - b2) < 2e-4, (a1, a2, b1, b2)
